// Channel mutation (Sec. 2.3): one weight per layer on a path from input unit
// u_0 to class u_L changes at once (re-drawn with the He amplitude of its
// fan-in, or set to zero).  From the cached local fields the change is:
//  - first layer: column u_1 of the field moves by de_0 * x[:, u_0];
//  - every later layer m: its field moves by W_m times the change of its
//    input (rank-1 through column W_m[:, u_1] for m = 1, a dense product
//    after that) plus the path weight's own change, de_m times the new
//    activation of the input unit u_m, at unit u_{m+1}
//    (W'_m a' - W_m a = W_m (a' - a) + (w'_m - w_m) a'[u_m]);
//  - the logits' change gives each sample's loss change with the cached
//    softmax (ce_change).
//
// Most of that is one unit at a time.  Where the first unit's activation does not
// change (its input is zero on four of five samples of an image, or a ReLU unit
// stays off), the second field moves at the path's unit alone, by its own
// weight's change; if that unit's activation does not change either, so does the
// third, and so on.  k_channel_rows walks every sample along the path up to the
// layer f that first receives a changed activation: layer f moves by the rank-1
// term of that one unit, and only the layers after it need dense products.
// Samples whose walk reaches the logits are done there (a rank-1 logit change; in a
// net of two layers all of them, k_channel_two);
// the others are listed, those of f = 1 first, and blocks of k_channel take tiles
// of T of them (dense_tile.hpp).  On 784-1024x3-10 with ReLU a tenth of the
// samples need the dense layer, a fifth a rank-1 second layer: 16 channels on 8192
// samples, with the products on bf16 parts, 5.4 -> 0.41 ms.
// The commit runs the same arithmetic for the chosen channel and moves every
// cached field by its change; a last kernel writes the path's weights.
#include <algorithm>
#include <type_traits>

#include "dense_tile.hpp"
#include "channel_kernels.hpp"

namespace mca {

namespace {

// Blocks of k_channel per unit of residency: one a CU, and a second round's worth
// so that a slow one is not waited for.
constexpr int kChannelBlocks = 512;

// Samples of a listing block, and its tile sums: the tiles of its two lists, at
// most one part-filled tile more, and the walked samples.
constexpr int kSegU = 2, kSegment = kSegU * kListThreads;
__host__ __device__ constexpr int segment_slots(int T) { return (kSegment + T - 1) / T + 2; }
// Samples of a block of k_channel_two: one wave.
constexpr int kTwo = 64;

// The channel of draw (t, k): 2L + 1 words of the Philox blocks at counters
// (t, k, 2 + b, 0), four words per block, in order.
__device__ mca_channel draw_channel(const NetDev& net, uint64_t t, uint64_t k) {
  mca_channel ch;
  const int L = net.L, nw = 2 * L + 1;
  for (int q = 0; q <= MCA_MAX_LAYERS; ++q) ch.units[q] = 0;
  for (int m = 0; m < MCA_MAX_LAYERS; ++m) ch.w_new[m] = 0.0f;
  for (int q0 = 0; q0 < nw; q0 += 4) {
    const Words w = philox4x64_10(t, k, 2 + (uint64_t)(q0 / 4), 0, net.seed, net.tag);
    const uint64_t ws[4] = {w.w0, w.w1, w.w2, w.w3};
    for (int e = 0; e < 4 && q0 + e < nw; ++e) {
      const int q = q0 + e;
      if (q <= L) {
        ch.units[q] = (int32_t)__umul64hi(ws[e], (uint64_t)net.widths[q]);
      } else if (net.mutation == MCA_MUTATE_CHANNEL_REDRAW) {
        const int m = q - L - 1;
        const float r = (float)(uint32_t)(ws[e] >> 40) * 0x1p-23f - 1.0f;
        ch.w_new[m] = net.chan_amp[m] * r;
      }
    }
  }
  return ch;
}

// Acceptance data of a channel: the weight bound (every re-drawn weight must
// stay inside it, Eq. 1) and the selection threshold.
__device__ Aux channel_aux(const NetDev& net, const mca_channel& ch) {
  Aux a;
  a.w_old = a.w_new = a.de = 0.0f;
  int ok = 1;
  for (int m = 0; m < net.L; ++m) ok &= !(net.bound > 0.f && fabsf(ch.w_new[m]) >= net.bound);
  a.valid = ok;
  a.theta = 0.0;
  return a;
}

__device__ __forceinline__ mca_cand placeholder() {
  mca_cand c;
  c.flat = 0;
  c.layer = 0;
  c.j = c.i = 0;
  c.d = 0.0f;
  c.code = 0;
  c.flags = 0;
  return c;
}

}  // namespace

__global__ void k_channel_propose(NetDev net_arg, uint64_t t_host, int use_dev_t,
                                  const DevState* st, int K, mca_channel* chans, mca_cand* cands,
                                  Aux* aux, mca_channel* host) {
  __shared__ NetDev net;
  stage_net(net, net_arg);
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= K) return;
  const uint64_t t = use_dev_t ? st->t : t_host;
  const mca_channel ch = draw_channel(net, t, (uint64_t)k);
  chans[k] = ch;
  if (host != nullptr) host[k] = ch;
  Aux a = channel_aux(net, ch);
  a.theta = accept_theta(net.rule, net.beta, net.seed, net.tag, t, (uint64_t)k);
  aux[k] = a;
  cands[k] = placeholder();
}

__global__ void k_channel_prepare(NetDev net_arg, mca_channel* chans, int K,
                                  mca_cand* cands, Aux* aux, const mca_channel* host) {
  __shared__ NetDev net;
  stage_net(net, net_arg);
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= K) return;
  const mca_channel ch = host != nullptr ? host[k] : chans[k];
  if (host != nullptr) chans[k] = ch;
  aux[k] = channel_aux(net, ch);
  cands[k] = placeholder();
}

// The path and the increments fl32(w' - w) of its weights (committed weights: a
// commit writes the new ones only after the field kernels).  By every thread.
__device__ __forceinline__ void load_path(const NetDev& net, const mca_channel& ch, int* units, float* de) {
  const int tid = threadIdx.x;
  if (tid <= net.L) units[tid] = ch.units[tid];
  __syncthreads();
  if (tid < net.L) {
    const float wo = net.W[tid][(int64_t)units[tid + 1] * net.widths[tid] + units[tid]];
    de[tid] = ch.w_new[tid] - wo;
  }
  __syncthreads();
}

// Block (s, k) (eval) or (s, 0) for the committed channel: the walk of the samples
// of segment s along the path.  Samples that break off at layer f <= L-2 are
// listed in sample order, f = 1 from the front of the segment's part of the
// channel's lists, later ones from its back: the sample, the changed activation
// entering layer f, the path unit's new one, f.  The others' loss changes are
// summed here, the segment's last tile sum.  The grid's last block then adds up
// the tiles of all lists (those of f = 1 first): lists.first[e], e = (list K + k)
// S + s.  A commit stores the walked fields.  Segments of 2048 samples: the walk
// is a chain of dependent loads, so its time is one block's; more samples a block
// take longer, fewer leave more part-filled tiles (8192 samples, 16 channels: 76
// us with one block a channel, 24 with these).
__global__ __launch_bounds__(kListThreads) void k_channel_rows(NetDev net_arg, const mca_channel* chans,
                                                               const Aux* aux, ChannelLists lists, float* partial,
                                                               int nchan, int T, int K, int k_mode, DevState* st) {
  __shared__ NetDev net;
  stage_net(net, net_arg);
  __shared__ int units[MCA_MAX_LAYERS + 1];
  __shared__ float de[MCA_MAX_LAYERS];
  __shared__ int counts[2][32];  // [list][u][wave]
  __shared__ double sums[kListThreads / 64];
  __shared__ int last;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool commit = k_mode != -2;
  const int k = commit ? ((k_mode >= 0) ? k_mode : st->chosen) : (int)blockIdx.y;
  const int S = (int)gridDim.x, seg = (int)blockIdx.x, nl = commit ? 1 : K;
  if (k < 0) {
    if (tid == 0) lists.first[2 * S] = 0;
    return;
  }
  const int L = net.L, C = net.C, act = net.act;
  const float gamma = net.gamma;
  const int64_t N = net.N, Ns = net.Ns;
  const bool scored = commit || aux[k].valid;  // rejected unevaluated: selection gives +inf
  int count[2] = {0, 0};
  double sum = 0.0;
  float* const sums_out = partial + (int64_t)k * nchan + seg * segment_slots(T);
  if (!commit && tid < segment_slots(T)) sums_out[tid] = 0.f;
  if (scored) {
    load_path(net, chans[k], units, de);
    const int64_t n0 = (int64_t)seg * kSegment;
    const int64_t part = (int64_t)(commit ? 0 : k) * N + n0,  // (a commit's lists are the first)
                   part_n = N - n0 < kSegment ? N - n0 : kSegment;
    {
      int64_t ns[kSegU];
      float d[kSegU], ap[kSegU];  // the last walked unit's change and new activation
      int f[kSegU];                // the layer they enter
      {
        float* z0 = net.Z[0] + (int64_t)units[1] * Ns;
        float x[kSegU], z[kSegU];
#pragma unroll
        for (int u = 0; u < kSegU; ++u) {
          const int64_t n = n0 + u * kListThreads + tid;
          ns[u] = n < N ? n : N - 1;
          x[u] = gload(&net.XT[(int64_t)units[0] * Ns + ns[u]]);
          z[u] = gload(&z0[ns[u]]);
        }
#pragma unroll
        for (int u = 0; u < kSegU; ++u) {
          const float dz = de[0] * x[u];
          d[u] = dphi(z[u], dz, act, gamma);
          ap[u] = act_fn(z[u] + dz, act, gamma);
          f[u] = 1;
          if (commit && dz != 0.f && n0 + u * kListThreads + tid < N) gstore(&z0[ns[u]], z[u] + dz);
        }
      }
      for (int m = 1; m <= L - 2; ++m) {
        float* zm = net.Z[m] + (int64_t)units[m + 1] * Ns;
        float z[kSegU];
#pragma unroll
        for (int u = 0; u < kSegU; ++u) z[u] = gload(&zm[ns[u]]);
#pragma unroll
        for (int u = 0; u < kSegU; ++u) {
          if (f[u] == m && d[u] == 0.f) {
            const float dz = de[m] * ap[u];
            d[u] = dphi(z[u], dz, act, gamma);
            ap[u] = act_fn(z[u] + dz, act, gamma);
            f[u] = m + 1;
            if (commit && dz != 0.f && n0 + u * kListThreads + tid < N) gstore(&zm[ns[u]], z[u] + dz);
          }
        }
      }
      uint64_t b[2][kSegU];
#pragma unroll
      for (int u = 0; u < kSegU; ++u) {
        const bool in = n0 + u * kListThreads + tid < N;
        b[0][u] = __ballot(in && f[u] <= L - 2 && f[u] == 1);
        b[1][u] = __ballot(in && f[u] <= L - 2 && f[u] > 1);
        if (lane < 2) counts[lane][u * (kListThreads / 64) + wave] = (int)__popcll(lane ? b[1][u] : b[0][u]);
        if (in && f[u] == L - 1) {
          // a rank-1 change of the logits
          const float* WL = net.W[L - 1] + units[L - 1];
          const float dp = de[L - 1] * ap[u];
          if (d[u] != 0.f || dp != 0.f) {
            const int64_t n = ns[u];
            const int y = gload(&net.y[n]), cls = units[L];
            float dz[kCMax], p[kCMax], dzy = 0.f;
#pragma unroll
            for (int c = 0; c < kCMax; ++c) {
              dz[c] = 0.f;
              p[c] = (c < C) ? gload(&net.prob[(int64_t)c * Ns + n]) : 0.f;
              if (c < C) {
                dz[c] = d[u] * gload(&WL[(int64_t)c * net.widths[L - 1]]);
                if (c == cls) dz[c] = fmaf(de[L - 1], ap[u], dz[c]);
              }
              dzy = (c == y) ? dz[c] : dzy;
            }
            sum += (double)ce_change<kCMax>(p, dz, C, dzy);
            if (commit) {
              float* ZL = net.Z[L - 1];
              float z[kCMax], pn[kCMax];
#pragma unroll
              for (int c = 0; c < kCMax; ++c) z[c] = (c < C) ? gload(&ZL[(int64_t)c * Ns + n]) + dz[c] : 0.f;
              const float ln = softmax_ce<kCMax>(z, C, y, pn);
#pragma unroll
              for (int c = 0; c < kCMax; ++c)
                if (c < C) {
                  gstore(&ZL[(int64_t)c * Ns + n], z[c]);
                  gstore(&net.prob[(int64_t)c * Ns + n], pn[c]);
                }
              gstore(&net.ell[n], ln);
            }
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const int mine = lane < 32 ? counts[g][lane] : 0;
        int incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int w = __shfl_up(incl, o, 64);
          if (lane >= o) incl += w;
        }
#pragma unroll
        for (int u = 0; u < kSegU; ++u) {
          const int off = __shfl(incl - mine, u * (kListThreads / 64) + wave, 64);
          if ((b[g][u] >> lane) & 1ull) {
            const int64_t e = off + (int)__popcll(b[g][u] & ((1ull << lane) - 1ull));
            const int64_t at = part + (g == 0 ? e : part_n - 1 - e);
            gstore(&lists.rows[at], (int)ns[u]);
            gstore(&lists.d[at], d[u]);
            gstore(&lists.ap[at], ap[u]);
            gstore(&lists.f[at], f[u]);
          }
        }
        count[g] = __shfl(incl, 63, 64);
      }
    }
  }
  if (!commit && scored) {
    // the walked samples' sum: lanes by a butterfly, waves in order
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (lane == 0) sums[wave] = sum;
    __syncthreads();
    if (tid == 0) {
      double s = 0.0;
      for (int w = 0; w < kListThreads / 64; ++w) s += sums[w];
      sums_out[segment_slots(T) - 1] = (float)s;
    }
  }
  // the tiles of every list, in order (a commit: of its channel's)
  const int ne = 2 * nl * S, e_k = (commit ? 0 : k) * S + seg;
  if (tid == 0) {
    __hip_atomic_store(&lists.cnt[e_k], count[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&lists.cnt[nl * S + e_k], count[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __threadfence();
    last = atomicAdd(&st->list_done, 1u) == gridDim.x * gridDim.y - 1;
  }
  __syncthreads();
  if (!last || wave != 0) return;
  __threadfence();
  int total = 0;
  for (int e0 = 0; e0 < ne; e0 += 64) {
    const int e = e0 + lane;
    const int c = e < ne ? __hip_atomic_load(&lists.cnt[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    const int tiles = (c + T - 1) / T;
    int incl = tiles;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int w = __shfl_up(incl, o, 64);
      if (lane >= o) incl += w;
    }
    if (e < ne) lists.first[e + 1] = total + incl;
    total += __shfl(incl, 63, 64);
  }
  if (lane == 0) {
    lists.first[0] = 0;
    st->list_done = 0u;
  }
}

// A net of two layers: every sample's walk ends at the logits and nothing is listed.
// Block (b, k) (eval) or (b, 0) for the committed channel: 64 samples, their changes'
// sum the block's one tile sum.  A step of such a net is a chain of short launches,
// so a sample's loads all leave together and a block is one wave: walked as segments
// of 2048 samples on one CU each, 380-256-12 with one channel a step on 1585 samples
// took 37 us a step (24 here), 400-512-10 with 64 channels on 10000 samples 86 (43).
__global__ __launch_bounds__(kTwo) void k_channel_two(NetDev net_arg, const mca_channel* chans, const Aux* aux,
                                                      float* partial, int nchan, int k_mode, const DevState* st) {
  __shared__ NetDev net;
  stage_net(net, net_arg);
  __shared__ int units[MCA_MAX_LAYERS + 1];
  __shared__ float de[MCA_MAX_LAYERS];
  const int tid = threadIdx.x;
  const bool commit = k_mode != -2;
  const int k = commit ? ((k_mode >= 0) ? k_mode : st->chosen) : (int)blockIdx.y;
  if (k < 0) return;
  if (!commit && !aux[k].valid) {  // rejected unevaluated: selection gives +inf
    if (tid == 0) partial[(int64_t)k * nchan + blockIdx.x] = 0.f;
    return;
  }
  load_path(net, chans[k], units, de);
  const int C = net.C, act = net.act, cls = units[2];
  const float gamma = net.gamma;
  const int64_t N = net.N, Ns = net.Ns, at = (int64_t)blockIdx.x * kTwo + tid, n = at < N ? at : N - 1;
  float* zp = net.Z[0] + (int64_t)units[1] * Ns + n;
  const float* WL = net.W[1] + units[1];
  const float x = gload(&net.XT[(int64_t)units[0] * Ns + n]), z0 = gload(zp);
  const int y = gload(&net.y[n]);
  float p[kCMax], w[kCMax];
#pragma unroll
  for (int c = 0; c < kCMax; ++c) {
    p[c] = (c < C) ? gload(&net.prob[(int64_t)c * Ns + n]) : 0.f;
    w[c] = (c < C) ? gload(&WL[(int64_t)c * net.widths[1]]) : 0.f;
  }
  const float dz0 = de[0] * x, d = dphi(z0, dz0, act, gamma), ap = act_fn(z0 + dz0, act, gamma);
  float change = 0.f;
  if (at < N && (d != 0.f || de[1] * ap != 0.f)) {
    float dz[kCMax], dzy = 0.f;
#pragma unroll
    for (int c = 0; c < kCMax; ++c) {
      dz[c] = d * w[c];
      if (c == cls) dz[c] = fmaf(de[1], ap, dz[c]);
      dzy = (c == y) ? dz[c] : dzy;
    }
    change = ce_change<kCMax>(p, dz, C, dzy);
    if (commit) {
      float* ZL = net.Z[1];
      float z[kCMax], pn[kCMax];
#pragma unroll
      for (int c = 0; c < kCMax; ++c) z[c] = (c < C) ? gload(&ZL[(int64_t)c * Ns + n]) + dz[c] : 0.f;
      const float ln = softmax_ce<kCMax>(z, C, y, pn);
#pragma unroll
      for (int c = 0; c < kCMax; ++c)
        if (c < C) {
          gstore(&ZL[(int64_t)c * Ns + n], z[c]);
          gstore(&net.prob[(int64_t)c * Ns + n], pn[c]);
        }
      gstore(&net.ell[n], ln);
    }
  }
  if (commit) {
    if (at < N && dz0 != 0.f) gstore(zp, z0 + dz0);
    return;
  }
  double sum = (double)change;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if (tid == 0) partial[(int64_t)k * nchan + blockIdx.x] = (float)sum;
}

// Tiles of the lists, shared out to the grid's blocks in list order.
template <int W, int ACT, bool commit>
__global__ __launch_bounds__((Dense<W, commit>::threads), (Dense<W, commit>::blocks_per_cu)) void k_channel(
    NetDev net_arg, const mca_channel* chans, ChannelLists lists, float* partial, int nchan, int K,
    int S, int k_mode, const DevState* st) {
  typedef Dense<W, commit> D;
  constexpr int T = D::T, SB = D::SB, H = D::H, NW = D::NW;
  const int nl = commit ? 1 : K, ne = 2 * nl * S;
  if ((int)blockIdx.x >= lists.first[ne]) return;
  __shared__ NetDev net;
  stage_net(net, net_arg);
  __shared__ __attribute__((aligned(16))) typename D::Tile ta;
  __shared__ int rown[T], rowf[T];
  __shared__ float rowd[T], rowa[T], dls[T];
  __shared__ int units[MCA_MAX_LAYERS + 1];
  __shared__ float de[MCA_MAX_LAYERS];
  __shared__ int item[2];
  auto logit = reinterpret_cast<float (*)[T][17]>(ta);
  static_assert(sizeof(float) * NW * T * 17 <= sizeof(ta), "the logits' sums take the tile's place");
  const int tid = threadIdx.x, L = net.L;
  const float gamma = net.gamma;
  const int64_t N = net.N, Ns = net.Ns;
  const int total = lists.first[ne];
  for (int w = blockIdx.x; w < total; w += gridDim.x) {
    __syncthreads();  // the last item's rows and sums are read
    if (tid < 64) {   // the list of item w: the first whose end lies past it
      for (int e0 = 0; e0 < ne; e0 += 64) {
        const int e = e0 + tid;
        const uint64_t past = __ballot(e < ne && lists.first[e + 1] > w);
        if (past != 0ull) {
          if (tid == 0) {
            const int e1 = e0 + (int)__ffsll((unsigned long long)past) - 1;
            item[0] = e1;
            item[1] = w - lists.first[e1];
          }
          break;
        }
      }
    }
    __syncthreads();
    const int e1 = item[0], tile = item[1];
    const bool front = e1 < nl * S;
    const int ks = front ? e1 : e1 - nl * S, seg = ks % S;
    const int k = commit ? ((k_mode >= 0) ? k_mode : st->chosen) : ks / S;
    const int n_rows = lists.cnt[e1];
    load_path(net, chans[k], units, de);
    if (tid < T) {
      const int e = tile * T + tid;
      const bool in = e < n_rows;
      const int64_t n0 = (int64_t)seg * kSegment, n1 = N - n0 < kSegment ? N : n0 + kSegment;
      const int64_t at = (int64_t)(commit ? 0 : k) * N + (front ? n0 + (in ? e : 0) : n1 - 1 - (in ? e : 0));
      rown[tid] = in ? gload(&lists.rows[at]) : -1;
      rowd[tid] = in ? gload(&lists.d[at]) : 0.f;
      rowa[tid] = in ? gload(&lists.ap[at]) : 0.f;
      rowf[tid] = in ? gload(&lists.f[at]) : L;
    }
    __syncthreads();
    D t;
    t.init(rown);
    int m0 = front ? 1 : L;
    if (!front)
      for (int r = 0; r < T; ++r) m0 = rowf[r] < m0 ? rowf[r] : m0;
    typename D::Acc acc, zc;
    for (int m = m0; m <= L - 2; ++m) {
      const int jn = units[m + 1];
      // (a 1024-unit product has no registers for the fields beside it)
      if constexpr (!D::kF32) t.fields(net.Z[m], Ns, zc);
      if (m > m0) {
        t.product(net, m, ta, acc);
      } else {
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
          for (int sb = 0; sb < SB; ++sb)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) acc[h][sb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      if constexpr (D::kF32) t.fields(net.Z[m], Ns, zc);
      if (m > m0) t.unscale(acc);
      // the rank-1 term of the rows whose changed unit enters here, and the path
      // weight's own change
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
          const int u = t.unit(h, cb);
          if (m == m0 || !front) {
            const float wm = gload(&net.W[m][(int64_t)u * W + units[m]]);
#pragma unroll
            for (int sb = 0; sb < SB; ++sb)
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const int r = 16 * sb + 4 * t.q + v;
                if (rowf[r] == m) acc[h][sb][cb][v] = rowd[r] * wm;
              }
          }
          if (u == jn) {
#pragma unroll
            for (int sb = 0; sb < SB; ++sb)
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const int r = 16 * sb + 4 * t.q + v;
                if (rowf[r] <= m) {
                  const float dz = fmaf(de[m], rowa[r], acc[h][sb][cb][v]);
                  acc[h][sb][cb][v] = dz;
                  rowa[r] = act_fn(zc[h][sb][cb][v] + dz, ACT, gamma);
                }
              }
          }
        }
      if (commit) t.store_fields(net.Z[m], Ns, zc, acc);
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int sb = 0; sb < SB; ++sb)
#pragma unroll
          for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[h][sb][cb][v] = dphi(zc[h][sb][cb][v], acc[h][sb][cb][v], ACT, gamma);
      __syncthreads();  // every wave has read the tile
      t.write_tile(ta, acc);
      __syncthreads();
    }
    f32x4 lg[SB][1];
    t.logit_part(net, ta, lg);
    __syncthreads();  // every wave has read the tile: the sums take its place
    const int cls = units[L];
#pragma unroll
    for (int sb = 0; sb < SB; ++sb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 16 * sb + 4 * t.q + v;
        float s = lg[sb][0][v];
        if (t.wave == 0 && t.li == cls) s = fmaf(de[L - 1], rowa[r], s);
        logit[t.wave][r][t.li] = s;
      }
    __syncthreads();
    if (tid < T) dls[tid] = rown[tid] < 0 ? 0.f : sample_change<NW, T>(net, rown[tid], logit, tid, commit);
    __syncthreads();
    if (!commit && tid == 0) {
      float v = 0.f;
      for (int r = 0; r < T; ++r) v += dls[r];
      // front tiles from the start of the segment's sums, back tiles after them
      const int slot = front ? tile : (lists.cnt[ks] + T - 1) / T + tile;
      partial[(int64_t)k * nchan + seg * segment_slots(T) + slot] = v;
    }
  }
}

int channel_segments(int64_t n_samples) { return (int)((n_samples + kSegment - 1) / kSegment); }

int channel_tiles(int64_t n_samples, int w, int n_layers) {
  if (n_layers == 2) return (int)((n_samples + kTwo - 1) / kTwo);
  const int T = w == 256 ? Dense<256, false>::T : (w == 512 ? Dense<512, false>::T : Dense<1024, false>::T);
  return channel_segments(n_samples) * segment_slots(T);
}

// After the field commit: the path's new weights (and the transposed copy of
// W_{L-2} where one is kept), the committed loss and the count.
__global__ void k_channel_weights(NetDev net, const mca_channel* chans, int k_mode, DevState* st,
                                  const double* dL) {
  const int k = (k_mode >= 0) ? k_mode : st->chosen;
  if (k < 0) return;
  const int m = threadIdx.x;
  if (m < net.L) {
    const int j = chans[k].units[m + 1], i = chans[k].units[m];
    const float w = chans[k].w_new[m];
    put_weight(net, m, j, i, w);
    if (net.WT != nullptr && m == net.L - 2) net.WT[(int64_t)i * net.widths[m + 1] + j] = w;
  }
  if (m == 0) {
    st->L += dL[k];
    st->accepted += 1;
  }
}

hipError_t launch_channel_propose(const NetDev& net, uint64_t t, bool use_dev_t,
                                  const DevState* st, int K, mca_channel* ch, mca_cand* cands,
                                  Aux* aux, hipStream_t s, mca_channel* host) {
  hipLaunchKernelGGL(k_channel_propose, dim3((K + 63) / 64), dim3(64), 0, s, net, t,
                     use_dev_t ? 1 : 0, st, K, ch, cands, aux, host);
  return hipGetLastError();
}

hipError_t launch_channel_prepare(const NetDev& net, mca_channel* ch, int K,
                                  mca_cand* cands, Aux* aux, hipStream_t s, const mca_channel* host) {
  hipLaunchKernelGGL(k_channel_prepare, dim3((K + 63) / 64), dim3(64), 0, s, net, ch, K, cands,
                     aux, host);
  return hipGetLastError();
}

hipError_t launch_channel(const NetDev& net, const mca_channel* ch, const Aux* aux, int K,
                          const ChannelLists& lists, float* partial, int nchan, int k_mode,
                          DevState* st, const double* dL, hipStream_t s) {
  const bool commit = k_mode != -2;
  const int group = list_group(net.N);
  if (!commit && K > group) {  // the lists hold `group` channels: one group after the other
    for (int g = 0; g < K; g += group) {
      const hipError_t e = launch_channel(net, ch + g, aux + g, std::min(K - g, group), lists,
                                          partial + (int64_t)g * nchan, nchan, k_mode, st, dL, s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  auto go = [&](auto w, auto act) {
    constexpr int W = decltype(w)::value, ACT = decltype(act)::value;
    auto run = [&](auto com) {
      typedef Dense<W, decltype(com)::value> D;
      if (net.L == 2) {
        hipLaunchKernelGGL(k_channel_two, dim3((unsigned)((net.N + kTwo - 1) / kTwo), commit ? 1u : (unsigned)K),
                           dim3(kTwo), 0, s, net, ch, aux, partial, nchan, k_mode, st);
        return;
      }
      const int S = channel_segments(net.N);
      hipLaunchKernelGGL(k_channel_rows, dim3(S, commit ? 1 : K), dim3(kListThreads), 0, s, net, ch, aux, lists,
                         partial, nchan, D::T, K, k_mode, st);
      const int64_t tiles = (int64_t)S * segment_slots(D::T) * (commit ? 1 : K);
      const int64_t most = kChannelBlocks * D::blocks_per_cu;
      hipLaunchKernelGGL((k_channel<W, ACT, decltype(com)::value>), dim3((unsigned)(tiles < most ? tiles : most)),
                         dim3(D::threads), 0, s, net, ch, lists, partial, nchan, K, S, k_mode, st);
    };
    if (commit) run(std::true_type{});
    else run(std::false_type{});
    return hipGetLastError();
  };
  auto by_act = [&](auto w) {
    if (net.act == MCA_ACT_TANH) return go(w, std::integral_constant<int, MCA_ACT_TANH>{});
    if (net.act == MCA_ACT_RELU) return go(w, std::integral_constant<int, MCA_ACT_RELU>{});
    return go(w, std::integral_constant<int, MCA_ACT_GAUSS>{});
  };
  hipError_t e;
  switch (net.widths[1]) {
    case 256: e = by_act(std::integral_constant<int, 256>{}); break;
    case 512: e = by_act(std::integral_constant<int, 512>{}); break;
    case 1024: e = by_act(std::integral_constant<int, 1024>{}); break;
    default: return hipErrorInvalidValue;  // the context's validation admits no other width
  }
  if (e != hipSuccess || !commit) return e;
  hipLaunchKernelGGL(k_channel_weights, dim3(1), dim3(64), 0, s, net, ch, k_mode, st, dL);
  return hipGetLastError();
}

}  // namespace mca

// Single mutations in the deep nets of Sec. 2.1: every layer may carry a bias
// per unit, and every hidden field may be normalized over its layer, sample
// by sample, before the transfer function.  Normalization couples the units
// of a layer: changing one field moves that sample's mean and variance, so
// every unit of the layer (and of each later layer) changes.  A candidate in
// layer l therefore moves column j of z_l by de times its input (1 for a
// bias), and from there the kernel carries dense changes layer to layer:
//   normalization, for each sample with mean mu, S = var + eps, c = z - mu:
//     dmu = mean(dz), e = dz - dmu, dS = mean(e (2c + e))   (exact identity),
//     dh = e / sqrt(S + dS) - c dS / (sqrt S sqrt(S + dS) (sqrt S + sqrt(S + dS))),
//   so that h + dh = (z' - mu') / sqrt(S') with no difference of near-equal
//   values; then da = phi(h + dh) - phi(h) (dphi), and the next field's change
//   W_m da as six products of bf16 parts (split_mma.hpp); the logits' change
//   gives each sample's loss change with the cached softmax (ce_change).
// k_norm_rows lists, per candidate and in sample order, the samples the change
// moves (a first-layer weight's input is zero on most: about 81 % of the images)
// with the size of their move; a block of k_norm takes a tile of them
// (dense_tile.hpp).  The row sums of the normalization add the lanes that hold
// a row by a fixed butterfly, then the waves in order.  A net without
// normalization starts at layer l+1, with the rank-1 term of the one moved
// unit.  The commit runs the same arithmetic, stores the moved fields and
// recomputes each moved sample's statistics from them.
#include <algorithm>
#include <type_traits>

#include "dense_tile.hpp"
#include "norm_kernels.hpp"

namespace mca {

namespace {

__device__ __forceinline__ float inv_sqrt(float s) { return 1.0f / sqrtf(s); }

// Activation of hidden unit i of layer l for sample n from the caches.
__device__ __forceinline__ float hidden_act(const NetDev& net, const NormDev& nd, int l, int i,
                                            int64_t n) {
  const float z = gload(&net.Z[l][(int64_t)i * net.Ns + n]);
  if (!net.ln) return act_fn(z, net.act, net.gamma);
  const float h = (z - gload(&nd.MU[l][n])) * inv_sqrt(gload(&nd.S[l][n]));
  return act_fn(h, net.act, net.gamma);
}

}  // namespace

// Block k (eval) or the committed candidate: the samples it moves, with the
// change of the one field (normalized nets, logit-layer parameters) or
// activation (a hidden unit without normalization) it enters by; cnt[k] their
// number, cnt[K + r] the candidate that is r-th by layer.  An evaluation lists
// the step's minibatch only.  A commit also stores the moved field where the
// tile kernel starts past it, the parameter and the state.
__global__ __launch_bounds__(kListThreads) void k_norm_rows(NetDev net_arg, NormDev nd, const mca_cand* cands,
                                                            const Aux* aux, int k_mode, DevState* st,
                                                            const double* dL, int* rows, float* vals,
                                                            int* cnt, int K) {
  __shared__ NetDev net;
  stage_net(net, net_arg);
  const bool commit = k_mode != -2;
  const int k = commit ? ((k_mode >= 0) ? k_mode : st->chosen) : (int)blockIdx.x;
  if (k < 0) return;
  const int slot = commit ? 0 : k;  // a commit's list is the first
  const mca_cand c = cands[k];
  const int L = net.L, l = c.layer;
  if (!commit && threadIdx.x < 64) {
    const int r = layer_rank(cands, K, k, l);
    if (threadIdx.x == 0) cnt[K + r] = k;
  }
  if (!commit && !aux[k].valid) {  // rejected unevaluated: selection gives +inf
    if (threadIdx.x == 0) cnt[slot] = 0;
    return;
  }
  const float de = aux[k].de;
  const int64_t N = net.N, Ns = net.Ns;
  const bool is_bias = c.i == net.widths[l];
  const bool unit = !net.ln && l < L - 1;  // lists the unit's activation change
  float* zrow = net.Z[l] + (int64_t)c.j * Ns;
  const int64_t sub0 = subset_start(net, commit ? 0 : st->t);
  const int n_rows = list_rows(N, rows + (int64_t)slot * N, vals + (int64_t)slot * N, [&](int64_t n, bool in) {
    const float x = is_bias ? 1.0f
                            : (l == 0 ? gload(&net.XT[(int64_t)c.i * Ns + n]) : hidden_act(net, nd, l - 1, c.i, n));
    float v = de * x;
    if (unit) {
      const float z = gload(&zrow[n]);
      if (commit && in && v != 0.f) gstore(&zrow[n], z + v);
      v = dphi(z, v, net.act, net.gamma);
    }
    return (commit || in_subset(net, sub0, n)) ? v : 0.f;
  });
  if (threadIdx.x == 0) {
    cnt[slot] = n_rows;
    if (commit) {
      const float w = aux[k].w_new;
      if (is_bias) gstore(&net.B[l][c.j], w);
      else put_weight(net, l, c.j, c.i, w);
      if (net.sub_size == 0) st->L += dL[k];  // a minibatch's change is not the loss's
      st->accepted += 1;
    }
  }
}

// grid (ntiles, K) for an evaluation (row y: the y-th candidate by layer),
// (ntiles, 1) for a commit.
template <int W, int ACT, bool LN, bool commit>
__global__ __launch_bounds__((Dense<W, commit>::threads), (Dense<W, commit>::blocks_per_cu)) void k_norm(
    NetDev net_arg, NormDev nd, const mca_cand* cands, const int* rows, const float* vals,
    const int* cnt, float* partial, int ntiles, int K, int k_mode, const DevState* st) {
  typedef Dense<W, commit> D;
  constexpr int T = D::T, SB = D::SB, H = D::H, NW = D::NW;
  __shared__ NetDev net;
  stage_net(net, net_arg);
  __shared__ __attribute__((aligned(16))) typename D::Tile ta;
  __shared__ int rown[T];
  __shared__ float rowv[T];
  __shared__ __attribute__((aligned(16))) float red[2][NW][T];  // row sums by wave
  __shared__ __attribute__((aligned(16))) float4 rowc[T];       // dmu, 1/sqrt S, 1/sqrt S', f
  __shared__ float rowmu[T], dls[T];
  auto logit = reinterpret_cast<float (*)[T][17]>(ta);
  static_assert(sizeof(float) * NW * T * 17 <= sizeof(ta), "the logits' sums take the tile's place");

  const int tid = threadIdx.x;
  const int k = commit ? ((k_mode >= 0) ? k_mode : st->chosen) : cnt[K + (int)blockIdx.y];
  if (k < 0) return;
  const int slot = commit ? 0 : k;
  const int tile = blockIdx.x, n_rows = cnt[slot], e0 = tile * T;
  if (e0 >= n_rows) {
    if (!commit && tid == 0) partial[(int64_t)k * ntiles + tile] = 0.f;
    return;
  }
  const mca_cand c = cands[k];
  const int L = net.L, l = c.layer;
  const float gamma = net.gamma;
  const int64_t N = net.N, Ns = net.Ns;
  if (tid < T) {
    const int e = e0 + tid;
    rown[tid] = (e < n_rows) ? gload(&rows[(int64_t)slot * N + e]) : -1;
    rowv[tid] = (e < n_rows) ? gload(&vals[(int64_t)slot * N + e]) : 0.f;
  }
  __syncthreads();
  D t;
  t.init(rown);
  if (l == L - 1) {
    // a logit-layer parameter: only logit j moves
    for (int e = tid; e < T * 16; e += D::threads) logit[0][e >> 4][e & 15] = ((e & 15) == c.j) ? rowv[e >> 4] : 0.f;
  } else {
    typename D::Acc acc, zc;
    // sum of x over the units of each of this lane's rows
    int buf = 0;
    auto row_sums = [&](auto&& x, float (&out)[SB][4]) {
#pragma unroll
      for (int sb = 0; sb < SB; ++sb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          float s = 0.f;
#pragma unroll
          for (int h = 0; h < H; ++h)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) s += x(h, sb, cb, v);
          s = lanes16_sum(s);
          if (t.li == 0) red[buf][t.wave][16 * sb + 4 * t.q + v] = s;
        }
      __syncthreads();
#pragma unroll
      for (int sb = 0; sb < SB; ++sb) {
        f32x4 s = *reinterpret_cast<const f32x4*>(&red[buf][0][16 * sb + 4 * t.q]);
#pragma unroll
        for (int w = 1; w < NW; ++w) s += *reinterpret_cast<const f32x4*>(&red[buf][w][16 * sb + 4 * t.q]);
#pragma unroll
        for (int v = 0; v < 4; ++v) out[sb][v] = s[v];
      }
      buf ^= 1;  // the other buffer next: no wave still reads it two sums later
    };
    // the layer's changes from its field's change acc, into the tile; `read`:
    // other waves may still read the tile
    auto finish = [&](int m, bool read) {
      if constexpr (LN) {
        float mu1 = 0.f, S1 = 0.f;
        bool moved = false;
        if (commit) {
          // the moved samples' statistics from their new fields
          float s[SB][4], m1[SB][4], v1[SB][4];
          row_sums([&](int h, int sb, int cb, int v) { return fabsf(acc[h][sb][cb][v]); }, s);
          row_sums([&](int h, int sb, int cb, int v) { return zc[h][sb][cb][v] + acc[h][sb][cb][v]; }, m1);
#pragma unroll
          for (int sb = 0; sb < SB; ++sb)
#pragma unroll
            for (int v = 0; v < 4; ++v) m1[sb][v] *= 1.0f / W;
          row_sums([&](int h, int sb, int cb, int v) {
            const float d = (zc[h][sb][cb][v] + acc[h][sb][cb][v]) - m1[sb][v];
            return d * d;
          }, v1);
          if (t.wave == 0 && t.li < 4)  // lane (q, v): row 4 q + v of each block of 16
#pragma unroll
            for (int sb = 0; sb < SB; ++sb)
#pragma unroll
              for (int v = 0; v < 4; ++v)
                if (v == t.li && t.nrow[sb][v] >= 0 && s[sb][v] != 0.f) {
                  rowc[16 * sb + 4 * t.q + v] = make_float4(m1[sb][v], v1[sb][v] * (1.0f / W) + net.ln_eps, 1.f, 0.f);
                } else if (v == t.li) {
                  rowc[16 * sb + 4 * t.q + v] = make_float4(0.f, 0.f, 0.f, 0.f);
                }
          __syncthreads();
          if (tid < T) {
            mu1 = rowc[tid].x;
            S1 = rowc[tid].y;
            moved = rowc[tid].z != 0.f;
          }
        }
        float S = 1.f;
        if (tid < T) {
          const int n = rown[tid] >= 0 ? rown[tid] : 0;
          rowmu[tid] = gload(&nd.MU[m][n]);
          S = gload(&nd.S[m][n]);
        }
        float dmu[SB][4], dS[SB][4];
        row_sums([&](int h, int sb, int cb, int v) { return acc[h][sb][cb][v]; }, dmu);  // (rowmu with its barrier)
        float mu[SB][4];
#pragma unroll
        for (int sb = 0; sb < SB; ++sb)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            dmu[sb][v] *= 1.0f / W;
            mu[sb][v] = rowmu[16 * sb + 4 * t.q + v];
          }
        row_sums([&](int h, int sb, int cb, int v) {
          const float c1 = zc[h][sb][cb][v] - mu[sb][v], e = acc[h][sb][cb][v] - dmu[sb][v];
          return e * (c1 + c1 + e);
        }, dS);
        // the row's factors by one thread a row
        if (t.wave == 0 && t.li == 0)
#pragma unroll
          for (int sb = 0; sb < SB; ++sb)
#pragma unroll
            for (int v = 0; v < 4; ++v) dls[16 * sb + 4 * t.q + v] = dS[sb][v] * (1.0f / W);
        __syncthreads();
        if (tid < T) {
          const float d = dls[tid];
          const float q0 = sqrtf(S), q1 = sqrtf(S + d);
          const float rs = 1.0f / q0, rs1 = 1.0f / q1;
          rowc[tid] = make_float4(rs, rs1, ((d * rs) * rs1) / (q0 + q1), 0.f);
          if (commit && moved) {
            gstore(&nd.MU[m][rown[tid]], mu1);
            gstore(&nd.S[m][rown[tid]], S1);
          }
        }
        __syncthreads();
        if (commit) t.store_fields(net.Z[m], Ns, zc, acc);
#pragma unroll
        for (int sb = 0; sb < SB; ++sb)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float4 r = rowc[16 * sb + 4 * t.q + v];
#pragma unroll
            for (int h = 0; h < H; ++h)
#pragma unroll
              for (int cb = 0; cb < 4; ++cb) {
                const float c1 = zc[h][sb][cb][v] - mu[sb][v], e = acc[h][sb][cb][v] - dmu[sb][v];
                acc[h][sb][cb][v] = dphi(c1 * r.x, e * r.y - c1 * r.z, ACT, gamma);
              }
          }
      } else {
        if (commit) t.store_fields(net.Z[m], Ns, zc, acc);
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
          for (int sb = 0; sb < SB; ++sb)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
#pragma unroll
              for (int v = 0; v < 4; ++v) acc[h][sb][cb][v] = dphi(zc[h][sb][cb][v], acc[h][sb][cb][v], ACT, gamma);
        if (read) __syncthreads();  // every wave has read the tile
      }
      t.write_tile(ta, acc);
      __syncthreads();
    };
    // 1. the first layer: the one moved field (normalized), or the rank-1 term
    // of the moved unit in the next layer
    const int s = LN ? l : l + 1;
    if (LN || s <= L - 2) {
      t.fields(net.Z[s], Ns, zc);
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
          const int u = t.unit(h, cb);
          const float w = LN ? (u == c.j ? 1.0f : 0.f) : gload(&net.W[s][(int64_t)u * W + c.j]);
#pragma unroll
          for (int sb = 0; sb < SB; ++sb)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[h][sb][cb][v] = rowv[16 * sb + 4 * t.q + v] * w;
        }
      finish(s, false);
      // 2. dense layers
      for (int m = s + 1; m <= L - 2; ++m) {
        // (a 1024-unit product has no registers for the fields beside it)
        if constexpr (!D::kF32) t.fields(net.Z[m], Ns, zc);
        t.product(net, m, ta, acc);
        if constexpr (D::kF32) t.fields(net.Z[m], Ns, zc);
        t.unscale(acc);
        finish(m, true);
      }
      // 3. the logits: the last hidden layer's change through W_{L-1}
      f32x4 lg[SB][1];
      t.logit_part(net, ta, lg);
      __syncthreads();  // every wave has read the tile: the sums take its place
#pragma unroll
      for (int sb = 0; sb < SB; ++sb)
#pragma unroll
        for (int v = 0; v < 4; ++v) logit[t.wave][16 * sb + 4 * t.q + v][t.li] = lg[sb][0][v];
    } else {
      // a unit of the last hidden layer without normalization: rank-1 logits
      const float* WL = net.W[L - 1];
      for (int e = tid; e < T * 16; e += D::threads) {
        const int r = e >> 4, cl = e & 15;
        logit[0][r][cl] = cl < net.C ? rowv[r] * gload(&WL[(int64_t)cl * W + c.j]) : 0.f;
      }
    }
  }
  __syncthreads();
  // 4. each sample's loss change; the tile's sum in row order
  const bool one = l == L - 1 || (!LN && l == L - 2);
  if (tid < T) {
    const int n = rown[tid];
    dls[tid] = n < 0 ? 0.f : (one ? sample_change<1, T>(net, n, logit, tid, commit)
                                  : sample_change<NW, T>(net, n, logit, tid, commit));
  }
  __syncthreads();
  if (!commit && tid == 0) {
    float v = 0.f;
    for (int r = 0; r < T; ++r) v += dls[r];
    partial[(int64_t)k * ntiles + tile] = v;
  }
}

int norm_tiles(int64_t n_samples, int w) {
  const int T = w == 256 ? Dense<256, false>::T : (w == 512 ? Dense<512, false>::T : Dense<1024, false>::T);
  return (int)((n_samples + T - 1) / T);
}

// Statistics of hidden layer l.  A block takes 16 samples (64 bytes of each
// unit's row) and shares their W units among 64 groups of lanes: a thread reads
// its W / 64 values once, and both sums meet in LDS in group order, by each
// sample's first thread.  A thread a sample ran 2 W dependent loads on N / 64
// waves (1024 units, 3000 samples: 339 us).
constexpr int kStatSamples = 16, kStatGroups = 64;
template <int PER>
__global__ __launch_bounds__(kStatSamples * kStatGroups) void k_norm_stats(NetDev net, NormDev nd, int l) {
  __shared__ float part[kStatGroups][kStatSamples];
  __shared__ float mean[kStatSamples];
  const int t = threadIdx.x % kStatSamples, g = threadIdx.x / kStatSamples;
  const int64_t n = (int64_t)blockIdx.x * kStatSamples + t;
  const int64_t nc = n < net.N ? n : net.N - 1;
  const float* Z = net.Z[l];
  const float inv = 1.0f / (float)(PER * kStatGroups);  // a power of two
  float z[PER], s = 0.f;
#pragma unroll
  for (int u = 0; u < PER; ++u) z[u] = gload(&Z[(int64_t)(g * PER + u) * net.Ns + nc]);
#pragma unroll
  for (int u = 0; u < PER; ++u) s += z[u];
  auto total = [&](float v) {  // in the first 16 threads, thread t sample t
    part[g][t] = v;
    __syncthreads();
    float a = 0.f;
    if (g == 0)
      for (int i = 0; i < kStatGroups; ++i) a += part[i][t];
    __syncthreads();
    return a;
  };
  const float a = total(s) * inv;
  if (g == 0) mean[t] = a;
  __syncthreads();
  const float mu = mean[t];
  float v = 0.f;
#pragma unroll
  for (int u = 0; u < PER; ++u) v += (z[u] - mu) * (z[u] - mu);
  const float q = total(v);
  if (g == 0 && n < net.N) {
    gstore(&nd.MU[l][n], mu);
    gstore(&nd.S[l][n], q * inv + net.ln_eps);
  }
}

// One layer's augmented matrix [rows][n + 1] (each row's weights, then its
// bias) from W [rows][n] and B, or (to_net) the other way: one contiguous copy
// between it and the host, where a strided copy moves a row at a time
// (784-256x3-10: 10.5 ms for the parameters as strided copies, 0.2 ms with this).
__global__ void k_augment(float* aug, float* W, float* B, int rows, int n, int to_net) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)rows * (n + 1)) return;
  const int64_t j = e / (n + 1);
  const int i = (int)(e - j * (n + 1));
  float* at = i < n ? &W[j * n + i] : &B[j];
  if (to_net) *at = aug[e];
  else aug[e] = *at;
}

hipError_t launch_augment(float* aug, float* W, float* B, int rows, int n, bool to_net, hipStream_t s) {
  const int64_t all = (int64_t)rows * (n + 1);
  hipLaunchKernelGGL(k_augment, dim3((unsigned)((all + 255) / 256)), dim3(256), 0, s, aug, W, B, rows, n,
                     to_net ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_norm_stats(const NetDev& net, const NormDev& nd, int l, hipStream_t s) {
  const dim3 grid((unsigned)((net.N + kStatSamples - 1) / kStatSamples)), block(kStatSamples * kStatGroups);
  switch (net.widths[l + 1]) {
    case 256: hipLaunchKernelGGL(k_norm_stats<4>, grid, block, 0, s, net, nd, l); break;
    case 512: hipLaunchKernelGGL(k_norm_stats<8>, grid, block, 0, s, net, nd, l); break;
    case 1024: hipLaunchKernelGGL(k_norm_stats<16>, grid, block, 0, s, net, nd, l); break;
    default: return hipErrorInvalidValue;  // the context's validation admits no other width
  }
  return hipGetLastError();
}

hipError_t launch_norm(const NetDev& net, const NormDev& nd, const mca_cand* cands,
                       const Aux* aux, int K, int* rows, float* vals, int* cnt, float* partial,
                       int ntiles, int k_mode, DevState* st, const double* dL, hipStream_t s) {
  const bool commit = k_mode != -2;
  const int group = list_group(net.N);
  if (!commit && K > group) {  // the lists hold `group` candidates: one group after the other
    for (int g = 0; g < K; g += group) {
      const hipError_t e = launch_norm(net, nd, cands + g, aux + g, std::min(K - g, group), rows, vals, cnt,
                                       partial + (int64_t)g * ntiles, ntiles, k_mode, st, dL, s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  hipLaunchKernelGGL(k_norm_rows, dim3(commit ? 1 : K), dim3(kListThreads), 0, s, net, nd, cands, aux,
                     k_mode, st, dL, rows, vals, cnt, K);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  constexpr int kCommitT = 16;
  const dim3 grid(commit ? (unsigned)((net.N + kCommitT - 1) / kCommitT) : (unsigned)ntiles,
                  commit ? 1u : (unsigned)K);
  auto go = [&](auto w, auto act) {
    constexpr int W = decltype(w)::value, ACT = decltype(act)::value;
    static_assert(Dense<W, true>::T == kCommitT, "a commit's grid");
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, dim3(Dense<W, false>::threads), 0, s, net, nd, cands, rows, vals, cnt,
                         partial, ntiles, K, k_mode, st);
    };
    if (net.ln) commit ? launch(k_norm<W, ACT, true, true>) : launch(k_norm<W, ACT, true, false>);
    else commit ? launch(k_norm<W, ACT, false, true>) : launch(k_norm<W, ACT, false, false>);
    return hipGetLastError();
  };
  auto by_act = [&](auto w) {
    if (net.act == MCA_ACT_TANH) return go(w, std::integral_constant<int, MCA_ACT_TANH>{});
    if (net.act == MCA_ACT_RELU) return go(w, std::integral_constant<int, MCA_ACT_RELU>{});
    return go(w, std::integral_constant<int, MCA_ACT_GAUSS>{});
  };
  switch (net.widths[1]) {
    case 256: return by_act(std::integral_constant<int, 256>{});
    case 512: return by_act(std::integral_constant<int, 512>{});
    case 1024: return by_act(std::integral_constant<int, 1024>{});
    default: return hipErrorInvalidValue;  // the context's validation admits no other width
  }
}

}  // namespace mca

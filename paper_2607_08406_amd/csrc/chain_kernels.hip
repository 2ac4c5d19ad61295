// Evaluation and commit of mutations in the deep layers of an MLP (layers
// 0..L-4, Sec. 2.1): changing W_l[j, i] moves unit j of layer l for every
// sample whose input a_{l-1}[n, i] is nonzero; its activation change da[n]
// moves every unit of layer l+1 by da[n] * W_{l+1}[:, j] (rank-1), and from
// there on every later layer changes densely.  The kernels carry the
// *changes*: dz_m = W_m dA_{m-1} for m = l+2 .. L-2, with
// dA_m = phi(z_m + dz_m) - phi(z_m) formed by dphi() from the cached field
// z_m, then the logit change dz_{L-1} = W_{L-1} dA_{L-2} and each sample's
// loss change from it and the cached softmax (ce_change).  A deep net with
// small weights changes its loss by 1e-11 per mutation; a recomputed loss
// minus the cached one would keep none of it in fp32.  The dense products are
// the dominant work and run on the matrix cores, in bf16 parts (split_mma.hpp).
//
// k_rows lists, per candidate and in increasing sample order, the samples
// whose activation changes, with their da.  A block of k_chain takes one
// candidate and 48 listed samples: it builds dA_{l+1} in an LDS tile
// ([3 parts][48][256], rows padded), runs the dense layers tile to tile (4
// waves, each 48 samples x 64 output units as 3 x 4 MFMA tiles), computes the
// logit changes and the loss change of each sample, and adds the 48 changes in
// list order.  The commit runs the same arithmetic for the chosen candidate
// and moves every cached field by its change.
//
// The hidden layers touched here must be exactly kChainUnits wide.
#include <type_traits>

#include "device_common.hpp"
#include "chain_kernels.hpp"
#include "split_mma.hpp"

namespace mca {

namespace {

constexpr int kRowsThreads = 1024;
constexpr int kChainThreads = 256;
constexpr int kCommitT = 16;  // listed samples per block of a commit
static_assert(kChainThreads == kChainUnits, "a wave takes 64 output units");

}  // namespace

// Block k (eval) or the committed candidate: samples n with a nonzero input
// a_{l-1}[n, i] and a changed activation, in increasing n: rows[k * N + e] =
// n, rda[k * N + e] = da; cnt[k] = their number (0 unless the candidate is in
// layers 0..L-4 and valid).  A commit also stores the new z_l[n, j] of every
// sample with a nonzero input, the new weight (and code) and the state.
__global__ __launch_bounds__(kRowsThreads) void k_rows(NetDev net_arg, const mca_cand* cands,
                                                       const Aux* aux, int k_mode,
                                                       DevState* st, const double* dL, int* rows,
                                                       float* rda, int* cnt, int K) {
  __shared__ NetDev net;
  stage_net(net, net_arg);
  __shared__ int wave_n[kRowsThreads / 64];
  const bool commit = k_mode != -2;
  const int k = commit ? ((k_mode >= 0) ? k_mode : st->chosen) : (int)blockIdx.x;
  if (k < 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const mca_cand c = cands[k];
  const int L = net.L, l = c.layer;
  if (!commit && wave == 0) {  // the candidate's place by layer, then by index
    int r = 0;
    for (int k1 = lane; k1 < K; k1 += 64) {
      const int l1 = cands[k1].layer;
      r += (l1 < l || (l1 == l && k1 < k)) ? 1 : 0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) r += __shfl_xor(r, o, 64);
    if (lane == 0) cnt[K + r] = k;
  }
  if (l > L - 4 || (!commit && !aux[k].valid)) {
    if (tid == 0) cnt[k] = 0;
    return;
  }
  const int act = net.act;
  const float gamma = net.gamma;
  const float de = aux[k].de;
  const int64_t N = net.N, Ns = net.Ns;
  const float* in = (l == 0) ? net.XT : net.Z[l - 1];
  float* zrow = net.Z[l] + (int64_t)c.j * Ns;
  // an evaluation lists the step's minibatch only; a commit moves every sample
  const int64_t sub0 = subset_start(net, commit ? 0 : st->t);
  int base = 0;
  for (int64_t n0 = 0; n0 < N; n0 += kRowsThreads) {
    const int64_t n = n0 + tid;
    float da = 0.f;
    if (n < N) {
      const float xr = gload(&in[(int64_t)c.i * Ns + n]);
      const float x = (l == 0) ? xr : act_fn(xr, act, gamma);
      if (x != 0.f) {
        const float zl = gload(&zrow[n]);
        const float dz = de * x;
        da = dphi(zl, dz, act, gamma);
        if (commit) gstore(&zrow[n], zl + dz);
      }
    }
    const bool take = da != 0.f && (commit || in_subset(net, sub0, n));
    const uint64_t b = __ballot(take);
    if (lane == 0) wave_n[wave] = (int)__popcll(b);
    __syncthreads();
    int off = base, tot = 0;
    for (int v = 0; v < kRowsThreads / 64; ++v) {
      if (v < wave) off += wave_n[v];
      tot += wave_n[v];
    }
    if (take) {
      const int e = off + (int)__popcll(b & ((1ull << lane) - 1ull));
      gstore(&rows[(int64_t)k * N + e], (int)n);
      gstore(&rda[(int64_t)k * N + e], da);
    }
    base += tot;
    __syncthreads();
  }
  if (tid == 0) {
    cnt[k] = base;
    if (commit) {
      const Aux a = aux[k];
      const int64_t idx = (int64_t)c.j * net.widths[l] + c.i;
      put_weight(net, l, c.j, c.i, a.w_new);
      if (net.ternary) gstore(&net.codes[l][idx], (int8_t)c.code);
      if (net.sub_size == 0) st->L += dL[k];
      st->accepted += 1;
    }
  }
}

// grid (nchain, K) for an evaluation (row y: the y-th candidate by layer, so
// that the longest chains start first and the short ones fill the last round),
// (nchain, 1) for a commit.
//
// What bounds it: the matrix cores and the L2 reads of the weights take about
// as long as each other.  The products run on bf16 parts (split_mma.hpp); the
// tile holds its parts in LDS (76 KB at 48 rows), so two blocks share a CU and
// one's products run beside the other's transfer functions.  More rows a block
// would halve the weights' reads but leave one block; 32 rows read too much.
// 784-24x256-10, 32 candidates on 4096 samples: 2.82 -> 1.33 ms a step against
// fp32 products on 64-row tiles, the same error against 64 bits (2.4e-7).
//
// T: rows of a block.  A commit has one candidate's rows: its time is the
// latency of one tile's layers one after another, all blocks at the same layer
// at once, so that every read of the weights is the first in its L2.  It takes
// 16 rows (4096 samples: a tile for every CU) and requests a whole layer ahead
// (its one block a CU has the registers).  Each row's sums are the same bits
// at every T.  784-24x256-10 on 4096 samples: 199 -> 96 us a commit on average.
template <int CM, int ACT, int T>
__global__ __launch_bounds__(kChainThreads, T == kCommitT ? 1 : 2) void k_chain(NetDev net_arg, const mca_cand* cands,
                                                         const Aux* aux, const int* rows,
                                                         const float* rda, const int* cnt,
                                                         float* partial, int nchain, int K,
                                                         int k_mode, const DevState* st) {
  constexpr int SB = T / 16, W = kChainUnits, RS = W + 8;
  __shared__ NetDev net;
  stage_net(net, net_arg);
  // activation changes in three bf16 parts, [part][sample][unit in k order],
  // rewritten in place layer by layer
  __shared__ __attribute__((aligned(16))) uint16_t ta[3 * T * RS];
  __shared__ int rown[T];
  __shared__ float rowda[T];
  __shared__ float dls[T];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool commit = k_mode != -2;
  const int k = commit ? ((k_mode >= 0) ? k_mode : st->chosen) : cnt[K + (int)blockIdx.y];
  if (k < 0) return;
  const mca_cand c = cands[k];
  const int L = net.L, l = c.layer;
  if (l > L - 4) return;  // scored by another kernel
  const int tile = blockIdx.x;
  const int nrows = cnt[k];
  const int e0 = tile * T;
  if (e0 >= nrows) {
    if (!commit && tid == 0) partial[(int64_t)k * nchain + tile] = 0.f;
    return;
  }
  const int C = (CM < kCMax) ? CM : net.C;
  const float gamma = net.gamma;
  const int64_t N = net.N, Ns = net.Ns;
  const int s = l + 1;  // the layer the rank-1 update reaches

  // 1. the tile's samples
  if (tid < T) {
    const int e = e0 + tid;
    rown[tid] = (e < nrows) ? gload(&rows[(int64_t)k * N + e]) : -1;
    rowda[tid] = (e < nrows) ? gload(&rda[(int64_t)k * N + e]) : 0.f;
  }
  __syncthreads();
  const int q = lane >> 4, li = lane & 15;
  // the samples of this lane's output rows 16 sb + 4 q + v (-1 for padding
  // rows: their changes are zero)
  int nrow[SB][4];
#pragma unroll
  for (int sb = 0; sb < SB; ++sb)
#pragma unroll
    for (int v = 0; v < 4; ++v) nrow[sb][v] = rown[16 * sb + 4 * q + v];
  // every row of the tile holds the next sample after the one before
  const bool rows_dense = rown[T - 1] == rown[0] + T - 1 && (rown[0] & 3) == 0;
  // The cached fields of layer m at this lane's outputs (D layout: lane (q,
  // li), element v -> row 16 sb + 4 q + v, unit 64 w + 16 cb + li).  A lane's
  // four rows are four consecutive samples whenever the tile lists every
  // sample (a candidate past the first layer): one 16-byte load each then
  // (16-byte aligned: the tile starts at a multiple of 16).
  auto fields = [&](int m, f32x4 (&zc)[SB][4]) {
    const float* Zm = net.Z[m];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const float* zu = Zm + (int64_t)(64 * wave + 16 * cb + li) * Ns;
      if (rows_dense) {
#pragma unroll
        for (int sb = 0; sb < SB; ++sb) zc[sb][cb] = gload(reinterpret_cast<const f32x4*>(zu + nrow[sb][0]));
      } else {
#pragma unroll
        for (int sb = 0; sb < SB; ++sb)
#pragma unroll
          for (int v = 0; v < 4; ++v) zc[sb][cb][v] = gload(zu + (nrow[sb][v] >= 0 ? nrow[sb][v] : 0));
      }
    }
  };
  // dA_m = phi(z_m + dz) - phi(z_m), times kPartScale, into the tile's parts; a commit stores
  // z_m + dz
  auto finish = [&](int m, const f32x4 (&dz)[SB][4], const f32x4 (&zc)[SB][4]) {
    float* Zm = net.Z[m];
#pragma unroll
    for (int sb = 0; sb < SB; ++sb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float d[4];
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
          d[cb] = dphi(zc[sb][cb][v], dz[sb][cb][v], ACT, gamma);
          if (commit && nrow[sb][v] >= 0)
            gstore(&Zm[(int64_t)(64 * wave + 16 * cb + li) * Ns + nrow[sb][v]], zc[sb][cb][v] + dz[sb][cb][v]);
        }
        const Split2 s0 = split2(d[0] * kPartScale, d[1] * kPartScale);
        const Split2 s1 = split2(d[2] * kPartScale, d[3] * kPartScale);
        uint16_t* at = ta + (16 * sb + 4 * q + v) * RS + 64 * wave + 4 * li;
#pragma unroll
        for (int p = 0; p < 3; ++p)
          *reinterpret_cast<uint2*>(at + p * T * RS) = make_uint2(s0.p[p], s1.p[p]);
      }
  };
  f32x4 acc[SB][4], zc[SB][4];
  // the split weights of the wave's 64 output units of layer m (s + 1 <= L - 2)
  auto weights = [&](int m) { return net.WF + split_layer(W, m) + (int64_t)4 * wave * (W / 32) * 3 * 512; };
  constexpr bool kAhead = T == kCommitT;
  bf16x8 held[kAhead ? W / 32 : 1][4][3];
  (void)held;
  if constexpr (kAhead) {
#pragma unroll
    for (int ks = 0; ks < W / 32; ++ks) fetch_weights<W>(weights(s + 1), lane, ks, held[ks]);
  }
  // 2. the rank-1 update: dz_s = da W_s[:, j]
  {
    fields(s, zc);
    const float* Ws = net.W[s];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const float w = gload(&Ws[(int64_t)(64 * wave + 16 * cb + li) * W + c.j]);
#pragma unroll
      for (int sb = 0; sb < SB; ++sb)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[sb][cb][v] = rowda[16 * sb + 4 * q + v] * w;
    }
    finish(s, acc, zc);
  }
  __syncthreads();
  // 3. dense layers m = s+1 .. L-2: dz = tile W_m^T, then the tile becomes
  // phi(z_m + dz) - phi(z_m); every wave has read the whole tile before any
  // writes its new values
  for (int m = s + 1; m <= L - 2; ++m) {
    fields(m, zc);
#pragma unroll
    for (int sb = 0; sb < SB; ++sb)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) acc[sb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (kAhead)
      split_product_ahead<W, T, RS>(ta, weights(m < L - 2 ? m + 1 : m), held, lane, acc);
    else
      split_product<W, T, RS>(ta, weights(m), lane, acc);
#pragma unroll
    for (int sb = 0; sb < SB; ++sb)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) acc[sb][cb] *= kPartUnscale;
    __syncthreads();
    finish(m, acc, zc);
    __syncthreads();
  }
  // 4. logit changes dz_{L-1} = W_{L-1} dA_{L-2}: wave w takes 64 of the k,
  // the four partial sums meet in wave order
  auto logit = reinterpret_cast<float (*)[T][17]>(ta);
  {
    f32x4 lg[SB];
#pragma unroll
    for (int sb = 0; sb < SB; ++sb) lg[sb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16x8* wl = reinterpret_cast<const bf16x8*>(net.WF + split_layer(W, L - 1)) + lane;
    constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int ks = 2 * wave; ks < 2 * wave + 2; ++ks) {
      bf16x8 b[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) b[p] = gload(wl + (ks * 3 + p) * 64);
#pragma unroll
      for (int sb = 0; sb < SB; ++sb) {
        bf16x8 a[3];
#pragma unroll
        for (int p = 0; p < 3; ++p)
          a[p] = *reinterpret_cast<const bf16x8*>(ta + (p * T + 16 * sb + li) * RS + 32 * ks + 8 * q);
#pragma unroll
        for (int t = 0; t < 6; ++t) lg[sb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[pa[t]], b[pb[t]], lg[sb], 0, 0, 0);
      }
    }
    __syncthreads();  // every wave has read the tile: the sums take its place
#pragma unroll
    for (int sb = 0; sb < SB; ++sb)
#pragma unroll
      for (int v = 0; v < 4; ++v) logit[wave][16 * sb + 4 * q + v][li] = lg[sb][v] * kPartUnscale;
  }
  __syncthreads();
  // 5. per-sample loss change from the logit change and the cached softmax;
  // the tile's sum in list order
  if (tid < T) {
    const int n = rown[tid];
    float d = 0.f;
    if (n >= 0) {
      const int y = gload(&net.y[n]);
      float dz[CM], p[CM], dzy = 0.f;
#pragma unroll
      for (int cc = 0; cc < CM; ++cc) {
        dz[cc] = (cc < C) ? (logit[0][tid][cc] + logit[1][tid][cc]) + (logit[2][tid][cc] + logit[3][tid][cc]) : 0.f;
        p[cc] = (cc < C) ? gload(&net.prob[(int64_t)cc * Ns + n]) : 0.f;
        dzy = (cc == y) ? dz[cc] : dzy;
      }
      d = ce_change<CM>(p, dz, C, dzy);
      if (commit) {
        float* ZL = net.Z[L - 1];
        float z[CM], pn[CM];
#pragma unroll
        for (int cc = 0; cc < CM; ++cc) z[cc] = (cc < C) ? gload(&ZL[(int64_t)cc * Ns + n]) + dz[cc] : 0.f;
        const float ln = softmax_ce<CM>(z, C, y, pn);
#pragma unroll
        for (int cc = 0; cc < CM; ++cc)
          if (cc < C) {
            gstore(&ZL[(int64_t)cc * Ns + n], z[cc]);
            gstore(&net.prob[(int64_t)cc * Ns + n], pn[cc]);
          }
        gstore(&net.ell[n], ln);
      }
    }
    dls[tid] = d;
  }
  __syncthreads();
  if (!commit && tid == 0) {
    float v = 0.f;
    for (int r = 0; r < T; ++r) v += dls[r];
    partial[(int64_t)k * nchain + tile] = v;
  }
}

namespace {
// One thread per pair of neighbours in a lane's eight values of a fragment.
__global__ void k_split_weights(NetDev net) {
  const int L = net.L, W = net.widths[1];
  const int64_t dense = (int64_t)(L - 2) * W * W / 2, all = dense + 16 * W / 2;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= all) return;
  const int64_t per = (int64_t)W * W / 2;
  const int m = e < dense ? 1 + (int)(e / per) : L - 1;
  const int64_t r = e < dense ? e % per : e - dense;
  const int rows = net.widths[m + 1];
  const int j = (int)(r / (W / 2)), kk = 2 * (int)(r % (W / 2));
  // k positions kk, kk + 1 hold units 16 apart (split_k's inverse)
  const int i0 = (kk & ~63) | ((kk >> 2) & 15) | ((kk & 3) << 4), i1 = i0 + 16;
  const float* row = net.W[m] + (int64_t)j * W;
  const Split2 v = j < rows ? split2(row[i0], row[i1]) : Split2{{0u, 0u, 0u}};
  uint16_t* at = net.WF + split_layer(W, m);
#pragma unroll
  for (int p = 0; p < 3; ++p) *reinterpret_cast<uint32_t*>(at + split_at(W, j, kk, p)) = v.p[p];
}
}  // namespace

hipError_t launch_split_weights(const NetDev& net, hipStream_t s) {
  const int W = net.widths[1];
  const int64_t n = (int64_t)(net.L - 2) * W * W / 2 + 16 * W / 2;
  hipLaunchKernelGGL(k_split_weights, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, net);
  return hipGetLastError();
}

hipError_t launch_chain(const NetDev& net, const mca_cand* cands, const Aux* aux, int K,
                        int* rows, float* rda, int* cnt, float* partial, int nchain, int k_mode,
                        DevState* st, const double* dL, hipStream_t s) {
  const bool commit = k_mode != -2;
  hipLaunchKernelGGL(k_rows, dim3(commit ? 1 : K), dim3(kRowsThreads), 0, s, net, cands, aux,
                     k_mode, st, dL, rows, rda, cnt, K);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto go = [&](auto kernel, int64_t tiles) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)tiles, commit ? 1u : (unsigned)K), dim3(kChainThreads), 0, s,
                       net, cands, aux, rows, rda, cnt, partial, nchain, K, k_mode, st);
  };
  auto pick = [&](auto cm, auto act) {
    constexpr int CM = decltype(cm)::value, ACT = decltype(act)::value;
    if (commit)
      go(k_chain<CM, ACT, kCommitT>, (net.N + kCommitT - 1) / kCommitT);
    else
      go(k_chain<CM, ACT, kChainT>, nchain);
  };
  auto by_act = [&](auto cm) {
    if (net.act == MCA_ACT_TANH) pick(cm, std::integral_constant<int, MCA_ACT_TANH>{});
    else if (net.act == MCA_ACT_RELU) pick(cm, std::integral_constant<int, MCA_ACT_RELU>{});
    else pick(cm, std::integral_constant<int, MCA_ACT_GAUSS>{});
  };
  if (net.C == 10) by_act(std::integral_constant<int, 10>{});
  else by_act(std::integral_constant<int, kCMax>{});
  return hipGetLastError();
}

}  // namespace mca

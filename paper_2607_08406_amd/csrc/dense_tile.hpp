// What the kernels of normalized nets and of channel mutations share: a block
// takes T listed samples of one candidate and carries their activation changes
// from one W-unit layer to the next.  The changes sit in LDS as bf16 parts
// (split_mma.hpp), the products' outputs and the cached fields beside them in
// registers, in the layout the matrix cores leave: lane (q, li) of wave w holds,
// for rows 16 sb + 4 q + v, units 64 (H w + h) + 16 cb + li.
//
// T by width.  Every block reads a layer's 6 W^2 bytes of weights, so fewer rows
// cost reads, of L2 and, where a layer's weights pass its 4 MiB, of the cache
// behind it.  256 units: 48 rows, two blocks a CU (one's products beside the
// other's transfer functions); 512: 32 rows; 1024: 32 rows whose changes stay
// fp32 in LDS (their parts would leave room for 16) and are split by each wave as
// it reads them, 88 instructions beside 96 matrix instructions (784-1024x3-10
// channels, 16 of them on 8192 samples: 537 -> 381 us).
#pragma once

#include "split_mma.hpp"

namespace mca {

//
// A commit has one candidate's rows: 16 of them a block at every width, so that
// all CUs share them (its time is the latency of one tile's layers).
template <int W, bool COMMIT>
struct Dense {
  static_assert(W == 256 || W == 512 || W == 1024, "hidden widths of the dense kernels");
  static constexpr int T = COMMIT ? 16 : (W == 256 ? 48 : 32);
  static constexpr bool kF32 = W == 1024;      // the tile holds fp32 changes, not their parts
  static constexpr int NW = W == 256 ? 4 : 8;  // waves
  static constexpr int H = W / 64 / NW;        // blocks of 64 units per wave
  static constexpr int SB = T / 16, RS = kF32 ? W + 4 : W + 8, threads = 64 * NW;
  static constexpr int tile_bytes = kF32 ? T * RS * 4 : 3 * T * RS * 2;
  typedef unsigned char Tile[tile_bytes];
  static constexpr int blocks_per_cu = W == 256 && !COMMIT ? 2 : 1;
  typedef f32x4 Acc[H][SB][4];

  int wave, lane, q, li;
  int nrow[SB][4];  // samples of this lane's rows (-1: padding, its changes are zero)
  bool dense;       // every row holds the next sample after the one before

  __device__ __forceinline__ void init(const int* rown) {
    wave = threadIdx.x >> 6;
    lane = threadIdx.x & 63;
    q = lane >> 4;
    li = lane & 15;
#pragma unroll
    for (int sb = 0; sb < SB; ++sb)
#pragma unroll
      for (int v = 0; v < 4; ++v) nrow[sb][v] = rown[16 * sb + 4 * q + v];
    dense = rown[0] >= 0 && rown[T - 1] == rown[0] + T - 1 && (rown[0] & 3) == 0;
  }
  __device__ __forceinline__ int unit(int h, int cb) const { return 64 * (H * wave + h) + 16 * cb + li; }

  // The cached fields of a layer at this lane's outputs; four rows that are
  // four consecutive samples come in one 16-byte load.
  __device__ __forceinline__ void fields(const float* Z, int64_t Ns, Acc& z) const {
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        const float* zu = Z + (int64_t)unit(h, cb) * Ns;
        if (dense) {
#pragma unroll
          for (int sb = 0; sb < SB; ++sb) z[h][sb][cb] = gload(reinterpret_cast<const f32x4*>(zu + nrow[sb][0]));
        } else {
#pragma unroll
          for (int sb = 0; sb < SB; ++sb)
#pragma unroll
            for (int v = 0; v < 4; ++v) z[h][sb][cb][v] = gload(zu + (nrow[sb][v] >= 0 ? nrow[sb][v] : 0));
        }
      }
  }
  __device__ __forceinline__ void store_fields(float* Z, int64_t Ns, const Acc& z, const Acc& dz) const {
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int sb = 0; sb < SB; ++sb)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (nrow[sb][v] >= 0) gstore(&Z[(int64_t)unit(h, cb) * Ns + nrow[sb][v]], z[h][sb][cb][v] + dz[h][sb][cb][v]);
  }
  // The changes d into the tile, times kPartScale.
  __device__ __forceinline__ void write_tile(Tile& tile, const Acc& d) const {
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int sb = 0; sb < SB; ++sb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int at = (16 * sb + 4 * q + v) * RS + 64 * (H * wave + h) + 4 * li;
          float x[4];
#pragma unroll
          for (int cb = 0; cb < 4; ++cb) x[cb] = d[h][sb][cb][v] * kPartScale;
          if constexpr (kF32) {
            *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(tile) + at) =
                f32x4{x[0], x[1], x[2], x[3]};
          } else {
            const Split2 s0 = split2(x[0], x[1]), s1 = split2(x[2], x[3]);
#pragma unroll
            for (int p = 0; p < 3; ++p)
              *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(tile) + at + p * T * RS) = make_uint2(s0.p[p], s1.p[p]);
          }
        }
  }
  // The product's sums as they are (after the loads that follow it are on their way).
  __device__ __forceinline__ void unscale(Acc& acc) const {
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int sb = 0; sb < SB; ++sb)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) acc[h][sb][cb] *= kPartUnscale;
  }
  // acc = tile x the split weights of dense layer m, times kPartScale.
  __device__ __forceinline__ void product(const NetDev& net, int m, const Tile& tile, Acc& acc) const {
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int sb = 0; sb < SB; ++sb)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) acc[h][sb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint16_t* wf = net.WF + split_layer(W, m) + (int64_t)4 * H * wave * (W / 32) * 3 * 512;
    if constexpr (kF32) {
      static_assert(H == 2, "the two blocks of units alternate, each in its own registers");
      constexpr int64_t kH = (int64_t)4 * (W / 32) * 3 * 512;
      constexpr int KS = W / 32;
      bf16x8 b0[4][3], b1[4][3];
      fetch_weights<W>(wf, lane, 0, b0);
#pragma unroll 1
      for (int ks = 0; ks < KS; ++ks) {
        bf16x8 a[SB][3];
        fetch_weights<W>(wf + kH, lane, ks, b1);
        split_rows<RS>(reinterpret_cast<const float*>(tile), lane, ks, a);
        multiply_parts(a, b0, acc[0]);
        fetch_weights<W>(wf, lane, ks + 1 < KS ? ks + 1 : 0, b0);
        multiply_parts(a, b1, acc[1]);
      }
    } else {
      static_assert(kF32 || H == 1, "one block of units a wave");
      split_product<W, T, RS>(reinterpret_cast<const uint16_t*>(tile), wf, lane, acc[0]);
    }
  }
  // The wave's share of the logits' change (64 H of the k): partial sums of
  // rows x 16 padded classes.
  __device__ __forceinline__ void logit_part(const NetDev& net, const Tile& tile, f32x4 (&lg)[SB][1]) const {
    const uint16_t* wf = net.WF + split_layer(W, net.L - 1);
#pragma unroll
    for (int sb = 0; sb < SB; ++sb) lg[sb][0] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 2 * H; ++u) {
      const int ks = 2 * H * wave + u;
      bf16x8 b[1][3];
      fetch_weights<W>(wf, lane, ks, b);
      if constexpr (kF32) {
        bf16x8 a[SB][3];
        split_rows<RS>(reinterpret_cast<const float*>(tile), lane, ks, a);
        multiply_parts(a, b, lg);
      } else {
        multiply_step<T, RS>(reinterpret_cast<const uint16_t*>(tile), lane, ks, b, lg);
      }
    }
#pragma unroll
    for (int sb = 0; sb < SB; ++sb) lg[sb][0] *= kPartUnscale;
  }
};

// Sum over the 16 lanes of a row of lanes, the same bits in each.
__device__ __forceinline__ float lanes16_sum(float v) {
  v += dpp_f32<0xB1>(v);   // lane ^ 1
  v += dpp_f32<0x4E>(v);   // lane ^ 2
  v += dpp_f32<0x141>(v);  // mirror within eight
  v += dpp_f32<0x140>(v);  // mirror within sixteen
  return v;
}

// Lists the samples n < N whose value(n) is not zero, in increasing order, with
// their values; returns their number (in every thread).  By a block of
// kListThreads; every thread calls value() for kListU samples at once (n past
// N: a clamped sample, its value is dropped), so their loads overlap.
constexpr int kListThreads = 1024, kListU = 4;
template <class F>
__device__ __forceinline__ int list_rows(int64_t N, int* rows, float* vals, F&& value) {
  static_assert(kListU * kListThreads / 64 == 64, "one count per lane");
  __shared__ int counts[64];  // [u][wave]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int base = 0;
  for (int64_t n0 = 0; n0 < N; n0 += kListU * kListThreads) {
    float v[kListU];
    uint64_t b[kListU];
#pragma unroll
    for (int u = 0; u < kListU; ++u) {
      const int64_t n = n0 + u * kListThreads + tid;
      v[u] = value(n < N ? n : N - 1, n < N);
    }
#pragma unroll
    for (int u = 0; u < kListU; ++u) {
      if (n0 + u * kListThreads + tid >= N) v[u] = 0.f;
      b[u] = __ballot(v[u] != 0.f);
      if (lane == 0) counts[u * (kListThreads / 64) + wave] = (int)__popcll(b[u]);
    }
    __syncthreads();
    const int mine = counts[lane];
    int incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int w = __shfl_up(incl, o, 64);
      if (lane >= o) incl += w;
    }
#pragma unroll
    for (int u = 0; u < kListU; ++u) {
      const int off = base + __shfl(incl - mine, u * (kListThreads / 64) + wave, 64);
      if (v[u] != 0.f) {
        const int e = off + (int)__popcll(b[u] & ((1ull << lane) - 1ull));
        gstore(&rows[e], (int)(n0 + u * kListThreads + tid));
        gstore(&vals[e], v[u]);
      }
    }
    base += __shfl(incl, 63, 64);
    __syncthreads();
  }
  return base;
}

// The place of candidate k among K by its layer, then by its index (so that a
// grid's longest chains start first), by one whole wave.
__device__ __forceinline__ int layer_rank(const mca_cand* cands, int K, int k, int layer) {
  int r = 0;
  for (int k1 = threadIdx.x & 63; k1 < K; k1 += 64) {
    const int l1 = cands[k1].layer;
    r += (l1 < layer || (l1 == layer && k1 < k)) ? 1 : 0;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) r += __shfl_xor(r, o, 64);
  return r;
}

// The loss change of one listed sample n from its logits' change (logit[0 ..
// parts-1][row], summed in order, or `one` for a single moved class); a commit
// also stores the sample's new logits, softmax and loss.
template <int PARTS, int T>
__device__ __forceinline__ float sample_change(const NetDev& net, int n, const float (*logit)[T][17], int row,
                                               bool commit) {
  const int C = net.C;
  const int64_t Ns = net.Ns;
  const int y = gload(&net.y[n]);
  float dz[kCMax], p[kCMax], dzy = 0.f;
#pragma unroll
  for (int c = 0; c < kCMax; ++c) {
    float a = 0.f;
    if (c < C) {
      a = logit[0][row][c];
#pragma unroll
      for (int w = 1; w < PARTS; ++w) a += logit[w][row][c];
    }
    dz[c] = a;
    p[c] = (c < C) ? gload(&net.prob[(int64_t)c * Ns + n]) : 0.f;
    dzy = (c == y) ? a : dzy;
  }
  const float d = ce_change<kCMax>(p, dz, C, dzy);
  if (commit) {
    float* ZL = net.Z[net.L - 1];
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
  return d;
}

}  // namespace mca

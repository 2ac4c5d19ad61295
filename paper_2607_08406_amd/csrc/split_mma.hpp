// fp32 products on the bf16 matrix cores: each operand is the exact sum of
// three bf16 values (hi + mid + lo, 24 significant bits), and a product of two
// fp32 matrices is the sum of the six bf16 products whose terms reach 2^-18
// of a term or more (hi hi, hi mid, mid hi, mid mid, hi lo, lo hi; Henry, Tang
// and Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For
// Higher-Precision Computations", ARITH 2019).  The three dropped ones are
// below 2^-26 of a term, under the rounding of the fp32 sums, which stay in
// fp32.  v_mfma_f32_16x16x32_bf16 takes 16 cycles for the 32 k that
// v_mfma_f32_16x16x4f32 takes 256 for, so six of them take 96: 2.7 times the
// fp32 rate.
//
// The matrix cores take bf16 values below 2^-126 as zero, so a value below 2^-103
// would lose its lowest bits.  Activation changes, which keep their relative
// accuracy down to where fp32 ends (a change can be all there is to a loss
// difference), and hidden activations of at most 1 (tanh, Gaussian) are therefore
// split times 2^24, which brings the last bit of the smallest fp32 value to 2^-125,
// and their products' sums taken times 2^-24, both exact.  Changes of 2^104 and
// more overflow that way, far past the logit change of 88 at which a sample's loss
// change is lost anyway.  Weights, inputs and ReLU activations are split as they
// are: below 2^-103 they lose their lowest bits, above 3.39e38 (bf16's largest) they
// become infinite.
//
// Hidden-layer weights are kept split beside their fp32 values (NetDev::WF), in
// the order the kernels read them: for each block of 16 output units and each
// 32 of the k order, the three parts, each a wave's 64 lanes of 8 values (lane
// (q, li): output unit 16 cb + li, k = 32 ks + 8 q + e).  The k order puts the
// four units 16 c + li (c = 0..3) of a block of 64 side by side, because a lane
// of the product's output holds exactly those four for its sample: its changes
// go back to the tile as one 8-byte store per part.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_common.hpp"

namespace mca {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr float kPartScale = 0x1p24f, kPartUnscale = 0x1p-24f;

// The parts of two fp32 values, each part a packed pair (a in the low half).
struct Split2 {
  uint32_t p[3];
};
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ Split2 split2(float a, float b) {
  Split2 s;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    s.p[i] = bf16_pair(a, b);
    a -= __uint_as_float(s.p[i] << 16);  // exact
    b -= __uint_as_float(s.p[i] & 0xFFFF0000u);
  }
  return s;
}

// Place of k in row r of a tile whose rows hold one part's 32 k (64 bytes): the
// row's four groups of 8 change places with r / 4, so that the 16 lanes that
// read one group of 16 rows (or store it) take all 64 banks.
__device__ __forceinline__ int part_at(int r, int k) { return ((((k >> 3) ^ (r >> 2)) & 3) << 3) | (k & 7); }

// Position of input unit i in the k order, and of element (row, k position,
// part) of a split matrix with W input units, in bf16 values.
__host__ __device__ inline int split_k(int i) { return (i & ~63) | ((i & 15) << 2) | ((i >> 4) & 3); }
__host__ __device__ inline int64_t split_at(int W, int row, int kk, int part) {
  return ((((int64_t)(row >> 4) * (W >> 5) + (kk >> 5)) * 3 + part) * 64 + ((kk >> 3) & 3) * 16 + (row & 15)) * 8 +
         (kk & 7);
}
// Split values of the dense layers m = 1 .. L-2 ([W][W] each), then of the
// logit layer (padded to 16 rows).
__host__ __device__ inline int64_t split_layer(int W, int m) { return (int64_t)(m - 1) * 3 * W * W; }
__host__ __device__ inline int64_t split_size(int W, int L) { return split_layer(W, L - 1) + (int64_t)3 * 16 * W; }

// W_l[j, i] = w, and its split copy where the net keeps one.
__device__ __forceinline__ void put_weight(const NetDev& net, int l, int j, int i, float w) {
  const int n_in = net.widths[l];
  gstore(&net.W[l][(int64_t)j * n_in + i], w);
  if (net.WF == nullptr || l == 0) return;
  uint16_t* at = net.WF + split_layer(n_in, l);
  const Split2 s = split2(w, 0.f);
#pragma unroll
  for (int p = 0; p < 3; ++p) gstore(&at[split_at(n_in, j, split_k(i), p)], (uint16_t)(s.p[p] & 0xFFFFu));
}

// Fills the split copy from the fp32 weights of every layer it holds.
hipError_t launch_split_weights(const NetDev& net, hipStream_t s);

// The 32 k of step ks of the weights of a wave's CB blocks of 16 output units.
template <int W, int CB>
__device__ __forceinline__ void fetch_weights(const uint16_t* wf, int lane, int ks, bf16x8 (&d)[CB][3]) {
  const bf16x8* wl = reinterpret_cast<const bf16x8*>(wf) + lane;
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int p = 0; p < 3; ++p) d[cb][p] = gload(wl + ((cb * (W / 32) + ks) * 3 + p) * 64);
}

// acc += a b over one step, from the parts of both; small terms first.
template <int SB, int CB>
__device__ __forceinline__ void multiply_parts(const bf16x8 (&a)[SB][3], const bf16x8 (&b)[CB][3],
                                               f32x4 (&acc)[SB][CB]) {
  constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
  for (int t = 0; t < 6; ++t)
#pragma unroll
    for (int sb = 0; sb < SB; ++sb)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        acc[sb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[sb][pa[t]], b[cb][pb[t]], acc[sb][cb], 0, 0, 0);
}

// acc[cb] += a b over one step, the product of the leading parts and the five
// smaller ones summed apart, each from zero, so that the running sum is rounded
// twice per 32 k and not six times.  For long sums of sparse inputs, where the
// chain on the running sum loses more than fp32 instructions, which skip the
// zeros' roundings (error over sum |w| |x|, 784 image inputs, 19 % of them lit:
// 2.3e-8 on fp32 instructions, 3.8e-8 with multiply_parts, 0.8e-8 here; 1024
// dense inputs: 2.6e-8, 2.0e-8, 0.7e-8).  Apart, because the instruction cuts an
// addend far below its products off towards minus infinity: with the small sum as
// the addend of the leading product every field came out low, by 3e-8 to 5e-8 of
// the mean |z| (apart: below 4e-10), which no average over samples removes (loss
// changes of 784-1024x3-10 ReLU channels: 1.5e-7 off 64 bits, 3.5e-8 apart).
template <int CB>
__device__ __forceinline__ void add_product(const bf16x8 (&a)[3], const bf16x8 (&b)[CB][3], f32x4 (&acc)[CB]) {
  constexpr int pa[5] = {2, 0, 1, 1, 0}, pb[5] = {0, 2, 1, 0, 1};
  f32x4 lead[CB], rest[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    rest[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    lead[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[cb][0], rest[cb], 0, 0, 0);
  }
#pragma unroll
  for (int t = 0; t < 5; ++t)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
      rest[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[pa[t]], b[cb][pb[t]], rest[cb], 0, 0, 0);
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[cb][v] += lead[cb][v] + rest[cb][v];
}

// acc += rows 16 sb + li of the tile (part p of row r at tile + (p * T + r) *
// RS, in bf16 values) times the weights b, over step ks.
template <int T, int RS, int SB, int CB>
__device__ __forceinline__ void multiply_step(const uint16_t* tile, int lane, int ks, const bf16x8 (&b)[CB][3],
                                              f32x4 (&acc)[SB][CB]) {
  const uint16_t* al = tile + (lane & 15) * RS + 8 * (lane >> 4) + 32 * ks;
  bf16x8 a[SB][3];
#pragma unroll
  for (int sb = 0; sb < SB; ++sb)
#pragma unroll
    for (int p = 0; p < 3; ++p) a[sb][p] = *reinterpret_cast<const bf16x8*>(al + (p * T + 16 * sb) * RS);
  multiply_parts(a, b, acc);
}

// The same from a tile of fp32 values (row r at tile + r * RS floats), split as
// they are read.
template <int RS, int SB>
__device__ __forceinline__ void split_rows(const float* tile, int lane, int ks, bf16x8 (&a)[SB][3]) {
  const float* al = tile + (lane & 15) * RS + 8 * (lane >> 4) + 32 * ks;
#pragma unroll
  for (int sb = 0; sb < SB; ++sb) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(al + 16 * sb * RS);
    const f32x4 y = *reinterpret_cast<const f32x4*>(al + 16 * sb * RS + 4);
    const Split2 s[4] = {split2(x[0], x[1]), split2(x[2], x[3]), split2(y[0], y[1]), split2(y[2], y[3])};
#pragma unroll
    for (int p = 0; p < 3; ++p)
      a[sb][p] = __builtin_bit_cast(bf16x8, make_uint4(s[0].p[p], s[1].p[p], s[2].p[p], s[3].p[p]));
  }
}

// acc += (T x W tile) x (weights wf of the wave's 16 CB output units), the
// next step's weights requested while the current ones multiply.
template <int W, int T, int RS, int SB, int CB>
__device__ __forceinline__ void split_product(const uint16_t* tile, const uint16_t* wf, int lane,
                                              f32x4 (&acc)[SB][CB]) {
  constexpr int KS = W / 32;
  bf16x8 b0[CB][3], b1[CB][3];
  fetch_weights<W>(wf, lane, 0, b0);
#pragma unroll 1
  for (int ks = 0; ks < KS; ks += 2) {
    fetch_weights<W>(wf, lane, ks + 1, b1);
    multiply_step<T, RS>(tile, lane, ks, b0, acc);
    fetch_weights<W>(wf, lane, ks + 2 < KS ? ks + 2 : 0, b0);
    multiply_step<T, RS>(tile, lane, ks + 1, b1, acc);
  }
}

// The same with a whole layer's weights in registers: b holds wf's on entry,
// and those of `next` are requested step by step in their place.
template <int W, int T, int RS, int SB, int CB>
__device__ __forceinline__ void split_product_ahead(const uint16_t* tile, const uint16_t* next,
                                                    bf16x8 (&b)[W / 32][CB][3], int lane,
                                                    f32x4 (&acc)[SB][CB]) {
#pragma unroll
  for (int ks = 0; ks < W / 32; ++ks) {
    multiply_step<T, RS>(tile, lane, ks, b[ks], acc);
    fetch_weights<W>(next, lane, ks, b[ks]);
  }
}

}  // namespace mca

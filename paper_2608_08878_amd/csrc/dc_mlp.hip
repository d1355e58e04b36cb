// Two-hidden-layer policy on matrix cores (Sec. 3.1.2 scoring with the App. D
// network: n_in -> h1 -> h2 -> 1, optional LayerNorm, widths up to 128), gfx950.
//
// Scoring every cached row is two dense contractions, [rows x n_in] x
// [n_in x h1] and [rows x h1] x [h1 x h2].  On this part the float32 matrix
// instructions run at the float32 vector rate and do not overlap the vector
// work around them, so both run on the bf16 matrix cores instead,
// at float32 accuracy: every float32 operand x is split exactly into three
// bf16 parts x = xh + xm + xl (8 significand bits each: 24 in all; |xm| and
// |xl| about 2^-8 and 2^-16 of |x|), and the product of an activation h and a
// weight w keeps the six part products down to about 2^-16 of it,
// hl wh + hm wm + hh wl + hm wh + hh wm + hh wh (each exact in float32,
// accumulated in float32 by v_mfma_f32_16x16x32_bf16); the three dropped ones
// (hm wl, hl wm, hl wl) come to about 2^-23 of the product, one float32
// rounding.  The hidden widths are padded to HP = 64 (both at most 64) or
// 128.  One wave takes 16 rows at a time:
//   layer 1 (MFMA, the same split, inputs padded to 32): per 16-unit block b,
//     W1 (16 units x 32 inputs) times the rows' features (32 x 16 rows), so
//     lane (i, g) receives units 16 b + 4 g + r (r < 4) of row i;
//   layer 2 (MFMA): HP / 16 column blocks x HP / 32 k-steps x 6 part products;
//     k-step t takes from lane (i, g) the units 32 t + 4 g + r and
//     32 t + 16 + 4 g + r (r < 4) that layer 1 left in it, and the weight
//     parts sit in LDS as three [n][k] bf16 arrays in that unit order, with
//     a row stride of 2 HP + 16 bytes (the 16 rows one read touches start 16
//     bytes apart in the banks); all weight parts are split once per
//     workgroup;
//   the accumulators hold row 4 (l / 16) + i, column 16 cb + l % 16: ReLU and the
//     output dot product reduce over the 16 lanes of a DPP row.
// HP = 128: 1024-thread workgroups (138 KB of LDS, one per CU, four waves per
// SIMD); HP = 64: 512 threads (44 KB, two per CU).  Padded units (k >= h1,
// n >= h2) are exact zeros.  Networks with LayerNorm have a kernel of their own
// (score_ln2_kernel below), which the normalised range of their activations allows
// two float16 parts instead.
#include <hip/hip_runtime.h>

#include "dc_mlp.hpp"
#include "dc_select.hpp"

#pragma clang fp contract(off)

namespace dc {

namespace {

constexpr int NX = 5;                // features per row (the fifth is 0 for four-input policies)
typedef float f32x4_v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const char lchar;

template <int HP>
struct Cfg {
  static constexpr int MT = HP == 128 ? 1024 : 512;    // threads per workgroup
  static constexpr int MINB = HP == 128 ? 1 : 2;       // workgroups per CU
  static constexpr int MW = MT / 64;                   // waves
};

// LDS layout for hidden widths padded to HP (64 or 128): the float arrays
// first, so that every per-lane read of them is a constant offset within the
// 64 KB reach of an LDS instruction, then the three bf16 parts of W2
template <int HP>
struct Lay {
  static constexpr int RS = 2 * HP + 16;              // bytes per W2 row (unit n, k in k-step order)
  static constexpr int RS1 = 64 + 16;                 // bytes per W1 row (unit, 32 padded inputs)
  static constexpr int O_B1 = 0;                      // floats: b1       [HP]
  static constexpr int O_B2 = O_B1 + HP;              // b2, wo   [HP] each
  static constexpr int FLOATS = O_B2 + 2 * HP;
  static constexpr int O_W2 = FLOATS * 4;             // bytes: parts h, m, l, [3][HP][RS]
  static constexpr int O_W1 = O_W2 + 3 * HP * RS;     // bytes: parts h, m, l, [3][HP][RS1]
  static constexpr int BYTES = O_W1 + 3 * HP * RS1;
};

// position, within its row of W2's parts, of unit k: k-step t = k / 32 holds
// lane group g's units 32 t + 4 g + r and 32 t + 16 + 4 g + r (r < 4) at
// bytes 2 (32 t + 8 g) .. + 16
__host__ __device__ constexpr int w2_pos(int k) {
  return (k & ~31) + ((k & 31) < 16 ? 8 * ((k & 15) >> 2) + (k & 3) : 8 * ((k & 15) >> 2) + 4 + (k & 3));
}

template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float sum16(float x) {    // over the 16 lanes of a DPP row
  x += dpp_f<0xB1>(x);    // quad_perm [1,0,3,2]
  x += dpp_f<0x4E>(x);    // quad_perm [2,3,0,1]
  x += dpp_f<0x141>(x);   // row_half_mirror
  x += dpp_f<0x140>(x);   // row_mirror
  return x;
}
__device__ __forceinline__ float sum4rows(float x) {  // over lanes l, l^16, l^32, l^48
  x += __shfl_xor(x, 16);
  x += __shfl_xor(x, 32);
  return x;
}

// x = h + m + l exactly (three round-to-nearest bf16 parts; each residual is
// exact in float32: it holds at most the 16, then 8, bits below the part taken)
__device__ __forceinline__ void split3(float x, __bf16& h, __bf16& m, __bf16& l) {
  h = (__bf16)x;
  const float r1 = x - (float)h;
  m = (__bf16)r1;
  const float r2 = r1 - (float)m;
  l = (__bf16)r2;
}

// the same for eight values, two at a time (one packed conversion per part
// and pair)
typedef float f32x2_v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split3x8(const float (&v)[8], bf16x8_t& h, bf16x8_t& m, bf16x8_t& l) {
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const f32x2_v x = {v[2 * p], v[2 * p + 1]};
    const bf16x2_t xh = __builtin_convertvector(x, bf16x2_t);
    const f32x2_v r1 = x - __builtin_convertvector(xh, f32x2_v);
    const bf16x2_t xm = __builtin_convertvector(r1, bf16x2_t);
    const f32x2_v r2 = r1 - __builtin_convertvector(xm, f32x2_v);
    const bf16x2_t xl = __builtin_convertvector(r2, bf16x2_t);
    h[2 * p] = xh[0];
    h[2 * p + 1] = xh[1];
    m[2 * p] = xm[0];
    m[2 * p + 1] = xm[1];
    l[2 * p] = xl[0];
    l[2 * p + 1] = xl[1];
  }
}

struct Feat {
  double num, den;
  int32_t pos;
  float al, vn, sg;
};
__device__ __forceinline__ void fetch_row(const EvictArgs& a, size_t ub, int r, int L, Feat& f) {
  const size_t gi = ub + (r < L ? r : L - 1);             // past the end: re-read, unused
  f.num = a.num[gi];
  f.den = a.den[gi];
  f.pos = a.pos[gi];
  f.al = a.alpha[gi];
  f.vn = a.vnorm[gi];
  f.sg = (a.n_in == 5 ? a.sigma : a.alpha)[gi];           // (a dummy read for four inputs)
}
__device__ __forceinline__ void inputs(const EvictArgs& a, const Feat& f, float invT, float (&x)[NX]) {
  const float H = f.den > 0.0 ? (float)(f.num / f.den) : 0.0f;
  const float ps = (float)f.pos * invT;
  const bool five = a.n_in == 5;
  x[0] = f.al;
  x[1] = f.vn;
  x[2] = five ? f.sg : H;
  x[3] = five ? H : ps;
  x[4] = five ? ps : 0.0f;
}

template <int HP>
__device__ void stage(const EvictArgs& a, float* sm) {
  using Y = Lay<HP>;
  constexpr int MT = Cfg<HP>::MT, RS = Y::RS, RS1 = Y::RS1, O_B1 = Y::O_B1, O_B2 = Y::O_B2;
  const cfloat* P = const_params(a.params);
  const int h1 = a.h1, h2 = a.h2, nin = a.n_in;
  const cfloat* W1 = P;
  const cfloat* b1 = W1 + h1 * nin;
  const cfloat* W2 = b1 + h1;
  const cfloat* b2 = W2 + h2 * h1;
  const cfloat* wo = b2 + h2;
  char* w2 = reinterpret_cast<char*>(sm) + Y::O_W2;
  for (int e = threadIdx.x; e < HP * HP; e += MT) {
    const int n = e / HP, k = e % HP;
    __bf16 wh, wm, wl;
    split3((k < h1 && n < h2) ? W2[n * h1 + k] : 0.0f, wh, wm, wl);
    const int q = 2 * w2_pos(k);
    *reinterpret_cast<__bf16*>(w2 + n * RS + q) = wh;
    *reinterpret_cast<__bf16*>(w2 + (HP + n) * RS + q) = wm;
    *reinterpret_cast<__bf16*>(w2 + (2 * HP + n) * RS + q) = wl;
  }
  char* w1 = reinterpret_cast<char*>(sm) + Y::O_W1;
  for (int e = threadIdx.x; e < HP * 32; e += MT) {
    const int k = e / 32, x = e % 32;
    __bf16 wh, wm, wl;
    split3((k < h1 && x < nin) ? W1[k * nin + x] : 0.0f, wh, wm, wl);
    *reinterpret_cast<__bf16*>(w1 + k * RS1 + 2 * x) = wh;
    *reinterpret_cast<__bf16*>(w1 + (HP + k) * RS1 + 2 * x) = wm;
    *reinterpret_cast<__bf16*>(w1 + (2 * HP + k) * RS1 + 2 * x) = wl;
  }
  for (int i = threadIdx.x; i < HP; i += MT) {
    sm[O_B2 + i] = i < h2 ? b2[i] : 0.0f;
    sm[O_B2 + HP + i] = i < h2 ? wo[i] : 0.0f;
    sm[O_B1 + i] = i < h1 ? b1[i] : 0.0f;
  }
}

template <int HP>
__global__ void __launch_bounds__(Cfg<HP>::MT, Cfg<HP>::MINB)
score_mlp2_kernel(EvictArgs a, uint64_t* keys, int kstride) {
  using Y = Lay<HP>;
  constexpr int MW = Cfg<HP>::MW, RS = Y::RS, RS1 = Y::RS1, O_B1 = Y::O_B1, O_B2 = Y::O_B2;
  constexpr int NT = HP / 32;    // MFMA k-steps (32 units each)
  constexpr int NB = HP / 16;    // 16-unit blocks of layer 1
  constexpr int NC = HP / 16;    // 16-column blocks of layer 2
  extern __shared__ float sm[];
  // a unit that keeps every row reads no key (the whole workgroup leaves)
  if (unit_rows(a, a.y0 + blockIdx.y) <= a.fused_rows) return;    // served by the single-launch step
  if (!a.scores_out && unit_budget(a, a.y0 + blockIdx.y) >= unit_rows(a, a.y0 + blockIdx.y)) return;
  stage<HP>(a, sm);
  __syncthreads();
  const int u = a.y0 + blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ri = lane & 15, kg = lane >> 4;
  const int h1 = a.h1, h2 = a.h2;
  const int L = unit_rows(a, u);   // this unit's rows (scores_out keeps stride a.L)
  const size_t ub = (size_t)u * a.cap;
  const float invT = 1.0f / (float)a.T;
  const float bout = const_params(a.params)[h1 * a.n_in + h1 + h2 * h1 + h2 + h2];
  // features of this lane's A row (the four lanes of a row load the same row);
  // the next row block's are requested while the current one is computed
  auto fetch = [&](int rbx, Feat& f) { fetch_row(a, ub, rbx + ri, L, f); };
  const int stride = gridDim.x * MW * 16;
  int rb = (blockIdx.x * MW + wave) * 16;
  Feat nxt;
  fetch(rb, nxt);
  for (; rb < L; rb += stride) {
    const Feat f = nxt;
    fetch(rb + stride, nxt);
    float x[NX];
    inputs(a, f, invT, x);
    // layer 1 on the matrix cores: per 16-unit block b, D = W1 x X^T with the
    // inputs padded to 32 (lanes kg > 0 supply zeros), so lane (ri, kg) gets
    // units 16 b + 4 kg + r of its row ri, accumulated onto their biases.
    // Padded units (k >= h1) have zero weights and bias, so they come out exactly 0
    // here and after the ReLU.
    typedef __attribute__((address_space(3))) const f32x4_v lfloat4;
    typedef __attribute__((address_space(3))) const bf16x8_t lbf16x8;
    bf16x8_t xh, xm, xl;
    {
      float v[8] = {x[0], x[1], x[2], x[3], x[4], 0.0f, 0.0f, 0.0f};
      split3x8(v, xh, xm, xl);
      if (kg != 0) {
        const bf16x8_t zero = {};
        xh = zero;
        xm = zero;
        xl = zero;
      }
    }
    const lfloat* p1 = (const lfloat*)sm + 4 * kg;   // LDS, this lane's unit offset in a block
    const lchar* w1 = (const lchar*)sm + Y::O_W1 + ri * RS1 + 16 * kg;
    asm volatile("" : "+v"(p1), "+v"(w1));
    f32x4_v hv[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const lchar* wb = w1 + 16 * b * RS1;
      const bf16x8_t wh = *reinterpret_cast<lbf16x8*>(wb);
      const bf16x8_t wm = *reinterpret_cast<lbf16x8*>(wb + HP * RS1);
      const bf16x8_t wl = *reinterpret_cast<lbf16x8*>(wb + 2 * HP * RS1);
      f32x4_v c = *reinterpret_cast<lfloat4*>(p1 + O_B1 + 16 * b);
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wl, xh, c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wm, xm, c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wh, xl, c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wm, xh, c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wh, xm, c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wh, xh, c, 0, 0, 0);
      hv[b] = c;
    }
    // layer 2 on the bf16 matrix cores, six part products per k-step and
    // block, accumulated onto the bias of the lane's column
    f32x4_v acc[NC];
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      const float bn = sm[O_B2 + 16 * cb + ri];
      acc[cb] = (f32x4_v){bn, bn, bn, bn};
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      bf16x8_t ah, am, al;
      float v[8];
#pragma unroll
      for (int r = 0; r < 4; ++r) {            // ReLU; units 32 t + 4 kg + r, then + 16
        v[r] = fmaxf(hv[2 * t][r], 0.0f);
        v[4 + r] = fmaxf(hv[2 * t + 1][r], 0.0f);
      }
      split3x8(v, ah, am, al);
      // the weight rows of column block cb, this lane's 8 units of k-step t, at
      // bytes 2 (32 t + 8 kg) .. + 16 of each row in that order (an
      // opaque pointer per k-step keeps the reads from being hoisted out of the
      // row loop: all of W2's parts would not fit in registers)
      const lchar* w2 = (const lchar*)sm + Y::O_W2 + ri * RS + (32 * t + 8 * kg) * 2;
      asm volatile("" : "+v"(w2));
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) {
        const bf16x8_t bh = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8_t*>(
            w2 + 16 * cb * RS);
        const bf16x8_t bm = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8_t*>(
            w2 + (HP + 16 * cb) * RS);
        const bf16x8_t bl = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8_t*>(
            w2 + (2 * HP + 16 * cb) * RS);
        f32x4_v c = acc[cb];
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, bm, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, bh, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bm, c, 0, 0, 0);
        acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, c, 0, 0, 0);
      }
    }
    // rows 4 kg + i of the block, columns 16 cb + ri (padded columns: weights,
    // bias and output weight 0)
    float score[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float o = 0.0f;
#pragma unroll
      for (int cb = 0; cb < NC; ++cb)
        o = __builtin_fmaf(sm[O_B2 + HP + 16 * cb + ri], fmaxf(acc[cb][i], 0.0f), o);
      score[i] = sum16(o) + bout;
    }
    // lanes ri < 4 of each row group write rows 4 kg + ri; lane 4 kg + ri
    // loaded that row's position with its features
    const int32_t p = __shfl(f.pos, 4 * kg + (ri & 3));
    if (ri < 4) {
      const int row = rb + 4 * kg + ri;
      float sc = score[0];
#pragma unroll
      for (int i = 1; i < 4; ++i) sc = ri == i ? score[i] : sc;
      if (row < L) {
        if (a.scores_out) a.scores_out[(size_t)u * a.L + row] = sc;
        keys[(size_t)u * kstride + row] = row_key(a.sample ? sampled_score(a, sc, p, u) : sc, p);
      }
    }
  }
}

// ---------------------------------------------------------------- LayerNorm
// With LayerNorm (the App. D network) both layers' means are taken out of the
// weights: z_n - mean_n z = sum_k (W[n][k] - mean_n W[n][k]) h_k + b_n - mean b,
// so the matrix cores deliver the centred values and no sum over the units but
// the variance's is formed (the weights are centred in binary64; nothing
// cancels at run time).
//
// Layer 1: the six part products of the bf16 split over at most five inputs are
// 30 of one MFMA's 32 k-slots, so a 16-unit block is one instruction.  Slot s
// holds input s mod 5 of part pair s / 5 in (xh wh, xm wh, xl wh, xh wm, xm wm,
// xh wl).
//
// Layer 2: behind the LayerNorm and the ReLU an activation is at most |gain| sqrt(h1)
// + shift, so a power of two per hidden unit puts it into float16's range and its
// inverse goes to the unit's column of W2: x = xh + xl in two float16 parts (11
// significand bits each, signed residual), all four part products kept.  What a unit's
// products lack of the largest unit's is shared evenly by the two scales, so that
// neither side reaches float16's subnormal range before the products lie 2^30 below the
// largest; a unit that its shift keeps off has no weights.  (With one scale for all, a
// unit of gain 1e8 cost the others 13 bits.)  The low products are accumulated first,
// over all k, and the high ones onto their sum: four roundings at the size of
// the result instead of 24, so the error against binary64 is below the bf16 split's
// with six products (rms, 128 units, in 2^-24 of the result: 1.73 and 1.84 for four and
// five inputs against 2.07 and 2.43; the same for gains of 1e6 and 1e8 in single units;
// 3.0 against 1.6 where one unit outweighs all others 1e9 times and is off).
// Networks of at most 64 units have fewer terms to round: there the weights have a
// third part, split from binary64, and the products of layer 1's high parts have an
// instruction of their own (its adder aligns a block's products to the largest).
// 64 units 1.31 and 1.50 against 1.50 and 1.64, 32 1.42 and 1.32 against 1.42 and 1.26;
// without the two 1.55, 1.67, 1.71 and 1.56, for a tenth to a sixth less time (1024 x
// 4097 rows, 64-64: 191 -> 223 us; six bf16 products 306).
//
// What bounds it: the sum of matrix and vector instructions, which do not overlap
// on a SIMD here (counters: 559 k MFMA cycles + 417 k vector cycles of 993 k; a
// probe with one wave of each agrees).  So the vector work is cut: a lane per
// row forms the inputs of 64 rows at a time, the means come out of the matrix
// product, a float16 residual is one mixed-precision instruction, and both layers'
// outputs lie along a row.  Two row blocks per weight read (halving the LDS
// reads) changed nothing, three products instead of four would save 55 us.
// One workgroup per CU stages the weights once and strides over all units' rows.
// Measured (1024 units x 4097 rows, 5 -> 128 -> 128 -> 1): 517-585 us against
// 748-950 us with the bf16 split of six products; the whole step with decode, global
// alpha and selection 1234 -> 962 us.
constexpr int LT = 1024;                              // threads: one workgroup per CU, four waves per SIMD

typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const f32x4_v lfloat4;
typedef __attribute__((address_space(3))) const bf16x8_t lbf16x8;
typedef __attribute__((address_space(3))) const f16x8_t lf16x8;

// LDS positions.  A 16-byte-per-lane read takes 16 lanes at a time, rows 0..3 and
// 12..15 of one lane group (kg) with rows 4..11 of its neighbour (kg ^ 1); so that
// they hit different banks, 16-byte chunk c of a W2 row (16 chunks, 8 for HP =
// 64) sits at c ^ (row mod that), and chunk c of a 64-byte row at c ^ swz64(row).
// (With rows padded by 16 bytes instead, 38 % of the LDS cycles were conflicts.)
__device__ __forceinline__ int swz64(int row) {       // 0, 2, 3, 1 by row / 4 mod 4
  const int j = (row >> 2) & 3;
  return (((j & 1) << 1) ^ (j & 2)) | (j >> 1);
}

template <int HP>
struct LayN {
  static constexpr int RS = 2 * HP;                   // bytes per W2 row (unit n, k in k-step order)
  static constexpr int CM = HP / 8 - 1;               // chunks of a W2 row - 1
  static constexpr int RS1 = 64;                      // bytes per W1 row (unit, 32 part slots)
  static constexpr int O_B1 = 0;                      // floats: b1, g1, be1       [HP] each
  static constexpr int O_B2 = O_B1 + 3 * HP;          // b2, g2, be2, wo           [HP] each
  static constexpr int O_C = O_B2 + 4 * HP;           // 1 / (activation scale x weight scale)
  static constexpr int FLOATS = O_C + 4;
  static constexpr int WP = HP == 64 ? 3 : 2;         // parts of a weight
  static constexpr int O_W2 = FLOATS * 4;             // bytes: parts h, l (, ll), [WP][HP][RS]
  static constexpr int O_W1 = O_W2 + WP * HP * RS;    // bytes: [HP][RS1]
  static constexpr int O_X = O_W1 + HP * RS1;         // input slots, [waves][64 rows][64 bytes]
  static constexpr int BYTES = O_X + LT / 64 * 64 * 64;
};

// exponent e with x < 2^e, x > 0
__device__ __forceinline__ int expo(float x) { return __builtin_amdgcn_frexp_expf(x); }

template <int HP>
__device__ void stage_ln(const EvictArgs& a, float* sm) {
  using Y = LayN<HP>;
  constexpr int RS = Y::RS, RS1 = Y::RS1, O_B1 = Y::O_B1, O_B2 = Y::O_B2;
  constexpr int PARTS = LT / HP, PER = HP / PARTS;    // threads per column of W2, rows per thread
  __shared__ double csum[PARTS][HP];
  __shared__ float cmax[PARTS][HP];
  __shared__ double m1[8];                            // means of W1's columns, of b1 and of b2
  __shared__ int wtop[LT / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int h1 = a.h1, h2 = a.h2, nin = a.n_in;
  const float* W1 = a.params;
  const float* b1 = W1 + h1 * nin;
  const float* g1 = b1 + h1;
  const float* be1 = g1 + h1;
  const float* W2 = be1 + h1;
  const float* b2 = W2 + h2 * h1;
  const float* g2 = b2 + h2;
  const float* be2 = g2 + h2;
  const float* wo = be2 + h2;
  // this thread's rows n = part + PARTS j of W2's column k, and the column's sum
  const int k = tid % HP, part = tid / HP;
  float w[PER];
  double cs = 0.0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int n = part + PARTS * j;
    w[j] = (k < h1 && n < h2) ? W2[n * h1 + k] : 0.0f;
    cs += (double)w[j];
  }
  csum[part][k] = cs;
  if (wave < 7) {                                     // wave c: mean of W1's column c, of b1 (5), of b2 (6)
    const int n = wave == 6 ? h2 : h1;
    double v = 0.0;
    if (wave >= 5 || wave < nin)
      for (int i = lane; i < n; i += 64)
        v += (double)(wave < 5 ? W1[i * nin + wave] : wave == 5 ? b1[i] : b2[i]);
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
    if (lane == 0) m1[wave] = v / n;
  }
  __syncthreads();
  double mean = csum[0][k];
  for (int q = 1; q < PARTS; ++q) mean += csum[q][k];
  mean /= h2;
  float mw = 0.0f;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int n = part + PARTS * j;
    const float c = (k < h1 && n < h2) ? (float)((double)w[j] - mean) : 0.0f;
    mw = fmaxf(mw, fabsf(c));
    if constexpr (Y::WP == 2) w[j] = c;
  }
  cmax[part][k] = mean - mean == 0.0 ? mw : 1.0f;     // (a column with a NaN or an infinity goes through)
  // unit k's activation is at most mh (none: the ReLU never lets it through)
  const float mh = k < h1 ? __builtin_fmaf(fabsf(g1[k]), __builtin_sqrtf((float)h1), be1[k]) : 0.0f;
  const float mb = tid < h2 ? fabsf((float)((double)b2[tid] - m1[6])) : 0.0f;
  __syncthreads();
  mw = cmax[0][k];
  for (int q = 1; q < PARTS; ++q) mw = fmaxf(mw, cmax[q][k]);
  // The largest product h W2 of the network is below 2^top, unit k's below
  // 2^(top - dk): scaled by 2^(30 - top) in all, half of dk is left to the
  // activation's scale 2^ek and half to the weights'.  The bias stays below 2^60 (no
  // variance overflows), and no network is scaled up by more than 2^120.
  const bool live = mh > 0.0f && mw > 0.0f;
  const int pk = live ? expo(mh) + expo(mw) : -90;
  int top = mb > 0.0f && expo(mb) - 30 > pk ? expo(mb) - 30 : pk;
  top = top < -90 ? -90 : top;
  for (int m = 32; m >= 1; m >>= 1) {
    const int o = __shfl_xor(top, m);
    top = o > top ? o : top;
  }
  if (lane == 0) wtop[wave] = top;
  __syncthreads();
  for (int q = 0; q < LT / 64; ++q) top = wtop[q] > top ? wtop[q] : top;
  top = top > 130 ? 130 : top;                        // (products beyond float32: no value either way)
  const int ek = live ? 15 - ((top - pk) >> 1) - expo(mh) : 0, ew = 30 - top - ek;
  char* w2 = reinterpret_cast<char*>(sm) + Y::O_W2;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int n = part + PARTS * j;
    _Float16 xh;
    float r;                              // what xh leaves
    if constexpr (Y::WP == 2) {
      const float x = live ? __builtin_ldexpf(w[j], ew) : 0.0f;
      xh = (_Float16)x;
      r = x - (float)xh;
    } else {                              // from binary64: the centred weight is not rounded first
      const double x = live && n < h2 ? __builtin_ldexp((double)w[j] - mean, ew) : 0.0;
      xh = (_Float16)(float)x;
      r = (float)(x - (double)xh);
    }
    const _Float16 xl = (_Float16)r;
    const int q = (2 * w2_pos(k)) ^ (16 * (n & Y::CM));
    *reinterpret_cast<_Float16*>(w2 + n * RS + q) = xh;
    *reinterpret_cast<_Float16*>(w2 + (HP + n) * RS + q) = xl;
    if constexpr (Y::WP == 3) *reinterpret_cast<_Float16*>(w2 + (2 * HP + n) * RS + q) = (_Float16)(r - (float)xl);
  }
  char* w1 = reinterpret_cast<char*>(sm) + Y::O_W1;
  for (int e = tid; e < HP * 8; e += LT) {            // unit e / 8, input e % 8 (five of them)
    const int n = e / 8, x = e % 8;
    __bf16 wh, wm, wl;
    split3((n < h1 && x < nin) ? (float)((double)W1[n * nin + x] - m1[x]) : 0.0f, wh, wm, wl);
    char* row = w1 + n * RS1;
    const int sw = 16 * swz64(n);
    if (x < 5) {
      const __bf16 parts[6] = {wh, wh, wh, wm, wm, wl};
#pragma unroll
      for (int q = 0; q < 6; ++q) *reinterpret_cast<__bf16*>(row + ((2 * (5 * q + x)) ^ sw)) = parts[q];
    } else if (x < 7) {
      *reinterpret_cast<__bf16*>(row + ((2 * (30 + x - 5)) ^ sw)) = (__bf16)0.0f;
    }
  }
  if (tid < HP) {                                     // (unit k = tid)
    const int i = tid;
    const bool v2 = i < h2, v1 = i < h1;
    sm[O_B1 + i] = v1 ? (float)((double)b1[i] - m1[5]) : 0.0f;
    sm[O_B1 + HP + i] = live ? __builtin_ldexpf(g1[i], ek) : 0.0f;
    sm[O_B1 + 2 * HP + i] = live ? __builtin_ldexpf(be1[i], ek) : 0.0f;
    sm[O_B2 + i] = v2 ? __builtin_ldexpf((float)((double)b2[i] - m1[6]), 30 - top) : 0.0f;
    sm[O_B2 + HP + i] = v2 ? g2[i] : 0.0f;
    sm[O_B2 + 2 * HP + i] = v2 ? be2[i] : 0.0f;
    sm[O_B2 + 3 * HP + i] = v2 ? wo[i] : 0.0f;
  }
  if (tid == 0) sm[Y::O_C] = __builtin_ldexpf(1.0f, top - 30);
}

// x - xh rounded to float16 for both halves of xh (one mixed-precision
// instruction per value: the difference is exact before its rounding)
__device__ __forceinline__ uint32_t residual2(uint32_t xh, float x0, float x1) {
  uint32_t r;
  asm("v_fma_mixlo_f16 %0, %1, -1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(xh), "v"(x0));
  asm("v_fma_mixhi_f16 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(r) : "v"(xh), "v"(x1));
  return r;
}

// (xh, xl) of eight values in float16
__device__ __forceinline__ void split2x8(const float (&v)[8], f16x8_t& h, f16x8_t& l) {
  uint4 hw, lw;
  uint32_t* hp = reinterpret_cast<uint32_t*>(&hw);
  uint32_t* lp = reinterpret_cast<uint32_t*>(&lw);
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const f32x2_v x = {v[2 * p], v[2 * p + 1]};
    hp[p] = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, f16x2_t));
    lp[p] = residual2(hp[p], v[2 * p], v[2 * p + 1]);
  }
  h = __builtin_bit_cast(f16x8_t, hw);
  l = __builtin_bit_cast(f16x8_t, lw);
}

// nq: 16-row blocks of a wave's item (1..4)
template <int HP>
__global__ void __launch_bounds__(LT, 1)
score_ln2_kernel(EvictArgs a, uint64_t* keys, int kstride, int nq) {
  using Y = LayN<HP>;
  constexpr int RS = Y::RS, RS1 = Y::RS1, O_B1 = Y::O_B1, O_B2 = Y::O_B2;
  constexpr int NT = HP / 32;    // MFMA k-steps of layer 2
  constexpr int NB = HP / 16;    // 16-unit blocks of either layer
  extern __shared__ float sm[];
  stage_ln<HP>(a, sm);
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ri = lane & 15, kg = lane >> 4;
  const int h1 = a.h1, h2 = a.h2;
  // the moments multiply by 1 / width and the scale uses the hardware
  // reciprocal square root (one rounding more each than a division)
  const float ih1 = 1.0f / (float)h1, ih2 = 1.0f / (float)h2;
  const float invT = 1.0f / (float)a.T;
  const float bout = const_params(a.params)[h1 * a.n_in + 3 * h1 + h2 * h1 + 3 * h2 + h2];
  const float cinv = sm[Y::O_C];
  char* xw = reinterpret_cast<char*>(sm) + Y::O_X + wave * 64 * 64;   // this wave's input slots
  const int rows = 16 * nq;
  const int per = (a.L + rows - 1) / rows;                 // items of the longest unit
  const int64_t total = (int64_t)per * a.units;
  const int stride = gridDim.x * (LT / 64);
  // items go to the workgroups first, so that few items spread over the CUs
  for (int64_t w0 = blockIdx.x + (int64_t)gridDim.x * wave; w0 < total; w0 += stride) {
    const int u = (int)(w0 / per), rb = (int)(w0 - (int64_t)u * per) * rows;
    const int L = unit_rows(a, u);
    // (a unit that keeps every row reads no key)
    if (rb >= L || L <= a.fused_rows || (!a.scores_out && unit_budget(a, u) >= L)) continue;
    const size_t ub = (size_t)u * a.cap;
    // the item's inputs, a lane per row: all 32 part slots to LDS
    Feat f;
    fetch_row(a, ub, rb + lane, L, f);
    {
      float x[NX];
      inputs(a, f, invT, x);
      __bf16 p[3][NX];
#pragma unroll
      for (int i = 0; i < NX; ++i) split3(x[i], p[0][i], p[1][i], p[2][i]);
      constexpr int PART[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        bf16x8_t v;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int s = 8 * c + j;
          v[j] = s < 30 ? p[PART[s / 5]][s % 5] : (__bf16)0.0f;
        }
        *reinterpret_cast<bf16x8_t*>(xw + 64 * lane + 16 * (c ^ swz64(lane))) = v;
      }
    }
    // (LDS operations of one wave complete in order)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    float sc = 0.0f;
#pragma unroll 1
    for (int q = 0; q < nq && rb + 16 * q < L; ++q) {
      // layer 1: lane (ri, kg) gets units 16 b + 4 kg + r of row ri, centred
      const lchar* xr = (const lchar*)xw + 64 * (16 * q + ri) + 16 * (kg ^ swz64(ri));
      const lfloat* p1 = (const lfloat*)sm + 4 * kg;
      const lchar* w1 = (const lchar*)sm + Y::O_W1 + ri * RS1 + 16 * (kg ^ swz64(ri));
      asm volatile("" : "+v"(p1), "+v"(w1));
      const bf16x8_t xs = *reinterpret_cast<lbf16x8*>(xr);
      // (narrow networks: the products of the high parts onto the sum of the others)
      bf16x8_t x0 = xs, x1 = {};
      if constexpr (Y::WP == 3) {
#pragma unroll
        for (int i = 0; i < 5; ++i) {
          x1[i] = kg == 0 ? xs[i] : (__bf16)0.0f;
          x0[i] = kg == 0 ? (__bf16)0.0f : xs[i];
        }
      }
      f32x4_v hv[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const bf16x8_t wv = *reinterpret_cast<lbf16x8*>(w1 + 16 * b * RS1);
        const f32x4_v c0 = *reinterpret_cast<lfloat4*>(p1 + O_B1 + 16 * b);
        hv[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv, x0, c0, 0, 0, 0);
        if constexpr (Y::WP == 3) hv[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv, x1, hv[b], 0, 0, 0);
      }
      float s2 = 0.0f;
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) s2 = __builtin_fmaf(hv[b][r], hv[b][r], s2);
      const float rs1 = __builtin_amdgcn_rsqf(__builtin_fmaf(sum4rows(s2), ih1, LN_EPS));
      // gain and shift (scaled), ReLU, the two parts: k-step t takes units
      // 32 t + 4 kg + r, then + 16 (padded units: gain and shift 0)
      f16x8_t ah[NT], al[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        float v[8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f32x4_v g = *reinterpret_cast<lfloat4*>(p1 + O_B1 + HP + 16 * (2 * t + h));
          const f32x4_v be = *reinterpret_cast<lfloat4*>(p1 + O_B1 + 2 * HP + 16 * (2 * t + h));
#pragma unroll
          for (int r = 0; r < 4; ++r)
            v[4 * h + r] = fmaxf(__builtin_fmaf(hv[2 * t + h][r] * rs1, g[r], be[r]), 0.0f);
        }
        split2x8(v, ah[t], al[t]);
      }
      // layer 2, the same way round (weights times activations^T): per block of 16
      // units the low products over all k-steps, then the high ones
      f32x4_v acc[NB];
      const lchar* w2[NT];                  // chunk 4 t + kg of the lane's weight row
#pragma unroll
      for (int t = 0; t < NT; ++t) w2[t] = (const lchar*)sm + Y::O_W2 + ri * RS + 16 * ((4 * t + kg) ^ (ri & Y::CM));
      // (opaque, so that the weight reads are not hoisted out of the row loop)
#pragma unroll
      for (int t = 0; t < NT; ++t) asm volatile("" : "+v"(w2[t]));
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        f16x8_t wh[NT];
        f32x4_v c = *reinterpret_cast<lfloat4*>(p1 + O_B2 + 16 * b);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          wh[t] = *reinterpret_cast<lf16x8*>(w2[t] + 16 * b * RS);
          const f16x8_t wl = *reinterpret_cast<lf16x8*>(w2[t] + (HP + 16 * b) * RS);
          if constexpr (Y::WP == 3) {
            const f16x8_t wn = *reinterpret_cast<lf16x8*>(w2[t] + (2 * HP + 16 * b) * RS);
            c = __builtin_amdgcn_mfma_f32_16x16x32_f16(wn, ah[t], c, 0, 0, 0);
          }
          c = __builtin_amdgcn_mfma_f32_16x16x32_f16(wl, al[t], c, 0, 0, 0);
          c = __builtin_amdgcn_mfma_f32_16x16x32_f16(wh[t], al[t], c, 0, 0, 0);
          c = __builtin_amdgcn_mfma_f32_16x16x32_f16(wl, ah[t], c, 0, 0, 0);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) c = __builtin_amdgcn_mfma_f32_16x16x32_f16(wh[t], ah[t], c, 0, 0, 0);
        acc[b] = c;
      }
      // units 16 b + 4 kg + r of row ri, centred (padded units 0)
      float t2 = 0.0f;
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) t2 = __builtin_fmaf(acc[b][r], acc[b][r], t2);
      const float rs2 = __builtin_amdgcn_rsqf(__builtin_fmaf(sum4rows(t2) * cinv * cinv, ih2, LN_EPS)) * cinv;
      float o = 0.0f;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const f32x4_v g = *reinterpret_cast<lfloat4*>(p1 + O_B2 + HP + 16 * b);
        const f32x4_v be = *reinterpret_cast<lfloat4*>(p1 + O_B2 + 2 * HP + 16 * b);
        const f32x4_v wo = *reinterpret_cast<lfloat4*>(p1 + O_B2 + 3 * HP + 16 * b);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          o = __builtin_fmaf(wo[r], fmaxf(__builtin_fmaf(acc[b][r] * rs2, g[r], be[r]), 0.0f), o);
      }
      // lane 16 q + i of the item takes row i's score from its own lane group
      const float got = sum4rows(o) + bout;
      sc = kg == q ? got : sc;
    }
    const int row = rb + lane;
    if (lane < rows && row < L) {
      if (a.scores_out) a.scores_out[(size_t)u * a.L + row] = sc;
      keys[(size_t)u * kstride + row] = row_key(a.sample ? sampled_score(a, sc, f.pos, u) : sc, f.pos);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the slots are read before the next item's
  }
}

}  // namespace

int launch_score_mlp2(const EvictArgs& a, uint64_t* keys, int kstride, void* stream) {
  // hidden widths up to 64 pad to 64: a quarter of the layer-2 work of 128
  const bool narrow = a.h1 <= 64 && a.h2 <= 64;
  if (a.ln) {
    // items of 64 rows where every wave of a workgroup per CU gets one, else of 16
    const int64_t b64 = (int64_t)a.units * ((a.L + 63) / 64);
    const int nq = b64 >= 256 * (LT / 64) ? 4 : 1;
    const int64_t items = nq == 4 ? b64 : (int64_t)a.units * ((a.L + 15) / 16);
    const int grid = (int)(items < 256 ? items : 256);
    const size_t lds = (size_t)(narrow ? LayN<64>::BYTES : LayN<128>::BYTES);
    auto kern = narrow ? score_ln2_kernel<64> : score_ln2_kernel<128>;
    hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(LT), lds, (hipStream_t)stream, a, keys, kstride, nq);
    return (int)hipGetLastError();
  }
  const int mw = narrow ? Cfg<64>::MW : Cfg<128>::MW;
  const int nblk = (a.L + mw * 16 - 1) / (mw * 16);
  // workgroups per unit: enough for about 2048 in all, each staging the weight
  // parts once for as many rows as possible
  int gx = (2048 + a.units - 1) / a.units;
  gx = gx < nblk ? gx : nblk;
  gx = gx > 0 ? gx : 1;
  const size_t lds = (size_t)(narrow ? Lay<64>::BYTES : Lay<128>::BYTES);
  auto launch = [&](auto kern, int mt) {
    hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    for_grid_y(a.units, [&](int y0, int ny) {
      EvictArgs b = a;
      b.y0 = y0;
      hipLaunchKernelGGL(kern, dim3(gx, ny), dim3(mt), lds, (hipStream_t)stream, b, keys, kstride);
    });
  };
  if (narrow) launch(score_mlp2_kernel<64>, Cfg<64>::MT);
  else launch(score_mlp2_kernel<128>, Cfg<128>::MT);
  return (int)hipGetLastError();
}

}  // namespace dc

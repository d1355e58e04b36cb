// Decode step for bfloat16 caches on gfx950 matrix cores, optionally fused with
// scoring, top-B selection and compaction (the whole of one Algorithm 1 step).
//
// Per unit (G query heads sharing one KV head, head_dim D):
//   pass A  stream K once.  One v_mfma_f32_16x16x32_bf16 chain per 16 keys gives
//           the logits of up to 16 query rows: rows 0..G-1 are this step's
//           queries, rows 8..8+G-1 the queries of the step leaving the entropy
//           window (from the ring), so the retired weights come out of the same
//           instructions that produced them w steps ago.  Logits s = scale q.k
//           go to LDS, the retired contributions are reduced per key.
//   pass P  with the block-wide max M_j: p = exp(s - M) (stored over s),
//           l_j = sum p, u_j = sum p (s - M);  H_j = ln l_j - u_j / l_j.
//   pass B  stream V once: o_j = sum_i p_ji v_i (fp32), one 16-lane group per row.
//   pass D  features per key (thread per key): alpha += mean_j a_ji,
//           den += sum_j a_ji - retired, num += sum_j a_ji H_j - retired,
//           a_ji = p_ji / l_j; with eviction fused, the policy score and the
//           64-bit ranking key of every row are formed here and the unit is
//           compacted before the workgroup exits.
// Caches too long for LDS use the chunked form of the same passes (two
// kernels, logits in the workspace).
#include "dc_select.hpp"

#pragma clang fp contract(off)

namespace dc {

constexpr int SNT = 512;              // threads per workgroup (two workgroups per CU)
constexpr int SNW = SNT / 64;
constexpr int SCHUNK = 2048;          // rows per workgroup on the chunked path
constexpr int S_KMAX = 10;            // fused step: row slots per thread (L <= 5120)
constexpr int S_LDS = 160 * 1024 - 4 * 1024;  // dynamic LDS budget (static LDS aside)

template <int D>
struct MG {
  static constexpr int NT = D / 32;   // MFMA k-steps per 16-key tile
  static constexpr int LB = D / 2;    // bytes of a key row one lane loads
  static constexpr int LPR = D / 8;   // lanes per row in the value pass (16 bytes each)
};

__device__ __forceinline__ float max16(float x) {
  x = fmaxf(x, dpp<DPP_XOR1>(x));
  x = fmaxf(x, dpp<DPP_XOR2>(x));
  x = fmaxf(x, dpp<DPP_HALF_MIRROR>(x));
  x = fmaxf(x, dpp<DPP_MIRROR>(x));
  return x;
}

// x + (x of lane l ^ 32), and l ^ 16, without the LDS pipe: after the swap of
// two copies' halves one holds the lower lanes' values twice, the other the
// upper ones'.
__device__ __forceinline__ float add_xor32(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_xor16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sum over the wave in butterfly order (32, 16, .. 1).  FAST: out of the LDS pipe.
// Past the first two levels a value repeats every 8, 4, 2 lanes of a row, so a
// rotation of the row by half a period is the butterfly's partner: the same bits.
template <bool FAST>
__device__ __forceinline__ float wave_sum(float x) {
  if constexpr (!FAST) {
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
    return x;
  }
  x = add_xor32(x);
  x = add_xor16(x);
  x += dpp<0x128>(x);    // row_ror:8
  x += dpp<0x124>(x);
  x += dpp<0x122>(x);
  x += dpp<0x121>(x);
  return x;
}

// A-operand fragments: lane l holds row i = l & 15 and, for MFMA t, the 8 dims
// of 16-byte chunk 4t + g (g = l >> 4) of that row.  The key rows are read
// with the same chunk assignment (so each load instruction covers 64
// contiguous bytes of 16 rows); which dims a lane contributes to an MFMA's
// reduction is free as long as both operands agree.  Rows 0..G-1 hold the
// current queries, rows 8..8+G-1 the retiring queries, other rows zero.
template <int D, int G>
__device__ __forceinline__ void load_qfrag(uint4 (&qa)[MG<D>::NT], const DecodeArgs& a, int u,
                                           bool retire) {
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  const char* src = nullptr;
  if (i < G) src = (const char*)a.q + ((size_t)u * G + i) * D * 2;
  else if (retire && i >= 8 && i < 8 + G)
    src = (const char*)a.qring + (((size_t)u * a.window + a.slot) * G + (i - 8)) * D * 2;
#pragma unroll
  for (int t = 0; t < MG<D>::NT; ++t)
    qa[t] = src ? ldg16(src + 16 * (4 * t + g)) : make_uint4(0, 0, 0, 0);
}

// Retiring step's statistics (uniform over the workgroup).
template <int G>
struct RetStats {
  float m[G], il[G], h[G];
};

template <int G>
__device__ __forceinline__ void load_ret(RetStats<G>& r, const DecodeArgs& a, int u) {
  const float* st = a.qstat + ((size_t)u * a.window + a.slot) * G * 3;
#pragma unroll
  for (int j = 0; j < G; ++j) {
    r.m[j] = st[3 * j];
    r.il[j] = st[3 * j + 1];
    r.h[j] = st[3 * j + 2];
  }
}

// ---------------------------------------------------------------- pass A
// Rows [r0, r1) of unit u in 16-key tiles.  Logits of the current heads go to
// s_sink[(i - sink0) * RS + j], running maxima per current head into mrun.  The
// retired contributions (z, n) of each key are either stored to
// r_sink[2 (i - sink0)] (tiles round-robin over the waves; chunked path) or, with
// GROUPED, kept in registers: rows then go in groups of 64 (four tiles), group
// b to wave b mod SNW, and after a group lane l of the wave holds the pair of
// the group's row l, in zr[k] / nr[k] for the wave's k-th group.
constexpr int S_GMAX = S_KMAX;        // 64-row groups per wave, at most (L <= 5120)

// Rows of unit u before this step (per unit for ragged caches).
// (Device lengths are clamped to [0, len_old], the host's bound, so that a bad
// value cannot take an access out of the buffers.)
__device__ __forceinline__ int len_old_of(const DecodeArgs& a, int u) {
  if (!a.unit_len) return a.len_old;
  const int n = a.unit_len[u];
  return n < 0 ? 0 : n > a.len_old ? a.len_old : n;
}

template <int D, int G, bool FEAT, bool GROUPED, int RS = G>
__device__ __forceinline__ void pass_a(const DecodeArgs& a, int u, int r0, int r1, float* s_sink,
                                       float* r_sink, int sink0, const uint4 (&qa)[MG<D>::NT],
                                       bool retire, const RetStats<G>& rs, float (&mrun)[4],
                                       float (&zr)[S_GMAX], float (&nr)[S_GMAX]) {
  constexpr int NT = MG<D>::NT;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
  const char* kc = (const char*)a.k + (size_t)u * a.cap * D * 2;
  const char* kn = a.append ? (const char*)a.k_new + (size_t)u * D * 2 : nullptr;
  const int newrow = a.append ? len_old_of(a, u) : -1;
  const int ntiles = (r1 - r0 + 15) / 16;
#pragma unroll
  for (int r = 0; r < 4; ++r) mrun[r] = NEG_BIG;
  auto clamp_tile = [&](int t) { return t < ntiles ? t : ntiles - 1; };
  auto load_tile = [&](int tile, uint4 (&kb)[NT]) {
    int key = r0 + tile * 16 + i;
    key = key < r1 ? key : r1 - 1;
    const char* kp = key == newrow ? kn : kc + (size_t)key * D * 2;
    // plain loads: instructions t and t+1 read the two halves of the same 128-byte
    // line, so the second one should find it in the vector L1
#pragma unroll
    for (int t = 0; t < NT; ++t) kb[t] = ldg16(kp + 16 * (4 * t + g));
  };
  // logits of tile tt; returns the retired pair of key (tile row i) in lanes
  // 32 + i (zero elsewhere or without a retiring step)
  auto process = [&](int tt, const uint4 (&kb)[NT], float& z, float& n) {
    f32x4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int t = 0; t < NT; ++t)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, qa[t]),
                                                    __builtin_bit_cast(bf16x8_t, kb[t]), acc, 0,
                                                    0, 0);
    const int key = r0 + tt * 16 + i;
    const bool valid = key < r1;
    float s[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) s[r] = acc[r] * a.scale;
    // rows 4g + r: current heads in groups g < 2, retiring heads in groups 2, 3
    if (4 * g < G && valid) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (4 * g + r < G) mrun[r] = fmaxf(mrun[r], s[r]);
      float* dst = s_sink + (size_t)(key - sink0) * RS + 4 * g;
      if constexpr (G >= 4) {
        *reinterpret_cast<f32x4_t*>(dst) = f32x4_t{s[0], s[1], s[2], s[3]};
      } else {
#pragma unroll
        for (int r = 0; r < G; ++r) dst[r] = s[r];
      }
    }
    z = 0.0f;
    n = 0.0f;
    if constexpr (FEAT) {
      if (retire && g >= 2 && 4 * (g - 2) < G) {
        const bool hi = G > 4 && g == 3;        // heads 4..7 (only when G == 8)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          constexpr int last = G - 1;
          const int jl = r < G ? r : last, jh = 4 + r < G ? 4 + r : last;
          if ((hi ? 4 + r : r) < G) {
            const float mm = hi ? rs.m[jh] : rs.m[jl];
            const float il = hi ? rs.il[jh] : rs.il[jl];
            const float hh = hi ? rs.h[jh] : rs.h[jl];
            const float w = attn_weight(s[r], mm, il);
            z = z + w;
            n = n + w * hh;
          }
        }
      }
      if constexpr (G > 4) {     // heads 4..7 live in group 3: add the blocks in order
        const float z1 = __shfl_down(z, 16), n1 = __shfl_down(n, 16);
        z = z + z1;
        n = n + n1;
      }
    }
  };
  // Two tiles in flight per wave: consume a buffer, then refill it.  Every load
  // is issued unconditionally (a tile past the end re-reads the last tile, which
  // the cache serves), so the wait before a tile's MFMAs covers only that
  // tile's loads and never drains the other buffer.
  if constexpr (GROUPED) {
    const int ngrp = (ntiles + 3) / 4;
    const int ngw = wave < ngrp ? (ngrp - 1 - wave) / SNW + 1 : 0;
#pragma unroll
    for (int k = 0; k < S_GMAX; ++k) {
      zr[k] = 0.0f;
      nr[k] = 0.0f;
    }
    if (ngw > 0) {
      uint4 kb0[NT], kb1[NT];
      load_tile(4 * wave, kb0);
      load_tile(clamp_tile(4 * wave + 1), kb1);
      for (int k = 0; k < ngw; ++k) {
        const int t0 = 4 * (wave + SNW * k), tn = t0 + 4 * SNW;
        float zz = 0.0f, nn = 0.0f;
        // tile j's pairs (lanes 32..47) move to lanes 16 j .. 16 j + 15
        auto take = [&](int j, float z, float n) {
          const float zj = __shfl(z, 32 + i), nj = __shfl(n, 32 + i);
          zz = g == j ? zj : zz;
          nn = g == j ? nj : nn;
        };
        float z, n;
        process(t0, kb0, z, n);
        if constexpr (FEAT) take(0, z, n);
        load_tile(clamp_tile(t0 + 2), kb0);
        process(t0 + 1, kb1, z, n);
        if constexpr (FEAT) take(1, z, n);
        load_tile(clamp_tile(t0 + 3), kb1);
        process(t0 + 2, kb0, z, n);
        if constexpr (FEAT) take(2, z, n);
        load_tile(clamp_tile(tn), kb0);
        process(t0 + 3, kb1, z, n);
        if constexpr (FEAT) take(3, z, n);
        load_tile(clamp_tile(tn + 1), kb1);
        if constexpr (FEAT) {
#pragma unroll
          for (int s2 = 0; s2 < S_GMAX; ++s2) {
            zr[s2] = s2 == k ? zz : zr[s2];
            nr[s2] = s2 == k ? nn : nr[s2];
          }
        }
      }
    }
  } else if (wave < ntiles) {
    uint4 kb0[NT], kb1[NT];
    load_tile(wave, kb0);
    // the loop stores one retired pair per tile between the two buffers' loads;
    // a store to the padding row here gives the loop's first wait the same
    // sequence of outstanding operations as every later one
    if constexpr (FEAT) *reinterpret_cast<float2*>(r_sink + 2 * (size_t)(a.lmax - 1 - sink0)) = make_float2(0.0f, 0.0f);
    load_tile(clamp_tile(wave + SNW), kb1);
    // every lane stores (a store under a branch would make the wait before the
    // next tile's matrix ops cover it too); lanes without a retired row of their
    // own write the padding row past the unit
    auto sink = [&](int tt, float z, float n) {
      if constexpr (FEAT) {
        const int key = r0 + tt * 16 + i;
        const int slot = (retire && g == 2 && key < r1) ? key - sink0 : a.lmax - 1 - sink0;
        *reinterpret_cast<float2*>(r_sink + 2 * (size_t)slot) = make_float2(z, n);
      }
    };
    for (int tile = wave; tile < ntiles; tile += 2 * SNW) {
      float z, n;
      process(tile, kb0, z, n);
      sink(tile, z, n);
      load_tile(clamp_tile(tile + 2 * SNW), kb0);
      // unconditional: a tile past the end has no valid key, so it writes no
      // logits and sends its retired pair to the padding row
      process(tile + SNW, kb1, z, n);
      sink(tile + SNW, z, n);
      load_tile(clamp_tile(tile + 3 * SNW), kb1);
    }
  }
}

// Block-wide max of the current heads' logits; stat: SNW * G + G floats of LDS.
// A few threads reduce over the waves (fixed order) and broadcast through LDS,
// so no thread holds all the per-wave partials at once.
template <int G>
__device__ __forceinline__ void block_max(const float (&mrun)[4], float* stat, float (&M)[G]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4;
  float mm[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) mm[r] = max16(mrun[r]);
  if ((lane & 15) == 0 && 4 * g < G) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * g + r < G) stat[wave * G + 4 * g + r] = mm[r];
  }
  __syncthreads();
  if (threadIdx.x < G) {
    float m = stat[threadIdx.x];
    for (int w = 1; w < SNW; ++w) m = fmaxf(m, stat[w * G + threadIdx.x]);
    stat[SNW * G + threadIdx.x] = m;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < G; ++j) M[j] = stat[SNW * G + j];
}

// pass P over LDS rows [0, n): p = exp(s - M) in place; returns the per-thread
// partial sums of p and p (s - M).
template <int G, int RS = G>
__device__ __forceinline__ void pass_p(float* sbuf, int n, const float (&M)[G], float (&ls)[G],
                                       float (&us)[G]) {
#pragma unroll
  for (int j = 0; j < G; ++j) {
    ls[j] = 0.0f;
    us[j] = 0.0f;
  }
  for (int i = threadIdx.x; i < n; i += SNT) {
#pragma unroll
    for (int j = 0; j < G; ++j) {
      const float d = sbuf[i * RS + j] - M[j];
      const float p = __builtin_amdgcn_exp2f(d * LOG2E);
      sbuf[i * RS + j] = p;
      ls[j] = ls[j] + p;
      us[j] = us[j] + p * d;
    }
  }
}

// Block sums of G-vectors (fixed order); stat: SNW * 2G + 2G floats of LDS.
template <int G, bool FAST>
__device__ __forceinline__ void block_sum2(float (&x)[G], float (&y)[G], float* stat) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < G; ++j) {
    x[j] = wave_sum<FAST>(x[j]);
    y[j] = wave_sum<FAST>(y[j]);
  }
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < G; ++j) {
      stat[wave * 2 * G + j] = x[j];
      stat[wave * 2 * G + G + j] = y[j];
    }
  }
  __syncthreads();
  if (threadIdx.x < 2 * G) {
    float acc = 0.0f;
    for (int w = 0; w < SNW; ++w) acc = acc + stat[w * 2 * G + threadIdx.x];
    stat[SNW * 2 * G + threadIdx.x] = acc;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < G; ++j) {
    x[j] = stat[SNW * 2 * G + j];
    y[j] = stat[SNW * 2 * G + G + j];
  }
}

// pass B: rows [r0, r1), p from pbuf[(i - p0) * G + j]; per-wave partial output
// o[j][e] for the lane's 8 dims (lanes 0..LPR-1 hold the wave total).
// The first PF rows of a group are requested by pass_b_first, ahead of pass P
// (they depend on nothing), so that their latency passes under it.
constexpr int PF = 8;

template <int D>
struct VRows {                          // where unit u's value rows are
  const char* vc;
  const char* vn;
  int newrow;
  __device__ __forceinline__ VRows(const DecodeArgs& a, int u)
      : vc((const char*)a.v + (size_t)u * a.cap * D * 2),
        vn(a.append ? (const char*)a.v_new + (size_t)u * D * 2 : nullptr),
        newrow(a.append ? len_old_of(a, u) : -1) {}
  // rows past r1 load row r1 - 1 again (no divergent loads)
  __device__ __forceinline__ uint4 load(int row, int r1, int lam) const {
    const int rc = row < r1 ? row : r1 - 1;
    return ldg16_nt((rc == newrow ? vn : vc + (size_t)rc * D * 2) + lam * 16);
  }
};

template <int D>
__device__ __forceinline__ void pass_b_first(const DecodeArgs& a, int u, int r0, int r1, uint4 (&vb)[PF]) {
  constexpr int LPR = MG<D>::LPR, NG = SNT / LPR;
  const VRows<D> v(a, u);
#pragma unroll
  for (int p = 0; p < PF; ++p) vb[p] = v.load(r0 + (int)threadIdx.x / LPR + p * NG, r1, threadIdx.x % LPR);
}

template <int D, int G, bool FAST, int RS = G>
__device__ __forceinline__ void pass_b(const DecodeArgs& a, int u, int r0, int r1,
                                       const float* pbuf, int p0, uint4 (&vb)[PF], float (&o)[G][8]) {
  constexpr int LPR = MG<D>::LPR, NG = SNT / LPR;
  const int tid = threadIdx.x, grp = tid / LPR, lam = tid % LPR;
  const VRows<D> vr(a, u);
#pragma unroll
  for (int j = 0; j < G; ++j)
#pragma unroll
    for (int e = 0; e < 8; ++e) o[j][e] = 0.0f;
  // (rows past r1 are given weight 0)
  auto accumulate = [&](int row, const uint4& vv) {
    const bool ok = row < r1;
    const int rc = ok ? row : r1 - 1;
    float pj[G];
    if constexpr (RS == 4 && G == 4) {
      const f32x4_t w = *reinterpret_cast<const f32x4_t*>(pbuf + (size_t)(rc - p0) * RS);
#pragma unroll
      for (int j = 0; j < G; ++j) pj[j] = ok ? w[j] : 0.0f;
    } else {
#pragma unroll
      for (int j = 0; j < G; ++j) {
        const float w = pbuf[(size_t)(rc - p0) * RS + j];
        pj[j] = ok ? w : 0.0f;
      }
    }
    float vf[8];
    unpack_slice<1>(vv, vf);
#pragma unroll
    for (int j = 0; j < G; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e) o[j][e] = __builtin_fmaf(pj[j], vf[e], o[j][e]);
  };
  const int nrows = r1 - r0;
  const int iters = (nrows + NG - 1) / NG;      // row slots per group (uniform)
  // Two halves of PF/2 rows per group in flight.  The loads are unconditional
  // (past the end they re-read the last row), and the scheduling barrier keeps
  // each half's refill between the halves, so while one half is consumed the
  // other half's loads are still outstanding; the last iters % PF rows are
  // consumed after the loop without new loads.
  constexpr int HF = PF / 2;
  const int full = iters / PF;
  for (int f = 0; f < full; ++f) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int q = 0; q < HF; ++q) accumulate(r0 + grp + (f * PF + h * HF + q) * NG, vb[h * HF + q]);
#pragma unroll
      for (int q = 0; q < HF; ++q) vb[h * HF + q] = vr.load(r0 + grp + ((f + 1) * PF + h * HF + q) * NG, r1, lam);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int p = 0; p < PF; ++p)
    if (full * PF + p < iters) accumulate(r0 + grp + (full * PF + p) * NG, vb[p]);
#pragma unroll
  for (int j = 0; j < G; ++j)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float x = o[j][e];
      if constexpr (!FAST) {
#pragma unroll
        for (int off = LPR; off < 64; off *= 2) x = x + __shfl_xor(x, off);
        o[j][e] = x;
        continue;
      }
      if constexpr (LPR == 8) x += dpp<0x128>(x);      // lane ^ 8: the row rotated by eight
      x = add_xor16(x);
      o[j][e] = add_xor32(x);
    }
}

// Norm of the appended value row (every thread receives it through LDS).
template <int D>
__device__ __forceinline__ float new_row_vnorm(const DecodeArgs& a, int u, float* slot) {
  constexpr int LPR = MG<D>::LPR;
  if (threadIdx.x < LPR) {
    float vf[8];
    unpack_slice<1>(ldg16((const char*)a.v_new + (size_t)u * D * 2 + threadIdx.x * 16), vf);
    float v2 = vf[0] * vf[0];
#pragma unroll
    for (int e = 1; e < 8; ++e) v2 = __builtin_fmaf(vf[e], vf[e], v2);
    v2 = row_sum<LPR>(v2);
    if (threadIdx.x == 0) *slot = __builtin_sqrtf(v2);
  }
  __syncthreads();
  return *slot;
}

// Feature state of one row.
struct RowState {
  float al, vn;
  double nu, de;
  int32_t p;
};
__device__ __forceinline__ void load_row_state(const DecodeArgs& a, size_t gi, RowState& x) {
  x.al = a.alpha[gi];
  x.nu = a.num[gi];
  x.de = a.den[gi];
  x.p = a.pos[gi];
  x.vn = a.vnorm[gi];
}

// Feature update of one row from its weights: x in, the updated state in x and in
// memory.
template <int G>
__device__ __forceinline__ void update_row(const DecodeArgs& a, size_t gi, bool is_new,
                                           const float (&pj)[G], const float (&invl)[G],
                                           const float (&H)[G], float2 ret, float newnorm,
                                           RowState& x) {
  constexpr float invG = 1.0f / G;
  float w[G];
#pragma unroll
  for (int j = 0; j < G; ++j) w[j] = pj[j] * invl[j];
  float cz, cn;
  contrib_from_weights<G>(w, H, cz, cn);
  if (is_new) {
    x = {cz * invG, newnorm, (double)cn, (double)cz, a.T - 1};
    a.pos[gi] = x.p;
    a.vnorm[gi] = x.vn;
  } else {
    x.al = (a.arec ? 0.0f : x.al) + cz * invG;
    x.de = x.de + (double)cz;
    x.nu = x.nu + (double)cn;
    if (a.retire && x.p <= a.pmax_ret) {
      x.de = x.de - (double)ret.x;
      x.nu = x.nu - (double)ret.y;
    }
  }
  a.alpha[gi] = x.al;
  a.den[gi] = x.de;
  a.num[gi] = x.nu;
  if (a.sigma) a.sigma[gi] = head_variance<G>(w);
}

template <int D, int G>
__device__ __forceinline__ void write_ring2(const DecodeArgs& a, int u, const float (&M)[G],
                                            const float (&invl)[G], const float (&H)[G]) {
  constexpr int N16 = G * D * 2 / 16;
  const int t = threadIdx.x;
  const size_t rs = (size_t)u * a.window + a.slot;
  if (t < N16) {
    const char* src = (const char*)a.q + (size_t)u * G * D * 2;
    char* dst = (char*)a.qring + rs * G * D * 2;
    *reinterpret_cast<uint4*>(dst + t * 16) = ldg16(src + t * 16);
  }
  if (t < G) {
#pragma unroll
    for (int j = 0; j < G; ++j)
      if (j == t) {
        a.qstat[(rs * G + j) * 3 + 0] = M[j];
        a.qstat[(rs * G + j) * 3 + 1] = invl[j];
        a.qstat[(rs * G + j) * 3 + 2] = H[j];
      }
  }
}

template <int D>
__device__ __forceinline__ void append_rows(const DecodeArgs& a, int u) {
  constexpr int N16 = D * 2 / 16;
  const int t = threadIdx.x;
  if (t < 2 * N16) {
    const bool isv = t >= N16;
    const int c = isv ? t - N16 : t;
    const char* src = (const char*)(isv ? a.v_new : a.k_new) + (size_t)u * D * 2;
    char* dst = (char*)(isv ? a.v : a.k) + ((size_t)u * a.cap + len_old_of(a, u)) * D * 2;
    *reinterpret_cast<uint4*>(dst + c * 16) = ldg16(src + c * 16);
  }
}

// ---------------------------------------------------------------- unit kernel
// One workgroup per unit, sized so that two fit on a CU (one computes while the
// other streams).  Dynamic LDS: [L * RS floats: logits -> weights -> u64 keys]
// [SNW/2 * G * D output partials][2 ints per compaction move]; the retired
// contributions (cz, cn) of pass A stay in registers (lane l holds those of
// row l of each of its wave's 64-row groups) until the feature pass.
template <int G>
struct RowStride {
  static constexpr int RS = G < 2 ? 2 : G;     // floats per row in LDS (a u64 key must fit)
  static constexpr int KS = RS / 2;            // u64 per row
};

// SMP: training-mode ranking by the Gumbel-perturbed score; the unperturbed
// score is kept in the row's LDS slot beside its key (needs RS >= 4, G >= 4).
// RAG: ragged cache with per-unit budgets (e.budgets).  Unit u has its own rows
// (unit_len[u] + the append) and budget; a.L bounds the rows a workgroup serves
// (it sizes the LDS), and a unit with more rows leaves at once (the chunked
// kernels serve it).  The compaction plan sits in the free half of the rows'
// LDS slots beside the keys (move j beside row j's key: at most L / 2 moves,
// however many rows the unit evicts), so it needs RS >= 4 (G >= 4).
// EARLY: value rows are requested ahead of pass P, the state ahead of the output
// combination, and the sums stay out of the LDS pipe, since a step waits for its
// own chain of passes.  Measured per step, off -> on: 2304 units of 187 rows 81.1 ->
// 73.0 us, 2048 of 513 139.4 -> 131.9 (G = 8: 232.8 -> 215.0), 2048 of 1025 236.4 ->
// 232.8, 1024 of 2049 224.7 -> 223.0, of 3342 368.1 -> 367.9, 256 of 1025 37.5 -> 35.4,
// 8 of 1025 28.2 -> 27.4; G = 8: 1024 of 2049 295 -> 284.  Where just two workgroups per CU cover each other's
// waits, and on long rows, it costs instead: 512 of 1025 60.0 -> 60.7 us, 4096 of
// 4097 1701 -> 1712.  The bits are the same.
template <int D, int G, bool FEAT, bool EVICT, bool SIG, bool SMP, bool RAG, bool EARLY>
__device__ __forceinline__ void step_unit_body(const DecodeArgs& a, const EvictArgs& e, const int u,
                                               float* lds) {
  static_assert(!SIG || (FEAT && !EVICT), "sigma is stored by the decode-only variant");
  static_assert(!SMP || (EVICT && RowStride<G>::RS >= 4), "sampling keeps the score beside the key");
  static_assert(!RAG || (FEAT && EVICT && !SIG && !SMP && RowStride<G>::RS >= 4),
                "the ragged variant plans its moves beside the keys");
  constexpr int LPR = MG<D>::LPR;
  constexpr int RS = RowStride<G>::RS, KS = RowStride<G>::KS;
  __shared__ SelShared sh;
  __shared__ float stat[SNW * 2 * G + 2 * G];
  __shared__ float newnorm_slot;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int L = RAG ? len_old_of(a, u) + a.append : a.L;
  if constexpr (RAG) {
    if (L > a.L || L < 1) return;                     // whole workgroup: the chunked kernels' unit
  }
  float* sbuf = lds;                                  // row stride RS
  float* obuf = lds + (size_t)L * RS;                 // (SNW / 2) * G * D
  int* mv = (int*)(obuf + (SNW / 2) * G * D);
  const size_t ub = (size_t)u * a.cap;

  if (a.append) append_rows<D>(a, u);
  const bool retire = FEAT && a.retire;
  float M[G], invl[G], H[G];
  float zr[S_GMAX], nr[S_GMAX];     // retired pairs of the wave's 64-row groups (lane = row)
  {
    uint4 qa[MG<D>::NT];
    load_qfrag<D, G>(qa, a, u, retire);
    RetStats<G> rs;
    if (retire) load_ret<G>(rs, a, u);
    float mrun[4];
    pass_a<D, G, FEAT, true, RS>(a, u, 0, L, sbuf, nullptr, 0, qa, retire, rs, mrun, zr, nr);
    block_max<G>(mrun, stat, M);
  }
  uint4 vb[PF];
  if constexpr (EARLY) pass_b_first<D>(a, u, 0, L, vb);
  {
    float ls[G], us[G];
    pass_p<G, RS>(sbuf, L, M, ls, us);
    __syncthreads();
    block_sum2<G, EARLY>(ls, us, stat);
#pragma unroll
    for (int j = 0; j < G; ++j) {
      invl[j] = 1.0f / ls[j];
      H[j] = __logf(ls[j]) - us[j] * invl[j];
    }
  }
  // the feature state of pass A's 64-row groups (see the feature pass); the
  // first group's is requested before the outputs are combined
  const int ngrp = (L + 63) / 64;
  const int ngw = wave < ngrp ? (ngrp - 1 - wave) / SNW + 1 : 0;
  auto load_row = [&](int k, RowState& x) {
    const int r = 64 * (wave + SNW * k) + lane;
    load_row_state(a, ub + (r < L ? r : L - 1), x);
  };
  RowState cur = {};
  {
    float o[G][8];
    if constexpr (!EARLY) pass_b_first<D>(a, u, 0, L, vb);
    pass_b<D, G, EARLY, RS>(a, u, 0, L, sbuf, 0, vb, o);
    if (FEAT && EARLY && ngw > 0) load_row(0, cur);
    // tree over the waves through SNW/2 partial slots
    if (wave >= SNW / 2 && lane < LPR) {
#pragma unroll
      for (int j = 0; j < G; ++j)
#pragma unroll
        for (int x = 0; x < 8; ++x) obuf[((wave - SNW / 2) * G + j) * D + lane * 8 + x] = o[j][x];
    }
    __syncthreads();
    if (wave < SNW / 2 && lane < LPR) {
#pragma unroll
      for (int j = 0; j < G; ++j)
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          float* slot = &obuf[(wave * G + j) * D + lane * 8 + x];
          *slot = o[j][x] + *slot;
        }
    }
  }
  __syncthreads();
  for (int t = tid; t < G * D; t += SNT) {
    const int j = t / D;
    float acc = obuf[t];
    for (int w = 1; w < SNW / 2; ++w) acc = acc + obuf[w * G * D + t];
    float il = invl[0];
#pragma unroll
    for (int jj = 1; jj < G; ++jj) il = (jj == j) ? invl[jj] : il;
    ((uint16_t*)a.out)[(size_t)u * G * D + t] = (uint16_t)f32_to_bf16_bits(acc * il);
  }
  if constexpr (FEAT) {
    const float newnorm = a.append ? new_row_vnorm<D>(a, u, &newnorm_slot) : 0.0f;
    const int newrow = a.append ? len_old_of(a, u) : -1;
    const float invT = 1.0f / (float)a.T;
    constexpr float invG = 1.0f / G;
    uint64_t* keys = reinterpret_cast<uint64_t*>(sbuf);   // row i's key replaces its weights
    // The rows of pass A's 64-row groups, one per lane: group b (wave b mod SNW)
    // row 64 b + lane, whose retired pair this lane kept in registers.  The next
    // group's state is requested before the current one is updated; in full
    // groups every load and store is unconditional, only the unit's partial last
    // group (one wave) guards its stores.
    const bool part = ngw > 0 && wave + SNW * (ngw - 1) == ngrp - 1 && (L & 63) != 0;
    const int nfull = ngw - (part ? 1 : 0);
    auto update = [&](int k, const RowState& x, bool guard) {
      const int r = 64 * (wave + SNW * k) + lane;
      const bool valid = r < L;
      const int ic = valid ? r : L - 1;
      const size_t gi = ub + ic;
      float w[G];
#pragma unroll
      for (int j = 0; j < G; ++j) w[j] = sbuf[ic * RS + j] * invl[j];
      float cz, cn;
      contrib_from_weights<G>(w, H, cz, cn);
      float rz = zr[0], rn = nr[0];
#pragma unroll
      for (int s2 = 1; s2 < S_GMAX; ++s2) {
        rz = s2 == k ? zr[s2] : rz;
        rn = s2 == k ? nr[s2] : rn;
      }
      float al = (a.arec ? 0.0f : x.al) + cz * invG;
      double de = x.de + (double)cz;
      double nu = x.nu + (double)cn;
      int32_t ps = x.p;
      float vn = x.vn;
      if (retire && ps <= a.pmax_ret) {
        de = de - (double)rz;
        nu = nu - (double)rn;
      }
      if (ic == newrow) {
        al = cz * invG;
        de = (double)cz;
        nu = (double)cn;
        ps = a.T - 1;
        vn = newnorm;
      }
      if (!guard || valid) {
        a.alpha[gi] = al;
        a.den[gi] = de;
        a.num[gi] = nu;
        if constexpr (SIG) a.sigma[gi] = head_variance<G>(w);
      }
      if constexpr (EVICT) {
        float f[1][4], sc[1];
        make_features(al, vn, nu, de, ps, invT, f[0]);
        policy_scores<1>(e, f, sc, 1);
        if constexpr (SMP) {
          const float ks = sampled_score(e, sc[0], ps, u);
          if (!guard || valid) {
            keys[(size_t)r * KS] = row_key(ks, ps);
            sbuf[(size_t)r * RS + 2] = sc[0];
          }
        } else {
          if (!guard || valid) keys[(size_t)r * KS] = row_key(sc[0], ps);
        }
      }
    };
    if (ngw > 0) {
      RowState nxt;
      if constexpr (!EARLY) load_row(0, cur);
      for (int k = 0; k < nfull; ++k) {
        load_row(k + 1 < ngw ? k + 1 : k, nxt);
        update(k, cur, false);
        cur = nxt;
      }
      if (part) update(nfull, cur, true);
    }
    // the appended row's position and value norm (the other rows keep theirs)
    if (a.append && tid == 0) {
      a.pos[ub + newrow] = a.T - 1;
      a.vnorm[ub + newrow] = newnorm;
    }
    if (a.window > 0) write_ring2<D, G>(a, u, M, invl, H);
    if constexpr (EVICT) {
      __syncthreads();
      // row stride of scores_out: the unit's rows, or the bound of a ragged cache
      const size_t lso = RAG ? (size_t)e.L : (size_t)L;
      if (e.scores_out) {
        // the scores: beside the keys when sampling, else recovered from the
        // ranking keys (-0 reads back as +0)
        for (int r = tid; r < L; r += SNT) {
          if constexpr (SMP) {
            e.scores_out[(size_t)u * lso + r] = sbuf[(size_t)r * RS + 2];
          } else {
            const uint32_t k = (uint32_t)(keys[(size_t)r * KS] >> 32);
            const uint32_t bits = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
            e.scores_out[(size_t)u * lso + r] = __uint_as_float(bits);
          }
        }
      }
      const int nslots = (L + SNT - 1) / SNT;
      LdsKeys<S_KMAX, SNT> lk{keys, KS};
      if constexpr (RAG) {
        const int Bu = unit_budget(e, u);
        if (Bu < L) {
          select_compact<LdsKeys<S_KMAX, SNT>, 1, D, SNT, RS>(e, u, L, Bu, lk, nslots, sh,
                                                             reinterpret_cast<int*>(sbuf) + 2);
          if (e.kept_out)     // slots past this unit's budget
            for (int r = Bu + tid; r < e.ld_kept; r += SNT) e.kept_out[(size_t)u * e.ld_kept + r] = -1;
        } else if (e.kept_out) {
          for (int r = tid; r < e.ld_kept; r += SNT) e.kept_out[(size_t)u * e.ld_kept + r] = r < L ? r : -1;
        }
      } else if (e.evict) {
        select_compact<LdsKeys<S_KMAX, SNT>, 1, D, SNT>(e, u, L, e.budget, lk, nslots, sh, mv);
      } else if (e.kept_out) {
        for (int r = tid; r < L; r += SNT) e.kept_out[(size_t)u * L + r] = r;
      }
    }
  }
}

template <int D, int G, bool FEAT, bool EVICT, bool SIG, bool SMP, bool RAG, bool EARLY>
__global__ void __launch_bounds__(SNT, G > 4 ? 2 : 4) step_unit_kernel(DecodeArgs a, EvictArgs e) {
  extern __shared__ float lds[];
  step_unit_body<D, G, FEAT, EVICT, SIG, SMP, RAG, EARLY>(a, e, blockIdx.x, lds);
}

// ---------------------------------------------------------------- chunked path
// ws_part per (unit, chunk): [G] chunk max m_c, [G] l_c, [G] u_c, [G*D] o_c, the
// sums taken relative to the chunk's own maximum (stepc_d rescales them).
// Passes A, P and B of one chunk in one workgroup: K streamed once (logits and
// retired pairs to the workspace), p = exp(s - m_c) against the chunk maximum,
// then V streamed once.  The chunk's logits come back from the workspace
// while still in L2 (this workgroup stored them moments before).  RET: the
// step retires a step leaving the window; without one no retired pair is
// stored (the feature pass reads them only when the step retires).
template <int D, int G>
struct ChunkLds {                         // floats of LDS of one chunk's workgroup
  float p[SCHUNK * G], o[SNW * G * D], stat[SNW * 2 * G + 2 * G];
};

template <int D, int G, bool FEAT, bool RET>
__device__ __forceinline__ void stepc_ab_body(const DecodeArgs& a, const int c, const int u,
                                              ChunkLds<D, G>& sm) {
  constexpr int LPR = MG<D>::LPR;
  float* pbuf = sm.p;
  float* obuf = sm.o;
  float* stat = sm.stat;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int Lu = len_old_of(a, u) + a.append;       // this unit's rows (ragged caches: per unit)
  if (Lu <= a.fused_rows) return;                   // served by the single-launch kernel
  const int r0 = c * a.chunk, r1 = min(Lu, r0 + a.chunk), n = r1 - r0;
  if (c == 0 && a.append) append_rows<D>(a, u);
  float* part = a.ws_part + ((size_t)u * a.nchunks + c) * (3 * G + G * D);
  if (n <= 0) {
    // a chunk past this unit's rows: neutral partials (max -inf, sums 0, no output)
    for (int t = tid; t < 3 * G + G * D; t += SNT) part[t] = t < G ? NEG_BIG : 0.0f;
    return;
  }
  constexpr bool FR = FEAT && RET;
  const bool retire = FR && a.retire;
  uint4 qa[MG<D>::NT];
  load_qfrag<D, G>(qa, a, u, retire);
  RetStats<G> rs;
  if (retire) load_ret<G>(rs, a, u);
  float mrun[4];
  float zr[S_GMAX], nr[S_GMAX];   // unused on this path
  pass_a<D, G, FR, false>(a, u, r0, r1, a.ws_s + (size_t)u * a.lmax * G,
                          FR ? a.ws_r + (size_t)u * a.lmax * 2 : nullptr, 0, qa, retire, rs,
                          mrun, zr, nr);
  float M[G];
  block_max<G>(mrun, stat, M);    // (its barriers also order the logit stores before the reads)
  const float* src = a.ws_s + ((size_t)u * a.lmax + r0) * G;
  for (int t = tid; t < n * G; t += SNT) pbuf[t] = src[t];
  __syncthreads();
  uint4 vb[PF];
  pass_b_first<D>(a, u, r0, r1, vb);
  float ls[G], us[G];
  pass_p<G>(pbuf, n, M, ls, us);
  __syncthreads();
  block_sum2<G, true>(ls, us, stat);
  float o[G][8];
  pass_b<D, G, true>(a, u, r0, r1, pbuf, r0, vb, o);
  if (lane < LPR) {
#pragma unroll
    for (int j = 0; j < G; ++j)
#pragma unroll
      for (int x = 0; x < 8; ++x) obuf[(wave * G + j) * D + lane * 8 + x] = o[j][x];
  }
  __syncthreads();
  for (int t = tid; t < G * D; t += SNT) {
    float acc = 0.0f;
    for (int w = 0; w < SNW; ++w) acc = acc + obuf[w * G * D + t];
    part[3 * G + t] = acc;
  }
  if (tid < G) {
#pragma unroll
    for (int j = 0; j < G; ++j)
      if (j == tid) {
        part[j] = M[j];
        part[G + j] = ls[j];
        part[2 * G + j] = us[j];
      }
  }
}

template <int D, int G, bool FEAT, bool RET>
__global__ void __launch_bounds__(SNT) stepc_ab_kernel(DecodeArgs a) {
  __shared__ ChunkLds<D, G> sm;
  stepc_ab_body<D, G, FEAT, RET>(a, blockIdx.x, a.y0 + blockIdx.y, sm);
}

// A ragged step's two decode kernels in one launch: workgroups 0 .. units - 1 take
// the units that fit on chip (step_unit_body, RAG), the others the longer units'
// chunks.  The first kind alone leaves half the chip idle in its last round (768
// units on 512 places), which the chunks fill.  Measured (one launch after the other
// -> here): 768 units of 4097 rows and 256 of 16385 840 -> 815 us; the step of 96 units
// of 4001 and 32 of 16001 rows 247 -> 210, of 512 of 501 and 512 of 5001 431 -> 392.
template <int D, int G, bool RET, bool EARLY>
__global__ void __launch_bounds__(SNT, 4) step_mixed_kernel(DecodeArgs a, EvictArgs e, DecodeArgs ac) {
  extern __shared__ float lds[];
  if ((int)blockIdx.x < a.units) {
    step_unit_body<D, G, true, true, false, false, true, EARLY>(a, e, blockIdx.x, lds);
  } else {
    const int b = blockIdx.x - a.units;
    stepc_ab_body<D, G, true, RET>(ac, b % ac.nchunks, b / ac.nchunks,
                                   *reinterpret_cast<ChunkLds<D, G>*>(lds));
  }
}

// SCORE: the one-hidden-layer policy and the ranking key of every row are formed
// where its features are, so the selection that follows needs no scoring pass over
// the state (28 B a row).  A row's key takes the place of its retired pair, which
// only this thread reads (8 B a row at row stride lmax).  Rows are requested before
// the chunks' sums are combined, one thread per head combines (not every thread
// all heads).  FEW: all of a thread's rows at once, sharing the policy's weights, for
// grids of at most three workgroups a CU; a larger one takes a row at a time in half
// the registers (G = 4: 51 for 91), where the waves in flight hide the loads: 1024
// units of 16001 rows that keep every row 315 -> 265 us (G = 8 416 -> 365), steps of
// 104-127 units of 8193 rows 2-5 % less; the 480 workgroups of a scoring step of 40
// units take 4 % longer by it, so they stay with the first.  Measured per step
// (decode, scores, selection), with a scoring pass of its own -> here: 8 units of
// 4097 rows 46.7 -> 30.1 us, of 12001 60.1 -> 42.6, 64 of 4097 67.8 -> 54.5; this
// kernel and the scoring pass on 1024 units of 16385 rows 395 -> 299 us.
template <int D, int G, bool FEAT, bool SCORE, bool FEW>
__global__ void __launch_bounds__(SNT, FEW || !FEAT ? 1 : G > 4 ? 6 : 8) stepc_d_kernel(DecodeArgs a, EvictArgs e) {
  static_assert(FEAT || !SCORE, "scores need the features");
  __shared__ float newnorm_slot;
  __shared__ float comb[3][G];          // M, 1 / l, H
  const int c = blockIdx.x, u = a.y0 + blockIdx.y, tid = threadIdx.x;
  const int Lu = len_old_of(a, u) + a.append;
  if (Lu <= a.fused_rows) return;                   // served by the single-launch kernel
  const int r0 = c * a.chunk, r1 = min(Lu, r0 + a.chunk);
  const int PART = 3 * G + G * D;
  const float* parts = a.ws_part + (size_t)u * a.nchunks * PART;
  const int newrow = a.append ? len_old_of(a, u) : -1;
  const size_t ub = (size_t)u * a.cap;
  const float* s_src = FEAT ? a.ws_s + (size_t)u * a.lmax * G : nullptr;
  float* r_src = FEAT ? a.ws_r + (size_t)u * a.lmax * 2 : nullptr;
  // this thread's rows i0 + tid + k SNT, RB at a time (rows past r1 re-read the
  // last one, unused); the first are requested before the chunks' sums are combined
  constexpr int RB = FEW ? SCHUNK / SNT : 1;
  RowState x[RB];
  float sj[RB][G];
  float2 ret[RB] = {};
  auto request = [&](int i0) {
#pragma unroll
    for (int k = 0; k < RB; ++k) {
      const int i = i0 + tid + k * SNT, ic = i < r1 ? i : r1 - 1;
      load_row_state(a, ub + ic, x[k]);
      if constexpr (G >= 4) {
#pragma unroll
        for (int j = 0; j < G; j += 4) {
          const f32x4_t v = *reinterpret_cast<const f32x4_t*>(s_src + (size_t)ic * G + j);
#pragma unroll
          for (int r = 0; r < 4; ++r) sj[k][j + r] = v[r];
        }
      } else {
#pragma unroll
        for (int j = 0; j < G; ++j) sj[k][j] = s_src[(size_t)ic * G + j];
      }
      if (a.retire) ret[k] = *reinterpret_cast<const float2*>(r_src + 2 * (size_t)ic);
    }
  };
  if (FEAT && r0 < r1) request(r0);
  // chunk c's sums move to the common maximum M: with f = e^(m_c - M),
  // l += f l_c, u += f (u_c + (m_c - M) l_c), o += f o_c (a neutral chunk: f = 0);
  // one thread per head, the chunks in order
  if (tid < G) {
    float m = parts[tid];
#pragma unroll 4
    for (int cc = 1; cc < a.nchunks; ++cc) m = fmaxf(m, parts[(size_t)cc * PART + tid]);
    float il, h;
    if (a.comb64) {
      // short chunks: where one row takes nearly all the weight, l is 1 plus little
      // and the entropy lives in the little, which many float32 additions would eat
      double l = 0.0, uu = 0.0;
#pragma unroll 4
      for (int cc = 0; cc < a.nchunks; ++cc) {
        const float* pc = parts + (size_t)cc * PART + tid;
        const float dm = pc[0] - m;
        const double f = (double)__builtin_amdgcn_exp2f(dm * LOG2E);
        l += f * (double)pc[G];
        uu += f * ((double)pc[2 * G] + (double)dm * (double)pc[G]);
      }
      il = (float)(1.0 / l);
      h = (float)(log(l) - uu / l);
    } else {
      float l = 0.0f, uu = 0.0f;
#pragma unroll 4
      for (int cc = 0; cc < a.nchunks; ++cc) {
        const float* pc = parts + (size_t)cc * PART + tid;
        const float dm = pc[0] - m;
        const float f = __builtin_amdgcn_exp2f(dm * LOG2E);
        l = l + f * pc[G];
        uu = uu + f * (pc[2 * G] + dm * pc[G]);
      }
      il = 1.0f / l;
      h = __logf(l) - uu * il;
    }
    comb[0][tid] = m;
    comb[1][tid] = il;
    comb[2][tid] = h;
  }
  const float newnorm = FEAT && a.append && newrow >= r0 && newrow < r1
                            ? new_row_vnorm<D>(a, u, &newnorm_slot) : 0.0f;
  __syncthreads();
  float M[G], invl[G], H[G];
#pragma unroll
  for (int j = 0; j < G; ++j) {
    M[j] = comb[0][j];
    invl[j] = comb[1][j];
    H[j] = comb[2][j];
  }
  if constexpr (FEAT) {
    auto update = [&](int i0) {
#pragma unroll
      for (int k = 0; k < RB; ++k) {
        const int i = i0 + tid + k * SNT;
        if (i >= r1) continue;
        float pj[G];
#pragma unroll
        for (int j = 0; j < G; ++j) pj[j] = __builtin_amdgcn_exp2f((sj[k][j] - M[j]) * LOG2E);
        update_row<G>(a, ub + i, i == newrow, pj, invl, H, ret[k], newnorm, x[k]);
      }
    };
    auto score = [&](int i0) {            // (past the last row of a chunk the state is that of its last row)
      const float invT = 1.0f / (float)a.T;
      float f[RB][4], sc[RB];
#pragma unroll
      for (int k = 0; k < RB; ++k) make_features(x[k].al, x[k].vn, x[k].nu, x[k].de, x[k].p, invT, f[k]);
      policy_scores<RB>(e, f, sc, (r1 - i0 + SNT - 1) / SNT);
#pragma unroll
      for (int k = 0; k < RB; ++k) {
        const int i = i0 + tid + k * SNT;
        if (i >= r1) continue;
        if (e.scores_out) e.scores_out[(size_t)u * e.L + i] = sc[k];
        reinterpret_cast<uint64_t*>(r_src)[i] =
            row_key(e.sample ? sampled_score(e, sc[k], x[k].p, u) : sc[k], x[k].p);
      }
    };
    // (a unit that keeps every row needs no key)
    const bool scored = SCORE && (e.scores_out || unit_budget(e, u) < Lu);
    if constexpr (FEW) {                  // one batch is a chunk
      update(r0);
      if constexpr (SCORE)
        if (r0 < r1 && scored) score(r0);
    } else {
#pragma unroll 1
      for (int i0 = r0; i0 < r1; i0 += SNT) {
        if (i0 > r0) request(i0);
        update(i0);
        if constexpr (SCORE)
          if (scored) score(i0);
      }
    }
  }
  if (c != 0) return;
  for (int t = tid; t < G * D; t += SNT) {
    const int j = t / D;
    float mj = M[0];
#pragma unroll
    for (int jj = 1; jj < G; ++jj) mj = (jj == j) ? M[jj] : mj;
    float acc = 0.0f;
    for (int cc = 0; cc < a.nchunks; ++cc) {
      const float* pc = parts + (size_t)cc * PART;
      acc = acc + __builtin_amdgcn_exp2f((pc[j] - mj) * LOG2E) * pc[3 * G + t];
    }
    float il = invl[0];
#pragma unroll
    for (int jj = 1; jj < G; ++jj) il = (jj == j) ? invl[jj] : il;
    ((uint16_t*)a.out)[(size_t)u * G * D + t] = (uint16_t)f32_to_bf16_bits(acc * il);
  }
  if (FEAT && a.window > 0) write_ring2<D, G>(a, u, M, invl, H);
}

// ---------------------------------------------------------------- ragged caches
__global__ void unit_len_add_kernel(int32_t* len, int units, int add) {
  const int u = blockIdx.x * 256 + threadIdx.x;
  if (u < units) len[u] += add;
}

__global__ void unit_len_min_kernel(int32_t* len, const int32_t* budgets, int b, int add, int units) {
  const int u = blockIdx.x * 256 + threadIdx.x;
  if (u < units) {
    int bu = budgets ? budgets[u] : b;
    bu = bu < 1 ? 1 : bu > b ? b : bu;            // the clamp the selection applies
    const int n = len[u] + add;
    len[u] = bu < n ? bu : n;
  }
}

int launch_unit_len_add(int32_t* len, int units, int add, void* stream) {
  hipLaunchKernelGGL(unit_len_add_kernel, dim3((units + 255) / 256), dim3(256), 0,
                     (hipStream_t)stream, len, units, add);
  return (int)hipGetLastError();
}

int launch_unit_len_min(int32_t* len, const int32_t* budgets, int b, int add, int units, void* stream) {
  hipLaunchKernelGGL(unit_len_min_kernel, dim3((units + 255) / 256), dim3(256), 0,
                     (hipStream_t)stream, len, budgets, b, add, units);
  return (int)hipGetLastError();
}

// ---------------------------------------------------------------- dispatch
// ints of the compaction move list (a multiple of four, so what follows it in
// LDS stays 16-byte aligned)
static int move_list_ints(int nmoves) { return (2 * (nmoves > 0 ? nmoves : 1) + 3) / 4 * 4; }

size_t step_lds_bytes(int L, int G, int D, bool feat, int nmoves) {
  const size_t rs = G < 2 ? 2 : G;
  const size_t b = ((size_t)L * rs + (size_t)(SNW / 2) * G * D) * sizeof(float);
  return b + (size_t)move_list_ints(nmoves) * sizeof(int);
}

bool step_fits(int L, int G, int D, bool feat, int nmoves) {
  return (!feat || L <= S_KMAX * SNT) && step_lds_bytes(L, G, D, feat, nmoves) <= (size_t)S_LDS;
}

int step_chunk_rows() { return SCHUNK; }

int step_ragged_rows(int G, int D) {
  if (G < 4) return 0;                            // keys fill the row slots: no room for the plan
  // two workgroups per CU: half the dynamic LDS budget; rows in registers: S_KMAX per thread
  int L = S_KMAX * SNT;
  while (L > 0 && step_lds_bytes(L, G, D, true, 0) > (size_t)S_LDS / 2) --L;
  return L;
}

// One workgroup per CU at most (G > 4: its registers allow no second), or more rounds
// than one of not too long rows.  Measured on / off, 17 unit counts by nine lengths by
// five shapes: up to 256 units 0.82-1.00 everywhere; G = 8 0.83-0.98 everywhere; over
// 512 units 0.77-0.99 to 2049 rows, 0.94-1.01 at 3001, 0.95-1.005 from 3585; 257-512
// units with rows of 128 elements 0.97-1.00 at 129 rows, 0.98-1.05 from 257 to 1025, then
// 0.98-1.00 (with rows of 64 0.85-1.00).
static bool step_early(const DecodeArgs& a, int G, int D) {
  if (G > 4 || a.units <= 256) return true;
  return a.units > 512 ? a.L <= 3584 : a.L <= (D > 64 ? 192 : 512);
}

template <int D, int G>
static int launch_step_t(const DecodeArgs& a, const EvictArgs* e, bool feat, bool chunked,
                         hipStream_t s) {
  if (!chunked) {
    // (the ragged variant plans its moves beside the keys: no separate list)
    const int nm = e && e->evict && !a.unit_len ? (a.L - e->budget < e->budget ? a.L - e->budget : e->budget) : 0;
    EvictArgs ee;
    if (e) ee = *e;
    else __builtin_memset(&ee, 0, sizeof(ee));
    ee.mv_ints = move_list_ints(nm);
    const size_t lds = step_lds_bytes(a.L, G, D, feat, nm);
    auto pick = [&](auto kern) {
      allow_lds((const void*)kern, lds);
      hipLaunchKernelGGL(kern, dim3(a.units), dim3(SNT), lds, s, a, ee);
    };
    // (the fused evicting variants serve the one-hidden-layer four-input policy)
    const bool early = step_early(a, G, D);
#define DC_STEP(...) do { if (early) pick(step_unit_kernel<D, G, __VA_ARGS__, true>); else pick(step_unit_kernel<D, G, __VA_ARGS__, false>); } while (0)
    if (!feat) DC_STEP(false, false, false, false, false);
    else if (e && e->sample) {
      if constexpr (RowStride<G>::RS >= 4) DC_STEP(true, true, false, true, false);
      else return (int)hipErrorInvalidValue;     // the caller takes the separate path
    }
    else if (e && a.unit_len) {
      if constexpr (RowStride<G>::RS >= 4) DC_STEP(true, true, false, false, true);
      else return (int)hipErrorInvalidValue;     // the caller takes the separate path
    }
    else if (e) DC_STEP(true, true, false, false, false);
    else if (a.sigma) DC_STEP(true, false, true, false, false);
    else DC_STEP(true, false, false, false, false);
#undef DC_STEP
  } else {
    // every slice of one pass before the next (stream order)
    for_grid_y(a.units, [&](int y0, int ny) {
      DecodeArgs b = a;
      b.y0 = y0;
      if (feat && a.retire)
        hipLaunchKernelGGL((stepc_ab_kernel<D, G, true, true>), dim3(a.nchunks, ny), dim3(SNT), 0, s, b);
      else if (feat)
        hipLaunchKernelGGL((stepc_ab_kernel<D, G, true, false>), dim3(a.nchunks, ny), dim3(SNT), 0, s, b);
      else
        hipLaunchKernelGGL((stepc_ab_kernel<D, G, false, false>), dim3(a.nchunks, ny), dim3(SNT), 0, s, b);
    });
    for_grid_y(a.units, [&](int y0, int ny) {
      DecodeArgs b = a;
      b.y0 = y0;
      const EvictArgs none = {};
      const bool few = (long)a.units * a.nchunks <= 768;
      auto pick = [&](auto kern, const EvictArgs& ev) {
        hipLaunchKernelGGL(kern, dim3(a.nchunks, ny), dim3(SNT), 0, s, b, ev);
      };
      if (!feat) few ? pick(stepc_d_kernel<D, G, false, false, true>, none) : pick(stepc_d_kernel<D, G, false, false, false>, none);
      else if (e) few ? pick(stepc_d_kernel<D, G, true, true, true>, *e) : pick(stepc_d_kernel<D, G, true, true, false>, *e);
      else few ? pick(stepc_d_kernel<D, G, true, false, true>, none) : pick(stepc_d_kernel<D, G, true, false, false>, none);
    });
  }
  return (int)hipGetLastError();
}

// The two kinds of workgroup share a launch for the group size whose chunks need no
// more registers than the unit kernel (G = 8: 202 a thread).
bool step_mixed_fits(int units, int nchunks, int G) {
  return G == 4 && (long)units * (1 + nchunks) <= 1l << 30;
}

// The ragged step in one launch for the decode of all units, then the features and
// scores of the longer ones.
template <int D>
static int launch_step_mixed_t(const DecodeArgs& a, const EvictArgs& e, const DecodeArgs& ac,
                               const EvictArgs& el, hipStream_t s) {
  constexpr int G = 4;
  // (a.L is at most step_ragged_rows: half the LDS)
  static_assert(sizeof(ChunkLds<D, G>) <= (size_t)S_LDS / 2, "two workgroups of either kind per CU");
  size_t lds = step_lds_bytes(a.L, G, D, true, 0);
  lds = lds > sizeof(ChunkLds<D, G>) ? lds : sizeof(ChunkLds<D, G>);
  auto pick = [&](auto kern) {
    allow_lds((const void*)kern, lds);
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.units * (1 + ac.nchunks))), dim3(SNT), lds, s, a, e, ac);
  };
  const bool early = step_early(a, G, D);
  if (ac.retire) early ? pick(step_mixed_kernel<D, G, true, true>) : pick(step_mixed_kernel<D, G, true, false>);
  else early ? pick(step_mixed_kernel<D, G, false, true>) : pick(step_mixed_kernel<D, G, false, false>);
  for_grid_y(ac.units, [&](int y0, int ny) {
    DecodeArgs b = ac;
    b.y0 = y0;
    // (most chunks are those of units served above and leave at once)
    auto kern = (long)ac.units * ac.nchunks <= 2048 ? stepc_d_kernel<D, G, true, true, true>
                                                    : stepc_d_kernel<D, G, true, true, false>;
    hipLaunchKernelGGL(kern, dim3(ac.nchunks, ny), dim3(SNT), 0, s, b, el);
  });
  return (int)hipGetLastError();
}

int launch_step_mixed(const DecodeArgs& a, const EvictArgs& e, const DecodeArgs& ac, const EvictArgs& el,
                      int D, int G, void* stream) {
  if (!step_mixed_fits(a.units, ac.nchunks, G)) return (int)hipErrorInvalidValue;
  if (D == 128) return launch_step_mixed_t<128>(a, e, ac, el, (hipStream_t)stream);
  if (D == 64) return launch_step_mixed_t<64>(a, e, ac, el, (hipStream_t)stream);
  return (int)hipErrorInvalidValue;
}

template <int D>
static int launch_step_g(const DecodeArgs& a, const EvictArgs* e, int G, bool feat, bool chunked,
                         hipStream_t s) {
  switch (G) {
    case 1: return launch_step_t<D, 1>(a, e, feat, chunked, s);
    case 2: return launch_step_t<D, 2>(a, e, feat, chunked, s);
    case 4: return launch_step_t<D, 4>(a, e, feat, chunked, s);
    case 8: return launch_step_t<D, 8>(a, e, feat, chunked, s);
  }
  return (int)hipErrorInvalidValue;
}

int launch_step(const DecodeArgs& a, const EvictArgs* e, int D, int G, bool feat, bool chunked,
                void* stream) {
  hipStream_t s = (hipStream_t)stream;
  if (D == 128) return launch_step_g<128>(a, e, G, feat, chunked, s);
  if (D == 64) return launch_step_g<64>(a, e, G, feat, chunked, s);
  return (int)hipErrorInvalidValue;
}

}  // namespace dc

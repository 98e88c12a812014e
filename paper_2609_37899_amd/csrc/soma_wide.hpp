// soma_wide.hpp -- the body of the paper's wider fixed-size controls
// (SOMA_ARCH_WIDE; Appendix C, counting rules and Table
// fixed-parameter-counts; Appendix E): D pre-norm residual blocks (a
// bias-free LSTM and a GELU MLP of hidden width 4 d_t, gain-only LayerNorm)
// at width d_t, between an input projection P_in from the head width d_E and
// an output projection P_out back to it, decoded by the expert's own tied
// matrix E [256][d_E], which is never perturbed.
//
// Canonical parameter order of one expert (every matrix row a multiple of 4
// long, so that a probe quad lies in one row of one matrix):
//   P_in [d_t][d_E]; per block A, R, U, V [d_t][4 d_t] (LSTM input and
//   recurrent weights with columns j = g d_t + u for gates g = i, f, g, o;
//   MLP up weights; MLP down weights, row = output feature); P_out [d_t][d_E];
//   gains g1, g2 per block, then g_f (each d_t long).
//
// A pass of this body runs, for every slot (expert, direction, sign):
//   k_wide_form   perturbed weights, gains folded into the matrices that
//                 read a normalised vector, zero-padded to d_p = 64 ceil(d_t
//                 / 64), and each expert's E, in fragment order (once per
//                 pass)
//   k_mm          U = E P_in^T (the input projection per byte value)
//   k_wide_ln     x = U[byte], n = LN(x)   (the gain sits in the weights)
//   per block:    k_mm gin = n A'           (gate inputs, units interleaved)
//                 k_rec_xchg or k_rec_persist h   (recurrent weights pre-formed)
//                 k_wide_ln x += h, n = LN(x)
//                 k_mm m = GELU(n U')
//                 k_mm x += m V^T
//   k_wide_ln     n = LN(x)
//   k_mm          u = n P_out'^T (the final gain folded into P_out)
//   k_wide_head   logits = u E^T, cross entropy
// Padded units have zero weights and zero gate inputs, so their cell state
// and h stay exactly 0 and every padded column of x stays 0.
#pragma once

#include "soma_kernels.hpp"
#include "soma_body.hpp"
#include "soma_mm.hpp"

namespace soma {

constexpr int kWideHeadWidth = 32;   // d_E of the GPU path (the paper's head width)
constexpr int kWidePad = 64;         // d_p: d_t rounded up to a multiple of this

__host__ __device__ constexpr int wide_padded(int dt) { return (dt + kWidePad - 1) / kWidePad * kWidePad; }

// Floats of one slot's pre-formed weights and their offsets.
struct WideForm {
  int64_t pin, blk0, blk_stride, pout, total;   // blk_stride: one block's four matrices
};

__host__ __device__ inline WideForm wide_form_layout(int dp, int D) {
  WideForm f{};
  const int64_t m = 4 * int64_t(dp) * dp;
  // Every matrix is stored output-major, split and in fragment order (the
  // bytes of the fp32 matrix): the rows of the gate matrices are interleaved
  // (row 4 u + g is gate g of unit u).
  f.pin = 0;                                   // P_in   [d_p][32]
  f.blk0 = int64_t(dp) * kWideHeadWidth;       // per block: A' [4 d_p][d_p], R [4 d_p][d_p],
  f.blk_stride = 4 * m;                        //   U' [4 d_p][d_p], V [d_p][4 d_p]
  f.pout = f.blk0 + int64_t(D) * f.blk_stride; // P_out' [32][d_p]
  f.total = f.pout + int64_t(dp) * kWideHeadWidth;
  return f;
}

struct WideArgs {
  const float* theta;     // [N][d]
  const uint64_t* seeds;  // [N]
  const uint8_t* bytes;   // [A][N][B][T]
  const float* E;         // tied matrices, expert e at E + e * e_stride, [256][32]
  int64_t e_stride;
  float* wform;           // pre-formed weights, [slots][WideForm::total]
  float* esplit;          // E in fragment order, [N][256][32] split pairs
  float* U;               // [slots][256][d_p]
  float* x;               // [slots][R][d_p] residual stream
  float* n;               // [slots][ceil(R / 16) 16][d_p] normalised x in fragment order (also h of the recurrence, fp32)
  float* gin;             // [slots][R][4 d_p] gate inputs, then the MLP hidden layer
  double* part;           // [slots][row_tiles] cross-entropy sums
  float* fdec;            // evaluation: decoder inputs u [N][B][T-1][32] (position b (T-1) + t)
  float* lse;             // evaluation: log-sum-exps [N][B][T-1]
  int64_t d;              // parameters per expert
  uint64_t step;
  const float* eps_v;     // radius of expert e: eps_v[e * eps_stride]
  int eps_stride;
  unsigned* err;          // the step's sticky abort flag
  int probe;
  int ppb;                // directions per accumulation batch
  int64_t bstride;        // bytes per accumulation batch, N B T
  int N, D, dt, dp, B, T, PC, pcs, j0, NS;   // NS: signs per direction (2; 1 for an evaluation)
  int row_tiles;          // 64-row tiles of the head per slot
};

// Sum and max over the 64 lanes of a wave (butterfly; every lane gets the
// same value, each pair adding its two values in either order).
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}

// Orders a wave's LDS writes before its later LDS reads of other lanes'
// words (a wave's LDS accesses execute in order; this keeps the compiler
// from moving them).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Slot s of the pass: (expert, direction in the pass, sign).
__device__ __forceinline__ void wide_slot(const WideArgs& a, int s, int& e, int& jl, int& sg) {
  sg = s % a.NS;
  const int pj = s / a.NS;
  jl = pj % a.pcs;
  e = pj / a.pcs;
}

__device__ __forceinline__ int64_t wide_slot_index(const WideArgs& a, int e, int jl, int sg) {
  return (int64_t(e) * a.PC + jl) * a.NS + sg;
}

// The perturbed value of canonical coordinate k of expert e (one probe quad
// drawn for it): theta_k + seps z_k.
__device__ __forceinline__ float wide_coord(const float* th, int64_t k, int64_t gain0, int law, uint2 key,
                                            uint32_t pair, uint32_t step_lo, float seps) {
  if (seps == 0.0f) return th[k];
  const int lw = (k >= gain0 && law == kProbeSparseRademacher) ? kProbeRademacher : law;
  const float4 z = probe_quad(lw, key, pair, step_lo, static_cast<uint64_t>(k & ~int64_t(3)));
  const float zz[4] = {z.x, z.y, z.z, z.w};
  return __builtin_fmaf(seps, zz[k & 3], th[k]);
}

// ---------------------------------------------------------------------------
// Pre-formed weights of every slot, and E, in fragment order.  A thread forms 16-byte
// words, so that stores are words and not halves:
//  * matrices whose canonical rows run along K's other side (A, R, U [c][j] and
//    P_out [c][q]; K index c): eight rows c of one column quad, i.e. eight
//    probe quads, giving one hi and one lo word for each of its four columns
//    (blockIdx.y: matrix and group of eight rows);
//  * V [c][j] and P_in [c][q] (K index j, q): eight columns of one row, two
//    quads, one hi and one lo word.
// The gains are not stored: the matrices that read a normalised vector
// multiply by the perturbed gain of their K index (drawn once per block).
// Padded entries are zeroed beforehand (k_fill_f32) or written as zeros.  A
// formed weight outside the split products' range, or NaN, sets the step's
// abort flag.
// ---------------------------------------------------------------------------
constexpr int kFormThreads = 128;

// Row groups along c, and the rows of blockIdx.y: 3 D matrices (A, R, U of
// each block) and P_out by groups of eight c, then V and P_in by rows c, then
// the words of the experts' E.
__host__ __device__ inline int wide_form_groups(int dt) { return (dt + 7) / 8; }
__host__ __device__ inline int wide_form_rows(int dt, int D) {
  return (3 * D + 1) * wide_form_groups(dt) + (D + 1) * dt;
}
constexpr int kFormSplitRows = kVocab * 4 / kFormThreads;

// Each expert's tied matrix E [256][32] in fragment order (256 x 32 split
// pairs at esplit + expert * 8192): one word per thread.
__device__ __forceinline__ bool wide_split_word(const float* E, _Float16* esplit, int i) {
  constexpr int K = kWideHeadWidth;
  const int row = i >> 2, g = i & 3;                    // 4 words of hi a row
  const float* src = E + row * K + 8 * g;
  const float4 x = *reinterpret_cast<const float4*>(src), y = *reinterpret_cast<const float4*>(src + 4);
  uint4 hi, lo;
  split8v(x, y, hi, lo);
  _Float16* w = esplit + int64_t(row >> 4) * 2 * 512 + (16 * g + (row & 15)) * 8;
  *reinterpret_cast<uint4*>(w) = hi;
  *reinterpret_cast<uint4*>(w + 512) = lo;
  return split_range_ok(x) && split_range_ok(y);
}

template <bool kPert>
__global__ __launch_bounds__(kFormThreads) void k_wide_form(WideArgs a) {
  __shared__ float gains[8];
  const int dt = a.dt, dp = a.dp, D = a.D;
  const int64_t dt4 = 4 * int64_t(dt), mat = dt4 * dt;
  const int64_t blk0 = int64_t(dt) * kWideHeadWidth, pout0 = blk0 + D * 4 * mat;
  const int64_t gain0 = pout0 + int64_t(dt) * kWideHeadWidth;
  int e, jl, sg;
  wide_slot(a, blockIdx.z, e, jl, sg);
  const int64_t slot = wide_slot_index(a, e, jl, sg);
  const float* th = a.theta + int64_t(e) * a.d;
  const uint2 key = kPert ? stream_key(a.seeds[e], a.step) : make_uint2(0u, 0u);
  const uint32_t pair = static_cast<uint32_t>(a.j0 + jl), step_lo = static_cast<uint32_t>(a.step);
  const float eps = kPert ? a.eps_v[int64_t(e) * a.eps_stride] : 0.0f;
  const float seps = sg == 0 ? eps : -eps;
  // The perturbed canonical quad at k (a multiple of 4).
  auto quad = [&](int64_t k) {
    const float4 t = make_float4(th[k], th[k + 1], th[k + 2], th[k + 3]);
    return kPert ? fma4(seps, probe_quad(a.probe, key, pair, step_lo, static_cast<uint64_t>(k)), t) : t;
  };
  const WideForm F = wide_form_layout(dp, D);
  _Float16* out = reinterpret_cast<_Float16*>(a.wform + slot * F.total);
  bool ok = true;
  // Eight values k .. k + 7 of row `row` of the matrix at element offset base with K columns.
  auto put = [&](int64_t base, int row, int k, int K, const float4& x, const float4& y) {
    ok = ok && split_range_ok(x) && split_range_ok(y);
    uint4 hi, lo;
    split8v(x, y, hi, lo);
    _Float16* w = out + 2 * base + (int64_t(row >> 4) * 2 * (K / 32) + (k >> 5)) * 512 +
                  (16 * ((k >> 3) & 3) + (row & 15)) * 8;
    *reinterpret_cast<uint4*>(w) = hi;
    *reinterpret_cast<uint4*>(w + (K / 32) * 512) = lo;
  };
  const int groups = wide_form_groups(dt);
  const int i = blockIdx.x * kFormThreads + threadIdx.x;
  int y = blockIdx.y;
  if (y < (3 * D + 1) * groups) {                       // block-uniform
    const int mi = y / groups, c0 = 8 * (y % groups);
    const bool is_out = mi == 3 * D;
    const int l = mi / 3, which = is_out ? 0 : mi % 3;  // A, R, U
    const bool gained = is_out || which != 1;           // A reads LN(x; g1), U LN(x; g2), P_out LN(x; g_f)
    if (threadIdx.x < 8) {
      float g = 1.0f;
      const int64_t gk = gain0 + (is_out ? 2 * D : 2 * l + (which == 2 ? 1 : 0)) * int64_t(dt) + c0 + threadIdx.x;
      if (gained && c0 + static_cast<int>(threadIdx.x) < dt)
        g = wide_coord(th, gk, gain0, a.probe, key, pair, step_lo, seps);
      gains[threadIdx.x] = g;
    }
    __syncthreads();
    const int ncol = is_out ? kWideHeadWidth : 4 * dt;
    const int j = 4 * i;
    if (j < ncol) {
      const int64_t src = is_out ? pout0 : blk0 + l * 4 * mat + which * mat;
      float v[8][4];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        float4 w = make_float4(0.f, 0.f, 0.f, 0.f);
        if (c0 + r < dt) w = quad(src + int64_t(c0 + r) * ncol + j);
        const float g = gains[r];
        v[r][0] = w.x * g; v[r][1] = w.y * g; v[r][2] = w.z * g; v[r][3] = w.w * g;
      }
      const int64_t base = is_out ? F.pout : F.blk0 + l * F.blk_stride + which * (4 * int64_t(dp) * dp);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int jj = j + q;
        // gate column g d_t + u -> row 4 u + g (A' and R); U' and P_out': row j
        const int row = !is_out && which <= 1 ? 4 * (jj % dt) + jj / dt : jj;
        put(base, row, c0, dp, make_float4(v[0][q], v[1][q], v[2][q], v[3][q]),
            make_float4(v[4][q], v[5][q], v[6][q], v[7][q]));
      }
    }
  } else if (y >= wide_form_rows(dt, D)) {              // E, once per expert
    if (blockIdx.x == 0 && jl == 0 && sg == 0)
      ok = wide_split_word(a.E + int64_t(e) * a.e_stride,
                           reinterpret_cast<_Float16*>(a.esplit + int64_t(e) * kVocab * kWideHeadWidth),
                           (y - wide_form_rows(dt, D)) * kFormThreads + static_cast<int>(threadIdx.x));
  } else {
    y -= (3 * D + 1) * groups;
    const int l = y / dt, c = y % dt;                   // V of block l, or P_in (l == D)
    const bool is_in = l == D;
    const int K = is_in ? kWideHeadWidth : 4 * dt, j = 8 * i;
    if (j < K) {
      const int64_t src = (is_in ? 0 : blk0 + l * 4 * mat + 3 * mat) + int64_t(c) * K + j;
      const float4 x = quad(src);
      const float4 w = j + 4 < K ? quad(src + 4) : make_float4(0.f, 0.f, 0.f, 0.f);
      const int64_t base = is_in ? F.pin : F.blk0 + l * F.blk_stride + 3 * (4 * int64_t(dp) * dp);
      put(base, c, j, is_in ? kWideHeadWidth : 4 * dp, x, w);
    }
  }
  report_split_range(a.err, ok);
}

// out[i] = 0 for i < n (a fill kernel, so that callers may capture it).
__global__ void k_fill_f32(float* out, int64_t n) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
    out[i] = 0.0f;
}

// ---------------------------------------------------------------------------
// Gain-free LayerNorm of every row of x, a row tile of 16 per block, RPW rows a
// wave one after another, d_p <= 64 kMaxC:
//   kMode 0: x = U[byte]          (the embedding's projection per byte value)
//   kMode 1: x += h               (the LSTM sublayer's residual; h in n)
//   kMode 2: x as it is
// then n = (x - mean) / sqrt(var + 1e-5) over the first d_t features (biased
// variance), 0 on the padded ones and on rows past the last, gathered in LDS
// and written in fragment order over the 16 fp32 rows of h it replaces (read by
// this block alone, before its barrier).  Rows are r = t B + b.
// ---------------------------------------------------------------------------
template <int kMode, int RPW, int kMaxC>
__global__ __launch_bounds__(1024 / RPW) void k_wide_ln(WideArgs a) {
  constexpr int LD = 64 * kMaxC + 4;                    // LDS row in split pairs
  __shared__ uint32_t tile[16][LD];                     // (hi, lo) of every value
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t R = int64_t(a.T - 1) * a.B;
  const int64_t r0 = int64_t(blockIdx.x) * 16;
  const int s = blockIdx.y;
  int e, jl, sg;
  wide_slot(a, s, e, jl, sg);
  const int64_t slot = wide_slot_index(a, e, jl, sg);
  const int dp = a.dp, dt = a.dt, nc = dp / 64;
  const int64_t n_rows = (R + 15) / 16 * 16;
  // The wave's rows are all requested before the first is used.
  float v[RPW][kMaxC];
#pragma unroll
  for (int rr = 0; rr < RPW; ++rr) {
    const int64_t r = r0 + wave * RPW + rr;
#pragma unroll
    for (int i = 0; i < kMaxC; ++i) v[rr][i] = 0.0f;
    if (r >= R) continue;                               // wave-uniform
    const float* src = a.x + (slot * R + r) * dp;
    if (kMode == 0) {
      const int64_t t = r / a.B, b = r % a.B;
      const uint8_t* by = a.bytes + int64_t((a.j0 + jl) / a.ppb) * a.bstride + (int64_t(e) * a.B + b) * a.T;
      src = a.U + (slot * kVocab + by[t]) * dp;
    }
#pragma unroll
    for (int i = 0; i < kMaxC; ++i)
      if (i < nc) v[rr][i] = src[64 * i + lane];
  }
  if (kMode == 1) {
    float h[RPW][kMaxC];
#pragma unroll
    for (int rr = 0; rr < RPW; ++rr) {
      const int64_t r = r0 + wave * RPW + rr;
      const float* nr = a.n + (slot * n_rows + r) * dp;
#pragma unroll
      for (int i = 0; i < kMaxC; ++i) h[rr][i] = i < nc && r < R ? nr[64 * i + lane] : 0.0f;
    }
#pragma unroll
    for (int rr = 0; rr < RPW; ++rr)
#pragma unroll
      for (int i = 0; i < kMaxC; ++i) v[rr][i] += h[rr][i];
  }
#pragma unroll
  for (int rr = 0; rr < RPW; ++rr) {
    const int row = wave * RPW + rr;
    const int64_t r = r0 + row;
    if (kMode != 2 && r < R) {
      float* xr = a.x + (slot * R + r) * dp;
#pragma unroll
      for (int i = 0; i < kMaxC; ++i)
        if (i < nc) xr[64 * i + lane] = v[rr][i];
    }
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < kMaxC; ++i)
      if (i < nc && 64 * i + lane < dt) sum += v[rr][i];
    sum = wave_sum(sum);
    const float mean = sum / static_cast<float>(dt);
    float sq = 0.0f;
#pragma unroll
    for (int i = 0; i < kMaxC; ++i)
      if (i < nc && 64 * i + lane < dt) {
        const float c = v[rr][i] - mean;
        sq = __builtin_fmaf(c, c, sq);
      }
    sq = wave_sum(sq);
    const float inv = 1.0f / __builtin_sqrtf(sq / static_cast<float>(dt) + 1e-5f);
#pragma unroll
    for (int i = 0; i < kMaxC; ++i)
      if (i < nc) {
        const float y = 64 * i + lane < dt && r < R ? (v[rr][i] - mean) * inv : 0.0f;
        uint32_t hi, lo;
        split2(y, 0.0f, hi, lo);
        tile[row][64 * i + lane] = (hi & 0xFFFFu) | (lo << 16);
      }
  }
  __syncthreads();
  // Word w of the tile's d_p / 32 chunks: chunk w >> 6, word w & 63 of its hi
  // and lo blocks.
  _Float16* dst = reinterpret_cast<_Float16*>(a.n + (slot * n_rows + r0) * dp);
  const int KC = dp / 32;
  for (int w = threadIdx.x; w < KC * 64; w += 1024 / RPW) {
    const int kc = w >> 6, row = w & 15, g = (w >> 4) & 3;
    const uint4 p0 = *reinterpret_cast<const uint4*>(&tile[row][32 * kc + 8 * g]);
    const uint4 p1 = *reinterpret_cast<const uint4*>(&tile[row][32 * kc + 8 * g + 4]);
    const uint4 hi = make_uint4((p0.x & 0xFFFFu) | (p0.y << 16), (p0.z & 0xFFFFu) | (p0.w << 16),
                                (p1.x & 0xFFFFu) | (p1.y << 16), (p1.z & 0xFFFFu) | (p1.w << 16));
    const uint4 lo = make_uint4((p0.x >> 16) | (p0.y & 0xFFFF0000u), (p0.z >> 16) | (p0.w & 0xFFFF0000u),
                                (p1.x >> 16) | (p1.y & 0xFFFF0000u), (p1.z >> 16) | (p1.w & 0xFFFF0000u));
    *reinterpret_cast<uint4*>(dst + kc * 512 + (w & 63) * 8) = hi;
    *reinterpret_cast<uint4*>(dst + (KC + kc) * 512 + (w & 63) * 8) = lo;
  }
}

// ---------------------------------------------------------------------------
// The decoder: logits = u E^T over the 256 byte values and the cross entropy
// against the next byte, u = n P_out'^T from the products above ([R][32] per
// slot, row stride u_ld).  One wave per row; lane l keeps rows l, l + 64,
// l + 128, l + 192 of the expert's E in registers, and u is broadcast from
// the lanes that loaded it.  A block covers kWideHeadRows rows of a slot and
// writes their sum of cross entropies to part[slot][tile] (fp64, rows in
// order).  Evaluations also write u and the log-sum-exp per position
// b (T-1) + t for the delta rule.  fp32 products on the vector ALU.
// ---------------------------------------------------------------------------
constexpr int kWideHeadRows = 256;

template <bool kEval>
__global__ __launch_bounds__(256) void k_wide_head(WideArgs a, const float* u_base, int64_t u_slot, int u_ld) {
  constexpr int EW = kWideHeadWidth;
  constexpr int RPW = kWideHeadRows / 4;     // rows per wave
  __shared__ double ce_w[4];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int tile = blockIdx.x, s = blockIdx.y;
  int e, jl, sg;
  wide_slot(a, s, e, jl, sg);
  const int64_t slot = wide_slot_index(a, e, jl, sg);
  const int64_t R = int64_t(a.T - 1) * a.B;
  const float* Ee = a.E + int64_t(e) * a.e_stride;
  float ev[4][EW];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int k = 0; k < EW; k += 4) {
      const float4 v = *reinterpret_cast<const float4*>(Ee + (lane + 64 * j) * EW + k);
      ev[j][k] = v.x; ev[j][k + 1] = v.y; ev[j][k + 2] = v.z; ev[j][k + 3] = v.w;
    }
  const uint8_t* by = a.bytes + int64_t((a.j0 + jl) / a.ppb) * a.bstride + int64_t(e) * a.B * a.T;
  const float* ub = u_base + slot * u_slot;
  double ce_sum = 0.0;
  for (int i = 0; i < RPW; ++i) {
    const int64_t r = int64_t(tile) * kWideHeadRows + wave * RPW + i;
    if (r >= R) break;                                 // wave-uniform
    const float u = lane < EW ? ub[r * u_ld + lane] : 0.0f;
    float lg[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < EW; ++k) {
      const float uk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(u), k));
#pragma unroll
      for (int j = 0; j < 4; ++j) lg[j] = __builtin_fmaf(ev[j][k], uk, lg[j]);
    }
    float mx = fmaxf(fmaxf(lg[0], lg[1]), fmaxf(lg[2], lg[3]));
    mx = wave_max(mx);
    float se = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) se += __expf(lg[j] - mx);
    se = wave_sum(se);
    const float lse = __logf(se) + mx;
    const int64_t t = r / a.B, b = r % a.B;
    const int y = by[b * a.T + t + 1];
    const float ly = __shfl(lg[y >> 6], y & 63);
    ce_sum += static_cast<double>(lse - ly);
    if (kEval) {
      const int64_t pos = int64_t(e) * R + b * (a.T - 1) + t;
      if (lane < EW) a.fdec[pos * EW + lane] = u;
      if (lane == 0) a.lse[pos] = lse;
    }
  }
  if (lane == 0) ce_w[wave] = ce_sum;
  __syncthreads();
  if (threadIdx.x == 0) a.part[slot * a.row_tiles + tile] = ((ce_w[0] + ce_w[1]) + ce_w[2]) + ce_w[3];
}

}  // namespace soma

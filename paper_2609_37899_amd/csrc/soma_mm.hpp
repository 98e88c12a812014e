// soma_mm.hpp -- batched products of split fp32 matrices on the fp16 matrix
// cores, both operands stored in MFMA fragment order:
//   C[s][m][n] (= | += | GELU of) sum_k A[s][m][k] W[s][n][k].
//
// Fragment order: a matrix [rows][K] is 1 KiB blocks [row / 16][hi, lo][k / 32]
// of 64 words of 8 halves, word 16 lg + lr holding row lr, k 8 lg .. + 7 -- the
// bytes of the fp32 matrix, and exactly what lane (lr, lg) feeds an MFMA.  The
// exchange recurrence stores its h so, the LayerNorm of the wide body its rows,
// the GELU epilogue its result, and the form kernels the weights.  Every block
// then moves to LDS by one DMA (contiguous, no registers, no bank conflicts on
// either side), which is all the staging there is.
//
// Two shapes of block:
//  * 8 waves, 256 (n) x 256 (m) or 384 x 128, one block per compute unit that
//    works through its tiles one after another.  A chunk of 32 columns is 64
//    KiB of DMA, in two LDS buffers, for 3,072 (2,304) clocks of MFMA on each
//    SIMD: with 128 x 128 tiles the DMA's bytes per product are twice that and
//    bound the kernel.  The next chunk, also the next tile's first, is in
//    flight under the products, and a tile's stores under the next tile's.
//  * 4 waves, 128 x 128, two blocks per compute unit, where N is smaller than
//    a large tile or no multiple of one.
// Tiles are dealt so that each XCD (blocks go to the 8 XCDs round-robin) works
// through a contiguous range of them: the n tiles of one m tile, and the m
// tiles of one slot, share its L2.  Each sum runs over the chunks in order, in
// a chunk over lo hi, hi lo, hi hi, in either shape.
//
// Measured (MI355X; a bf16 library product of 16,384^3 reaches 1,370 TF/s here):
// gate inputs of the wide control, 64 x (65,472 x 1,536 x 384), 13.0 ms = 1,140
// TF/s of fp16 products (before, 128 x 128 tiles staged through registers into
// padded LDS rows: 20.7 ms); with GELU 15.1 (24.5), the down projection 13.5
// (18.1); H = 704, 256 x (16,320 x 2,816 x 704), 40.4 ms with the forming of
// the weights (register-resident weights: 61).  Bound by the matrix cores and
// the barrier and first fragment reads of each chunk.
#pragma once

#include "soma_body.hpp"
#include "soma_kernels.hpp"

namespace soma {

enum MmEpi { kEpiStore = 0, kEpiGelu = 1, kEpiAdd = 2, kEpiGates = 3 };

struct MmArgs {
  const _Float16* A;  // activations, fragment order, ceil(M / 16) row tiles
  int64_t a_slot;     // elements (split pairs) between consecutive A matrices (slots, or experts)
  int a_expert;       // A is per expert rather than per slot
  const _Float16* W;  // weights, fragment order, N / 16 row tiles
  int64_t w_slot;     // elements between slots' matrices
  void* C;            // kEpiStore, kEpiAdd: fp32 [M][N]; kEpiGelu: fragment order; kEpiGates: tiled gate inputs
  int64_t c_slot;     // elements between slots' outputs
  int M, N, K;        // N % 16 == 0, K % 32 == 0
  int pcs, PC, NS;    // the pass's slots
  int ntn, ntm;       // n tiles, m tiles
  int64_t tiles;      // ntn * ntm * slots
  int B;              // kEpiGates: sequences; row m is sequence m % B of step m / B (0: whole tiles, row tile m / 16)
  unsigned* err;
};

constexpr int kXcds = 8;

// TN x TM row tiles of 16 (n, m) per block, WN x WM waves.
template <int kEpi, int TN, int TM, int WN, int WM>
__global__ __launch_bounds__(64 * WN * WM) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mm(MmArgs p) {
  constexpr int NW = WN * WM, tn = TN / WN, tm = TM / WM;   // waves; row tiles of a wave
  constexpr int BLK = 512;                              // halves per 1 KiB block
  constexpr int BUF = 2 * (TN + TM) * BLK;              // one chunk: hi and lo of every row tile
  constexpr int DPW = 2 * (TN + TM) / NW;               // blocks a wave moves per chunk
  constexpr int WWAVES = TN * NW / (TN + TM);           // waves that move the weights
  static_assert(DPW * NW == 2 * (TN + TM) && WWAVES * DPW == 2 * TN && DPW % 2 == 0, "whole row tiles per wave");
  constexpr int kStores = tn * tm * (kEpi == kEpiGelu ? 2 : 1);   // a tile's stores per wave, at most
  constexpr bool kLoop = NW == 8;                       // one block per compute unit works through its tiles
  extern __shared__ __attribute__((aligned(16))) unsigned char mm_lds[];
  _Float16* const lds = reinterpret_cast<_Float16*>(mm_lds);   // 2 BUF halves
  const int64_t per_xcd = (p.tiles + kXcds - 1) / kXcds;
  const int64_t first = (blockIdx.x % kXcds) * per_xcd;
  const int64_t last = first + per_xcd < p.tiles ? first + per_xcd : p.tiles;   // this XCD's tiles: first .. last - 1
  const int64_t stride = gridDim.x / kXcds;
  int64_t tile = first + blockIdx.x / kXcds;
  if (tile >= last) return;                             // block-uniform
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int wn = wave % WN, wm = wave / WN;
  const int M = p.M, N = p.N, KC = p.K / 32;

  struct Where {
    int nt, mt;     // tile
    int64_t s;      // slot
    int e;
  };
  auto where = [&](int64_t t) {
    Where w;
    w.nt = static_cast<int>(t % p.ntn);
    const int64_t rest = t / p.ntn;
    w.mt = static_cast<int>(rest % p.ntm);
    const int z = static_cast<int>(rest / p.ntm);
    const int sg = z % p.NS, jl = (z / p.NS) % p.pcs;
    w.e = z / (p.NS * p.pcs);
    w.s = (int64_t(w.e) * p.PC + jl) * p.NS + sg;
    return w;
  };
  // The first waves move the weights' row tiles, the others the activations'.
  // Every offset is per lane and checked against the matrix: row tiles past
  // its end read as zeros and nothing is stored from them.
  const bool weights = wave < WWAVES;
  i32x4 rs;
  uint32_t voff[DPW];
  auto aim = [&](int64_t t) {
    const Where w = where(t);
    const _Float16* base = weights ? p.W + 2 * w.s * p.w_slot : p.A + 2 * (p.a_expert ? int64_t(w.e) : w.s) * p.a_slot;
    const int rt_all = weights ? N / 16 : (M + 15) / 16;
    rs = buffer_words(base, static_cast<uint32_t>(rt_all) * 2u * KC * BLK * 2u);
    const int rt0 = weights ? w.nt * TN + wave * (DPW / 2) : w.mt * TM + (wave - WWAVES) * (DPW / 2);
#pragma unroll
    for (int i = 0; i < DPW; ++i)
      voff[i] = static_cast<uint32_t>(((rt0 + (i >> 1)) * 2 + (i & 1)) * KC) * (BLK * 2) + lane * 16;
  };
  const uint32_t dst0 = lds_address(lds + wave * DPW * BLK);
  auto issue = [&](int buf) {
#pragma unroll
    for (int i = 0; i < DPW; ++i) {
      dma16(rs, voff[i], 0u, dst0 + static_cast<uint32_t>((buf * BUF + i * BLK) * 2));
      voff[i] += BLK * 2;
    }
  };
  const _Float16* const wl0 = lds + wn * tn * 2 * BLK + lane * 8;           // this wave's weight tiles
  const _Float16* const al0 = lds + (TN + wm * tm) * 2 * BLK + lane * 8;    // and activation tiles

  bool ok = true;
  aim(tile);
  issue(0);
  int buf = 0;
  bool stored = false;                                  // the last accesses are a tile's stores
  for (;;) {
    f32x4 acc[tn][tm];
#pragma unroll
    for (int i = 0; i < tn; ++i)
#pragma unroll
      for (int j = 0; j < tm; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const Where w = where(tile);
    const int64_t next = tile + stride;
    const bool more = kLoop && next < last;             // block-uniform
    for (int c = 0; c < KC; ++c) {
      // Chunk c has landed (a wave's accesses complete in order: only a tile's
      // stores, issued after it, may still be out), and every wave is done
      // with the other buffer.
      if (stored)
        wait_vmem_but<(kStores < 63 ? kStores : 63)>();
      else
        wait_vmem();
      stored = false;
      __syncthreads();
      if (c + 1 < KC) {
        issue(buf ^ 1);
      } else if (more) {
        aim(next);
        issue(buf ^ 1);
      }
      uint4 bh[tm], bl[tm];
#pragma unroll
      for (int mt = 0; mt < tm; ++mt) {
        bh[mt] = *reinterpret_cast<const uint4*>(al0 + buf * BUF + 2 * mt * BLK);
        bl[mt] = *reinterpret_cast<const uint4*>(al0 + buf * BUF + (2 * mt + 1) * BLK);
      }
#pragma unroll
      for (int ntl = 0; ntl < tn; ++ntl) {
        const uint4 wh = *reinterpret_cast<const uint4*>(wl0 + buf * BUF + 2 * ntl * BLK);
        const uint4 wl = *reinterpret_cast<const uint4*>(wl0 + buf * BUF + (2 * ntl + 1) * BLK);
        mfma3_batch<tm>(wh, wl, bh, bl, acc[ntl]);
      }
      buf ^= 1;
    }

    // acc[ntl][mt][i] = C[16 (TM w.mt + tm wm + mt) + lr][16 (TN w.nt + tn wn + ntl) + 4 lg + i]
#pragma unroll
    for (int ntl = 0; ntl < tn; ++ntl) {
      const int ntile = w.nt * TN + wn * tn + ntl;
      if (ntile * 16 >= N) continue;                    // wave-uniform
      const int n = ntile * 16 + 4 * lg;
#pragma unroll
      for (int mt = 0; mt < tm; ++mt) {
        const int rt = w.mt * TM + wm * tm + mt, m = rt * 16 + lr;
        if (m >= M) continue;
        float4 v = make_float4(acc[ntl][mt][0], acc[ntl][mt][1], acc[ntl][mt][2], acc[ntl][mt][3]);
        if constexpr (kEpi == kEpiGelu) {
          // the next product's A: K there is N here
          v = make_float4(gelu_f(v.x), gelu_f(v.y), gelu_f(v.z), gelu_f(v.w));
          ok = ok && split_range_ok(v);
          uint2 hi, lo;
          split4(v, hi, lo);
          _Float16* C = reinterpret_cast<_Float16*>(p.C) + 2 * w.s * p.c_slot +
                        (int64_t(rt) * 2 * (N / 32) + ntile / 2) * BLK +
                        (16 * (2 * (ntile & 1) + (lg >> 1)) + lr) * 8 + 4 * (lg & 1);
          *reinterpret_cast<uint2*>(C) = hi;
          *reinterpret_cast<uint2*>(C + (N / 32) * BLK) = lo;
        } else if constexpr (kEpi == kEpiGates) {
          int64_t t16 = rt;                             // row tile and lane of the tiled order
          int l = lane;
          if (p.B > 0) {
            const int t = m / p.B, b = m - t * p.B;
            t16 = int64_t(t) * ((p.B + 15) / 16) + (b >> 4);
            l = (b & 15) + 16 * lg;
          }
          *reinterpret_cast<float4*>(reinterpret_cast<float*>(p.C) + w.s * p.c_slot +
                                     (t16 * (N / 16) + ntile) * 256 + l * 4) = v;
        } else {
          float4* c = reinterpret_cast<float4*>(reinterpret_cast<float*>(p.C) + w.s * p.c_slot + int64_t(m) * N + n);
          if constexpr (kEpi == kEpiAdd) {
            const float4 o = *c;
            v = make_float4(o.x + v.x, o.y + v.y, o.z + v.z, o.w + v.w);
          }
          *c = v;
        }
      }
    }
    if (!more) break;
    tile = next;
    stored = kEpi != kEpiAdd && w.mt * TM + TM <= M / 16 && w.nt * TN + TN <= N / 16;   // every store was issued
  }
  if constexpr (kEpi == kEpiGelu) report_split_range(p.err, ok);
}

// Dynamic LDS of a block.
constexpr unsigned mm_lds_bytes(int TN, int TM) { return 2u * 2u * static_cast<unsigned>(TN + TM) * 1024u; }

// ---------------------------------------------------------------------------
// Perturbed input weights of layer l >= 2 of the stacked LSTM for k_mm: rows
// 4 u + g (gate g of unit u) of W_l+-'s columns [0, K), split, in fragment
// order, slot by slot.  A wave forms one 16-row tile's chunk of 32 columns for
// both signs of a direction from one draw of its probes and stores each as two
// 1 KiB blocks (grid: 4 chunks a block, then directions).  Bound by the
// probes' arithmetic (Gaussian): one draw per weight and direction, where the
// register-resident projection draws once per weight and sign.
// ---------------------------------------------------------------------------
template <bool kRad>
__global__ __launch_bounds__(256) void k_form_gates(FwdArgs a, _Float16* out) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int H = a.H, K = a.in_l, KC = K / 32;
  const int b = blockIdx.x * 4 + wave;                  // row tile b / KC, chunk b % KC (4H/16 KC is a multiple of 4)
  const int e = blockIdx.y / a.pcs, jl = blockIdx.y % a.pcs;
  const int row = (b / KC) * 16 + lr;
  const int64_t kk = a.off_l + static_cast<int64_t>((row & 3) * H + (row >> 2)) * (K + H) + 32 * (b % KC) + 8 * lg;
  const float* th = a.theta + static_cast<int64_t>(e) * a.d + kk;
  const uint2 key = stream_key(a.seeds[e], a.step);
  const uint32_t pair = static_cast<uint32_t>(a.j0 + jl), step_lo = static_cast<uint32_t>(a.step);
  const float eps = eps_of(a, e, kGroupLstm);
  float4 z[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
    z[i] = kRad ? rademacher_quad(key, pair, step_lo, static_cast<uint64_t>(kk + 4 * i), a.probe == kProbeRademacher)
                : gauss_quad(key, pair, step_lo, static_cast<uint64_t>(kk + 4 * i) >> 2);
  const float4 t0 = *reinterpret_cast<const float4*>(th), t1 = *reinterpret_cast<const float4*>(th + 4);
  bool ok = true;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const float4 w0 = fma4(s == 0 ? eps : -eps, z[0], t0), w1 = fma4(s == 0 ? eps : -eps, z[1], t1);
    ok = ok && split_range_ok(w0) && split_range_ok(w1);
    uint4 hi, lo;
    split8v(w0, w1, hi, lo);
    const int64_t slot = (static_cast<int64_t>(e) * a.PC + jl) * 2 + s;
    _Float16* dst = out + slot * 8 * H * K + (static_cast<int64_t>(b / KC) * 2 * KC + b % KC) * 512 + lane * 8;
    *reinterpret_cast<uint4*>(dst) = hi;
    *reinterpret_cast<uint4*>(dst + static_cast<int64_t>(KC) * 512) = lo;
  }
  report_split_range(a.err, ok);
}

}  // namespace soma

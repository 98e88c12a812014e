// soma_xchg.hpp -- the persistent recurrence with the pipelined split exchange.
#pragma once

#include <type_traits>
#include <utility>

#include "soma_kernels.hpp"

namespace soma {

// ---------------------------------------------------------------------------
// Persistent recurrence with a pipelined split exchange (k_rec_xchg): the
// per-step arithmetic of k_rec_persist -- G_t = G_in,t + h_{t-1} W_h+-^T on
// the fp16 matrix cores from split operands, the cell update in the lane
// that holds a unit's four gates -- organised so that neither the exchange of
// h between the blocks of a group nor the cell update waits in front of the
// products.
//
//  * The batch's row tiles (16 sequences each, four of them: 64 sequences, a
//    larger batch being cut into several jobs) are independent recurrences
//    that share the block's resident weights.  A block runs sub-steps
//    s = (t, k) in the order t, then tile k: the products of tile k at step
//    t need only tile k's h_{t-1}, published in sub-step s - 3, so its
//    exchange is hidden behind the products of the other tiles.
//  * Eight waves: row group rg = wave & 3 (32 gate rows: eight units, two
//    MFMA row tiles) and K half kh = wave >> 2.  Each fragment of h read from
//    LDS feeds two row tiles (six MFMAs), so the products of a sub-step read
//    4 waves x 2 halves x H / 2 x 64 bytes of LDS instead of eight times all
//    of h: with one row tile per wave the reads (256 KiB a sub-step at
//    H = 512, 2,048 clocks) took longer than the MFMAs (1,536 clocks).
//  * The two K halves have two roles, because a wave's memory accesses
//    complete in order.  The second half's waves read the gate inputs and
//    nothing else, two sub-steps ahead (they come from HBM, or at layer 1 by
//    byte value from the folded table: in the queue of a wave that also waits
//    for its DMA and stores every sub-step they held it up by 900 of 3,700
//    clocks); their sums start from them, and go through LDS to the first
//    half's waves.  Those finish the
//    units (two cells a lane), publish h and move it: DMA, stores, flags.
//  * The tail of sub-step s - 1 (partner's sums, cell update, publication)
//    is cut into stages that run between the MFMAs of sub-step s, so one
//    block barrier separates the sub-steps and only the hand-over of the
//    partial sums, the wait and the flags stand outside the products.
//  * Each block publishes its 32 units of h_t of a tile (one 32-wide K
//    chunk) already split into fp16 hi and lo parts in MFMA fragment order:
//    per part 64 words of 8 halves, word 16 lg + lr holding row lr, columns
//    8 lg .. + 7 -- row group lg's eight units, brought into one lane by lane
//    swaps, so a wave stores whole 128-byte lines straight from the cell
//    lanes.  A group keeps two steps per tile (parity t mod 2) in L2.  h_t
//    also goes to the layer's hseq for the kernels that read the whole
//    sequence: in fp32 rows, or (split_out, where the next layer's projection
//    is k_mm) as the same split words, in fragment order, every time step in
//    whole row tiles (rows past the batch are finite and used by nobody).
//  * The tile's h_{t-1} reaches LDS by DMA (buffer_load_dwordx4 ... lds):
//    each 1 KiB block lands unchanged.  The DMA of sub-step s + 2 is issued
//    after the block barrier that ends the products of sub-step s, into the
//    LDS buffer they have released (two buffers).
//  * Arrival is a per-(tile, block) flag word holding the steps published.
//    The stores of sub-step s - 1's publication go out during the products of
//    sub-step s and are covered by the wait that ends them (the sequence's
//    store, issued last, is left in flight); a block barrier follows and
//    thread 0 raises the flag at once.  The flags the DMA of sub-step s + 2
//    needs (raised a sub-step earlier) are read by one load during the
//    products of s and checked after the barrier.
//
// Every wait is bounded: a wave that polls longer than the spin limit, or
// that sees the step's abort flag, sets the flag and stops waiting; every
// wave then runs to the end without waiting (on stale data), so the grid
// drains, and the losses read NaN.  A block owns 128 gate rows (32 units); a
// group of H / 32 blocks sits on one XCD; one block per compute unit, claimed
// at start from the compute unit it runs on.
//
// Measured (MI355X): H = 512, B = 64, 16 groups, 8 jobs of 255 steps each:
// 11.8 ms a layer, 1.44 us a sub-step of which the MFMAs (two waves a SIMD)
// take 0.75 (one row tile per wave, the tail after the products, gate inputs
// in rows of 4 H: 12.8 ms); H = 704, 32 jobs a group: 67 ms (layer 1) and 55 ms
// (68.5 before); wide body, H = 384: 18.5 ms against 22.6 on the staged
// recurrence.  What remains of a sub-step: the DMA's issue (0.25 us: 32 KiB
// through a 64-byte path), the tail's vector work in the finishing waves, and
// the hand-over and barrier (0.2 us).
//
// The LDS DMA is issued through inline assembly: the compiler assumes that a
// pending LDS DMA may alias every later LDS read and would wait for it
// before each fragment read.  Its completion is covered by the sub-step's
// wait and the block barrier that follows.
// ---------------------------------------------------------------------------
// Perturbed weights of the exchange recurrence's wave (rg, kh), one sign, as
// split fragments: gate rows r0 + 32 rg + 16 m + lr (m < 2; row 4u + g is
// gate g of unit u) over the K chunks kh NCH .. + NCH - 1 of H = 64 NCH
// columns from col0.  As resident_weights_split otherwise: the probes of a
// piece (the same chunks of both K halves, so that every wave takes its share
// of every piece) are drawn once by the block into the scratch zs.
template <int NCH, bool kRad>
__device__ __forceinline__ void resident_weights_khalf(uint4 (&wh)[2][NCH], uint4 (&wl)[2][NCH], float* zs,
                                                       const float* th, int64_t off_l, int ld, int col0, int H, int r0,
                                                       int law, uint2 key, uint32_t pair, uint32_t step_lo, float seps,
                                                       unsigned* err) {
  constexpr int ZC = NCH % 2 == 0 ? 2 : 1;              // chunks of each half per piece
  constexpr int ZLD = 64 * ZC + 8;                      // scratch row in floats (an odd multiple of 32 bytes)
  bool in_range = true;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int rg = wave & 3, kh = wave >> 2;
  auto canon = [&](int r) { return (r & 3) * H + (r >> 2); };
#pragma unroll
  for (int piece = 0; piece < NCH / ZC; ++piece) {
    __syncthreads();
    for (int q = threadIdx.x; q < 128 * 16 * ZC; q += 512) {
      const int m = q / (16 * ZC), k4 = q % (16 * ZC), half = k4 / (8 * ZC), kq = k4 % (8 * ZC);
      const uint64_t kk = static_cast<uint64_t>(off_l + static_cast<int64_t>(canon(r0 + m)) * ld + col0 +
                                                32 * (half * NCH + piece * ZC) + 4 * kq);
      *reinterpret_cast<float4*>(&zs[m * ZLD + 4 * k4]) =
          kRad ? rademacher_quad(key, pair, step_lo, kk, law == kProbeRademacher) : gauss_quad(key, pair, step_lo, kk >> 2);
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const int row = 32 * rg + 16 * m + lr;
      const float* tr = th + off_l + static_cast<int64_t>(canon(r0 + row)) * ld + col0 + 32 * kh * NCH + 8 * lg;
#pragma unroll
      for (int c2 = 0; c2 < ZC; ++c2) {
        const int c = piece * ZC + c2;
        const float* zr = &zs[row * ZLD + 32 * (kh * ZC + c2) + 8 * lg];
        const float4 w0 = fma4(seps, *reinterpret_cast<const float4*>(zr), *reinterpret_cast<const float4*>(tr + 32 * c));
        const float4 w1 =
            fma4(seps, *reinterpret_cast<const float4*>(zr + 4), *reinterpret_cast<const float4*>(tr + 32 * c + 4));
        in_range = in_range && split_range_ok(w0) && split_range_ok(w1);
        split8v(w0, w1, wh[m][c], wl[m][c]);
      }
    }
  }
  report_split_range(err, in_range);
  __syncthreads();
}

// kL1: the layer reads its inputs from the folded table by byte value (layer
// 1) rather than from the time-parallel gate inputs; kPre: the recurrent
// weights come pre-formed (a.wpre), a pass may run one sign per direction
// (a.ns == 1).  Template parameters, so that each instance loads its inputs
// on one path and keeps its registers.
template <int NCH, bool kRad, bool kL1, bool kPre>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_rec_xchg(XchgArgs p) {
  constexpr int NU = 32;                                // units per block (one K chunk of h)
  constexpr int NB = kXchgTiles;
  constexpr int KC = 2 * NCH;                           // 32-wide k chunks: H = 64 NCH
  constexpr int FRAG = 512;                             // halves per 1 KiB block (one part of a chunk of a tile)
  constexpr int TBUF = KC * 2 * FRAG;                   // halves of one tile's h (in LDS, and published)
  constexpr int XSLOT = 2 * NB * TBUF;                  // halves per group: parity x tile
  constexpr int ZS_BYTES = kPre ? 0 : 128 * (64 * (NCH % 2 == 0 ? 2 : 1) + 8) * 4;
  constexpr int RING_BYTES = 2 * TBUF * 2;
  constexpr int LDS_BYTES = RING_BYTES > ZS_BYTES ? RING_BYTES : ZS_BYTES;
  constexpr int NBLK = 2 * KC;                          // 1 KiB blocks per tile
  constexpr int BPW = NBLK / 4;                         // of them per wave of the first K half
  // Registers: 16 NCH of weights.  Above 512 columns they leave room for two
  // fragments read ahead instead of three and for one sum per row tile
  // instead of two (cross terms apart from hi x hi).
  constexpr bool kLean = NCH > 8;
  __shared__ __attribute__((aligned(16))) unsigned char lds[LDS_BYTES];
  __shared__ __attribute__((aligned(16))) float4 part[2][4][2][64];   // sums handed over: [parity][rg][row tile]
  __shared__ int role[2];
  _Float16* ring = reinterpret_cast<_Float16*>(lds);
  const FwdArgs& a = p.a;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int rg = wave & 3, kh = wave >> 2;
  const int H = a.H, B = a.B, T = a.T, in = a.in_l;
  const int UT = H / NU;                                // blocks per group

  // Claim (group, unit tile): rank r = how many blocks started on this
  // compute unit before this one, i = how many blocks of rank r on this XCD
  // claimed before; position r * cus_per_xcd + i of the XCD's per_cu *
  // cus_per_xcd blocks, UT consecutive positions per group, positions past
  // the XCD's whole groups idle.  The host launches with per_cu = 1 only: a
  // launch that placed two blocks on each compute unit faulted the device (H =
  // 128, B = 10, cause not found).  (per_cu as a constant costs two to three per
  // cent at H = 640 and 704: the main loop spills more.)
  if (threadIdx.x == 0) {
    const unsigned hw = __builtin_amdgcn_s_getreg((31 << 11) | 4);         // HW_ID
    const unsigned xcc = __builtin_amdgcn_s_getreg((31 << 11) | 20) & 15;  // XCC_ID
    const unsigned cu = ((hw >> 13) & 3) * 16 + ((hw >> 8) & 15);          // shader engine, compute unit
    int grp = -2, tile = 0;                             // -2: unplaced (an error), -1: idle
    if (xcc < 8) {
      const unsigned r = __hip_atomic_fetch_add(&p.cu_count[xcc * 64 + cu], 1u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
      if (r < static_cast<unsigned>(p.per_cu)) {
        const unsigned i = __hip_atomic_fetch_add(&p.rank_count[xcc * kXchgMaxPerCu + r], 1u, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
        if (i < static_cast<unsigned>(p.cus_per_xcd)) {
          const int pos = static_cast<int>(r) * p.cus_per_xcd + static_cast<int>(i);
          grp = pos < (p.groups / 8) * UT ? (pos / UT) * 8 + static_cast<int>(xcc) : -1;
          tile = pos % UT;
        }
      }
    }
    if (grp == -2) __hip_atomic_fetch_or(p.err, kAbortPlace, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    role[0] = grp;
    role[1] = tile;
  }
  __syncthreads();
  const int grp = __builtin_amdgcn_readfirstlane(role[0]), utile = __builtin_amdgcn_readfirstlane(role[1]);
  if (grp < 0) return;
  unsigned* const flags = p.flag + grp * kXchgFlagWords;   // [tile][block]
  // This group's part of the published ring: offsets stay small, and every
  // access is checked against it.
  const uint32_t xbytes = XSLOT * 2u;
  _Float16* const xg = p.xh + static_cast<int64_t>(grp) * XSLOT;
  const i32x4 xrs = buffer_words(xg, xbytes);              // the same buffer for the DMA (scalar words)
  const __amdgpu_buffer_rsrc_t xbuf = buffer_of(xg, xbytes);
  const int unit = utile * NU + rg * 8 + lg;            // this lane's unit of row tile 0; row tile 1: unit + 4
  const int64_t R = static_cast<int64_t>(T - 1) * B;
  const int64_t H4 = 4 * static_cast<int64_t>(H);
  const int RT = (B + 15) / 16;                         // row tiles of a time step
  const int64_t gin_rows = static_cast<int64_t>(T - 1) * RT * 16;
  const uint32_t slot_bytes = static_cast<uint32_t>((p.split_out ? gin_rows : R) * H * sizeof(float));   // < 2^31 (host check)
  constexpr int kGiChunk = NCH / 2;                     // chunk after which the next inputs are requested
  constexpr uint32_t kOut = 0x80000000u;                // past every buffer: a store there is dropped
  bool failed = false;                                  // this wave stopped waiting (abort)

  // Poll until every block of the group has published `target` steps of
  // tile k (flag words [k][0 .. UT)), or give up.  Every wave polls for
  // itself; after an abort nothing waits any more.  One load per poll: lane
  // 63 reads the abort flag, the others their flag word.
  auto ready = [&](unsigned target, unsigned v) { return __builtin_amdgcn_ballot_w64(lane < UT && v < target) == 0; };
  auto wait_flags = [&](int k, unsigned target) {
    unsigned polls = 0;
    const unsigned* addr = lane == 63 ? p.err : flags + k * 64 + lane;
    while (!failed) {
      const unsigned v = __hip_atomic_load(addr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const unsigned f = __builtin_amdgcn_readlane(v, 63);
      if (ready(target, v)) break;
      if (f != 0u || ++polls > p.spin_limit) {
        if (lane == 0) __hip_atomic_fetch_or(p.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        failed = true;
      } else {
        __builtin_amdgcn_s_sleep(1);
      }
    }
  };

  const bool one_sign = kPre && a.ns == 1;
  const int seq_step = p.split_out ? RT * 16 : B;       // rows of a time step in hseq
  const uint32_t split_mask = p.split_out ? 0xFFFFFFFFu : 0u;
  // Published word of this lane's row (lane groups 0, 1: the hi and lo word
  // for the ring; 2, 3: the same, or in fp32 the two unit quads, for the
  // layer's sequence).
  const uint32_t ring_lane =
      lg < 2 ? static_cast<uint32_t>(((utile * 2 + lg) * FRAG + (16 * rg + lr) * 8) * 2) : kOut;
  const _Float16* const blane = ring + lane * 8 + kh * NCH * 2 * FRAG;   // this lane's fragment words in LDS

  unsigned base = 0;                                    // steps of every tile published in earlier jobs

  using std::integral_constant;
  using Yes = std::true_type;
  using No = std::false_type;

  // The products of one sub-step, tile in LDS buffer `buf`, onto cr (cross
  // terms; kLean: everything) and mn (hi x hi); between(c) runs after chunk c.
  auto products = [&](auto Pc, const uint4 (&wh)[2][NCH], const uint4 (&wl)[2][NCH], int buf, f32x4 (&cr)[2],
                      f32x4 (&mn)[kLean ? 1 : 2], auto between) {
    constexpr int PF = decltype(Pc)::value < NCH ? decltype(Pc)::value : NCH;   // fragments read ahead
    const _Float16* const src = blane + buf * TBUF;
    uint4 bh[PF], bl[PF];
#pragma unroll
    for (int c = 0; c < PF; ++c) {
      bh[c] = *reinterpret_cast<const uint4*>(src + c * 2 * FRAG);
      bl[c] = *reinterpret_cast<const uint4*>(src + c * 2 * FRAG + FRAG);
    }
    auto chunk = [&](auto Cc) {
      constexpr int c = decltype(Cc)::value;
      const h8 BH = __builtin_bit_cast(h8, bh[c % PF]), BL = __builtin_bit_cast(h8, bl[c % PF]);
      const h8 A0 = __builtin_bit_cast(h8, wh[0][c]), A1 = __builtin_bit_cast(h8, wh[1][c]);
      f32x4& m0 = kLean ? cr[0] : mn[0];
      f32x4& m1 = kLean ? cr[1] : mn[kLean ? 0 : 1];
      cr[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, wl[0][c]), BH, cr[0], 0, 0, 0);
      cr[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, wl[1][c]), BH, cr[1], 0, 0, 0);
      m0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(A0, BH, m0, 0, 0, 0);
      m1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(A1, BH, m1, 0, 0, 0);
      cr[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A0, BL, cr[0], 0, 0, 0);
      cr[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A1, BL, cr[1], 0, 0, 0);
      if constexpr (c + PF < NCH) {
        bh[c % PF] = *reinterpret_cast<const uint4*>(src + (c + PF) * 2 * FRAG);
        bl[c % PF] = *reinterpret_cast<const uint4*>(src + (c + PF) * 2 * FRAG + FRAG);
      }
      between(Cc);
    };
    [&]<int... C>(std::integer_sequence<int, C...>) {
      (chunk(integral_constant<int, C>{}), ...);
    }(std::make_integer_sequence<int, NCH>{});
  };
  auto clear = [&](f32x4 (&cr)[2], f32x4 (&mn)[kLean ? 1 : 2]) {
#pragma unroll
    for (int m = 0; m < 2; ++m) cr[m] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int m = 0; m < (kLean ? 1 : 2); ++m) mn[m] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  };
  auto total = [&](const f32x4 (&cr)[2], const f32x4 (&mn)[kLean ? 1 : 2], int m) {
    return kLean ? cr[m] : cr[m] + mn[kLean ? 0 : m];
  };
  // Four sub-steps of step t, then the next: sub(k, products?, tail?, t).
  auto all_steps = [&](auto sub) {
    sub(integral_constant<int, 0>{}, No{}, No{}, 0);
    sub(integral_constant<int, 1>{}, No{}, Yes{}, 0);
    sub(integral_constant<int, 2>{}, No{}, Yes{}, 0);
    sub(integral_constant<int, 3>{}, No{}, Yes{}, 0);
    for (int t = 1; t + 1 < T; ++t) {
      sub(integral_constant<int, 0>{}, Yes{}, Yes{}, t);
      sub(integral_constant<int, 1>{}, Yes{}, Yes{}, t);
      sub(integral_constant<int, 2>{}, Yes{}, Yes{}, t);
      sub(integral_constant<int, 3>{}, Yes{}, Yes{}, t);
    }
  };

  // The second K half: gate inputs of the tile's rows (row lr, units unit and
  // unit + 4), read two sub-steps ahead; the sums start from them.
  auto input_half = [&](const uint4 (&wh)[2][NCH], const uint4 (&wl)[2][NCH], __amdgpu_buffer_rsrc_t gbuf,
                        __amdgpu_buffer_rsrc_t bbuf, int b0) {
    // This lane's part of the block's 512 bytes of a table row (layer 1), or
    // of its 8 KiB of a row tile's gate inputs.
    const uint32_t gi_lane = kL1 ? static_cast<uint32_t>(utile * kVocab * 512 + (rg * 8 + lg) * 16)
                                 : static_cast<uint32_t>(((b0 / 16) * UT + utile) * 8192 + rg * 2048 + lane * 16);
    const uint32_t byte_lane = static_cast<uint32_t>((b0 + lr) * T);
    float4 gi[2][2];                                    // by sub-step parity
    int vb[NB];                                         // layer 1: byte of the tile's next step to gather
    auto load_byte = [&](int t, int k) {
      if constexpr (kL1)
        vb[k] = __builtin_amdgcn_raw_buffer_load_b8(bbuf, byte_lane + static_cast<uint32_t>(k * 16 * T + t), 0, 0);
    };
    auto load_inputs = [&](int t, int k) {
      const uint32_t off =
          gi_lane + (kL1 ? static_cast<uint32_t>(vb[k] * 512) : static_cast<uint32_t>((t * RT + k) * UT * 8192));
      gi[k & 1][0] = buffer_load_f4<0>(gbuf, off);
      gi[k & 1][1] = buffer_load_f4<0>(gbuf, off + (kL1 ? 64 : 1024));
    };
#pragma unroll
    for (int k = 0; k < NB; ++k) load_byte(0, k);
    load_inputs(0, 0);
    load_byte(1, 0);
    load_inputs(0, 1);
    load_byte(1, 1);
    all_steps([&](auto Kc, auto Mulc, auto, int t) {
      constexpr int k = decltype(Kc)::value;
      f32x4 cr[2], mn[kLean ? 1 : 2];
      clear(cr, mn);
#pragma unroll
      for (int m = 0; m < 2; ++m) cr[m] = f32x4{gi[k & 1][m].x, gi[k & 1][m].y, gi[k & 1][m].z, gi[k & 1][m].w};
      // The inputs of sub-step s + 2 = (t2, k2), and the byte of its tile's
      // step after that.
      constexpr int k2 = (k + 2) % NB;
      const int t2 = k < 2 ? t : t + 1;
      auto next = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        load_inputs(t2, k2);
        load_byte(t2 + 1, k2);
        __builtin_amdgcn_sched_barrier(0);
      };
      if constexpr (decltype(Mulc)::value) {
        products(integral_constant<int, kLean ? 2 : 3>{}, wh, wl, k & 1, cr, mn, [&](auto Cc) {
          if constexpr (decltype(Cc)::value == kGiChunk) next();
        });
      } else {
        next();
      }
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const f32x4 s = total(cr, mn, m);
        part[k & 1][rg][m][lane] = make_float4(s[0], s[1], s[2], s[3]);
      }
      __syncthreads();
    });
    __syncthreads();                                    // the other half's last publication
  };

  // The first K half: cell updates, publication, exchange.
  auto finish_half = [&](const uint4 (&wh)[2][NCH], const uint4 (&wl)[2][NCH], __amdgpu_buffer_rsrc_t hbuf, int b0,
                         int nrows) {
    const uint32_t seq_lane =
        lg < 2 ? kOut
               : (p.split_out
                      ? static_cast<uint32_t>((((b0 / 16) * 2 + (lg & 1)) * KC + utile) * FRAG * 2 + (16 * rg + lr) * 16)
                      : static_cast<uint32_t>(((b0 + lr) * H + utile * NU + rg * 8 + (lg & 1) * 4) * 4));
    float cs[NB][2];                                    // cell state of this lane's two units, per tile
#pragma unroll
    for (int k = 0; k < NB; ++k) cs[k][0] = cs[k][1] = 0.0f;
    f32x4 own[2];                                       // this half's sums of the tail's sub-step
    unsigned v2 = 0;                                    // flag words read during the products
    // The tail of sub-step (t, k) in stages; k2: the tile whose flags the end
    // of the running sub-step needs.
    float4 pp[2];
    float sf[2], ig[2], h[2];
    float4 hv[2];
    auto tail = [&](auto Jc, auto Kc, int t, int k2) {
      constexpr int J = decltype(Jc)::value, k = decltype(Kc)::value;
      if constexpr (J == 0) {                           // lstm_cell in two stages, both units
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const float ef = exp2_f(-kLog2e * (own[m][1] + pp[m].y)), ei = exp2_f(-kLog2e * (own[m][0] + pp[m].x));
          const float pg = own[m][2] + pp[m].z, eg = exp2_f(-2.0f * kLog2e * __builtin_fabsf(pg));
          sf[m] = __builtin_amdgcn_rcpf(1.0f + ef);
          ig[m] = __builtin_copysignf((1.0f - eg) * __builtin_amdgcn_rcpf((1.0f + ei) * (1.0f + eg)), pg);
        }
      } else if constexpr (J == 1) {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const float eo = exp2_f(-kLog2e * (own[m][3] + pp[m].w));
          const float c = __builtin_fmaf(sf[m], cs[k][m], ig[m]);
          cs[k][m] = c;
          const float ec = exp2_f(-2.0f * kLog2e * __builtin_fabsf(c));
          h[m] = __builtin_copysignf((1.0f - ec) * __builtin_amdgcn_rcpf((1.0f + eo) * (1.0f + ec)), c);
        }
      } else if constexpr (J == 2) {
        // Every lane of a row takes the row group's eight units.
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const uint32_t x = __float_as_uint(h[m]);
          const auto p16 = __builtin_amdgcn_permlane16_swap(x, x, false, false);
          const auto qa = __builtin_amdgcn_permlane32_swap(p16[0], p16[0], false, false);   // units 0, 2
          const auto qb = __builtin_amdgcn_permlane32_swap(p16[1], p16[1], false, false);   // units 1, 3
          hv[m] = make_float4(__uint_as_float(qa[0]), __uint_as_float(qb[0]), __uint_as_float(qa[1]),
                              __uint_as_float(qb[1]));
        }
      } else if constexpr (J == 3) {
        typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
        uint4 hi, lo;
        split8v(hv[0], hv[1], hi, lo);
        const bool odd = (lg & 1) != 0;
        const u32x4 words = {odd ? lo.x : hi.x, odd ? lo.y : hi.y, odd ? lo.z : hi.z, odd ? lo.w : hi.w};
        __builtin_amdgcn_raw_buffer_store_b128(words, xbuf, ring_lane,
                                               static_cast<uint32_t>(((t & 1) * NB + k) * TBUF * 2), kCoherent);
        __builtin_amdgcn_sched_barrier(0);
        v2 = __hip_atomic_load(flags + k2 * 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_sched_barrier(0);
        // The layer's sequence, last: it is not waited for.  A select without
        // a branch; fp32 rows past the batch, and split row tiles past the
        // time step's, are dropped.
        const float4 q = odd ? hv[1] : hv[0];
        const u32x4 fp = {__float_as_uint(q.x), __float_as_uint(q.y), __float_as_uint(q.z), __float_as_uint(q.w)};
        const u32x4 sv = (words & split_mask) | (fp & ~split_mask);
        const uint32_t off = lg >= 2 && k * 16 + (p.split_out ? 0 : lr) < nrows
                                 ? seq_lane + static_cast<uint32_t>((t * seq_step + k * 16) * H * 4)
                                 : kOut;
        __builtin_amdgcn_raw_buffer_store_b128(sv, hbuf, off, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    constexpr int kStages = 4;
    auto whole_tail = [&](auto Kc, int t, int k2) {
      tail(integral_constant<int, 0>{}, Kc, t, k2);
      tail(integral_constant<int, 1>{}, Kc, t, k2);
      tail(integral_constant<int, 2>{}, Kc, t, k2);
      tail(integral_constant<int, 3>{}, Kc, t, k2);
    };
    auto take_part = [&](int parity) {
      pp[0] = part[parity][rg][0][lane];
      pp[1] = part[parity][rg][1][lane];
    };

    // Sub-step (t, k): the products of tile k with h_{t-1} from LDS buffer
    // k & 1 (not at t = 0: h_{-1} = 0), between them the tail of sub-step
    // s - 1.
    all_steps([&](auto Kc, auto Mulc, auto Tailc, int t) {
      constexpr int k = decltype(Kc)::value;
      constexpr bool kMul = decltype(Mulc)::value, kTail = decltype(Tailc)::value;
      constexpr int kp = (k + NB - 1) % NB, k2 = (k + 2) % NB;
      const int tp = k == 0 ? t - 1 : t;                // step of the tail
      const int t2 = k < 2 ? t : t + 1;                 // sub-step s + 2 is (t2, k2)
      f32x4 cr[2], mn[kLean ? 1 : 2];
      clear(cr, mn);
      if constexpr (kTail) take_part(kp & 1);
      if constexpr (kMul) {
        products(integral_constant<int, kLean ? 1 : 3>{}, wh, wl, k & 1, cr, mn, [&](auto Cc) {
          constexpr int c = decltype(Cc)::value;
          constexpr int span = NCH < kStages ? NCH : kStages;   // chunks that carry the stages
          if constexpr (c < span) {
            constexpr int first = c * kStages / span, last = (c + 1) * kStages / span;
            [&]<int... I>(std::integer_sequence<int, I...>) {
              (tail(integral_constant<int, first + I>{}, integral_constant<int, kp>{}, tp, k2), ...);
            }(std::make_integer_sequence<int, last - first>{});
          }
          __builtin_amdgcn_sched_barrier(0);
        });
      } else if constexpr (kTail) {
        whole_tail(integral_constant<int, kp>{}, tp, k2);
      }
      own[0] = total(cr, mn, 0);
      own[1] = total(cr, mn, 1);
      // Complete: the DMA of sub-step s + 1, the tail's store to the ring, the
      // flag load; the store to the sequence may stay in flight.
      __builtin_amdgcn_sched_barrier(0);
      wait_vmem_but<kTail ? 1 : 0>();
      __syncthreads();
      // Raise the flag of the tail's publication: every wave's stores of it
      // completed before the barrier.
      if constexpr (kTail) {
        if (threadIdx.x == 0)
          __hip_atomic_store(flags + kp * 64 + utile, base + static_cast<unsigned>(tp + 1), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
      }
      // Every wave's products of this sub-step are done: its LDS buffer takes
      // the DMA of sub-step s + 2, tile k2's h_{t2 - 1}, once every block has
      // published it.  (Issued between the products instead, by either half's
      // waves, it costs them as much: LDS takes its writes in the same time.)
      if (t2 >= 1 && t2 + 1 < T) {
        const unsigned target = base + static_cast<unsigned>(t2);
        if (!ready(target, v2)) wait_flags(k2, target);
        const uint32_t src = static_cast<uint32_t>((((t2 - 1) & 1) * NB + k2) * TBUF * 2 + rg * FRAG * 2);
        const uint32_t dst = lds_address(ring + (k & 1) * TBUF + rg * FRAG);
#pragma unroll
        for (int i = 0; i < BPW; ++i)
          dma16(xrs, static_cast<uint32_t>(lane * 16), src + static_cast<uint32_t>(4 * i * FRAG * 2),
                dst + static_cast<uint32_t>(4 * i * FRAG * 2));
      }
    });
    // The last sub-step's tail and publication (tile NB - 1 at step T - 2).
    take_part((NB - 1) & 1);
    whole_tail(integral_constant<int, NB - 1>{}, T - 2, 0);
    wait_vmem();
    __syncthreads();
    if (threadIdx.x == 0)
      __hip_atomic_store(flags + (NB - 1) * 64 + utile, base + static_cast<unsigned>(T - 1), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  };

  for (int job = grp; job < p.jobs; job += p.groups, base += static_cast<unsigned>(T - 1)) {
    const int bb = job % p.bblocks, sj = job / p.bblocks;
    const int b0 = bb * kXchgRows;                      // this job's sequences of the batch: b0 .. b0 + nb_rows - 1
    const int nrows = B - b0 < kXchgRows ? B - b0 : kXchgRows;
    const int sg = one_sign ? 0 : sj & 1, pj = one_sign ? sj : sj >> 1;
    const int e = pj / a.pcs, jl = pj % a.pcs;
    const int64_t slot = (static_cast<int64_t>(e) * a.PC + jl) * (one_sign ? 1 : 2) + sg;
    const __amdgpu_buffer_rsrc_t hbuf = buffer_of(a.hseq + slot * a.hrows * H, slot_bytes);
    const __amdgpu_buffer_rsrc_t gbuf =
        kL1 ? buffer_of(a.U + slot * kVocab * H4, static_cast<uint32_t>(kVocab * H4 * sizeof(float)))
            : buffer_of(a.gin + slot * gin_rows * H4, static_cast<uint32_t>(gin_rows * H4 * sizeof(float)));
    const __amdgpu_buffer_rsrc_t bbuf = buffer_of(bytes_of(a, e, jl), static_cast<uint32_t>(B * T));

    // The ring slots this job writes were read in the previous job: every
    // block must have finished it (its last publication of every tile).
    if (base > 0) {
      for (int k = 0; k < NB; ++k) wait_flags(k, base);
    }
    // Recurrent weights of this wave's gate rows and K half, split, for the
    // whole sequence (the probe scratch overlays the LDS ring; the barriers
    // inside order it after the previous job's last fragment reads).
    uint4 wh[2][NCH], wl[2][NCH];
    if constexpr (kPre) {
      // Fragments as the pre-formed matrix stores them (soma_mm.hpp).
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const _Float16* wr = reinterpret_cast<const _Float16*>(a.wpre + slot * a.wpre_slot) +
                             (static_cast<int64_t>(utile * 8 + 2 * rg + m) * 2 * KC + kh * NCH) * FRAG + lane * 8;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          wh[m][c] = *reinterpret_cast<const uint4*>(wr + c * FRAG);
          wl[m][c] = *reinterpret_cast<const uint4*>(wr + (KC + c) * FRAG);
        }
      }
    } else {
      const float seps = sg == 0 ? eps_of(a, e, kGroupLstm) : -eps_of(a, e, kGroupLstm);
      resident_weights_khalf<NCH, kRad>(wh, wl, reinterpret_cast<float*>(lds), a.theta + static_cast<int64_t>(e) * a.d,
                                        a.off_l, in + H, in, H, utile * 128, a.probe, stream_key(a.seeds[e], a.step),
                                        static_cast<uint32_t>(a.j0 + jl), static_cast<uint32_t>(a.step), seps, p.err);
    }
    if (kh == 0)
      finish_half(wh, wl, hbuf, b0, nrows);
    else
      input_half(wh, wl, gbuf, bbuf, b0);
  }
}

}  // namespace soma

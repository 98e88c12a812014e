// soma_narrow.hpp -- the narrow stacked LSTM whose width is no multiple of 64
// (fp32 products): the recurrence of a layer in one launch where the width is an
// odd multiple of 16 (k_rec_narrow), and the projection and the head with
// weights drawn once (k_proj_narrow, k_head_narrow).
//
// These widths keep fp32 operands (k_rec_step's products, sums and cell, in the
// same order: the same results bit for bit), but not its launch per time step,
// which drew every probe of the recurrent weights again and cost 9 us at any
// size.  A block owns 16 NB batch rows of one (expert, direction, sign) slot
// for the whole sequence: its weights are drawn once and stay in registers (4 H
// gate rows = 4 KG tiles of 16, dealt round the waves: the KG tiles that each
// SIMD gets are equal), h goes round through a double-buffered LDS tile with
// one barrier a step, c stays in registers.  Bound by the fp32 matrix
// instruction: KG tiles x 4 KG of 32 clocks a SIMD and step (1.3 us at H = 80).
// H <= 144: beyond it the weights (16 H^2 bytes) leave no registers.
//
// Measured against the launch per step (whole steps): 48 slots of 10 sequences
// x 64 steps, two layers, H = 80: 1196 -> 385 us (2.4 us a time step, of which
// 1.3 the products and 0.5 the cells); 2048 slots of 64 x 64, H = 80: 20.7 ->
// 14.0 ms; 1024 slots of 48 x 64, H = 144: 17.9 -> 10.2 ms; 4 slots of 1 x 63,
// H = 16: 373 -> 87 us.  Nowhere slower in that range.
#pragma once

#include "soma_kernels.hpp"

namespace soma {

constexpr int kNarrowMaxH = 144;

// Waves per block: four a SIMD while the weights, accumulators and gate inputs
// of a wave's tiles fit its 128 registers; three at H = 144 (168 registers),
// two where two row tiles share the weights at H = 112.
__host__ __device__ constexpr int narrow_waves(int kg, int nb) {
  return kg == 9 ? 12 : (kg == 7 && nb == 2 ? 8 : (4 * kg < 16 ? 4 * kg : 16));
}

template <int KG, int NB>
__global__ __launch_bounds__(64 * narrow_waves(KG, NB), 1) void k_rec_narrow(FwdArgs a, int pert) {
  constexpr int H = 16 * KG, NT = 4 * KG, NW = narrow_waves(KG, NB), MT = (NT + NW - 1) / NW;
  constexpr int ROWS = 16 * NB, LD = H + 8;             // an odd multiple of 8 floats: conflict-free b128 reads
  __shared__ __attribute__((aligned(16))) float hs[2][ROWS][LD];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int B = a.B, T = a.T, in = a.in_l;
  const int64_t R = static_cast<int64_t>(T - 1) * B;
  const int bt = (B + ROWS - 1) / ROWS;
  const int b0 = static_cast<int>(blockIdx.x % bt) * ROWS, ps = blockIdx.x / bt;
  const int sg = ps % a.ns, pj = ps / a.ns;
  const int e = pj / a.pcs, jl = pj % a.pcs;
  const int64_t slot = (static_cast<int64_t>(e) * a.PC + jl) * a.ns + sg;

  // Row lr of tile i is gate lr & 3 of unit 4 (wave + NW i) + (lr >> 2).
  float4 w[MT][KG];
  {
    const float* th = a.theta + static_cast<int64_t>(e) * a.d;
    const uint2 key = pert ? stream_key(a.seeds[e], a.step) : make_uint2(0u, 0u);
    const uint32_t pair = static_cast<uint32_t>(a.j0 + jl), step_lo = static_cast<uint32_t>(a.step);
    const float eps = pert ? eps_of(a, e, kGroupLstm) : 0.0f, seps = sg == 0 ? eps : -eps;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int tile = wave + NW * i;
      if (tile >= NT) continue;                         // wave-uniform
      const int prow = tile * 16 + lr;
      const int64_t wrow = a.off_l + static_cast<int64_t>((prow & 3) * H + (prow >> 2)) * (in + H) + in;
#pragma unroll
      for (int g = 0; g < KG; ++g) {
        const int64_t kk = wrow + 16 * g + 4 * lg;
        w[i][g] = *reinterpret_cast<const float4*>(th + kk);
        if (pert) w[i][g] = fma4(seps, probe_quad(a.probe, key, pair, step_lo, static_cast<uint64_t>(kk)), w[i][g]);
      }
    }
  }

  // Rows past the batch compute on row B - 1's inputs and are never stored.
  const uint8_t* by[NB];
  const float* gp[NB];                                  // gate inputs of this lane's row: U's slot, or gin's row
  float* hp[NB];
  int v[NB];
  float cs[MT][NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int b = b0 + nb * 16 + lr, bc = b < B ? b : B - 1;
    by[nb] = bytes_of(a, e, jl) + static_cast<int64_t>(bc) * T;
    gp[nb] = (a.layer == 0 ? a.U + slot * kVocab * (4 * H) : a.gin + (slot * R + bc) * (4 * H)) + 16 * wave + 4 * lg;
    hp[nb] = a.hseq + (slot * R + bc) * H + 4 * wave + lg;
    v[nb] = a.layer == 0 ? by[nb][0] : 0;
#pragma unroll
    for (int i = 0; i < MT; ++i) cs[i][nb] = 0.0f;
  }
  float4 gi[MT][NB];
  // Gate inputs of step t; layer 1 also fetches the bytes of step t + 1 (the
  // last step's byte index is T - 1, inside the row).
  auto load_inputs = [&](int t) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const float* p = gp[nb] + (a.layer == 0 ? static_cast<int64_t>(v[nb]) * (4 * H)
                                              : static_cast<int64_t>(t) * B * (4 * H));
#pragma unroll
      for (int i = 0; i < MT; ++i)
        if (wave + NW * i < NT) gi[i][nb] = *reinterpret_cast<const float4*>(p + 16 * NW * i);
      if (a.layer == 0) v[nb] = by[nb][t + 1];
    }
  };
  load_inputs(0);

  for (int t = 0; t + 1 < T; ++t) {
    f32x4 acc[MT][NB];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[i][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (t > 0) {
#pragma unroll
      for (int g = 0; g < KG; ++g) {
        float4 x[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          x[nb] = *reinterpret_cast<const float4*>(&hs[(t - 1) & 1][nb * 16 + lr][16 * g + 4 * lg]);
#pragma unroll
        for (int i = 0; i < MT; ++i)
          if (wave + NW * i < NT)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[i][nb] = mfma_k16(w[i][g], x[nb], acc[i][nb]);
      }
    }
    float h[MT][NB];
#pragma unroll
    for (int i = 0; i < MT; ++i)
      if (wave + NW * i < NT)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const float ai = acc[i][nb][0] + gi[i][nb].x, af = acc[i][nb][1] + gi[i][nb].y;
          const float ag = acc[i][nb][2] + gi[i][nb].z, ao = acc[i][nb][3] + gi[i][nb].w;
          cs[i][nb] = sigmoid_f(af) * cs[i][nb] + sigmoid_f(ai) * tanh_f(ag);
          h[i][nb] = sigmoid_f(ao) * tanh_f(cs[i][nb]);
          hs[t & 1][nb * 16 + lr][4 * (wave + NW * i) + lg] = h[i][nb];
        }
    // The next step's inputs are requested before this step's stores, which a
    // wait for them would otherwise include.
    if (t + 2 < T) load_inputs(t + 1);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      if (b0 + nb * 16 + lr < B)
#pragma unroll
        for (int i = 0; i < MT; ++i)
          if (wave + NW * i < NT) hp[nb][static_cast<int64_t>(t) * B * H + 4 * NW * i] = h[i][nb];
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Projection and head of the widths that keep fp32 operands (H % 64 != 0, up to
// kNarrowMaxH): a block forms the perturbed rows of one (expert, direction,
// sign) slot once, in registers, and takes runs of 64 rows of h past them,
// requested a tile ahead and staged through LDS.  k_proj and k_head_ce draw the
// probes again for every 128 or 64 rows, half of their time; products, sums
// and their order are theirs, so the results are the same bit for bit.  Bound by
// the fp32 matrix instruction.
// ---------------------------------------------------------------------------

// Rows [64 tile, +64) of a slot's h: 64 H consecutive floats, KG float4 a thread.
template <int KG>
struct NarrowRows {
  static constexpr int H = 16 * KG, LD = H + 8;
  float4 pre[KG];
  __device__ __forceinline__ void request(const float* h, int64_t R, int64_t tile) {
    const int64_t left = (R - 64 * tile) * (H / 4);     // float4 up to the slot's end
    const float4* p = reinterpret_cast<const float4*>(h + 64 * tile * H);
#pragma unroll
    for (int i = 0; i < KG; ++i) {
      const int q = threadIdx.x + i * kThreads;
      pre[i] = q < left ? p[q] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  __device__ __forceinline__ void stage(float (&xs)[64][LD]) const {
#pragma unroll
    for (int i = 0; i < KG; ++i) {
      const int q = threadIdx.x + i * kThreads;
      *reinterpret_cast<float4*>(&xs[q / (4 * KG)][4 * (q % (4 * KG))]) = pre[i];
    }
  }
};

// Weight quads of one row starting at canonical coordinate wrow.
template <int KG>
__device__ __forceinline__ void narrow_row(float4 (&w)[KG], const FwdArgs& a, const float* th, int64_t wrow, bool pert,
                                           uint2 key, uint32_t pair, float seps) {
  const uint32_t step_lo = static_cast<uint32_t>(a.step);
  const int lg = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int g = 0; g < KG; ++g) {
    const int64_t kk = wrow + 16 * g + 4 * lg;
    w[g] = *reinterpret_cast<const float4*>(th + kk);
    if (pert) w[g] = fma4(seps, probe_quad(a.probe, key, pair, step_lo, static_cast<uint64_t>(kk)), w[g]);
  }
}

// Gate row tiles of 16 per wave: all 4 KG of them in one block of four waves
// while their weights and sums fit, else two to four blocks a slot.
__host__ __device__ constexpr int narrow_proj_tiles(int kg) { return kg == 7 ? 2 : (kg < 3 ? kg : 3); }
__host__ __device__ constexpr int narrow_proj_blocks(int kg) {
  return (kg + narrow_proj_tiles(kg) - 1) / narrow_proj_tiles(kg);
}

// Measured against k_proj (second layers; floor at 157 TFLOP/s): 1024 slots of
// 8,192 rows at H = 80 7.23 -> 4.96 ms (2.7), of 3,072 at H = 144 7.66 -> 4.87
// (3.3), 2048 slots of 4,096 at H = 48 3.29 -> 1.97 (1.0).
template <int KG>
__global__ __launch_bounds__(kThreads, 2) void k_proj_narrow(FwdArgs a, int pert, int tiles) {
  constexpr int H = 16 * KG, NT = 4 * KG, MT = narrow_proj_tiles(KG), MB = narrow_proj_blocks(KG), LD = H + 8;
  __shared__ __attribute__((aligned(16))) float xs[64][LD];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int64_t R = static_cast<int64_t>(a.T - 1) * a.B;
  const int ps = blockIdx.x / MB, tw = static_cast<int>(blockIdx.x % MB) * 4 + wave;   // tiles tw, tw + 4 MB, ..
  const int sg = ps % a.ns, pj = ps / a.ns;
  const int e = pj / a.pcs, jl = pj % a.pcs;
  const int64_t slot = (static_cast<int64_t>(e) * a.PC + jl) * a.ns + sg;
  const float* h = a.hseq + slot * R * H;
  const int64_t t0 = static_cast<int64_t>(tiles) * blockIdx.y / gridDim.y;
  const int64_t t1 = static_cast<int64_t>(tiles) * (blockIdx.y + 1) / gridDim.y;
  NarrowRows<KG> rows;
  rows.request(h, R, t0);

  float4 w[MT][KG];
  {
    const uint2 key = pert ? stream_key(a.seeds[e], a.step) : make_uint2(0u, 0u);
    const float eps = pert ? eps_of(a, e, kGroupLstm) : 0.0f;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int tile = tw + 4 * MB * i < NT ? tw + 4 * MB * i : NT - 1;   // past the last: formed, never stored
      const int prow = tile * 16 + lr;
      narrow_row<KG>(w[i], a, a.theta + static_cast<int64_t>(e) * a.d,
                     a.off_l + static_cast<int64_t>((prow & 3) * H + (prow >> 2)) * (2 * H), pert != 0, key,
                     static_cast<uint32_t>(a.j0 + jl), sg == 0 ? eps : -eps);
    }
  }
  for (int64_t tile = t0; tile < t1; ++tile) {
    __syncthreads();
    rows.stage(xs);
    __syncthreads();
    if (tile + 1 < t1) rows.request(h, R, tile + 1);
    f32x4 acc[MT][4];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) acc[i][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < KG; ++g)
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) {
        const float4 x = *reinterpret_cast<const float4*>(&xs[nb * 16 + lr][16 * g + 4 * lg]);
#pragma unroll
        for (int i = 0; i < MT; ++i)
          if (4 * KG % (4 * MB) == 0 || tw + 4 * MB * i < NT) acc[i][nb] = mfma_k16(w[i][g], x, acc[i][nb]);
      }
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      const int64_t row = tile * 64 + nb * 16 + lr;
      if (row >= R) continue;
#pragma unroll
      for (int i = 0; i < MT; ++i)
        if (tw + 4 * MB * i < NT)
          *reinterpret_cast<float4*>(a.gin + (slot * R + row) * (4 * H) + 16 * (tw + 4 * MB * i) + 4 * lg) =
              make_float4(acc[i][nb][0], acc[i][nb][1], acc[i][nb][2], acc[i][nb][3]);
    }
  }
}

// Blocks per compute unit: two while the weights, sums and requested rows fit
// 256 registers.
__host__ __device__ constexpr int narrow_head_blocks(int kg) { return kg <= 5 ? 2 : 1; }

// Wave w holds vocabulary rows [64 w, +64).  Measured against k_head_ce (floor):
// 1024 slots of 8,192 rows at H = 80 8.07 -> 3.28 ms (2.2), of 3,072 at H = 144
// 4.51 -> 2.36 (1.5), 2048 slots of 4,096 at H = 48 6.32 -> 2.56 (1.3).
template <int KG>
__global__ __launch_bounds__(kThreads, narrow_head_blocks(KG)) void k_head_narrow(FwdArgs a, int pert) {
  constexpr int H = 16 * KG, LD = H + 8;
  __shared__ __attribute__((aligned(16))) float xs[64][LD];
  __shared__ float red[4][64];
  __shared__ float tgt[64];
  __shared__ float ces[64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int B = a.B, T = a.T;
  const int64_t R = static_cast<int64_t>(T - 1) * B;
  const int ps = blockIdx.x, sg = ps % a.ns, pj = ps / a.ns;
  const int e = pj / a.pcs, jl = pj % a.pcs;
  const int64_t slot = (static_cast<int64_t>(e) * a.PC + jl) * a.ns + sg;
  const float* h = a.hseq + slot * R * H;
  const int64_t t0 = static_cast<int64_t>(a.row_tiles) * blockIdx.y / gridDim.y;
  const int64_t t1 = static_cast<int64_t>(a.row_tiles) * (blockIdx.y + 1) / gridDim.y;
  NarrowRows<KG> rows;
  rows.request(h, R, t0);

  float4 w[4][KG];
  {
    const uint2 key = pert ? stream_key(a.seeds[e], a.step) : make_uint2(0u, 0u);
    const float eps = pert ? eps_of(a, e, kGroupHead) : 0.0f;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
      narrow_row<KG>(w[mb], a, a.theta + static_cast<int64_t>(e) * a.d,
                     a.off_head + static_cast<int64_t>(wave * 64 + mb * 16 + lr) * H, pert != 0, key,
                     static_cast<uint32_t>(a.j0 + jl), sg == 0 ? eps : -eps);
  }
  // Time step and sequence of this lane's next row, 16 rows on at a time.
  const uint8_t* by = bytes_of(a, e, jl);
  int64_t yt = (t0 * 64 + lr) / B;
  int yb = static_cast<int>((t0 * 64 + lr) % B);
  const int dt = 16 / B, db = 16 % B;
  for (int64_t tile = t0; tile < t1; ++tile) {
    __syncthreads();                                    // the last tile's rows and sums have been read
    rows.stage(xs);
    __syncthreads();
    if (tile + 1 < t1) rows.request(h, R, tile + 1);
    int y[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      y[nb] = tile * 64 + nb * 16 + lr < R ? by[static_cast<int64_t>(yb) * T + yt + 1] : -1;
      yt += dt;
      yb += db;
      if (yb >= B) {
        yb -= B;
        ++yt;
      }
    }
    f32x4 acc[4][4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < KG; ++g)
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) {
        const float4 x = *reinterpret_cast<const float4*>(&xs[nb * 16 + lr][16 * g + 4 * lg]);
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) acc[mb][nb] = mfma_k16(w[mb][g], x, acc[mb][nb]);
      }
    float mx[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      float m = acc[0][nb][0];
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) m = fmaxf(m, acc[mb][nb][r]);
      m = fmaxf(m, __shfl_xor(m, 16));
      m = fmaxf(m, __shfl_xor(m, 32));
      mx[nb] = m;
      if (lg == 0) red[wave][nb * 16 + lr] = m;
      // the target's logit, from the lane that holds it (y = -1 past the rows: none does)
      if ((y[nb] >> 6) == wave && ((y[nb] >> 2) & 3) == lg) {
        const int ymb = (y[nb] >> 4) & 3, yr = y[nb] & 3;
        float v = 0.0f;
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (mb == ymb && r == yr) v = acc[mb][nb][r];
        tgt[nb * 16 + lr] = v;
      }
    }
    __syncthreads();
    float se[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      const int n = nb * 16 + lr;
      mx[nb] = fmaxf(fmaxf(red[0][n], red[1][n]), fmaxf(red[2][n], red[3][n]));
      float sum = 0.0f;
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) sum += __expf(acc[mb][nb][r] - mx[nb]);
      sum += __shfl_xor(sum, 16);
      sum += __shfl_xor(sum, 32);
      se[nb] = sum;
    }
    __syncthreads();                                    // the maxima have been read
    if (lg == 0) {
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) red[wave][nb * 16 + lr] = se[nb];
    }
    __syncthreads();
    if (wave == 0) {
      if (lg == 0) {
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
          const int n = nb * 16 + lr;
          float ce = 0.0f;
          if (tile * 64 + n < R) {
            const float sum = ((red[0][n] + red[1][n]) + red[2][n]) + red[3][n];
            ce = __logf(sum) + mx[nb] - tgt[n];
          }
          ces[n] = ce;
        }
      }
      // One wave writes and reads ces: its LDS operations complete in order.
      __builtin_amdgcn_wave_barrier();
      if (lane == 0) {
        double tot = 0.0;
        for (int n = 0; n < 64; ++n) tot += static_cast<double>(ces[n]);
        a.part[slot * a.row_tiles + tile] = tot;
      }
    }
  }
}

}  // namespace soma

// soma_narrow.hpp -- the recurrence of the narrow stacked LSTM whose width is an
// odd multiple of 16 (k_rec_narrow): one launch per layer, fp32 products.
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

}  // namespace soma

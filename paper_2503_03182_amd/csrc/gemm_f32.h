// f32 GEMM for problems that fill at most half the chip with 128 x 128 tiles (the
// f32 workload's products are 256 x 256..1024): one 32 x 32 block of C per
// workgroup, its 8 waves sharing the contraction, added up through LDS in
// ascending order.
//
// What bounds it: latency.  A 128 x 128 tile puts a 256 x 256 product on 4 of
// 256 CUs, and each of its K tiles passes through LDS behind two barriers.  Here
// a wave loads its operands straight into registers (no LDS, no barrier in the
// K loop): 32 k per step, the next step's loads in flight beside 16 MFMAs of
// 32x32x2.  Any pairing of k between the operands serves as long as both use
// the same: lane half h takes k = 8 j + 4 h + i, so that a K-contiguous operand
// is read in 16-byte pieces.  Measured: 256 x 256 x 1024 89 -> 12 us, 256 x 1024 x
// 256 35 -> 5 us, TN 512 x 2048 x 1024 (64 tiles of 128) 118 -> 45 us, 1024 x 2048
// x 512 (128 tiles) 56 -> 49 us; at 512 tiles of 128 those are twice as fast.  A
// 64 x 64 block of 2 x 2 such blocks with the contraction in two was no faster
// anywhere (14 us at 256 x 1024 x 256).
#pragma once
#include "kernels.h"
#include "tps_device.h"

namespace tps {

namespace gf {

constexpr int KU = 32;     // k per step
constexpr int WK = 8;      // waves sharing the contraction
constexpr int LDP = 40;    // f32 pitch of a parked block (the two lane halves hit different banks)

// One operand's 32 rows (columns) x 32 k of a step.  KC: contiguous along k.
template <bool KC>
struct Oper {
  const float* p;
  int64_t ld;
  __device__ __forceinline__ void init(const float* base, int64_t ld_, int row0, int rows, int lane) {
    ld = ld_;
    const int row = min(row0 + (lane & 31), rows - 1);   // rows past the end are not stored
    p = KC ? base + (int64_t)row * ld : base + row;
  }
  // v[4 j + i] = element at k = k0 + 8 j + 4 h + i, zero at and past K
  __device__ __forceinline__ void load(float (&v)[16], int k0, int K, int h) const {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = k0 + 8 * j + 4 * h;
      if constexpr (KC) {
        f32x4 t = {0.f, 0.f, 0.f, 0.f};
        if (k < K) t = *reinterpret_cast<const f32x4*>(p + k);   // K % 4 == 0
#pragma unroll
        for (int i = 0; i < 4; ++i) v[4 * j + i] = t[i];
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[4 * j + i] = k + i < K ? p[(int64_t)(k + i) * ld] : 0.f;
      }
    }
  }
};

}  // namespace gf

template <int LAYOUT>
__global__ __launch_bounds__(64 * gf::WK) void gemm_f32_kernel(GemmArgs g) {
  using namespace gf;
  __shared__ float park[WK][32 * LDP];
  const int tile_m = blockIdx.x / g.tiles_n, tile_n = blockIdx.x % g.tiles_n;
  const int m0 = tile_m * 32, n0 = tile_n * 32;
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  Oper<LAYOUT != TPS_GEMM_TN> a;
  Oper<LAYOUT == TPS_GEMM_NT> b;
  a.init(static_cast<const float*>(g.A), g.lda, m0, g.M, lane);
  b.init(static_cast<const float*>(g.B), g.ldb, n0, g.N, lane);
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  float va[2][16], vb[2][16];
  // step s of this wave: k = (s WK + wave) KU ..
  const int k0 = wave * KU;
  if (k0 < g.K) {
    a.load(va[0], k0, g.K, h);
    b.load(vb[0], k0, g.K, h);
  }
  auto step = [&](int k, float (&ca)[16], float (&cb)[16], float (&na)[16], float (&nb)[16]) {
    if (k + WK * KU < g.K) {
      a.load(na, k + WK * KU, g.K, h);
      b.load(nb, k + WK * KU, g.K, h);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) acc = Mma<float>::run(ca[i], cb[i], acc);
  };
  for (int k = k0; k < g.K; k += 2 * WK * KU) {
    step(k, va[0], vb[0], va[1], vb[1]);
    if (k + WK * KU < g.K) step(k + WK * KU, va[1], vb[1], va[0], vb[0]);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) park[wave][acc_row(r, lane) * LDP + (lane & 31)] = acc[r];
  __syncthreads();

  // the block's sums, 32 columns of a row per half wave
  const int epi = g.epi;
  for (int e = threadIdx.x; e < 32 * 32; e += 64 * WK) {
    const int c = e & 31, r = e >> 5, row = m0 + r, col = n0 + c;
    if (row >= g.M || col >= g.N) continue;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < WK; ++w) v += park[w][r * LDP + c];
    float* cp = static_cast<float*>(g.C) + (int64_t)row * g.ldc + col;
    if (epi == TPS_EPI_ACC_F32) {
      v += g.overwrite ? 0.f : *cp;
    } else if (epi == TPS_EPI_GELU_GRAD) {
      v *= gelu_grad_f(static_cast<const float*>(g.aux)[(int64_t)row * g.ldaux + col]);
    } else if (epi != TPS_EPI_STORE) {
      v += static_cast<const float*>(g.bias)[col];
      if (epi == TPS_EPI_BIAS_RESID) v += static_cast<const float*>(g.resid)[(int64_t)row * g.ldr + col];
      if (epi == TPS_EPI_BIAS_GELU) {
        if (g.aux) static_cast<float*>(g.aux)[(int64_t)row * g.ldaux + col] = v;
        v = gelu_f(v);
      }
    }
    *cp = v;
  }
}

template <int LAYOUT>
static hipError_t launch_f32(GemmArgs g, hipStream_t stream) {
  g.tiles_m = (g.M + 31) / 32;
  g.tiles_n = (g.N + 31) / 32;
  hipLaunchKernelGGL((gemm_f32_kernel<LAYOUT>), dim3(g.tiles_m * g.tiles_n), dim3(64 * gf::WK), 0, stream, g);
  return hipGetLastError();
}

}  // namespace tps

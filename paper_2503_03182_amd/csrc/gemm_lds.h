// Building blocks of the bf16 GEMM (gemm_quad.h) and the attention kernels on
// gfx950: LDS fragment reads issued as inline assembly with explicit waits,
// and the GEMM epilogue, which parks accumulators in LDS to apply bias /
// residual / GeLU / GeLU' / f32 accumulation with 16-byte accesses.
#pragma once
#include <utility>

#include "kernels.h"
#include "tps_device.h"

namespace tps {

namespace gl {

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((ext_vector_type(4))) short s16x4;

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// LDS fragment reads are issued as inline assembly.  The compiler orders
// every LDS read it can see after all outstanding direct-to-LDS loads
// (s_waitcnt vmcnt(0)), which would drain the load pipeline once per K tile;
// reads it cannot see are ordered by the explicit lgkmcnt / vmcnt waits and
// barriers below instead.
__device__ __forceinline__ uint32_t lds_u32(const void* p) {
  return (uint32_t)(uintptr_t)((const __attribute__((address_space(3))) char*)p);
}
template <int OFF>
__device__ __forceinline__ bf16x8 ds_b128(uint32_t a) {
  bf16x8 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(a), "i"(OFF));
  return v;
}
template <int OFF>
__device__ __forceinline__ s16x4 ds_tr16(uint32_t a) {
  s16x4 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(a), "i"(OFF));
  return v;
}
// Wait until at most N LDS reads are outstanding (LDS reads complete in
// issue order; no scalar loads are in flight inside the K loop).
template <int N>
__device__ __forceinline__ void wait_lgkm() {
  static_assert(N >= 0 && N < 16, "lgkmcnt");
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
}
// The value is not consumed before this point (pins uses after a wait).
__device__ __forceinline__ void pin(bf16x8& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void pin(f32x4& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void lds_barrier() { asm volatile("s_barrier" ::: "memory"); }

template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
// f(integral_constant<int, i>) for i = 0 .. N-1, unrolled at compile time.
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

}  // namespace gl

// Epilogue through LDS: per 32-row strip, each wave parks its accumulators
// ([32][WN] f32) in its own LDS region, reads them back row-contiguous and
// applies the epilogue on 8 consecutive columns with 16-byte accesses.  The
// global inputs of a strip (old f32 sums, residual, kept pre-activation) are
// loaded one strip ahead, before the stores of the current strip: the
// compiler cannot move loads of one pass above the (possibly aliasing)
// stores of the previous one, so issuing them in program order first keeps
// them all in flight together.
// LDS_BYTES: LDS the kernel owns (all of it is free when this runs).
template <int EPI, int P>
struct EpiIn {
  // per pass: f32 sums (ACC_F32) or one 16-byte bf16 vector (residual / aux)
  f32x4 c0[EPI == TPS_EPI_ACC_F32 ? P : 1], c1[EPI == TPS_EPI_ACC_F32 ? P : 1];
  Vec16<bf16> v[(EPI == TPS_EPI_BIAS_RESID || EPI == TPS_EPI_GELU_GRAD) ? P : 1];
};

// acc: 16 x 16 blocks [2 TA][4]; lane l holds row l % 16 and columns 4 (l / 16)
// .. +4 of each.  Strip i is blocks 2 i and 2 i + 1 of the wave's rows.
// row_of(i, r): output row of row r of strip i; col_of(c): output column of
// column c of the wave's 64 (groups of 8 columns stay together).
// RAGGED: rows at or past M and groups of 8 columns at or past N (N a multiple
// of 8) are neither read nor written.
template <int EPI, bool RAGGED, int NWAVES, int TA, int LDS_BYTES, typename RowOf, typename ColOf>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& g, f32x4 (&acc)[2 * TA][4], char* smem, RowOf&& row_of,
                                              ColOf&& col_of, int lane, int wave) {
  constexpr int WN = 64, TM = TA;   // strips
  constexpr int LDE = WN + 4;       // f32 row pitch: the parking writes are conflict-free, rows 16-byte aligned
  static_assert(NWAVES * 32 * LDE * 4 <= LDS_BYTES, "epilogue staging must fit in LDS");
  float* strip = reinterpret_cast<float*>(smem) + wave * 32 * LDE;
  constexpr int CPR = WN / 8;             // 8-column chunks per row
  constexpr int RPP = 64 / CPR;           // rows per pass
  constexpr int P = 32 / RPP;             // passes per strip
  const int rl0 = lane / CPR, cl = (lane % CPR) * 8;
  const int col = col_of(cl);
  const bool col_ok = !RAGGED || col < g.N;
  auto ok = [&](int64_t row) { return !RAGGED || (col_ok && row < g.M); };
  Vec16<bf16> bias;
  if constexpr (EPI == TPS_EPI_BIAS || EPI == TPS_EPI_BIAS_RESID || EPI == TPS_EPI_BIAS_GELU)
    bias = col_ok ? load16(static_cast<const bf16*>(g.bias) + col) : zero16<bf16>();

  auto load_strip = [&](int i, EpiIn<EPI, P>& in) {
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const int64_t row = row_of(i, rl0 + q * RPP);
      if constexpr (EPI == TPS_EPI_ACC_F32) {
        if (g.overwrite || !ok(row)) {
          in.c0[q] = f32x4{0.f, 0.f, 0.f, 0.f};
          in.c1[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        } else {
          const f32x4* c = reinterpret_cast<const f32x4*>(static_cast<const float*>(g.C) + row * g.ldc + col);
          in.c0[q] = c[0];
          in.c1[q] = c[1];
        }
      } else if constexpr (EPI == TPS_EPI_BIAS_RESID) {
        in.v[q] = ok(row) ? load16(static_cast<const bf16*>(g.resid) + row * g.ldr + col) : zero16<bf16>();
      } else if constexpr (EPI == TPS_EPI_GELU_GRAD) {
        in.v[q] = ok(row) ? load16(static_cast<const bf16*>(g.aux) + row * g.ldaux + col) : zero16<bf16>();
      }
    }
  };
  EpiIn<EPI, P> in[2];
  load_strip(0, in[0]);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        *reinterpret_cast<f32x4*>(strip + (b * 16 + (lane & 15)) * LDE + j * 16 + (lane >> 4) * 4) = acc[2 * i + b][j];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (i + 1 < TM) load_strip(i + 1, in[(i + 1) & 1]);
    const EpiIn<EPI, P>& cur = in[i & 1];
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const int rl = q * RPP + rl0;
      const f32x4 v0 = *reinterpret_cast<const f32x4*>(strip + rl * LDE + cl);
      const f32x4 v1 = *reinterpret_cast<const f32x4*>(strip + rl * LDE + cl + 4);
      const float v[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
      const int64_t row = row_of(i, rl0 + q * RPP);
      if (!ok(row)) continue;
      if constexpr (EPI == TPS_EPI_ACC_F32) {
        f32x4* c = reinterpret_cast<f32x4*>(static_cast<float*>(g.C) + row * g.ldc + col);
        f32x4 c0 = cur.c0[q], c1 = cur.c1[q];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          c0[t] += v[t];
          c1[t] += v[4 + t];
        }
        c[0] = c0;
        c[1] = c1;
      } else {
        float out[8];
        Vec16<bf16> aux;
        if constexpr (EPI == TPS_EPI_GELU_GRAD) aux = cur.v[q];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          if constexpr (EPI == TPS_EPI_STORE) {
            out[t] = v[t];
          } else if constexpr (EPI == TPS_EPI_BIAS) {
            out[t] = v[t] + to_f32(bias.get(t));
          } else if constexpr (EPI == TPS_EPI_BIAS_RESID) {
            out[t] = v[t] + to_f32(bias.get(t)) + to_f32(cur.v[q].get(t));
          } else if constexpr (EPI == TPS_EPI_BIAS_GELU) {
            const bf16 u = from_f32<bf16>(v[t] + to_f32(bias.get(t)));
            aux.set(t, u);
            out[t] = gelu_f(to_f32(u));
          } else {
            out[t] = v[t] * gelu_grad_f(to_f32(aux.get(t)));
          }
        }
        if constexpr (EPI == TPS_EPI_BIAS_GELU)
          if (g.aux) store16(static_cast<bf16*>(g.aux) + row * g.ldaux + col, aux);
        Vec16<bf16> o;
#pragma unroll
        for (int t = 0; t < 8; ++t) o.set(t, from_f32<bf16>(out[t]));
        store16(static_cast<bf16*>(g.C) + row * g.ldc + col, o);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

}  // namespace tps

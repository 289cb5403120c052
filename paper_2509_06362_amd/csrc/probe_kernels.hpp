// Sustained vector-ALU rate of a latency evaluation's instruction mix (fma, add, minimum), measured on
// the device the library runs on: fixed instruction sequences in a loop with nothing else - no LDS, no
// memory, no branches beyond the loop's own.  What these kernels reach is the practical ceiling of
// vector issue on this chip; the nominal peak is one instruction per SIMD every two cycles.
// Instrumentation only: no entry point of the scoring path uses them.
#pragma once

#include "sweep_kernels.hpp"

namespace maaso {

constexpr int kProbeThreads = 256;

// Two records {p, a, wait} folded into the running minimum of eight requests: per request fma, fma (each
// followed by the add of the wait where there is one) and one three-input minimum, two requests
// interleaved so that no instruction reads the result of the one just before it.
// Operands: %0-%(N-1) running minima, then 4 temporaries, then N prompt lengths, then p, a of the two
// records (and their waits).
#define MAASO_FOLD2(MA, MB, LA, LB, T0, T1, T2, T3, RX, RY, UX, UY)                                  \
  "v_fma_f32 " T0 ", " RX ", " LA ", " RY "\n\t" "v_fma_f32 " T1 ", " UX ", " LA ", " UY "\n\t"        \
  "v_fma_f32 " T2 ", " RX ", " LB ", " RY "\n\t" "v_fma_f32 " T3 ", " UX ", " LB ", " UY "\n\t"        \
  "v_min3_f32 " MA ", " MA ", " T0 ", " T1 "\n\t" "v_min3_f32 " MB ", " MB ", " T2 ", " T3 "\n\t"
#define MAASO_FOLD2W(MA, MB, LA, LB, T0, T1, T2, T3, RX, RY, UX, UY, RZ, UZ)                         \
  "v_fma_f32 " T0 ", " RX ", " LA ", " RY "\n\t" "v_fma_f32 " T1 ", " UX ", " LA ", " UY "\n\t"        \
  "v_fma_f32 " T2 ", " RX ", " LB ", " RY "\n\t" "v_fma_f32 " T3 ", " UX ", " LB ", " UY "\n\t"        \
  "v_add_f32 " T0 ", " RZ ", " T0 "\n\t" "v_add_f32 " T1 ", " UZ ", " T1 "\n\t"                       \
  "v_add_f32 " T2 ", " RZ ", " T2 "\n\t" "v_add_f32 " T3 ", " UZ ", " T3 "\n\t"                       \
  "v_min3_f32 " MA ", " MA ", " T0 ", " T1 "\n\t" "v_min3_f32 " MB ", " MB ", " T2 ", " T3 "\n\t"

template <bool kWait>
__device__ __forceinline__ void fold_pair_n(float (&m)[8], const float (&L)[8], const float4& r,
                                            const float4& u) {
  float t0, t1, t2, t3;
  if (kWait)
    asm(MAASO_FOLD2W("%0", "%1", "%12", "%13", "%8", "%9", "%10", "%11", "%20", "%21", "%22", "%23", "%24", "%25")
        MAASO_FOLD2W("%2", "%3", "%14", "%15", "%8", "%9", "%10", "%11", "%20", "%21", "%22", "%23", "%24", "%25")
        MAASO_FOLD2W("%4", "%5", "%16", "%17", "%8", "%9", "%10", "%11", "%20", "%21", "%22", "%23", "%24", "%25")
        MAASO_FOLD2W("%6", "%7", "%18", "%19", "%8", "%9", "%10", "%11", "%20", "%21", "%22", "%23", "%24", "%25")
        : "+v"(m[0]), "+v"(m[1]), "+v"(m[2]), "+v"(m[3]), "+v"(m[4]), "+v"(m[5]), "+v"(m[6]), "+v"(m[7]),
          "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3)
        : "v"(L[0]), "v"(L[1]), "v"(L[2]), "v"(L[3]), "v"(L[4]), "v"(L[5]), "v"(L[6]), "v"(L[7]), "v"(r.x),
          "v"(r.y), "v"(u.x), "v"(u.y), "v"(r.z), "v"(u.z));
  else
    asm(MAASO_FOLD2("%0", "%1", "%12", "%13", "%8", "%9", "%10", "%11", "%20", "%21", "%22", "%23")
        MAASO_FOLD2("%2", "%3", "%14", "%15", "%8", "%9", "%10", "%11", "%20", "%21", "%22", "%23")
        MAASO_FOLD2("%4", "%5", "%16", "%17", "%8", "%9", "%10", "%11", "%20", "%21", "%22", "%23")
        MAASO_FOLD2("%6", "%7", "%18", "%19", "%8", "%9", "%10", "%11", "%20", "%21", "%22", "%23")
        : "+v"(m[0]), "+v"(m[1]), "+v"(m[2]), "+v"(m[3]), "+v"(m[4]), "+v"(m[5]), "+v"(m[6]), "+v"(m[7]),
          "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3)
        : "v"(L[0]), "v"(L[1]), "v"(L[2]), "v"(L[3]), "v"(L[4]), "v"(L[5]), "v"(L[6]), "v"(L[7]), "v"(r.x),
          "v"(r.y), "v"(u.x), "v"(u.y));
}


// pattern 0: pair body without a queue wait (two fma, one three-input minimum per request), 24
//            instructions per trip;  1: with the wait's add, 40 per trip;  2: pattern 0 four times
//            per trip (96);  3: eight compares that write a lane mask, each followed by an add that
//            keeps it alive (16 per trip);  4: eight fma with a scalar-register operand.
template <int kPattern>
__global__ __launch_bounds__(kProbeThreads, 8) void valu_probe_kernel(float* out, uint32_t trips, float seed) {
  float m[8], L[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) { m[q] = 1.0e30f; L[q] = seed + (float)(threadIdx.x + q); }
  float4 r = make_float4(seed * 1.0e-5f, seed * 1.0e-2f, seed * 1.0e-3f, 0.0f);
  float4 u = make_float4(seed * 2.0e-5f, seed * 2.0e-2f, seed * 2.0e-3f, 0.0f);
  uint32_t hits = 0;
  for (uint32_t t = 0; t < trips; ++t) {
    if (kPattern == 0) fold_pair_n<false>(m, L, r, u);
    if (kPattern == 1) fold_pair_n<true>(m, L, r, u);
    if (kPattern == 2) {
      fold_pair_n<false>(m, L, r, u);
      fold_pair_n<false>(m, L, u, r);
      fold_pair_n<false>(m, L, r, u);
      fold_pair_n<false>(m, L, u, r);
    }
    if (kPattern == 3) {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        uint32_t h;
        asm volatile("v_cmp_le_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, 0, %3, vcc"
                     : "=v"(h) : "v"(L[q]), "v"(m[q]), "v"(hits) : "vcc");
        hits = h;
      }
    }
    if (kPattern == 4) {
      const float k = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, r.x)));
#pragma unroll
      for (int q = 0; q < 8; ++q) asm volatile("v_fma_f32 %0, %1, %2, %0" : "+v"(m[q]) : "s"(k), "v"(L[q]));
    }
    asm volatile("" : "+v"(r.x), "+v"(u.x));  // the records are not loop constants to the compiler
  }
  float s = (float)hits;
#pragma unroll
  for (int q = 0; q < 8; ++q) s += m[q];
  out[(size_t)blockIdx.x * kProbeThreads + threadIdx.x] = s;
}

}  // namespace maaso

// gpuos_device.h -- device code shared by the library's own kernels (gpuos_kernels.hip) and by the
// worker kernels that are compiled at run time for operators defined as programs (the source of
// this file is embedded in the library for that): memory access policy, element conversions, the
// operator library, the execution paths, the chunk executor and the worker loop.  Device code only;
// compiles under hipcc and under the run-time compiler.
#pragma once
#if !defined(__HIPCC_RTC__)
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "../../include/gpuos.h"
#endif
#include "gpuos_internal.h"

namespace gpuos {


#define SC_AGENT __HIP_MEMORY_SCOPE_AGENT
#define SC_SYSTEM __HIP_MEMORY_SCOPE_SYSTEM

#define DEV __device__ __forceinline__
// The per-path executors are real functions (not inlined into the worker loop): each gets a
// register allocation of its own, so the streaming loops do not inherit the worker loop's live values.
#define PATHFN __device__ __attribute__((noinline))

// ---------------------------------------------------------------------------
// memory access policy
//
// The persistent kernel never reaches a kernel boundary, and the 8 XCDs have
// one L2 each that are not coherent with each other for ordinary accesses.
// Agent-scope acquire / release fences would make a task's data visible, but
// they write back / invalidate a whole L2 on every chunk, which costs more than
// half of the HBM bandwidth when a thousand workgroups do it.  Instead every
// access to task data, descriptors and work units made by the persistent
// kernel carries the system-scope cache policy (sc0 sc1: stores write through
// to memory, loads do not hit stale lines).  With that, "release" is: wait until this wave's stores are
// acknowledged (s_waitcnt), then publish with a relaxed atomic store; "acquire"
// is: observe the flag with a relaxed atomic load, then read with the same
// policy.  No L2-wide maintenance happens in the steady state.
//
// 16-byte accesses go through buffer instructions whose resource is rebased to
// the chunk being processed: the hardware bounds-checks them (out-of-range
// loads return 0, stores are dropped).  The ordinary one-launch-per-task kernel
// uses POL_PLAIN (kernel-boundary coherence as for any kernel).
//
// The non-temporal hint (nt) keeps a line out of the memory-side cache (256 MB): what the next operation reads
// is then in memory, and the parts of a line that two stores write each go there by themselves.  So:
//   * contiguous aligned elementwise operations load and store with it (their stores are whole lines) where a task reads much
//     (RF_STREAM: 4 MB; EXP, DIV and SUB_EXP 16 MB), so that it leaves what is there in place; both GELUs never, they are bound
//     by their instructions;
//   * those by rows or by pairs load with it from 1 MB on and store without; ROW2D, transposed tiles and the gather path have
//     it on nothing;
//   * reductions load with it from 4 MB on, of whole aligned rows of up to 64 vectors from 16 MB on, of rows that go by way of
//     the LDS never;
//   * runs have it on nothing (each link's result is read by no one but may be, their inputs are the chain's);
//   * row operations store with it and load without: the rows' readers are a matrix product away, and the inputs stay.
// Measured against nt on every 16-byte access, three sets of buffers in turn / one set over and over: 24 chains of six
// tasks 155.6 us, 134; masked softmax 38.4 and 32.3 / 37.9 and 32.4; layer norm 41.0 and 36.5; 24 layout changes 57.7 and 57.9 / 57.5 and 49.8
// (rows of 363 bf16 copied into a wider matrix, 149 MB: 86 and 52); integers 51.5 and 45.6 / 51.4 and 44.3; softmax over 32,003
// columns 139 and 134 / 139 and 117; forty streaming operations of 503 MB 110.3 and 111.6 / 110 and 95.7.  With the stores of large
// contiguous tasks, and 4 MB and 1 MB in place of 8, those took 101.2 / 98.8, the layout changes 53.1 / 50.5, and 20,000 streaming
// operations over 4 GB of inputs 55.5 ms instead of 57.7.  (From 2 MB on everywhere: 101.5 / 101.4, layout changes 55.7.)
// Streams of one operation, 1-4 GB in tasks of 8M elements, without it and with it: DIV and SUB_EXP fp32 590 and 547 us, 16-bit 298 and
// 282; EXP fp32 779 and 759; an interpreted addition 611 and 561; sums of 24 fp32 451 and 411, of 256 fp32 413 and 359, of 256 bf16 220 and
// 189.  The 16 MB: on buffers used over and over EXP of 8 MB takes 22.5 us with it, 21.7 without, four of 16 MB 36.9 and
// 37.9; DIV of 8 MB 21.2 and 20.7, of 64 MB 79.4 and 83.5.  ROW2D of 4 GB: 726 and 729 on every access, in tasks of 2 MB 487 and 479.
// By rows, on stores too: rows of 2,049 fp32 less a scalar each 928 and 972, of 1,025 bf16 in tasks of 1 MB 378 and 371.  Gathered, on
// every access: products with every third fp32 element 504 and 530, bf16 438 and 443; the gather's rounds would need two executors for it.
// ---------------------------------------------------------------------------
enum { POL_PLAIN = 0, POL_COHERENT = 1 };
typedef int v4i __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;

DEV rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, 0x00020000);
}

template <int POL, bool LOADS_NT = false, bool STORES_NT = false> struct Mem {
  static constexpr int BASE = POL == POL_COHERENT ? 17 : 0, AUX = BASE | (LOADS_NT ? 2 : 0), AUXS = BASE | (STORES_NT ? 2 : 0);     // sc0|sc1, nt
  static DEV v4i ld16(rsrc_t r, uint32_t off) { return __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, AUX); }
  static DEV v4i ld16(rsrc_t r, uint32_t off, uint32_t more) { return __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, (int)more, AUX); }      // (`more`: the same in every lane)
  // (No store of the kind: with an offset in a scalar register the compiler lets the next instruction overwrite the stored registers,
  // and on gfx950 a 16-byte store still reads them then: softmax of 16-bit rows wrote pieces of the next vector's arguments.)
  static DEV void st16(rsrc_t r, uint32_t off, v4i q) { __builtin_amdgcn_raw_buffer_store_b128(q, r, (int)off, 0, AUXS); }
  static DEV void st8(rsrc_t r, uint32_t off, uint32_t w0, uint32_t w1) {
    typedef int v2i __attribute__((ext_vector_type(2)));
    const v2i q = {(int)w0, (int)w1};
    __builtin_amdgcn_raw_buffer_store_b64(q, r, (int)off, 0, AUXS);
  }
  static DEV v4i ld8(rsrc_t r, uint32_t off) {
    const auto q = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, AUX);
    return v4i{(int)q[0], (int)q[1], 0, 0};
  }
  static DEV void stb4(rsrc_t r, uint32_t off, uint32_t w) { __builtin_amdgcn_raw_buffer_store_b32(w, r, (int)off, 0, AUXS); }
  static DEV void stb2(rsrc_t r, uint32_t off, uint32_t h) { __builtin_amdgcn_raw_buffer_store_b16((uint16_t)h, r, (int)off, 0, AUXS); }
  static DEV uint32_t ldb2(rsrc_t r, uint32_t off) { return (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)off, 0, AUX); }
  static DEV uint32_t ldb4(rsrc_t r, uint32_t off) { return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, AUX); }
  static DEV uint32_t ld4(const void* p, uint32_t i) {
    if (POL == POL_COHERENT) return __hip_atomic_load((const uint32_t*)p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return ((const uint32_t*)p)[i];
  }
  static DEV uint32_t ld2(const void* p, uint32_t i) {
    if (POL == POL_COHERENT) return __hip_atomic_load((const uint16_t*)p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return ((const uint16_t*)p)[i];
  }
  static DEV void st4(void* p, uint32_t i, uint32_t v) {
    if (POL == POL_COHERENT) __hip_atomic_store((uint32_t*)p + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    else ((uint32_t*)p)[i] = v;
  }
  static DEV void st2(void* p, uint32_t i, uint32_t v) {
    if (POL == POL_COHERENT) __hip_atomic_store((uint16_t*)p + i, (uint16_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    else ((uint16_t*)p)[i] = (uint16_t)v;
  }
};

// This wave's stores (all write-through) have been acknowledged when this returns.
DEV void drain_stores() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");   // keeps the compiler from moving stores below
  __builtin_amdgcn_s_waitcnt(0);                           // vmcnt = expcnt = lgkmcnt = 0
}
DEV void order_loads() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup"); }
// Between lanes of ONE wavefront that hand data to each other through LDS: its LDS operations execute
// in order, so this only keeps the compiler from moving them across (and waits for the counter).
DEV void lds_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------
// element conversions (fp16 / bf16 <-> fp32; RNE, denormals kept)
// ---------------------------------------------------------------------------
DEV float h2f(uint32_t b) { return (float)__builtin_bit_cast(_Float16, (uint16_t)b); }
DEV uint32_t f2h(float f) {
  // The empty asm keeps the fp32 value opaque: without it the compiler folds the producing
  // multiply / fma and this conversion into one mixed-precision instruction that rounds the
  // exact result straight to fp16 (one rounding), while the defined result is fp32 first.
  asm("" : "+v"(f));
  return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)f);
}
DEV float b2f(uint32_t b) { return __builtin_bit_cast(float, b << 16); }
DEV uint32_t f2b(float f) {
  // round-to-nearest-even, NaN stays a (quiet) NaN: gfx950 has the conversion in hardware
  // (v_cvt_pk_bf16_f32), which the compiler selects for this cast; done by hand it is six
  // integer operations per element, and the 16-bit paths are the ones short of ALU time
  return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)f);
}

template <int DT> struct Elem;
template <> struct Elem<GPUOS_F32> {
  static constexpr int V = 4, ES = 4;
  static DEV float get(const v4i& q, int k) {
    const int w = q[k];      // read the lane into a scalar first: bit-casting the element lvalue directly reads lane 0
    return __builtin_bit_cast(float, w);
  }
  static DEV void put(v4i& q, int k, float f) { q[k] = __builtin_bit_cast(int, f); }
  template <int POL> static DEV float load1(const void* p, uint32_t i) { return __builtin_bit_cast(float, Mem<POL>::ld4(p, i)); }
  template <int POL> static DEV void store1(void* p, uint32_t i, float f) { Mem<POL>::st4(p, i, __builtin_bit_cast(uint32_t, f)); }
  template <int POL> static DEV void copy1(void* o, const void* a, uint32_t i) { Mem<POL>::st4(o, i, Mem<POL>::ld4(a, i)); }
};
template <> struct Elem<GPUOS_I32> { static constexpr int V = 4, ES = 4; };      // moved and combined as words
// 16-bit elements are taken out of and put into a 32-bit word as the halves of a two-element vector:
// the compiler then reads a half with the conversion instruction's own operand selector and writes
// two converted values with one pack (fp16) or one packed conversion (bf16), where shifts and
// masks on integers cost three to four operations per element.
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bfloat2_t __attribute__((ext_vector_type(2)));
DEV float opaque_f32(float f) {
  // keeps the fp32 value a value of its own: without it the compiler folds the producing multiply /
  // fma and the conversion into one mixed-precision instruction that rounds the exact result
  // straight to 16 bits (one rounding), while the defined result is fp32 first
  asm("" : "+v"(f));
  return f;
}
template <> struct Elem<GPUOS_F16> {
  static constexpr int V = 8, ES = 2;
  static DEV float get(const v4i& q, int k) {
    const int w = q[k >> 1];
    return (float)__builtin_bit_cast(half2_t, w)[k & 1];
  }
  static DEV void put(v4i& q, int k, float f) {
    const int w = q[k >> 1];
    half2_t h = __builtin_bit_cast(half2_t, w);
    h[k & 1] = (_Float16)opaque_f32(f);
    q[k >> 1] = __builtin_bit_cast(int, h);
  }
  template <int POL> static DEV float load1(const void* p, uint32_t i) { return h2f(Mem<POL>::ld2(p, i)); }
  template <int POL> static DEV void store1(void* p, uint32_t i, float f) { Mem<POL>::st2(p, i, f2h(f)); }
  template <int POL> static DEV void copy1(void* o, const void* a, uint32_t i) { Mem<POL>::st2(o, i, Mem<POL>::ld2(a, i)); }
};
template <> struct Elem<GPUOS_BF16> {
  static constexpr int V = 8, ES = 2;
  static DEV float get(const v4i& q, int k) {
    const uint32_t w = (uint32_t)q[k >> 1];
    return __builtin_bit_cast(float, (k & 1) ? (w & 0xffff0000u) : (w << 16));
  }
  static DEV void put(v4i& q, int k, float f) {
    const int w = q[k >> 1];
    bfloat2_t h = __builtin_bit_cast(bfloat2_t, w);
    h[k & 1] = (__bf16)f;
    q[k >> 1] = __builtin_bit_cast(int, h);
  }
  template <int POL> static DEV float load1(const void* p, uint32_t i) { return b2f(Mem<POL>::ld2(p, i)); }
  template <int POL> static DEV void store1(void* p, uint32_t i, float f) { Mem<POL>::st2(p, i, f2b(f)); }
  template <int POL> static DEV void copy1(void* o, const void* a, uint32_t i) { Mem<POL>::st2(o, i, Mem<POL>::ld2(a, i)); }
};

// Element i of a float tensor whose dtype is known at run time only.  Whatever the dtype, the load
// is that of the aligned 32-bit word that holds the element (same page as the element, so it
// cannot fault; for a 16-bit element the other half of the word is dropped): one form of load, no
// branch on the dtype in front of it, so that the loads of several elements or operands can be in
// flight together.
template <int POL> DEV float load_rt(const void* p, uint32_t i, uint32_t dt) {
  const uint64_t at = (uint64_t)(__UINTPTR_TYPE__)p + (uint64_t)i * (dt == GPUOS_F32 ? 4u : 2u);
  const uint32_t w = Mem<POL>::ld4((const void*)(__UINTPTR_TYPE__)(at & ~3ull), 0);
  const uint32_t h = ((uint32_t)at & 2u) ? (w >> 16) : (w & 0xffffu);
  const uint32_t m_f32 = dt == GPUOS_F32 ? ~0u : 0u, m_f16 = dt == GPUOS_F16 ? ~0u : 0u, m_bf16 = dt == GPUOS_BF16 ? ~0u : 0u;
  return __builtin_bit_cast(float, (w & m_f32) | (__builtin_bit_cast(uint32_t, h2f(h)) & m_f16) | ((h << 16) & m_bf16));
}
template <int POL> DEV void store_rt(void* p, uint32_t i, uint32_t dt, float f) {
  if (dt == GPUOS_F32) Mem<POL>::st4(p, i, __builtin_bit_cast(uint32_t, f));
  else if (dt == GPUOS_F16) Mem<POL>::st2(p, i, f2h(f));
  else Mem<POL>::st2(p, i, f2b(f));
}

// ---------------------------------------------------------------------------
// operator library (paper Section 5.2).  fp32 in, fp32 out; the caller rounds
// to the output dtype.  GELU is evaluated in fp64 in a cancellation-free form
// and rounded once: an fp32 evaluation cannot hold 2 ulp
// for x < 0, where 1 + tanh(u) and 1 + erf(u) cancel.
// ---------------------------------------------------------------------------
template <int IMPL> struct Op;
template <> struct Op<GPUOS_IMPL_ADD> { static constexpr int N = 2; static DEV float f(float x, float y, float, float) { return x + y; } };
template <> struct Op<GPUOS_IMPL_SUB> { static constexpr int N = 2; static DEV float f(float x, float y, float, float) { return x - y; } };
template <> struct Op<GPUOS_IMPL_MUL> { static constexpr int N = 2; static DEV float f(float x, float y, float, float) { return x * y; } };
template <> struct Op<GPUOS_IMPL_DIV> { static constexpr int N = 2; static DEV float f(float x, float y, float, float) { return x / y; } };
template <> struct Op<GPUOS_IMPL_RELU> { static constexpr int N = 1; static DEV float f(float x, float, float, float) { return (x != x) ? x : (x > 0.0f ? x : 0.0f); } };
template <> struct Op<GPUOS_IMPL_EXP> { static constexpr int N = 1; static DEV float f(float x, float, float, float) { return expf(x); } };
// Both GELUs are bound by arithmetic: the fp64 library functions erfc, exp and divide cost 150-250
// instructions an element (8.4M bf16 elements, four times: 112 us; 77 now).  What is evaluated
// instead, in fp64 for every dtype:
//   ERF   x Phi(x), with Phi(-a) = 2^(-a^2 log2(e)/2) P(t) / (a + k), t = (a - k) / (a + k): the scaled
//         complementary error function times (a + k) is smooth in t over all a >= 0, and P is its
//         Chebyshev fit over [0, 14.5] (beyond, x Phi(-a) is 0 in every output format).
//   TANH  x / (1 + 2^z), z = -2 log2(e) u.
// P (k = 6, degree 18) and 2^r (degree 11) hold 2^-52.9 and 2^-55.5.  Measured against 113 bits over
// 60,000 values in each of nine ranges of either sign: ERF at most 2^-50.2 off everywhere (the
// library form 2^-52 to 2^-44.8), TANH as the library form within a quarter of a bit; no fp32 result
// of either was rounded otherwise than the exact value.
DEV double rcp64(double v) {                           // (the hardware's reciprocal is good to 2^-23: one step of third order)
  const double d = __builtin_amdgcn_rcp(v), e = __builtin_fma(-v, d, 1.0);
  return __builtin_fma(d, __builtin_fma(e, e, e), d);
}
DEV double exp2_64(double k, double s) {               // 2^(k s), |k s| <= 1020; the product is rounded for its integer part only
  const double n = __builtin_rint(k * s), r = __builtin_fma(k, s, -n);
  double p = 4.4558179083360645e-10;
  p = __builtin_fma(p, r, 7.0741942972885211e-09);
  p = __builtin_fma(p, r, 1.0178057087733941e-07);
  p = __builtin_fma(p, r, 1.3215432535912375e-06);
  p = __builtin_fma(p, r, 1.5252733841556773e-05);
  p = __builtin_fma(p, r, 0.00015403530463724353);
  p = __builtin_fma(p, r, 0.0013333558146406471);
  p = __builtin_fma(p, r, 0.0096181291075872564);
  p = __builtin_fma(p, r, 0.055504108664821625);
  p = __builtin_fma(p, r, 0.24022650695910158);
  p = __builtin_fma(p, r, 0.69314718055994529);
  p = __builtin_fma(p, r, 1.0);
  return __builtin_ldexp(p, (int)n);
}
constexpr double kHalfLog2e = 0.72134752044448170368;                 // log2(e) / 2
constexpr double kTanhZ1 = -2.30220819814432489;                      // -2 log2(e) sqrt(2/pi)
constexpr double kTanhZ3 = kTanhZ1 * 0.044715;
template <> struct Op<GPUOS_IMPL_GELU_ERF> {
  static constexpr int N = 1;
  static DEV float f(float x, float, float, float) {
    const double xd = (double)x, a = __builtin_fabs(xd), c = __builtin_fmin(a, 14.5);
    const double d = rcp64(c + 6.0), t = __builtin_fma(-12.0, d, 1.0);
    double p = 9.4493983714996806e-08;
    p = __builtin_fma(p, t, 3.313519355067924e-07);
    p = __builtin_fma(p, t, -5.3093212564717683e-07);
    p = __builtin_fma(p, t, -1.9020061133223297e-06);
    p = __builtin_fma(p, t, 6.7987559520099021e-06);
    p = __builtin_fma(p, t, 1.1248503341662688e-06);
    p = __builtin_fma(p, t, -6.4735423425417934e-05);
    p = __builtin_fma(p, t, 0.00018135137862420019);
    p = __builtin_fma(p, t, 3.286459436615171e-05);
    p = __builtin_fma(p, t, -0.0021316045793056183);
    p = __builtin_fma(p, t, 0.010029821405329551);
    p = __builtin_fma(p, t, -0.030985315502152118);
    p = __builtin_fma(p, t, 0.075171915614156148);
    p = __builtin_fma(p, t, -0.15268023206701492);
    p = __builtin_fma(p, t, 0.26797424584358071);
    p = __builtin_fma(p, t, -0.41390358577550523);
    p = __builtin_fma(p, t, 0.56896889181475718);
    p = __builtin_fma(p, t, -0.7010090295908662);
    p = __builtin_fma(p, t, 0.77735177189336224);
    const double q = p * d * exp2_64(-kHalfLog2e, c * c);
    // max(x, 0) - a Phi(-a), with c for a (infinite a; beyond 14.5 the term is 0 in every format) and NaN for -inf,
    // as the definition has it; the sign is x's, also of a zero
    return __builtin_copysignf((float)__builtin_fma(-c, q, 0.5 * (xd + a)), x);
  }
};
template <> struct Op<GPUOS_IMPL_GELU_TANH> {
  static constexpr int N = 1;
  static DEV float f(float x, float, float, float) {
    const double xd = (double)x, z = xd * __builtin_fma(kTanhZ3, xd * xd, kTanhZ1);
    const double r = rcp64(1.0 + exp2_64(1.0, __builtin_fmax(__builtin_fmin(z, 600.0), -600.0)));
    return (float)(xd * (z > 600.0 ? 0.0 : r));
  }
};
template <> struct Op<GPUOS_IMPL_SCALE> { static constexpr int N = 1; static DEV float f(float x, float, float, float a) { return x * a; } };
template <> struct Op<GPUOS_IMPL_FMA> { static constexpr int N = 3; static DEV float f(float x, float y, float z, float) { return __builtin_fmaf(x, y, z); } };
template <> struct Op<GPUOS_IMPL_SUB_EXP> { static constexpr int N = 2; static DEV float f(float x, float y, float, float) { const float d = x - y; return expf(d); } };
template <> struct Op<GPUOS_IMPL_COPY> { static constexpr int N = 1; static DEV float f(float x, float, float, float) { return x; } };

// ---------------------------------------------------------------------------
// operator programs: elementwise operators defined at run time, interpreted.  The program of
// the chunk being executed sits in LDS (exec_program puts it there); every lane runs the same
// instruction on its own element, so opcode and register numbers are wavefront-uniform and the
// loop over the instructions is scalar control flow.  One IEEE binary32 operation per instruction.
// ---------------------------------------------------------------------------
__shared__ ProgramImage g_prog;

// internal implementation tags: "the program in LDS, taking N inputs"
enum { kImplProg1 = 201, kImplProg2 = 202, kImplProg3 = 203 };

// The same program over K elements at once: every instruction is decoded once (scalar work) and
// applied to the K elements a lane holds, so the interpreter's overhead is shared by a whole
// 16-byte vector instead of being paid per element.
template <int K>
DEV void run_program_vec(const float (&x)[K], const float (&y)[K], const float (&z)[K], float alpha, float (&o)[K]) {
  // The register file is eight separately named arrays selected by a switch on the (uniform)
  // register number: a dynamically indexed array would be placed in scratch memory.
  float r0[K], r1[K], r2[K], r3[K], r4[K], r5[K], r6[K], r7[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    r0[k] = x[k]; r1[k] = y[k]; r2[k] = z[k]; r3[k] = alpha;
    r4[k] = 0.f; r5[k] = 0.f; r6[k] = 0.f; r7[k] = 0.f;
  }
#define GPUOS_RF_COPY(dst, src) _Pragma("unroll") for (int k = 0; k < K; ++k) dst[k] = src[k];
#define GPUOS_RF_READ(dst, idx) switch (idx) { \
    case 0: GPUOS_RF_COPY(dst, r0) break; case 1: GPUOS_RF_COPY(dst, r1) break; \
    case 2: GPUOS_RF_COPY(dst, r2) break; case 3: GPUOS_RF_COPY(dst, r3) break; \
    case 4: GPUOS_RF_COPY(dst, r4) break; case 5: GPUOS_RF_COPY(dst, r5) break; \
    case 6: GPUOS_RF_COPY(dst, r6) break; default: GPUOS_RF_COPY(dst, r7) break; }
#define GPUOS_RF_WRITE(idx, src) switch (idx) { \
    case 0: GPUOS_RF_COPY(r0, src) break; case 1: GPUOS_RF_COPY(r1, src) break; \
    case 2: GPUOS_RF_COPY(r2, src) break; case 3: GPUOS_RF_COPY(r3, src) break; \
    case 4: GPUOS_RF_COPY(r4, src) break; case 5: GPUOS_RF_COPY(r5, src) break; \
    case 6: GPUOS_RF_COPY(r6, src) break; default: GPUOS_RF_COPY(r7, src) break; }
  const uint32_t n = __builtin_amdgcn_readfirstlane(g_prog.n_instr);
  for (uint32_t i = 0; i < n; ++i) {
    const uint32_t w = __builtin_amdgcn_readfirstlane(g_prog.code[2 * i]);
    const float imm = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(g_prog.code[2 * i + 1]));
    const uint32_t op = w & 0xffu, d = (w >> 8) & 7u, ia = (w >> 16) & 7u, ib = (w >> 24) & 7u;
    float a[K], b[K], v[K];
    GPUOS_RF_READ(a, ia)
    GPUOS_RF_READ(b, ib)
    switch (op) {
#define GPUOS_PC_CASE(code, expr) case code: _Pragma("unroll") for (int k = 0; k < K; ++k) v[k] = (expr); break;
      GPUOS_PC_CASE(GPUOS_PC_MOV, a[k])
      GPUOS_PC_CASE(GPUOS_PC_IMM, imm)
      GPUOS_PC_CASE(GPUOS_PC_ADD, a[k] + b[k])
      GPUOS_PC_CASE(GPUOS_PC_SUB, a[k] - b[k])
      GPUOS_PC_CASE(GPUOS_PC_MUL, a[k] * b[k])
      GPUOS_PC_CASE(GPUOS_PC_DIV, a[k] / b[k])
      GPUOS_PC_CASE(GPUOS_PC_MAX, (a[k] != a[k]) ? a[k] : ((b[k] != b[k]) ? b[k] : (a[k] > b[k] ? a[k] : b[k])))
      GPUOS_PC_CASE(GPUOS_PC_MIN, (a[k] != a[k]) ? a[k] : ((b[k] != b[k]) ? b[k] : (a[k] < b[k] ? a[k] : b[k])))
      GPUOS_PC_CASE(GPUOS_PC_NEG, -a[k])
      GPUOS_PC_CASE(GPUOS_PC_ABS, __builtin_fabsf(a[k]))
      GPUOS_PC_CASE(GPUOS_PC_RELU, (a[k] != a[k]) ? a[k] : (a[k] > 0.0f ? a[k] : 0.0f))
      GPUOS_PC_CASE(GPUOS_PC_EXP, expf(a[k]))
      GPUOS_PC_CASE(GPUOS_PC_SQRT, __builtin_sqrtf(a[k]))
#undef GPUOS_PC_CASE
      case GPUOS_PC_FMA: {
        float c[K];
        GPUOS_RF_READ(c, d)
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = __builtin_fmaf(a[k], b[k], c[k]);
      } break;
      default:
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = 0.f;
        break;
    }
    GPUOS_RF_WRITE(d, v)
  }
#pragma unroll
  for (int k = 0; k < K; ++k) o[k] = r0[k];
#undef GPUOS_RF_COPY
#undef GPUOS_RF_READ
#undef GPUOS_RF_WRITE
}

DEV float run_program(float x, float y, float z, float alpha) {      // one element (strided and ragged-tail paths)
  const float xs[1] = {x}, ys[1] = {y}, zs[1] = {z};
  float os[1];
  run_program_vec<1>(xs, ys, zs, alpha, os);
  return os[0];
}
template <> struct Op<kImplProg1> { static constexpr int N = 1; static DEV float f(float x, float, float, float a) { return run_program(x, 0.f, 0.f, a); } };
template <> struct Op<kImplProg2> { static constexpr int N = 2; static DEV float f(float x, float y, float, float a) { return run_program(x, y, 0.f, a); } };
template <> struct Op<kImplProg3> { static constexpr int N = 3; static DEV float f(float x, float y, float z, float a) { return run_program(x, y, z, a); } };

// The exponential when the result is going to be rounded to a 16-bit format: the hardware base-2
// exponential of x * log2(e).  Its relative error (2^-17 at the ends of the range: the product's
// rounding, times ln 2; one step of the hardware exponential on top) is far below half a step of
// either 16-bit format (2^-9, 2^-12), so the rounded result is the correctly rounded one or its
// neighbour, inside the 2 units allowed; the full-precision routine it replaces costs about twenty
// operations where this costs two (fp16) or seven (bf16).  The hardware exponential flushes results
// below fp32's normal range.  fp16 does not care (everything below 2^-25 rounds to zero there);
// bf16 shares fp32's range, so there the argument is raised by 64 and the result scaled back with an
// exact multiplication, which rounds into the subnormal range correctly.
template <int DT> DEV float exp_for_16bit(float x) {
  const float t = x * 1.44269504088896340736f;
  if (DT == GPUOS_F16) return __builtin_amdgcn_exp2f(t);
  const bool low = t < -120.0f;
  return __builtin_amdgcn_exp2f(low ? t + 64.0f : t) * (low ? 0x1.0p-64f : 1.0f);
}
// Op<IMPL> as it is evaluated when the output dtype is DT
template <int IMPL, int DT> struct OpOut : Op<IMPL> {};
template <> struct OpOut<GPUOS_IMPL_EXP, GPUOS_F16> { static constexpr int N = 1; static DEV float f(float x, float, float, float) { return exp_for_16bit<GPUOS_F16>(x); } };
template <> struct OpOut<GPUOS_IMPL_EXP, GPUOS_BF16> { static constexpr int N = 1; static DEV float f(float x, float, float, float) { return exp_for_16bit<GPUOS_BF16>(x); } };
template <> struct OpOut<GPUOS_IMPL_SUB_EXP, GPUOS_F16> { static constexpr int N = 2; static DEV float f(float x, float y, float, float) { const float d = x - y; return exp_for_16bit<GPUOS_F16>(d); } };
template <> struct OpOut<GPUOS_IMPL_SUB_EXP, GPUOS_BF16> { static constexpr int N = 2; static DEV float f(float x, float y, float, float) { const float d = x - y; return exp_for_16bit<GPUOS_BF16>(d); } };

// GELU_ERF of a vector of bf16 elements: evaluated in fp32 with a bound on its relative error, and in fp64, as above,
// where the two ends of that bound do not round to the same bf16 value (Ziv's rounding test).  Bound by arithmetic (half
// of it gone, a large tensor is bound by memory): what decides is instructions an element, 30 against 60.
// The formula of Op<GELU_ERF> with k = 3 and degree 8 (2^-25.1); a * a is exact for a 16-bit a, so the
// exponent is carried in two words.  2^-21 is no sum of worst cases (2^-21.7 for the formula in fp32, and the last
// bits of the hardware's reciprocal and exponential on top would pass it): there are 65,536 inputs, and the tests compare
// every one with fp64, bit for bit.  (Near zero, at infinity and for NaN both ends round alike.  bf16 reaches down
// to where fp32 has no more normal numbers: there, below -12, fp64 decides always.)
// It is for batches of several vectors a lane.  A wavefront falls back for one vector in 16, and waits for a chain of
// 60 dependent instructions then, which other vectors in flight hide and a lone one does not.  Not for f16 and not for
// GELU_TANH, which are in doubt 8 and 2 times as often (three more bits of a result; a bound that grows with the exponent):
// four tasks of 164K elements, fp64 against this, f16 ERF 26.1 and 27.7 us, f16 TANH 21.1 and 27.4, bf16 TANH 20.8 and 25.0;
// two of 8.4M, 54.4 and 52.1, 40.3 and 51.2, 40.0 and 45.3.  (bf16 ERF: 26.3 and 22.2; 54.9 and 38.8.)
DEV float gelu_erf_fp32(float x) {
  const float a = __builtin_fabsf(x), c = __builtin_fminf(a, 12.0f), s = c * c;
  const float d = __builtin_amdgcn_rcpf(c + 3.0f), t = __builtin_fmaf(-6.0f, d, 1.0f);
  float p = -0.00028271329938434064f;
  p = __builtin_fmaf(p, t, -0.0009280924568884075f);
  p = __builtin_fmaf(p, t, 0.0010787147330120206f);
  p = __builtin_fmaf(p, t, 0.0069399685598909855f);
  p = __builtin_fmaf(p, t, -0.01047808863222599f);
  p = __builtin_fmaf(p, t, -0.04725917801260948f);
  p = __builtin_fmaf(p, t, 0.23001901805400848f);
  p = __builtin_fmaf(p, t, -0.5093321204185486f);
  p = __builtin_fmaf(p, t, 0.7290836572647095f);
  constexpr float KH = (float)-kHalfLog2e, KL = (float)(-kHalfLog2e - (double)KH);
  const float z = s * KH, e = __builtin_fmaf(s, KL, __builtin_fmaf(s, KH, -z));        // the exponent is z + e
  float q = p * d * __builtin_amdgcn_exp2f(z);
  q = __builtin_fmaf(q, e * 0.6931472f, q);
  return __builtin_copysignf(__builtin_fmaf(-c, q, 0.5f * (x + a)), x);
}
DEV void gelu_erf_bf16(const float (&x)[8], float (&o)[8]) {
  using E = Elem<GPUOS_BF16>;
  constexpr float eps = 0x1p-21f, limit = -12.0f;
  v4i lo = {0, 0, 0, 0}, hi = {0, 0, 0, 0};
  float least = x[0];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    o[k] = gelu_erf_fp32(x[k]);
    E::put(lo, k, __builtin_fmaf(-eps, o[k], o[k]));
    E::put(hi, k, __builtin_fmaf(eps, o[k], o[k]));
    least = __builtin_fminf(least, x[k]);
  }
  const v4i diff = lo ^ hi;
  if (__ballot((diff[0] | diff[1] | diff[2] | diff[3]) != 0 || least < limit) == 0) return;
  // (one element of the eight after the other: few vectors have more than one in doubt, and the code is there once)
#pragma unroll 1
  for (int k = 0; k < 8; ++k) {
    float xk = x[0];
    int dk = diff[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) { xk = j == k ? x[j] : xk; dk = j == k ? diff[j >> 1] : dk; }
    const bool doubt = ((uint32_t)dk & (k & 1 ? 0xffff0000u : 0xffffu)) != 0 || xk < limit;
    if (__ballot(doubt) == 0) continue;
    const float y = Op<GPUOS_IMPL_GELU_ERF>::f(xk, 0.f, 0.f, 0.f);
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = doubt && j == k ? y : o[j];
  }
}

// o[k] = f(x[k], y[k], z[k], alpha) for the K elements a lane holds (one of BATCH vectors in flight): element by element for
// the built-in implementations (the compiler unrolls it back into straight code), instruction by
// instruction for a program.
template <int IMPL, int K, int DT = GPUOS_F32, int BATCH = 1>
DEV void apply_vec(const float (&x)[K], const float (&y)[K], const float (&z)[K], float alpha, float (&o)[K]) {
  if constexpr (IMPL == GPUOS_IMPL_GELU_ERF && DT == GPUOS_BF16 && K == 8 && BATCH > 1) {
    gelu_erf_bf16(x, o);
    return;
  }
  if (IMPL == kImplProg1 || IMPL == kImplProg2 || IMPL == kImplProg3) {
    run_program_vec<K>(x, y, z, alpha, o);
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) o[k] = OpOut<IMPL, DT>::f(x[k], y[k], z[k], alpha);
  }
}

template <int IMPL> DEV uint32_t int_op(uint32_t x, uint32_t y) {
  if (IMPL == GPUOS_IMPL_ADD) return x + y;
  if (IMPL == GPUOS_IMPL_SUB) return x - y;
  if (IMPL == GPUOS_IMPL_MUL) return x * y;
  return x;
}

DEV uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
DEV const char* uni_ptr(uint64_t p) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
  return (const char*)(((uint64_t)hi << 32) | lo);
}
// Arguments of a PATHFN function arrive in vector registers and pointers arrive generic.  Both
// facts are restored on entry: values the whole workgroup shares go back to scalar registers
// (uni / uni_ptr), and a pointer known to address LDS goes back to the LDS address space (so that
// it is read with LDS instructions, not flat ones).
template <class T> DEV T* lds_arg(T* p) {
  typedef __attribute__((address_space(3))) T* lds_t;
  uint32_t a = uni((uint32_t)(__UINTPTR_TYPE__)(lds_t)p);
  asm("" : "+s"(a));                 // (or the conversions fold away: the pointer is generic again, every access through it flat)
  return (T*)(lds_t)(__UINTPTR_TYPE__)a;
}
// This thread's index in the workgroup, from its wavefront's index (a scalar).  The executors get it as an
// argument, and the worker finds it anew for each unit (the empty asm keeps it from being carried over).
// threadIdx.x in an executor would make every call hand over the work-item id, and the worker kernel,
// which has to keep that across calls that preserve few vector registers, kept it in scratch
// memory: three loads from there in a row on every unit, 0.3 us, with one set of executors, none with another.
DEV uint32_t lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }
DEV uint32_t thread_index(uint32_t wave) {
  uint32_t zero = 0;
  asm volatile("" : "+v"(zero));
  return wave * 64u + __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
}

// K 16-byte vectors of one operand; or, under MixArg, one scalar per vector in their place (of any
// dtype: `word` holds the bits of an fp32 value, or an int32).
template <int DT, int K> struct VecArg {
  const v4i (&q)[K];
  DEV v4i raw(int u) const { return q[u]; }
  DEV float get(int u, int k) const { return Elem<DT>::get(q[u], k); }
  DEV uint32_t word(int u, int k) const { return (uint32_t)q[u][k]; }
};
template <int DT, int K> struct MixArg {
  const v4i (&q)[K];
  const uint32_t (&w)[K];
  bool scalar;
  DEV v4i raw(int u) const { return q[u]; }
  DEV float get(int u, int k) const { return scalar ? __builtin_bit_cast(float, w[u]) : Elem<DT>::get(q[u], k); }
  DEV uint32_t word(int u, int k) const { return scalar ? w[u] : (uint32_t)q[u][k]; }
};

// K vectors of an elementwise operation: floats through fp32, I32 word by word, COPY as it is (bits).
// Each result goes to sink(u, vector) as soon as it is there.
template <int IMPL, int DT, int K, class A, class B, class C, class S> DEV void ew_vectors(const A& a, const B& b, const C& c, float alpha, S sink) {
  using E = Elem<DT>;
  constexpr int V = E::V;
#pragma unroll
  for (int u = 0; u < K; ++u) {
    v4i q;
    if constexpr (IMPL == GPUOS_IMPL_COPY) q = a.raw(u);
    else if constexpr (DT == GPUOS_I32) {
#pragma unroll
      for (int k = 0; k < V; ++k) q[k] = (int)int_op<IMPL>(a.word(u, k), b.word(u, k));
    } else {
      constexpr int N = Op<IMPL>::N;
      float xa[V], xb[V], xc[V], xo[V];
#pragma unroll
      for (int k = 0; k < V; ++k) {
        xa[k] = a.get(u, k); xb[k] = N > 1 ? b.get(u, k) : 0.f; xc[k] = N > 2 ? c.get(u, k) : 0.f;
      }
      apply_vec<IMPL, V, DT, K>(xa, xb, xc, alpha, xo);
#pragma unroll
      for (int k = 0; k < V; ++k) E::put(q, k, xo[k]);
    }
    sink(u, q);
  }
}

// The operator as an executor sees it.  FixedOp: one implementation, the executor is instantiated for
// it (operators of many instructions, programs, native code).  ByArity: the built-in operators of N
// inputs and a few instructions share one executor, which decides between them when the round's loads
// are on their way: the decision costs nothing there.  (An executor per operator makes the choice
// among 12 x 3 x paths executors in front of the first load: every many-way branch of this kernel
// becomes a chain that is walked case by case, and each further path put 0.25 us on every unit.)
template <int IMPL> struct FixedOp {
  static constexpr int N = Op<IMPL>::N;
  template <int DT, int K, class A, class B, class C, class S> static DEV void vectors(uint32_t, const A& a, const B& b, const C& c, float alpha, S sink) {
    ew_vectors<IMPL, DT, K>(a, b, c, alpha, sink);
  }
};
template <int ARITY> struct ByArity {
  static constexpr int N = ARITY;
  template <int DT, int K, class A, class B, class C, class S> static DEV void vectors(uint32_t impl, const A& a, const B& b, const C& c, float alpha, S sink) {
    if constexpr (DT == GPUOS_I32) {
      if constexpr (N == 1) ew_vectors<GPUOS_IMPL_COPY, DT, K>(a, b, c, alpha, sink);
      else if (impl == GPUOS_IMPL_ADD) ew_vectors<GPUOS_IMPL_ADD, DT, K>(a, b, c, alpha, sink);
      else if (impl == GPUOS_IMPL_SUB) ew_vectors<GPUOS_IMPL_SUB, DT, K>(a, b, c, alpha, sink);
      else ew_vectors<GPUOS_IMPL_MUL, DT, K>(a, b, c, alpha, sink);
    } else if constexpr (N == 1) {
      if (impl == GPUOS_IMPL_COPY) ew_vectors<GPUOS_IMPL_COPY, DT, K>(a, b, c, alpha, sink);
      else if (impl == GPUOS_IMPL_SCALE) ew_vectors<GPUOS_IMPL_SCALE, DT, K>(a, b, c, alpha, sink);
      else if (impl == GPUOS_IMPL_RELU) ew_vectors<GPUOS_IMPL_RELU, DT, K>(a, b, c, alpha, sink);
      else ew_vectors<GPUOS_IMPL_EXP, DT, K>(a, b, c, alpha, sink);
    } else if constexpr (N == 2) {
      if (impl == GPUOS_IMPL_ADD) ew_vectors<GPUOS_IMPL_ADD, DT, K>(a, b, c, alpha, sink);
      else if (impl == GPUOS_IMPL_MUL) ew_vectors<GPUOS_IMPL_MUL, DT, K>(a, b, c, alpha, sink);
      else if (impl == GPUOS_IMPL_SUB) ew_vectors<GPUOS_IMPL_SUB, DT, K>(a, b, c, alpha, sink);
      else if (impl == GPUOS_IMPL_DIV) ew_vectors<GPUOS_IMPL_DIV, DT, K>(a, b, c, alpha, sink);
      else ew_vectors<GPUOS_IMPL_SUB_EXP, DT, K>(a, b, c, alpha, sink);
    } else {
      ew_vectors<GPUOS_IMPL_FMA, DT, K>(a, b, c, alpha, sink);
    }
  }
};

// ---------------------------------------------------------------------------
// PATH_CONTIG: out[i] = f(a[i], b[i], c[i]), all operands the same dtype.
// 16 bytes per lane per access, four accesses in flight per operand.
// ---------------------------------------------------------------------------
template <int POL, int IMPL, int DT, int U = 4>
PATHFN void ew_contig(const Record* r_v, uint32_t begin_v, uint32_t end_v, uint32_t tid) {
  const Record* r = lds_arg(r_v);
  uint32_t begin = uni(begin_v);
  const uint32_t end = uni(end_v);
  using E = Elem<DT>;
  using M = Mem<POL>;
  constexpr int V = E::V, N = Op<IMPL>::N;
  const char* pa = uni_ptr(r->ptr[0]);
  const char* pb = N > 1 ? uni_ptr(r->ptr[1]) : pa;
  const char* pc = N > 2 ? uni_ptr(r->ptr[2]) : pa;
  char* po = (char*)uni_ptr(r->ptr[3]);
  const float alpha = r->alpha;
  if (r->rflags & RF_VEC) {
    // buffer resources rebased to this chunk; begin is a multiple of V
    const uint32_t nvec = (end - begin) / V;
    const uint32_t bytes = nvec * 16u;
    const uint64_t boff = (uint64_t)begin * E::ES;
    const rsrc_t ra = make_rsrc(pa + boff, bytes), rb = make_rsrc(pb + boff, bytes), rc = make_rsrc(pc + boff, bytes);
    const rsrc_t ro = make_rsrc(po + boff, bytes);
    uint32_t v = tid;
    auto batches = [&](auto mem) {
      using ML = decltype(mem);
      for (; U > 1 && v + (U - 1) * kThreads < nvec; v += U * kThreads) {
        v4i qa[U], qb[U], qc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          qa[u] = ML::ld16(ra, (v + u * kThreads) * 16u);
          qb[u] = N > 1 ? ML::ld16(rb, (v + u * kThreads) * 16u) : qa[u];
          qc[u] = N > 2 ? ML::ld16(rc, (v + u * kThreads) * 16u) : qa[u];
        }
        typedef VecArg<DT, U> Arg;
        ew_vectors<IMPL, DT, U>(Arg{qa}, Arg{qb}, Arg{qc}, alpha, [&](int u, const v4i& q) { ML::st16(ro, (v + u * kThreads) * 16u, q); });
      }
    };
    // (both GELUs are bound by their instructions and take the same time either way)
    constexpr bool SHORT = IMPL != GPUOS_IMPL_GELU_ERF && IMPL != GPUOS_IMPL_GELU_TANH;
    if (SHORT && (uni(r->rflags) & RF_STREAM) != 0) batches(Mem<POL, SHORT, SHORT>{});
    else batches(M{});
    for (; v < nvec; v += kThreads) {
      v4i qa[1], qb[1], qc[1];
      qa[0] = M::ld16(ra, v * 16u);
      qb[0] = N > 1 ? M::ld16(rb, v * 16u) : qa[0];
      qc[0] = N > 2 ? M::ld16(rc, v * 16u) : qa[0];
      typedef VecArg<DT, 1> Arg;
      ew_vectors<IMPL, DT, 1>(Arg{qa}, Arg{qb}, Arg{qc}, alpha, [&](int, const v4i& q) { M::st16(ro, v * 16u, q); });
    }
    begin += nvec * V;                                // ragged tail below
  }
  for (uint32_t i = begin + tid; i < end; i += kThreads) {
    if constexpr (DT == GPUOS_I32) M::st4(po, i, int_op<IMPL>(M::ld4(pa, i), M::ld4(pb, i)));
    else if constexpr (IMPL == GPUOS_IMPL_COPY) E::template copy1<POL>(po, pa, i);
    else
      E::template store1<POL>(po, i, OpOut<IMPL, DT>::f(E::template load1<POL>(pa, i), N > 1 ? E::template load1<POL>(pb, i) : 0.f,
                                                 N > 2 ? E::template load1<POL>(pc, i) : 0.f, alpha));
  }
}
// ---------------------------------------------------------------------------
// PATH_ROW2D: contiguous [R, C] output of dtype DT, C a multiple of the vector
// width; each input is a full [R, C] tensor (dtype DT), a row vector [C]
// broadcast over rows (dtype DT), or one scalar per row (any float dtype).
// ---------------------------------------------------------------------------
constexpr uint32_t kScratchFloats = 7168;   // LDS scratch per workgroup (gather staging, transpose tiles, reduction partials): 28 KB,
                                            // still below what the dispatcher's workgroup needs, so the kernel's allocation does not grow

// KIND1 >= 0: a binary operation whose first operand is a full tensor and whose second is of that
// kind (the attention chain's layouts: full + row vector, full + per-row scalar); the kinds are then
// compile-time facts and the selects and branches on them disappear.  KIND1 < 0: kinds read from
// the descriptor.
template <int POL, int IMPL, int DT, int KIND1>
PATHFN void ew_row2d(const Record* r_v, uint32_t begin_v, uint32_t end_v, float* s_v, uint32_t tid) {
  const Record* r = lds_arg(r_v);
  const uint32_t begin = uni(begin_v), end = uni(end_v);
  float* s_scratch = lds_arg(s_v);
  using E = Elem<DT>;
  using M = Mem<POL>;
  constexpr int V = E::V, N = Op<IMPL>::N;
  const uint32_t C = uni(r->size[1]);
  const char* p[3];
  uint32_t kind[3], dt[3], st0[3];
  rsrc_t rs[3];
  const uint32_t nvec = (end - begin) / V;
  const uint64_t boff = (uint64_t)begin * E::ES;
  uint32_t n_scalar = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int kk = k < N ? k : 0;
    p[k] = uni_ptr(r->ptr[kk]);
    kind[k] = KIND1 < 0 ? uni(r->okind[kk]) : (kk == 0 ? (uint32_t)K_FULL : (uint32_t)KIND1);
    dt[k] = uni(r->dtype[kk]);
    st0[k] = uni(r->stride[kk][0]);
    // full operands: rebased to the chunk; row vectors: the whole vector
    rs[k] = kind[k] == K_FULL ? make_rsrc(p[k] + boff, nvec * 16u) : make_rsrc(p[k], C * E::ES);
    if (k < N && kind[k] == K_ROWSCALAR) ++n_scalar;
  }
  const rsrc_t ro = make_rsrc(uni_ptr(r->ptr[3]) + boff, nvec * 16u);
  const float alpha = r->alpha;
  // Per-row scalars (x - rowmax, e / rowsum): the rows of this chunk are gathered once into LDS
  // with coalesced loads and broadcast from there; without the staging every 16-byte vector would
  // cost one more uncached 4-byte memory request.
  const uint32_t row_first = begin / C, row_cnt = (end - 1) / C - row_first + 1;
  const bool staged = n_scalar != 0 && row_cnt * n_scalar <= kScratchFloats;
  // UN vectors per thread and round, all their loads issued before the first result is needed.
  // A chunk is one or two rounds, so the round is made long (a chunk of 12K 16-bit elements is
  // exactly one) and the first round's loads leave BEFORE the row scalars are staged: the chunk
  // then pays one memory latency, not three in a row.
  constexpr int UN = (N == 2 && KIND1 != (int)K_ROWVEC) ? 6 : 4;
  // (row, column) of a thread's vectors: one division per chunk, then steps with a carry
  const uint32_t step = kThreads * V;
  const uint32_t step_rows = step / C, step_cols = step - step_rows * C;
  uint32_t row, col;
  {
    const uint32_t i = begin + tid * V;
    row = i / C;
    col = i - row * C;
  }
  v4i q[UN][3];
  uint32_t rowu[UN];
  auto load_round = [&](uint32_t v0) {
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const uint32_t v = v0 + (uint32_t)u * kThreads;
      const bool act = v < nvec;
      rowu[u] = row;
#pragma unroll
      for (int k = 0; k < N; ++k) {
        if (kind[k] == K_FULL) q[u][k] = M::ld16(rs[k], act ? v * 16u : kNoLoad);
        else if (kind[k] == K_ROWVEC) q[u][k] = M::ld16(rs[k], act ? col * E::ES : kNoLoad);
      }
      row += step_rows;
      col += step_cols;
      if (col >= C) { col -= C; ++row; }
    }
  };
  auto compute_round = [&](uint32_t v0) {
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const uint32_t v = v0 + (uint32_t)u * kThreads;
      if (v < nvec) {
        float sc[3] = {0.f, 0.f, 0.f};
        uint32_t region = 0;
#pragma unroll
        for (int k = 0; k < N; ++k)
          if (kind[k] == K_ROWSCALAR) {
            if (staged) { sc[k] = s_scratch[region + rowu[u] - row_first]; region += row_cnt; }
            else sc[k] = load_rt<POL>(p[k], rowu[u] * st0[k], dt[k]);
          }
        v4i res;
        float xv[3][V], xo[V];
#pragma unroll
        for (int e = 0; e < V; ++e)
#pragma unroll
          for (int k = 0; k < 3; ++k) xv[k][e] = k < N ? ((kind[k] == K_ROWSCALAR) ? sc[k] : E::get(q[u][k], e)) : 0.f;
        apply_vec<IMPL, V, DT>(xv[0], xv[1], xv[2], alpha, xo);
#pragma unroll
        for (int e = 0; e < V; ++e) E::put(res, e, xo[e]);
        M::st16(ro, v * 16u, res);
      }
    }
  };
  load_round(tid);                           // (every thread, whatever nvec: the barrier below is for all)
  if (staged) {
    uint32_t region = 0;
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (kind[k] == K_ROWSCALAR) {
        for (uint32_t t = tid; t < row_cnt; t += kThreads)
          s_scratch[region + t] = load_rt<POL>(p[k], (row_first + t) * st0[k], dt[k]);
        region += row_cnt;
      }
    __syncthreads();
  }
  compute_round(tid);
  for (uint32_t v0 = tid + kThreads * UN; v0 < nvec; v0 += kThreads * UN) {
    load_round(v0);
    compute_round(v0);
  }
  if (staged) __syncthreads();        // the scratch may be reused by the next chunk
}

// ---------------------------------------------------------------------------
// PATH_TILE2D: contiguous [B, R, C] output where at least one input is stored with R as its
// unit-stride dim (a transposed view).  Such an input is gathered through a 32 x 32 LDS tile:
// it is read along ITS contiguous dim (coalesced), written to LDS, and read back transposed
// (pitch 33: no bank conflicts), so neither side of the transpose touches memory with a stride.
// Row-major inputs (unit stride along C, any row pitch, including 0 for a broadcast row) are
// read directly.  Any float dtype per operand.
// ---------------------------------------------------------------------------
constexpr uint32_t kTile = 32, kTilePitch = 33;

template <int POL, int IMPL>
PATHFN void ew_tile2d(const Record* r_v, uint32_t begin_v, uint32_t end_v, float* s_v, uint32_t tid) {
  const Record* r = lds_arg(r_v);
  const uint32_t tile_begin = uni(begin_v), tile_end = uni(end_v);
  float* s_scratch = lds_arg(s_v);
  constexpr int N = Op<IMPL>::N;
  const uint32_t R = uni(r->size[1]), C = uni(r->size[2]);
  const uint32_t tr = (R + kTile - 1) / kTile, tc = (C + kTile - 1) / kTile;
  const char* p[3];
  uint32_t kind[3], dt[3], sb[3], sr[3], sc[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int kk = k < N ? k : 0;
    p[k] = uni_ptr(r->ptr[kk]);
    kind[k] = uni(r->okind[kk]);
    dt[k] = uni(r->dtype[kk]);
    sb[k] = uni(r->stride[kk][0]); sr[k] = uni(r->stride[kk][1]); sc[k] = uni(r->stride[kk][2]);
  }
  char* po = (char*)uni_ptr(r->ptr[3]);
  const uint32_t odt = uni(r->dtype[3]);
  const float alpha = r->alpha;
  uint32_t m_f32[3], m_f16[3], m_bf16[3];                  // all ones for the input's dtype
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    m_f32[k] = dt[k] == GPUOS_F32 ? ~0u : 0u;
    m_f16[k] = dt[k] == GPUOS_F16 ? ~0u : 0u;
    m_bf16[k] = dt[k] == GPUOS_BF16 ? ~0u : 0u;
  }
  for (uint32_t t = tile_begin; t < tile_end; ++t) {
    const uint32_t b = t / (tr * tc), rem = t - b * tr * tc;
    const uint32_t ti = rem / tc, tj = rem - ti * tc;
    const uint32_t r0 = ti * kTile, c0 = tj * kTile;
    // Everything the tile needs is requested first, four elements per lane and input, and used
    // afterwards: one memory latency per tile, not one per element.  A transposed input is read
    // with the lanes along r (its contiguous dim), the others along c, where they are used; a lane
    // outside the tensor reads the tile's first element instead (in bounds) and drops it.  Whatever
    // the dtype, the load is that of the aligned 32-bit word that holds the element (same page, so
    // it cannot fault; the other half of the word is dropped): one form of load for every input,
    // no branch between the requests.
    uint32_t raw[3][4], upper[3][4];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const uint32_t es = dt[k] == GPUOS_F32 ? 4u : 2u;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t idx = tid + i * kThreads, lo5 = idx & (kTile - 1), hi5 = idx / kTile;
        uint32_t off;
        if (kind[k] == K_TRANSPOSED) {
          const bool in = r0 + lo5 < R && c0 + hi5 < C;
          off = b * sb[k] + r0 + c0 * sc[k] + (in ? lo5 + hi5 * sc[k] : 0u);
        } else {
          const bool in = r0 + hi5 < R && c0 + lo5 < C;
          off = b * sb[k] + r0 * sr[k] + c0 + (in ? hi5 * sr[k] + lo5 : 0u);
        }
        const uint64_t at = (uint64_t)(__UINTPTR_TYPE__)p[k] + (uint64_t)off * es;
        upper[k][i] = (uint32_t)at & 2u;
        raw[k][i] = Mem<POL>::ld4((const void*)(__UINTPTR_TYPE__)(at & ~3ull), 0);
      }
    }
    float x[3][4];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        // (masks, not branches on the dtype)
        const uint32_t w = k < N ? raw[k][i] : 0u;
        const uint32_t h = (k < N && upper[k][i]) ? (w >> 16) : (w & 0xffffu);
        const uint32_t bits = (w & m_f32[k]) | (__builtin_bit_cast(uint32_t, h2f(h)) & m_f16[k]) | ((h << 16) & m_bf16[k]);
        x[k][i] = k < N ? __builtin_bit_cast(float, bits) : 0.0f;
      }
    // the transposed operands go through LDS: written along r, read back along c
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (kind[k] == K_TRANSPOSED) {
        float* tile = s_scratch + k * (kTile * kTilePitch);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t idx = tid + i * kThreads, rr = idx & (kTile - 1), cc = idx / kTile;
          tile[cc * kTilePitch + rr] = x[k][i];
        }
      }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (kind[k] == K_TRANSPOSED) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t idx = tid + i * kThreads, cc = idx & (kTile - 1), rr = idx / kTile;
          x[k][i] = s_scratch[k * (kTile * kTilePitch) + cc * kTilePitch + rr];
        }
      }
    // compute: lanes run along c (the output's contiguous dim)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t idx = tid + i * kThreads, cc = idx & (kTile - 1), rr = idx / kTile;
      if (r0 + rr < R && c0 + cc < C)
        store_rt<POL>(po, (b * R + r0 + rr) * C + c0 + cc, odt, Op<IMPL>::f(x[0][i], x[1][i], x[2][i], alpha));
    }
    __syncthreads();                  // the tiles are rewritten by the next iteration
  }
}

// ---------------------------------------------------------------------------
// PATH_STAGED: contiguous [B, R, C] output (leading sizes may be 1: a matrix, a flat tensor), every
// input addressed by three strides of its own (any values, 0 on broadcast dims), any float dtype
// per operand, any alignment of the inputs: stride-2 slices, row and column vectors whatever C is,
// small transposes, operands of another dtype.  A round is 1024 consecutive output elements, four
// per lane.  For each input the workgroup first brings the contiguous span of memory that the
// round touches into LDS with coalesced 16-byte loads (every line is fetched once, whatever the
// stride), then each lane gathers its elements from LDS; the results leave as whole vectors.  An
// input whose span does not fit what is left of the LDS is read element by element for that
// round instead.
// ---------------------------------------------------------------------------
constexpr uint32_t kStageRound = 4u * kThreads;
constexpr int kStageLoads = 4;             // 16-byte loads per lane and input in flight while a window is staged

struct StagedCtx {     // what every round of a chunk shares (workgroup-uniform)
  const char* p[3];
  uint32_t dt[3], es[3], sb[3], sr[3], sc[3];
  uint32_t m_f32[3], m_f16[3], m_bf16[3];  // all ones for the input's dtype
  uint32_t R, C, RC, odt, oes, begin;
  char* po;
  rsrc_t ro;                               // the output rebased to the chunk: stores past it are dropped
  float alpha;
  char* lds;
};
template <int IMPL> DEV void staged_ctx(StagedCtx& c, const Record* r, uint32_t begin, uint32_t end, char* lds) {
  constexpr int N = Op<IMPL>::N;
  c.R = uni(r->size[1]); c.C = uni(r->size[2]); c.RC = c.R * c.C;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int kk = k < N ? k : 0;
    c.p[k] = uni_ptr(r->ptr[kk]);
    c.dt[k] = uni(r->dtype[kk]);
    c.es[k] = c.dt[k] == GPUOS_F32 ? 4u : 2u;
    c.sb[k] = uni(r->stride[kk][0]); c.sr[k] = uni(r->stride[kk][1]); c.sc[k] = uni(r->stride[kk][2]);
    c.m_f32[k] = c.dt[k] == GPUOS_F32 ? ~0u : 0u;
    c.m_f16[k] = c.dt[k] == GPUOS_F16 ? ~0u : 0u;
    c.m_bf16[k] = c.dt[k] == GPUOS_BF16 ? ~0u : 0u;
  }
  c.odt = uni(r->dtype[3]);
  c.oes = c.odt == GPUOS_F32 ? 4u : 2u;
  c.po = (char*)uni_ptr(r->ptr[3]);
  c.ro = make_rsrc(c.po + (uint64_t)begin * c.oes, (end - begin) * c.oes);
  c.alpha = r->alpha;
  c.begin = begin;
  c.lds = lds;
}

// One round's gather, arithmetic and store: the elements [c0, c1) of the output, inputs staged at
// g_region (element g_lo of input k lies at byte g_region[k] of the LDS scratch).  FULL: the round
// has all its 1,024 elements (every lane four live ones, one whole-vector store).  ALL_STAGED:
// every input is in LDS, and the round holds no memory load at all.
template <int POL, int IMPL, bool FULL, bool ALL_STAGED>
DEV void staged_round(const StagedCtx& c, uint32_t c0, uint32_t c1, const uint32_t (&g_lo)[3], const uint32_t (&g_region)[3],
                      const bool (&g_staged)[3], uint32_t tid) {
  using M = Mem<POL>;
  constexpr int N = Op<IMPL>::N;
  const uint32_t i = c0 + 4u * tid;
  if (!FULL && i >= c1) return;
  uint32_t b = i / c.RC;
  const uint32_t j = i - b * c.RC;
  uint32_t row = j / c.C, col = j - row * c.C;
  float x[3][4], o[4];
  // the four elements' offsets first, then every read of a staged input in one go (one LDS latency
  // per input, not one per element): the aligned word that holds the element is read whatever the
  // dtype and the element is cut out of it afterwards
  uint32_t off[3][4];
  bool live[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    live[e] = FULL || i + e < c1;
#pragma unroll
    for (int k = 0; k < N; ++k) off[k][e] = b * c.sb[k] + row * c.sr[k] + col * c.sc[k];
    if (++col == c.C) { col = 0; if (++row == c.R) { row = 0; ++b; } }
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (k >= N) {
#pragma unroll
      for (int e = 0; e < 4; ++e) x[k][e] = 0.0f;
    } else if (ALL_STAGED || g_staged[k]) {
      uint32_t w[4], at_byte[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        at_byte[e] = live[e] ? g_region[k] + (off[k][e] - g_lo[k]) * c.es[k] : g_region[k];
        w[e] = *(const uint32_t*)(c.lds + (at_byte[e] & ~3u));
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        // (masks, not branches on the dtype: the three decodings are a handful of operations)
        const uint32_t h = (at_byte[e] & 2u) ? (w[e] >> 16) : (w[e] & 0xffffu);
        const uint32_t bits = (w[e] & c.m_f32[k]) | (__builtin_bit_cast(uint32_t, h2f(h)) & c.m_f16[k]) | ((h << 16) & c.m_bf16[k]);
        x[k][e] = live[e] ? __builtin_bit_cast(float, bits) : 0.0f;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) x[k][e] = live[e] ? load_rt<POL>(c.p[k], off[k][e], c.dt[k]) : 0.0f;
    }
  }
  apply_vec<IMPL, 4>(x[0], x[1], x[2], c.alpha, o);
  const uint32_t rel = (i - c.begin) * c.oes;
  if (FULL) {
    // Both forms of the store are issued, the one that does not apply past the end of the window
    // (dropped, no traffic): the number of stores a wavefront has in flight after a full round is
    // then the same on every path, and the wait for the next round's vectors can leave them there.
    v4i qo;
#pragma unroll
    for (int e = 0; e < 4; ++e) qo[e] = __builtin_bit_cast(int, o[e]);
    uint32_t w0, w1;
    if (c.odt == GPUOS_F16) { w0 = f2h(o[0]) | (f2h(o[1]) << 16); w1 = f2h(o[2]) | (f2h(o[3]) << 16); }
    else { w0 = f2b(o[0]) | (f2b(o[1]) << 16); w1 = f2b(o[2]) | (f2b(o[3]) << 16); }
    M::st16(c.ro, c.odt == GPUOS_F32 ? rel : kNoLoad, qo);
    M::st8(c.ro, c.odt == GPUOS_F32 ? kNoLoad : rel, w0, w1);
  } else if (i + 4u <= c1) {
    if (c.odt == GPUOS_F32) {
      v4i qo;
#pragma unroll
      for (int e = 0; e < 4; ++e) qo[e] = __builtin_bit_cast(int, o[e]);
      M::st16(c.ro, rel, qo);
    } else {
      uint32_t w0, w1;
      if (c.odt == GPUOS_F16) { w0 = f2h(o[0]) | (f2h(o[1]) << 16); w1 = f2h(o[2]) | (f2h(o[3]) << 16); }
      else { w0 = f2b(o[0]) | (f2b(o[1]) << 16); w1 = f2b(o[2]) | (f2b(o[3]) << 16); }
      M::st8(c.ro, rel, w0, w1);
    }
  } else {
    for (uint32_t e = 0; i + e < c1; ++e) store_rt<POL>(c.po, i + e, c.odt, o[e]);      // the chunk's ragged end
  }
}

// A round with an input whose window does not fit the LDS scratch (that input is read element by
// element): a function of its own, so that its memory loads and the waits for them stay out of the
// common round's code.
template <int POL, int IMPL>
PATHFN void ew_staged_slow_round(const Record* r_v, uint32_t begin_v, uint32_t end_v, float* s_v, uint32_t c0_v, uint32_t c1_v,
                                 uint32_t lo0, uint32_t lo1, uint32_t lo2, uint32_t rg0, uint32_t rg1, uint32_t rg2, uint32_t staged_mask_v, uint32_t tid) {
  const Record* r = lds_arg(r_v);
  StagedCtx c;
  staged_ctx<IMPL>(c, r, uni(begin_v), uni(end_v), (char*)lds_arg(s_v));
  const uint32_t g_lo[3] = {uni(lo0), uni(lo1), uni(lo2)}, g_region[3] = {uni(rg0), uni(rg1), uni(rg2)};
  const uint32_t mask = uni(staged_mask_v);
  const bool g_staged[3] = {(mask & 1u) != 0, (mask & 2u) != 0, (mask & 4u) != 0};
  staged_round<POL, IMPL, false, false>(c, uni(c0_v), uni(c1_v), g_lo, g_region, g_staged, tid);
}

template <int POL, int IMPL>
PATHFN void ew_staged(const Record* r_v, uint32_t begin_v, uint32_t end_v, float* s_v, uint32_t tid) {
  const Record* r = lds_arg(r_v);
  const uint32_t begin = uni(begin_v), end = uni(end_v);
  char* lds = (char*)lds_arg(s_v);
  using M = Mem<POL>;
  constexpr int N = Op<IMPL>::N;
  StagedCtx c;
  staged_ctx<IMPL>(c, r, begin, end, lds);
  constexpr uint32_t kLdsBytes = kScratchFloats * 4u;
  constexpr uint32_t kBatchBytes = kStageLoads * kThreads * 16u;
  static_assert(kStageLoads == 4, "the pin in stash() names four vectors");
  // What a round stages (uniform): for every input the 16-byte window of memory its elements lie in.
  uint32_t lo[3] = {0, 0, 0}, region[3] = {0, 0, 0}, at[3], nbs[3], most = 0;
  bool staged[3] = {true, true, true};
  rsrc_t rs[3];
  auto plan = [&](uint32_t i0, uint32_t i1) {
    // indices of the first and the last element of the round
    const uint32_t ba = i0 / c.RC, ja = i0 - ba * c.RC, ra = ja / c.C, ca = ja - ra * c.C;
    const uint32_t bb = (i1 - 1) / c.RC, jb = (i1 - 1) - bb * c.RC, rb = jb / c.C, cb = jb - rb * c.C;
    uint32_t used = 0;
    most = 0;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      // bounds on the element offsets the round can touch (strides are non-negative): exact up to
      // the outermost index in which its first and last element differ, everything inside that
      uint32_t first, last;
      if (ba != bb) { first = ba * c.sb[k]; last = bb * c.sb[k] + (c.R - 1u) * c.sr[k] + (c.C - 1u) * c.sc[k]; }
      else if (ra != rb) { first = ba * c.sb[k] + ra * c.sr[k]; last = ba * c.sb[k] + rb * c.sr[k] + (c.C - 1u) * c.sc[k]; }
      else { first = ba * c.sb[k] + ra * c.sr[k] + ca * c.sc[k]; last = ba * c.sb[k] + ra * c.sr[k] + cb * c.sc[k]; }
      // the window in whole 16-byte vectors of the address space (the base need not be aligned)
      const uint64_t a_first = (uint64_t)(__UINTPTR_TYPE__)c.p[k] + (uint64_t)first * c.es[k];
      const uint64_t a_last = (uint64_t)(__UINTPTR_TYPE__)c.p[k] + (uint64_t)last * c.es[k] + c.es[k];
      const uint64_t v_first = a_first & ~15ull;
      const uint64_t bytes = ((a_last + 15ull) & ~15ull) - v_first;
      staged[k] = bytes <= (uint64_t)(kLdsBytes - used);
      lo[k] = first;
      // an input that is not staged gets an empty window: its loads fetch nothing
      nbs[k] = staged[k] ? (uint32_t)bytes : 0u;
      rs[k] = make_rsrc((const void*)(__UINTPTR_TYPE__)v_first, nbs[k]);
      at[k] = used;
      region[k] = used + (uint32_t)(a_first - v_first);            // where element `first` lies inside the staged bytes
      used += nbs[k];
      most = nbs[k] > most ? nbs[k] : most;
    }
  };
  // The windows of all inputs move together, kStageLoads vectors per lane and input in flight: every
  // load of a batch is issued before the first one is written to LDS (one memory latency per batch,
  // not one per vector and input).  Loads past a window's end are dropped by its bounds check.
  v4i q[N][kStageLoads];
  auto issue = [&](uint32_t b0) {
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
      for (int u = 0; u < kStageLoads; ++u) q[k][u] = M::ld16(rs[k], b0 + (tid + u * kThreads) * 16u);
  };
  auto stash = [&](uint32_t b0) {
    // (the values are pinned here: a load used only under the condition below would be moved there,
    // behind the waits of the stores before it)
#pragma unroll
    for (int k = 0; k < N; ++k) asm volatile("" : "+v"(q[k][0]), "+v"(q[k][1]), "+v"(q[k][2]), "+v"(q[k][3]));
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
      for (int u = 0; u < kStageLoads; ++u) {
        const uint32_t off = b0 + (tid + u * kThreads) * 16u;
        if (off < nbs[k]) *(v4i*)(lds + at[k] + off) = q[k][u];
      }
  };
  // Rounds are pipelined: the first batch of the NEXT round's windows is requested before this
  // round's elements are gathered and computed, so from the second round on the memory latency
  // hides behind the round before.  A round that has a successor is a full one, and every
  // wavefront issues exactly one store in it after those requests: the wait for the requested
  // vectors can leave that one store in flight.
  uint32_t i0 = begin, i1 = (end - begin < kStageRound) ? end : begin + kStageRound;
  plan(i0, i1);
  issue(0);
  stash(0);
  for (uint32_t b0 = kBatchBytes; b0 < most; b0 += kBatchBytes) { issue(b0); stash(b0); }
  __syncthreads();
  uint32_t c0, c1, g_lo[3], g_region[3];
  bool g_staged[3], all_staged;
  auto take = [&]() {                 // this round's share of the plan; the plan itself moves on
    c0 = i0; c1 = i1;
    all_staged = true;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      g_lo[k] = lo[k]; g_region[k] = region[k]; g_staged[k] = staged[k];
      if (k < N) all_staged = all_staged && staged[k];
    }
  };
  auto slow_round = [&]() {
    const uint32_t mask = (g_staged[0] ? 1u : 0u) | (g_staged[1] ? 2u : 0u) | (g_staged[2] ? 4u : 0u);
    ew_staged_slow_round<POL, IMPL>(r_v, begin, end, s_v, c0, c1, g_lo[0], g_lo[1], g_lo[2], g_region[0], g_region[1], g_region[2], mask, tid);
  };
  while (i1 < end) {                  // a round with a successor
    take();
    if (!all_staged) break;           // (rare) the rest of the chunk goes round by round below
    i0 = c1;
    i1 = (end - i0 < kStageRound) ? end : i0 + kStageRound;
    plan(i0, i1);
    issue(0);
    staged_round<POL, IMPL, true, true>(c, c0, c1, g_lo, g_region, g_staged, tid);
    __syncthreads();                  // the staged windows may be overwritten now
    stash(0);
    for (uint32_t b0 = kBatchBytes; b0 < most; b0 += kBatchBytes) { issue(b0); stash(b0); }
    __syncthreads();
  }
  // The chunk's last round, and every round from the first one on that has an input too wide to
  // stage: one after the other.
  for (;;) {
    take();
    if (all_staged) staged_round<POL, IMPL, false, true>(c, c0, c1, g_lo, g_region, g_staged, tid);
    else slow_round();
    __syncthreads();                  // the scratch may be reused (by the next round, by the next chunk)
    if (i1 >= end) break;
    i0 = c1;
    i1 = (end - i0 < kStageRound) ? end : i0 + kStageRound;
    plan(i0, i1);
    issue(0);
    stash(0);
    for (uint32_t b0 = kBatchBytes; b0 < most; b0 += kBatchBytes) { issue(b0); stash(b0); }
    __syncthreads();
  }
}

// PATH_STAGED under RF_PAIRS: contiguous output, inputs of its dtype that are contiguous or every second element of a buffer.  Both
// halves of each pair are read and one is dropped: no LDS, no rounds, nothing to wait for but memory.  A lane makes 8 bytes of the output
// from 16 of such an input, so that every access of a wavefront is one run of memory, and computes two of them together.
// (Gathered through LDS the rounds are latencies in a row: products of 400 x 579 fp32 with every other column took 61 us
// for 147 MB, 1,238 x 2,359 bf16 93 us for 140 MB; 52 and 55 so.)  The tensor's last vector goes element by element: behind
// its last element may be nothing to read.
template <int POL, class OPER, int DT>
PATHFN void ew_pairs(const Record* r_v, uint32_t begin_v, uint32_t end_v, uint32_t tid) {
  const Record* r = lds_arg(r_v);
  const uint32_t begin = uni(begin_v), end = uni(end_v);
  using E = Elem<DT>;
  using M = Mem<POL>;
  constexpr uint32_t V = E::V;
  constexpr int N = OPER::N, U = N > 2 ? 2 : 4;
  const uint32_t n = uni(r->size[2]), impl = uni(r->impl);
  const float alpha = __builtin_bit_cast(float, uni(__builtin_bit_cast(uint32_t, r->alpha)));
  uint32_t nvec = (end - begin) / V;
  if (end == n && nvec * V == end - begin) --nvec;
  const char* p[3];
  rsrc_t rs[3];
  uint32_t step[3];                                      // 1 or 2
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int kk = k < N ? k : 0;
    step[k] = uni(r->stride[kk][2]);
    p[k] = uni_ptr(r->ptr[kk]) + (uint64_t)begin * step[k] * E::ES;
    rs[k] = make_rsrc(p[k], (end < n ? (end - begin) * step[k] : (end - begin - 1u) * step[k] + 1u) * E::ES);
  }
  char* const po = (char*)uni_ptr(r->ptr[3]) + (uint64_t)begin * E::ES;
  const rsrc_t ro = make_rsrc(po, (end - begin) * E::ES);
  const uint32_t units = 2u * nvec;
  const bool stream = (uni(r->rflags) & RF_STREAM) != 0;
  auto ld16 = [&](rsrc_t q, uint32_t off) { return stream ? Mem<POL, true>::ld16(q, off) : M::ld16(q, off); };
  auto ld8 = [&](rsrc_t q, uint32_t off) { return stream ? Mem<POL, true>::ld8(q, off) : M::ld8(q, off); };
  for (uint32_t v = tid; v - tid < units; v += 2 * U * kThreads) {
    v4i q[3][U], h[3][U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t a = v + 2 * u * kThreads, b = a + kThreads;
#pragma unroll
      for (int k = 0; k < N; ++k) {
        if (step[k] == 2u) {
          q[k][u] = ld16(rs[k], a < units ? a * 16u : kNoLoad);
          h[k][u] = ld16(rs[k], b < units ? b * 16u : kNoLoad);
        } else {
          q[k][u] = ld8(rs[k], a < units ? a * 8u : kNoLoad);
          h[k][u] = ld8(rs[k], b < units ? b * 8u : kNoLoad);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const v4i a = q[k < N ? k : 0][u], b = h[k < N ? k : 0][u];
        if (k >= N) { q[k][u] = a; continue; }
        v4i c;
        if (E::ES == 4) c = v4i{a[0], a[2], b[0], b[2]};
        else {                                           // the low halves of two words
          c[0] = (int)__builtin_amdgcn_perm((uint32_t)a[1], (uint32_t)a[0], 0x05040100u);
          c[1] = (int)__builtin_amdgcn_perm((uint32_t)a[3], (uint32_t)a[2], 0x05040100u);
          c[2] = (int)__builtin_amdgcn_perm((uint32_t)b[1], (uint32_t)b[0], 0x05040100u);
          c[3] = (int)__builtin_amdgcn_perm((uint32_t)b[3], (uint32_t)b[2], 0x05040100u);
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) q[k][u][w] = step[k] == 2u ? c[w] : (w < 2 ? a[w] : b[w - 2]);
      }
    typedef VecArg<DT, U> Arg;
    OPER::template vectors<DT, U>(impl, Arg{q[0]}, Arg{q[1]}, Arg{q[2]}, alpha, [&](int u, const v4i& o) {
      const uint32_t a = v + 2 * u * kThreads, b = a + kThreads;
      M::st8(ro, a < units ? a * 8u : kNoLoad, (uint32_t)o[0], (uint32_t)o[1]);
      M::st8(ro, b < units ? b * 8u : kNoLoad, (uint32_t)o[2], (uint32_t)o[3]);
    });
  }
  for (uint32_t i = nvec * V + tid; i < end - begin; i += kThreads) {      // one element each, in the lowest place of a vector
    v4i q[3][1];
#pragma unroll
    for (int k = 0; k < 3; ++k) q[k][0] = v4i{(int)(E::ES == 4 ? M::ld4(p[k < N ? k : 0], i * step[k]) : M::ld2(p[k < N ? k : 0], i * step[k])), 0, 0, 0};
    typedef VecArg<DT, 1> Arg;
    OPER::template vectors<DT, 1>(impl, Arg{q[0]}, Arg{q[1]}, Arg{q[2]}, alpha, [&](int, const v4i& o) {
      if (E::ES == 4) M::st4(po, i, (uint32_t)o[0]);
      else M::st2(po, i, (uint32_t)o[0]);
    });
  }
}

// ---------------------------------------------------------------------------
// PATH_GENERIC: row-major index decomposition over <= 6 coalesced dims, per
// operand strides (0 on broadcast dims), per operand dtype.
// ---------------------------------------------------------------------------
template <int POL, int IMPL, bool INT>
PATHFN void ew_generic(const Record* r_v, uint32_t begin_v, uint32_t end_v, uint32_t tid) {
  const Record* r = lds_arg(r_v);
  const uint32_t begin = uni(begin_v), end = uni(end_v);
  using M = Mem<POL>;
  constexpr int N = INT ? 2 : Op<IMPL>::N;
  const int nd = (int)uni(r->ndim);
  const int nin = (int)uni(r->n_inputs);
  uint32_t size[GPUOS_MAX_DIMS], st[4][GPUOS_MAX_DIMS];
#pragma unroll
  for (int d = 0; d < GPUOS_MAX_DIMS; ++d) {
    size[d] = uni(r->size[d]);
#pragma unroll
    for (int k = 0; k < 4; ++k) st[k][d] = uni(r->stride[k][d]);
  }
  const char* p[3];
  uint32_t dt[4];
#pragma unroll
  for (int k = 0; k < 3; ++k) { p[k] = uni_ptr(r->ptr[k]); dt[k] = uni(r->dtype[k]); }
  dt[3] = uni(r->dtype[3]);
  char* po = (char*)uni_ptr(r->ptr[3]);
  const float alpha = r->alpha;
  for (uint32_t i = begin + tid; i < end; i += kThreads) {
    uint32_t rem = i, off[4] = {0, 0, 0, 0};
#pragma unroll
    for (int d = GPUOS_MAX_DIMS - 1; d >= 0; --d) {
      if (d < nd) {
        const uint32_t q = rem / size[d];
        const uint32_t idx = rem - q * size[d];
        rem = q;
#pragma unroll
        for (int k = 0; k < 4; ++k) off[k] += idx * st[k][d];
      }
    }
    if (INT) {
      const uint32_t x = M::ld4(p[0], off[0]);
      const uint32_t y = nin > 1 ? M::ld4(p[1], off[1]) : 0u;
      M::st4(po, off[3], int_op<IMPL>(x, y));
    } else if (IMPL == GPUOS_IMPL_COPY && dt[0] == dt[3]) {
      if (dt[0] == GPUOS_F32) M::st4(po, off[3], M::ld4(p[0], off[0]));
      else M::st2(po, off[3], M::ld2(p[0], off[0]));
    } else {
      const float x = load_rt<POL>(p[0], off[0], dt[0]);
      const float y = N > 1 ? load_rt<POL>(p[1], off[1], dt[1]) : 0.f;
      const float z = N > 2 ? load_rt<POL>(p[2], off[2], dt[2]) : 0.f;
      store_rt<POL>(po, off[3], dt[3], Op<IMPL>::f(x, y, z, alpha));
    }
  }
}

// ---------------------------------------------------------------------------
// PATH_ROWS: up to three outer dims of any strides over rows of C elements that are contiguous in
// every operand that is not one scalar per row: slices of a wider matrix (read or written), head
// splits, masks repeated over leading dims, per-row scalars, whatever the row length and the
// alignment of the rows are (an access of 16 bytes needs no alignment beyond its elements').
// Operands of dtype DTI, output of dtype DTO (they differ for COPY only); scalars of any float dtype.
// A row is cut into vectors of V elements from its first element on, one lane each; the last vector of
// a row that is no multiple of V covers the row's last V elements and stores those the vector
// before it does not hold.  The extent of every operand fits a buffer resource (checked on the host).
// ---------------------------------------------------------------------------
// DTI != DTO: the cast of a COPY.
template <int POL, class OPER, int DTI, int DTO, bool SCALARS>
PATHFN void ew_rows(const Record* r_v, uint32_t begin_v, uint32_t end_v, uint32_t tid) {
  const Record* r = lds_arg(r_v);
  const uint32_t begin = uni(begin_v), end = uni(end_v);
  using EI = Elem<DTI>;
  using EO = Elem<DTO>;
  using M = Mem<POL>;
  constexpr int V = EI::V > EO::V ? EI::V : EO::V;
  // A cast that widens gives each vector of eight elements to two lanes, four elements each, so that a wavefront's store is
  // one run of memory.  (One lane for both halves leaves every other 16 bytes to the next store, and memory takes each
  // for itself: 24M elements from bf16 to fp32 took 98 us, 45 so, 39 with plain stores.)
  constexpr int LN = EI::ES < EO::ES ? 2 : 1, VL = V / LN, NI = LN == 2 ? 1 : V / EI::V, NO = VL / EO::V;
  constexpr uint32_t kStep = kThreads / LN;
  constexpr int N = OPER::N;
  constexpr int U = 4;
  const uint32_t A = uni(r->size[0]), B = uni(r->size[1]), R = uni(r->size[2]), C = uni(r->size[3]);
  const uint32_t VR = (C + V - 1) / V, tail = C % V;
  rsrc_t rs[4];
  uint32_t st[4][3], dt[3], es[3], lead[3];
  bool scalar[3];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int kk = k < N || k == 3 ? k : 0;
    const char* p = uni_ptr(r->ptr[kk]);
    const uint32_t e = k == 3 ? (uint32_t)EO::ES : (uni(r->dtype[kk]) == GPUOS_F32 || DTI == GPUOS_I32 ? 4u : 2u);
    uint32_t extent = k < 3 && SCALARS && uni(r->okind[kk]) == K_ROWSCALAR ? 1u : C;      // elements from the first to the last
    extent += (A - 1) * uni(r->stride[kk][0]) + (B - 1) * uni(r->stride[kk][1]) + (R - 1) * uni(r->stride[kk][2]);
#pragma unroll
    for (int d = 0; d < 3; ++d) st[k][d] = uni(r->stride[kk][d]) * e;
    if (k < 3) {
      dt[k] = uni(r->dtype[kk]);
      es[k] = e;
      scalar[k] = SCALARS && uni(r->okind[kk]) == K_ROWSCALAR;
      // a scalar is read as the aligned word that holds it
      lead[k] = scalar[k] ? (uint32_t)(__UINTPTR_TYPE__)p & 3u : 0u;
      rs[k] = make_rsrc(p - lead[k], (lead[k] + extent * e + (scalar[k] ? 3u : 0u)) & (scalar[k] ? ~3u : ~0u));
    } else {
      rs[k] = make_rsrc(p, extent * e);
    }
  }
  const float alpha = __builtin_bit_cast(float, uni(__builtin_bit_cast(uint32_t, r->alpha)));
  const uint32_t impl = uni(r->impl);
  const bool stream = (uni(r->rflags) & RF_STREAM) != 0;
  auto load = [&](rsrc_t rs, uint32_t off) {
    typedef Mem<POL, true> S;
    if (LN == 2) return stream ? S::ld8(rs, off) : M::ld8(rs, off);
    return stream ? S::ld16(rs, off) : M::ld16(rs, off);
  };
  // (row, vector) of this lane's first unit by division, then steps of 256 units with carries
  const bool deep = A * B > 1;
  const uint32_t ti = tid / LN, half = LN == 2 ? (tid & 1u) * VL : 0u;
  uint32_t v = begin + ti;
  uint32_t row = v / VR, vc = v - row * VR, b = 0, a = 0;
  const uint32_t s_rows = kStep / VR, s_vc = kStep - s_rows * VR;
  uint32_t s_r = s_rows, s_b = 0, s_a = 0;
  if (deep) {
    const uint32_t t = row / R;
    row -= t * R;
    a = t / B;
    b = t - a * B;
    const uint32_t ts = s_rows / R;
    s_r = s_rows - ts * R;
    s_a = ts / B;
    s_b = ts - s_a * B;
  }
  for (; v - ti < end; ) {
    v4i q[3][U][NI];
    uint32_t w[3][U], oo[U];
    bool last[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool act = v + u * kStep < end;
      last[u] = tail != 0 && vc == VR - 1;
      const uint32_t col = (last[u] ? C - V : vc * V) + half;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (k < N || k == 3) {
          uint32_t o = row * st[k][2];
          if (deep) o += b * st[k][1] + a * st[k][0];
          if (k == 3) oo[u] = o + col * EO::ES;
          else {
            // (both forms of the load under SCALARS, the one that does not apply past the resource, where it
            // moves nothing: no branch between the loads of a round)
            const uint32_t of = act && !(SCALARS && scalar[k]) ? o + col * EI::ES : kNoLoad;
#pragma unroll
            for (int i = 0; i < NI; ++i) q[k][u][i] = load(rs[k], of + i * 16u);
            if (SCALARS) w[k][u] = M::ldb4(rs[k], act && scalar[k] ? (lead[k] + o) & ~3u : kNoLoad) >> (((lead[k] + o) & 2u) * 8u);
          }
        }
      }
      vc += s_vc;
      row += s_r;
      if (vc >= VR) { vc -= VR; ++row; }
      if (deep) {
        b += s_b;
        a += s_a;
        if (row >= R) { row -= R; ++b; }               // (one step and one carry: at most 2 R - 1)
        if (b >= B) { b -= B; ++a; }
      }
    }
    auto sink = [&](int u, const v4i (&qo)[NO]) {
      const bool act = v + u * kStep < end;
#pragma unroll
      for (int i = 0; i < NO; ++i) M::st16(rs[3], act && !last[u] ? oo[u] + i * 16u : kNoLoad, qo[i]);
      if (tail != 0 && act && last[u]) {
#pragma unroll
        for (int e = LN == 2 ? 0 : 1; e < VL; ++e)
          if (half + (uint32_t)e >= V - tail) {
            if (EO::ES == 4) M::stb4(rs[3], oo[u] + e * 4u, (uint32_t)qo[e / EO::V][e % EO::V]);
            else M::stb2(rs[3], oo[u] + e * 2u, (uint32_t)qo[e / EO::V][(e % EO::V) / 2] >> ((e & 1) * 16));
          }
      }
    };
    if constexpr (DTI != DTO) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        v4i qo[NO];
#pragma unroll
        for (int e = 0; e < VL; ++e) EO::put(qo[e / EO::V], e % EO::V, EI::get(q[0][u][e / EI::V], e % EI::V));
        sink(u, qo);
      }
    } else {
      v4i qv[3][U];
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int u = 0; u < U; ++u) qv[k][u] = q[k < N ? k : 0][u][0];
      auto sink1 = [&](int u, const v4i& r1) { const v4i qo[1] = {r1}; sink(u, qo); };
      if constexpr (SCALARS) {
        if constexpr (DTI != GPUOS_I32) {
#pragma unroll
          for (int k = 0; k < N; ++k)
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const uint32_t h = w[k][u] & 0xffffu;
              w[k][u] = dt[k] == GPUOS_F32 ? w[k][u] : __builtin_bit_cast(uint32_t, dt[k] == GPUOS_F16 ? h2f(h) : b2f(h));
            }
        }
        typedef MixArg<DTI, U> Arg;
        OPER::template vectors<DTI, U>(impl, Arg{qv[0], w[0], scalar[0]}, Arg{qv[1], w[N > 1 ? 1 : 0], scalar[N > 1 ? 1 : 0]},
                                       Arg{qv[2], w[N > 2 ? 2 : 0], scalar[N > 2 ? 2 : 0]}, alpha, sink1);
      } else {
        typedef VecArg<DTI, U> Arg;
        OPER::template vectors<DTI, U>(impl, Arg{qv[0]}, Arg{qv[1]}, Arg{qv[2]}, alpha, sink1);
      }
    }
    v += U * kStep;
  }
}

// Which executor takes a task is decided by halving: pick<LO, HI> calls F::run<K> for the K in [LO, HI)
// that equals k.  (The compiler turns a many-way branch into a chain that is walked case by case, with
// a flag to carry per case; a two-way choice whose sides meet again is left alone.)
template <int LO, int HI, class F, class... A> DEV void pick(uint32_t k, A... a) {
  if constexpr (HI - LO == 1) F::template run<LO>(a...);
  else {
    constexpr int MID = (LO + HI) / 2;
    if (k < (uint32_t)MID) pick<LO, MID, F>(k, a...);
    else pick<MID, HI, F>(k, a...);
  }
}

// ---------------------------------------------------------------------------
// reductions over the last dim
// ---------------------------------------------------------------------------
// The accumulator of a reduction over elements of dtype DT: fp32 for the float types, int32 for I32.
template <int DT> struct RedAcc { typedef float T; };
template <> struct RedAcc<GPUOS_I32> { typedef int32_t T; };
template <int RIMPL, class T> DEV T red_identity();
template <> DEV float red_identity<GPUOS_IMPL_SUM_LAST, float>() { return 0.0f; }
template <> DEV float red_identity<GPUOS_IMPL_MAX_LAST, float>() { return -__builtin_inff(); }
template <> DEV float red_identity<GPUOS_IMPL_MIN_LAST, float>() { return __builtin_inff(); }
template <> DEV int32_t red_identity<GPUOS_IMPL_SUM_LAST, int32_t>() { return 0; }
template <> DEV int32_t red_identity<GPUOS_IMPL_MAX_LAST, int32_t>() { return (int32_t)0x80000000; }
template <> DEV int32_t red_identity<GPUOS_IMPL_MIN_LAST, int32_t>() { return 0x7fffffff; }
template <int RIMPL> DEV float red_combine(float a, float b) {
  if (RIMPL == GPUOS_IMPL_SUM_LAST) return a + b;
  if (RIMPL == GPUOS_IMPL_MAX_LAST) return __builtin_elementwise_maximum(a, b);      // (IEEE maximum and minimum: NaN goes through)
  return __builtin_elementwise_minimum(a, b);
}
template <int RIMPL> DEV int32_t red_combine(int32_t a, int32_t b) {
  if (RIMPL == GPUOS_IMPL_SUM_LAST) return (int32_t)((uint32_t)a + (uint32_t)b);
  if (RIMPL == GPUOS_IMPL_MAX_LAST) return a > b ? a : b;
  return a < b ? a : b;
}

// Step OFF of an all-reduce butterfly over aligned groups of 2 * OFF lanes: a lane's own value and its
// partner's, in either order.  Steps 1 and 2 swap inside a quad and steps 4 and 8 mirror a half row / a row of
// 16 lanes (lane i with i ^ 7, i ^ 15), DPP operand modifiers; steps 16 and 32 swap rows and halves between two
// copies.  None takes a trip through the LDS crossbar as a shuffle does.  The masks 1, 2, 7, 15, 16, 32 are
// independent, so the steps reach every lane of the group.  All lanes must be active.
template <int OFF> DEV void butterfly_pair(int v, int& a, int& b) {
  a = v;
  if (OFF == 1) b = __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xf, 0xf, false);      // quad_perm [1,0,3,2]
  else if (OFF == 2) b = __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xf, 0xf, false); // quad_perm [2,3,0,1]
  else if (OFF == 4) b = __builtin_amdgcn_update_dpp(v, v, 0x141, 0xf, 0xf, false);     // row_half_mirror
  else if (OFF == 8) b = __builtin_amdgcn_update_dpp(v, v, 0x140, 0xf, 0xf, false);     // row_mirror
  else {
    auto two = OFF == 16 ? __builtin_amdgcn_permlane16_swap(v, v, false, false) : __builtin_amdgcn_permlane32_swap(v, v, false, false);
    a = (int)two[0];
    b = (int)two[1];
  }
}
template <int OFF> DEV void butterfly_pair(float v, float& a, float& b) {
  int x, y;
  butterfly_pair<OFF>(__builtin_bit_cast(int, v), x, y);
  a = __builtin_bit_cast(float, x);
  b = __builtin_bit_cast(float, y);
}

// all-reduce over the `width` lanes (power of two <= 64, aligned) a lane belongs to
template <int RIMPL, class T> DEV T wave_reduce(T acc, uint32_t width) {
  T a, b;
  if (width > 32) { butterfly_pair<32>(acc, a, b); acc = red_combine<RIMPL>(a, b); }
  if (width > 16) { butterfly_pair<16>(acc, a, b); acc = red_combine<RIMPL>(a, b); }
  if (width > 8) { butterfly_pair<8>(acc, a, b); acc = red_combine<RIMPL>(a, b); }
  if (width > 4) { butterfly_pair<4>(acc, a, b); acc = red_combine<RIMPL>(a, b); }
  if (width > 2) { butterfly_pair<2>(acc, a, b); acc = red_combine<RIMPL>(a, b); }
  if (width > 1) { butterfly_pair<1>(acc, a, b); acc = red_combine<RIMPL>(a, b); }
  return acc;
}

// PATH_RED_CONTIG: input is a contiguous [rows, n] matrix of dtype DT, output a
// contiguous vector [rows] of any float dtype (I32 for I32).  The rows of a chunk are read as one
// flat run of 16-byte vectors of the address space, whatever n and the base's alignment are: a
// vector that straddles a row boundary is loaded by both rows and masked per element.  (The first
// and the last vector of the run may hold bytes outside the tensor, in the same aligned 16 bytes as
// one of its elements and so in the same page; they are masked like another row's.)  I32 rows take
// the same way: with one wavefront per row and one word per lane and load, whatever the row length,
// 24 integer operations of 0.1-50 MB took 529 us, a 13,946 x 22 maximum among them 505; 95 with this,
// 62 with rows on 16-byte accesses besides (ew_rows).
// Four shapes of work:
//   whole short rows (<= 64 vectors, each a whole number of them): P lanes per row, 64 / P rows per
//               wavefront pass, eight passes at a time;
//   other short rows (<= 128): through LDS, by the piece of as many rows as fit;
//   medium rows: a wavefront reads its rows as one run, in groups of 64 vectors;
//   long rows   (>= 1024 vectors): the four wavefronts take a quarter of each row, partial
//               results meet in LDS once per chunk (one barrier per chunk, not per row).
// 134 MB of fp32 rows of 24, 75, 136, 256, 486, 1,060 and 2,634 took 67, 135, 121, 71, 92, 69 and 57 us (P lanes per row
// or one wavefront per row from memory, all requested before any was looked at and again nothing in flight while it was), 47, 49, 59,
// 46, 54, 49 and 53 so; 16-bit rows as much.
// Per-element accumulation.  SUM adds; MAX / MIN are IEEE maximum and minimum, one instruction of three operands for two
// elements, through which a NaN goes (red_finish gives it one form).  (With the hardware's older maximum, which skips NaNs, a
// flag beside it took a compare a pair, and combining lanes four operations a step: rows of 136 fp32 121 us for
// 134 MB, of which this and steps without shuffles took off 30.)
template <int RIMPL> DEV int32_t red_step(int32_t acc, int32_t x) { return red_combine<RIMPL>(acc, x); }
template <int RIMPL> DEV float red_step(float acc, float x) { return red_combine<RIMPL>(acc, x); }
template <int RIMPL> DEV int32_t red_finish(int32_t acc) { return acc; }
template <int RIMPL> DEV float red_finish(float acc) { return RIMPL != GPUOS_IMPL_SUM_LAST && acc != acc ? __builtin_nanf("") : acc; }
template <int RIMPL> DEV float red_step2(float acc, float x0, float x1) {
  float r;
  if (RIMPL == GPUOS_IMPL_MAX_LAST) asm("v_maximum3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(acc), "v"(x0), "v"(x1));
  else asm("v_minimum3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(acc), "v"(x0), "v"(x1));
  return r;
}

template <int DT> DEV typename RedAcc<DT>::T red_get(const v4i& q, int k) { return Elem<DT>::get(q, k); }
template <> DEV int32_t red_get<GPUOS_I32>(const v4i& q, int k) { return q[k]; }

template <int RIMPL, int DT>
DEV typename RedAcc<DT>::T red_vector(const v4i& q, uint32_t f0, uint32_t lo, uint32_t hi, bool edge, typename RedAcc<DT>::T acc) {
  // q holds elements f0 .. f0+V-1 of the flat run; the row is [lo, hi)
  using E = Elem<DT>;
  if (!edge) {
    if constexpr (RIMPL == GPUOS_IMPL_SUM_LAST || DT == GPUOS_I32) {
#pragma unroll
      for (int k = 0; k < E::V; ++k) acc = red_step<RIMPL>(acc, red_get<DT>(q, k));
    } else {
#pragma unroll
      for (int k = 0; k < E::V; k += 2) acc = red_step2<RIMPL>(acc, E::get(q, k), E::get(q, k + 1));
    }
  } else {
#pragma unroll
    for (int k = 0; k < E::V; ++k)
      if (f0 + k >= lo && f0 + k < hi) acc = red_step<RIMPL>(acc, red_get<DT>(q, k));
  }
  return acc;
}

// the result of one row: of any float dtype, or the bits of an int32
template <int POL> DEV void red_store(void* p, uint32_t i, uint32_t dt, float v) { store_rt<POL>(p, i, dt, v); }
template <int POL> DEV void red_store(void* p, uint32_t i, uint32_t, int32_t v) { Mem<POL>::st4(p, i, (uint32_t)v); }

struct RedArgs {       // what a row-reduction variant is called with (plain values: see lds_arg)
  const char* base;    // first byte of the run: the tensor base advanced to the chunk's first vector
  uint32_t bytes;      // length of the run, whole vectors
  uint32_t base_elem;  // first element of the run (multiple of V), counted from the 16-byte block the tensor begins in
  uint32_t lead;       // elements of that block in front of the tensor
  uint32_t n;
  char* po;
  uint32_t odt, row_begin, row_end, max_span;
  uint32_t stream;     // loads with nt
  uint32_t tid;
  float* s_part;       // LDS
};
struct RedRun {        // the chunk's rows as a flat run of vectors
  rsrc_t rin;
  uint32_t skew;       // row r begins at element r * n + skew of the run (modulo 2^32)
  uint32_t n;
};
DEV RedRun red_run(const RedArgs& a) {
  RedRun run;
  run.rin = make_rsrc(uni_ptr((uint64_t)a.base), uni(a.bytes));
  run.skew = uni(a.lead) - uni(a.base_elem);
  run.n = uni(a.n);
  return run;
}

// Row `i` of the chunk's results, where `act`: no branch round the store, and none under a condition of its own.  (The
// compiler counts what is in flight per path: where a store may or may not have been issued, the next wait for
// loads waits for it too.)
template <int POL> DEV void red_put(rsrc_t ro, uint32_t i, uint32_t odt, float v, bool act) {
  if (odt == GPUOS_F32) Mem<POL>::stb4(ro, act ? i * 4u : kNoLoad, __builtin_bit_cast(uint32_t, v));
  else Mem<POL>::stb2(ro, act ? i * 2u : kNoLoad, odt == GPUOS_F16 ? f2h(v) : f2b(v));
}
template <int POL> DEV void red_put(rsrc_t ro, uint32_t i, uint32_t, int32_t v, bool act) { Mem<POL>::stb4(ro, act ? i * 4u : kNoLoad, (uint32_t)v); }
DEV rsrc_t red_out(const RedArgs& a, uint32_t row_begin, uint32_t row_end, uint32_t odt) {
  const uint32_t os = odt == GPUOS_F16 || odt == GPUOS_BF16 ? 2u : 4u;
  return make_rsrc(uni_ptr((uint64_t)a.po) + (uint64_t)row_begin * os, (row_end - row_begin) * os);
}
// K elements join a lane's accumulator; sums in pairs (a shorter chain, and a smaller error).
template <int RIMPL, int K> DEV int32_t red_join(int32_t acc, const int32_t (&x)[K]) {
#pragma unroll
  for (int k = 0; k < K; ++k) acc = red_combine<RIMPL>(acc, x[k]);
  return acc;
}
template <int RIMPL, int K> DEV float red_join(float acc, const float (&x)[K]) {
  if constexpr (RIMPL == GPUOS_IMPL_SUM_LAST) {
    float t[K];
#pragma unroll
    for (int k = 0; k < K; ++k) t[k] = x[k];
#pragma unroll
    for (int w = K / 2; w > 0; w /= 2)
#pragma unroll
      for (int k = 0; k < w; ++k) t[k] += t[k + w];
    return acc + t[0];
  } else {
#pragma unroll
    for (int k = 0; k < K; k += 2) acc = red_step2<RIMPL>(acc, x[k], x[k + 1]);
    return acc;
  }
}

// Rows of more vectors than go by way of the LDS, whatever their alignment (1,024 and more where a chunk has more than 64 rows; else
// those go by quarters).  A wavefront takes a share of the chunk's rows, which is one
// dense run of memory, and reads it in groups of 64 vectors, four of them while it works on the four before; a row ends where
// it ends, within a group, and that group is looked at once for either row.  Bound by memory latency: what counts is
// that four to eight loads a lane are always in flight.  (Row by row, four rows' or one row's eight loads at a time and then
// all of their arithmetic with nothing in flight: 134 MB of fp32 rows of 1,060 69 us, of 2,634 57 us.)
template <int POL, int RIMPL, int DT>
PATHFN void red_rows_stream(RedArgs a) {
  const RedRun run = red_run(a);
  const uint32_t odt = uni(a.odt), row_begin = uni(a.row_begin), row_end = uni(a.row_end);
  using E = Elem<DT>;
  using A = typename RedAcc<DT>::T;
  using M = Mem<POL>;
  constexpr uint32_t V = E::V, U = 4;
  const uint32_t lane = a.tid & 63u, wave = uni(a.tid >> 6);
  const uint32_t n = run.n;
  const rsrc_t ro = red_out(a, row_begin, row_end, odt);
  const uint32_t per = (row_end - row_begin + 3u) / 4u, w0 = row_begin + wave * per, w1 = row_end - w0 < per ? row_end : w0 + per;
  if (wave * per >= row_end - row_begin) return;
  uint32_t row = w0, lo = w0 * n + run.skew, hi = lo + n;    // the row being read: elements [lo, hi) of the run
  const uint32_t j_last = (w1 * n + run.skew - 1u) / V;
  A acc = red_identity<RIMPL, A>(), res = 0;                 // (lane L of `res`: the L-th result since the last store)
  uint32_t kept = 0;
  const bool stream = uni(a.stream) != 0;
  auto fetch = [&](v4i (&q)[U], uint32_t j) {
    if (stream) {
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) q[u] = Mem<POL, true>::ld16(run.rin, j + u * 64u + lane <= j_last ? (j + u * 64u + lane) * 16u : kNoLoad);
    } else {
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) q[u] = M::ld16(run.rin, j + u * 64u + lane <= j_last ? (j + u * 64u + lane) * 16u : kNoLoad);
    }
  };
  auto take = [&](const v4i (&q)[U], uint32_t j) {           // true: the last row is complete
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const uint32_t g0 = (j + u * 64u) * V, g1 = g0 + 64u * V;
      while (true) {
        if (lo <= g0 && hi >= g1) {
          A x[V];
#pragma unroll
          for (uint32_t k = 0; k < V; ++k) x[k] = red_get<DT>(q[u], (int)k);
          acc = red_join<RIMPL>(acc, x);
        } else {
          A x[V];
          const uint32_t d = g0 + lane * V - lo;             // (unsigned: elements before the row are past its end)
#pragma unroll
          for (uint32_t k = 0; k < V; ++k) x[k] = d + k < n ? red_get<DT>(q[u], (int)k) : red_identity<RIMPL, A>();
          acc = red_join<RIMPL>(acc, x);
        }
        if (hi > g1) break;                                  // the row goes on
        const A t = wave_reduce<RIMPL>(red_finish<RIMPL>(acc), 64);
        if (lane == kept) res = t;
        ++kept;
        ++row;
        if (kept == 64u || row == w1) { red_put<POL>(ro, row - row_begin - kept + lane, odt, res, lane < kept); kept = 0; }
        if (row == w1) return true;
        acc = red_identity<RIMPL, A>();
        lo = hi;
        hi += n;
        if (lo >= g1) break;
      }
    }
    return false;
  };
  v4i qa[U], qb[U];
  uint32_t j = lo / V;
  fetch(qa, j);
  while (true) {
    fetch(qb, j + 64u * U);
    if (take(qa, j)) break;
    fetch(qa, j + 128u * U);
    if (take(qb, j + 64u * U)) break;
    j += 128u * U;
  }
}

constexpr uint32_t kRedPartialRows = 64;   // rows of partial results the LDS scratch holds
constexpr uint32_t kRedPieceVectors = 448; // ... and vectors of a wavefront's own rows
// Rows of up to this many vectors go by way of the LDS.  (Beyond, a group of 64 vectors holds few rows' ends and
// the wavefront reads them as they come: rows of 130 to 450 vectors take the same time either way, and longer ones no LDS holds.)
constexpr uint32_t kRedLdsSpan = 128;

// Rows of 1,024 vectors and more, a quarter of each row to a wavefront: four vectors a lane are worked on while the four behind them,
// or the next row's first, are on their way.  (Eight at a time with nothing in flight meanwhile, forty streaming operations: 101.6 us, 100.6 so.)
template <int POL, int RIMPL, int DT>
PATHFN void red_rows_quarter(RedArgs a) {
  const RedRun run = red_run(a);
  const uint32_t tid = a.tid;
  char* po = (char*)uni_ptr((uint64_t)a.po);
  const uint32_t odt = uni(a.odt), row_begin = uni(a.row_begin), row_end = uni(a.row_end);
  float* s_part = lds_arg(a.s_part);
  using E = Elem<DT>;
  using A = typename RedAcc<DT>::T;
  using M = Mem<POL>;
  constexpr uint32_t V = E::V, U = 4;
  const uint32_t lane = tid & 63u, wave = uni(tid >> 6);
  const uint32_t n = run.n;
  const bool stream = uni(a.stream) != 0;
  struct At { uint32_t row, v, end; };                       // 4 x 64 vectors from v on, below end, of this wavefront's quarter of a row
  auto quarter = [&](uint32_t row) {
    const uint32_t j0 = (row * n + run.skew) / V, j1 = (row * n + run.skew + n - 1u) / V;
    const uint32_t sq = (j1 - j0 + 4u) / 4u, v = j0 + wave * sq;
    return At{row, v, v + sq <= j1 + 1u ? v + sq : j1 + 1u};
  };
  auto behind = [&](const At& at) { return at.v + 64u * U < at.end ? At{at.row, at.v + 64u * U, at.end} : quarter(at.row + 1u); };
  auto fetch = [&](v4i (&q)[U], const At& at) {
    const uint32_t end = at.row < row_end ? at.end : 0u;
    if (stream) {
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) q[u] = Mem<POL, true>::ld16(run.rin, at.v + u * 64u + lane < end ? (at.v + u * 64u + lane) * 16u : kNoLoad);
    } else {
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) q[u] = M::ld16(run.rin, at.v + u * 64u + lane < end ? (at.v + u * 64u + lane) * 16u : kNoLoad);
    }
  };
  A a0 = red_identity<RIMPL, A>(), a1 = a0;
  auto take = [&](const v4i (&q)[U], const At& at, uint32_t next_row) {
    const uint32_t lo = at.row * n + run.skew, hi = lo + n, j0 = lo / V, j1 = (hi - 1u) / V;
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const uint32_t j = at.v + u * 64u + lane;
      if (j < at.end) {
        if ((u & 1) == 0) a0 = red_vector<RIMPL, DT>(q[u], j * V, lo, hi, j == j0 || j == j1, a0);
        else a1 = red_vector<RIMPL, DT>(q[u], j * V, lo, hi, j == j0 || j == j1, a1);
      }
    }
    if (next_row == at.row) return;
    const A t = wave_reduce<RIMPL>(red_finish<RIMPL>(red_combine<RIMPL>(a0, a1)), 64);
    if (lane == 0) s_part[(at.row - row_begin) * 4 + wave] = __builtin_bit_cast(float, t);
    a0 = a1 = red_identity<RIMPL, A>();
  };
  v4i qa[U], qb[U];
  At at = quarter(row_begin);
  fetch(qa, at);
  while (true) {
    const At b = behind(at);
    fetch(qb, b);
    take(qa, at, b.row);
    if (b.row >= row_end) break;
    at = behind(b);
    fetch(qa, at);
    take(qb, b, at.row);
    if (at.row >= row_end) break;
  }
  __syncthreads();
  const uint32_t nrows = row_end - row_begin;
  if (tid < nrows) {
    const float* p = s_part + tid * 4;
    auto part = [&](int k) { return __builtin_bit_cast(A, p[k]); };
    const A t = red_combine<RIMPL>(red_combine<RIMPL>(part(0), part(1)), red_combine<RIMPL>(part(2), part(3)));
    red_store<POL>(po, row_begin + tid, odt, t);
  }
  __syncthreads();
}

// Rows of up to 128 vectors, but for whole aligned ones of up to 64.  A wavefront takes a share of the chunk's rows and reads it
// densely, as many whole rows at a time as 448 vectors hold, puts them into its part of the LDS and
// requests the next; from there rows have no edges: P lanes a row, element by element.  Bound by memory latency: seven
// loads a lane are in flight throughout.  (P lanes a row straight from memory, masked element by element at either end, 64 lanes
// for the 35 vectors of a row of 136 fp32: 134 MB of those took 121 us.)
template <int POL, int RIMPL, int DT>
PATHFN void red_rows_lds(RedArgs a) {
  const RedRun run = red_run(a);
  const uint32_t odt = uni(a.odt), row_begin = uni(a.row_begin), row_end = uni(a.row_end);
  using E = Elem<DT>;
  using A = typename RedAcc<DT>::T;
  using M = Mem<POL>;
  constexpr uint32_t V = E::V, K = 8;
  const uint32_t lane = a.tid & 63u, wave = uni(a.tid >> 6);
  char* const mem = (char*)lds_arg(a.s_part) + wave * kRedPieceVectors * 16u;
  static_assert(kRedPieceVectors * 16 * 4 <= kScratchFloats * 4 && kRedPieceVectors % 64 == 0, "a piece per wavefront");
  constexpr uint32_t NV = kRedPieceVectors / 64u;
  const uint32_t n = run.n;
  const rsrc_t ro = red_out(a, row_begin, row_end, odt);
  const uint32_t per = (row_end - row_begin + 3u) / 4u, w0 = row_begin + wave * per, w1 = row_end - w0 < per ? row_end : w0 + per;
  if (wave * per >= row_end - row_begin) return;
  // rows a piece: the most that fit with a partly covered vector at either end, evened out over the pieces
  const uint32_t most = ((kRedPieceVectors - 1u) * V + 1u) / n, pieces = (per + most - 1u) / most, R = (per + pieces - 1u) / pieces;
  uint32_t P = 64;
  while (P > 1u && 64u / P < R) P >>= 1;
  const uint32_t rps = 64u / P, sub = lane / P, first = lane & (P - 1u), whole = n / (P * K);    // whole: rounds of K elements that every lane has
  v4i q[NV];
  auto fetch = [&](uint32_t row) {
    const uint32_t end = w1 - row < R ? w1 : row + R;
    const uint32_t j0 = (row * n + run.skew) / V, j1 = (end * n + run.skew - 1u) / V;
#pragma unroll
    for (uint32_t u = 0; u < NV; ++u) q[u] = M::ld16(run.rin, row < w1 && j0 + u * 64u + lane <= j1 ? (j0 + u * 64u + lane) * 16u : kNoLoad);
  };
  auto get = [&](uint32_t i) {
    if constexpr (DT == GPUOS_I32) return ((const int32_t*)mem)[i];
    else if constexpr (DT == GPUOS_F32) return ((const float*)mem)[i];
    else if constexpr (DT == GPUOS_F16) return h2f(((const uint16_t*)mem)[i]);
    else return b2f(((const uint16_t*)mem)[i]);
  };
  fetch(w0);
  for (uint32_t row = w0; row < w1; row += R) {
#pragma unroll
    for (uint32_t u = 0; u < NV; ++u) ((v4i*)mem)[u * 64u + lane] = q[u];
    lds_wave_sync();
    fetch(row + R);
    const uint32_t rows = w1 - row < R ? w1 - row : R, lead = (row * n + run.skew) & (V - 1u);
    for (uint32_t rb = 0; rb < rows; rb += rps) {
      const uint32_t mr = rb + sub, at = lead + (mr < rows ? mr : rows - 1u) * n;
      A acc = red_identity<RIMPL, A>();
      uint32_t e = first;
      A x[K];
      for (uint32_t b = 0; b < whole; ++b) {
#pragma unroll
        for (uint32_t k = 0; k < K; ++k) x[k] = get(at + e + k * P);
        e += K * P;
        acc = red_join<RIMPL>(acc, x);
      }
      if (whole * K * P < n) {                               // the last elements: of a maximum, some are taken twice
#pragma unroll
        for (uint32_t k = 0; k < K; ++k) {
          const uint32_t i = e + k * P;
          x[k] = get(at + (i < n ? i : n - 1u));
          if (RIMPL == GPUOS_IMPL_SUM_LAST) x[k] = i < n ? x[k] : (A)0;
        }
        acc = red_join<RIMPL>(acc, x);
      }
      const A t = wave_reduce<RIMPL>(red_finish<RIMPL>(acc), P);
      red_put<POL>(ro, row - row_begin + mr, odt, t, first == 0 && mr < rows);
    }
    lds_wave_sync();
  }
}

// The same when every row is a whole number of vectors and starts on one (the attention shapes: rows
// of 64 / 128 / 256 16-bit elements): no edges to mask and nothing to remember per pass but the
// loaded vector, so eight passes stay in registers.
template <int POL, int RIMPL, int DT, bool LOADS_NT>
PATHFN void red_rows_short_aligned(RedArgs a) {
  const RedRun run = red_run(a);
  const uint32_t tid = a.tid;
  const uint32_t odt = uni(a.odt), row_begin = uni(a.row_begin), row_end = uni(a.row_end), vpr = uni(a.max_span);
  using E = Elem<DT>;
  using A = typename RedAcc<DT>::T;
  using M = Mem<POL, LOADS_NT>;
  constexpr uint32_t UP = 8;
  const uint32_t lane = tid & 63u, wave = uni(tid >> 6);
  uint32_t P = 1;                                     // lanes per row: power of two >= vectors per row
  while (P < vpr) P <<= 1;
  const uint32_t rpw = 64u / P, sub = lane / P, j = lane & (P - 1u);
  const bool gather = UP * rpw <= 64u;                // the pass's rows fit one lane each
  const bool mine = j < vpr;
  const rsrc_t ro = red_out(a, row_begin, row_end, odt);
  // (four vectors a lane are requested while the four before are worked on)
  constexpr uint32_t H = UP / 2;
  v4i qa[H], qb[H];
  auto fetch = [&](v4i (&q)[H], uint32_t base) {
#pragma unroll
    for (uint32_t u = 0; u < H; ++u) {
      const uint32_t row = base + u * rpw + sub;
      q[u] = M::ld16(run.rin, row < row_end && mine ? ((row - row_begin) * vpr + j) * 16u : kNoLoad);
    }
  };
  A res = 0;                                   // lane L ends up with the result of row base + L
  auto take = [&](const v4i (&q)[H], uint32_t base, uint32_t u0) {
#pragma unroll
    for (uint32_t u = 0; u < H; ++u) {
      const uint32_t row = base + (u0 + u) * rpw + sub;
      A x[E::V], acc = red_identity<RIMPL, A>();
#pragma unroll
      for (int k = 0; k < E::V; ++k) x[k] = red_get<DT>(q[u], k);
      acc = red_join<RIMPL>(acc, x);
      acc = mine ? red_finish<RIMPL>(acc) : red_identity<RIMPL, A>();
      acc = wave_reduce<RIMPL>(acc, P);
      if (gather) {
        const A got = __shfl(acc, (int)((lane & (rpw - 1u)) * P), 64);
        if (lane / rpw == u0 + u) res = got;
      } else {
        red_put<POL>(ro, row - row_begin, odt, acc, row < row_end && j == 0);
      }
    }
  };
  uint32_t base = row_begin + wave * rpw * UP;
  fetch(qa, base);
  for (; base < row_end; base += 4 * rpw * UP) {
    fetch(qb, base + H * rpw);
    take(qa, base, 0);
    fetch(qa, base + 4 * rpw * UP);
    take(qb, base, H);
    if (gather) red_put<POL>(ro, base + lane - row_begin, odt, res, lane < UP * rpw && base + lane < row_end);
  }
}

template <int POL, int RIMPL, int DT>
DEV void red_contig(const Record* r, uint32_t row_begin, uint32_t row_end, float* s_part, uint32_t tid) {
  using E = Elem<DT>;
  constexpr uint32_t V = E::V;
  const uint32_t n = uni(r->red_n);
  const char* pin = uni_ptr(r->ptr[0]);
  RedArgs a;
  a.n = n;
  a.lead = ((uint32_t)(__UINTPTR_TYPE__)pin & 15u) / E::ES;
  a.base_elem = (a.lead + row_begin * n) / V * V;     // chunk start, aligned down to a vector
  // end rounded up to a whole vector: the padding stays inside the 16-byte block that holds the last
  // element; vector loads further out read zeros; both are masked per element
  a.base = pin - a.lead * E::ES + (uint64_t)a.base_elem * E::ES;
  a.bytes = ((a.lead + row_end * n - a.base_elem) * E::ES + 15u) & ~15u;
  a.po = (char*)uni_ptr(r->ptr[3]);
  a.stream = uni(r->rflags) & RF_STREAM; a.odt = uni(r->dtype[3]); a.row_begin = row_begin; a.row_end = row_end; a.s_part = s_part; a.tid = tid;
  const bool whole = n % V == 0 && a.lead == 0;       // every row is whole vectors
  a.max_span = whole ? n / V : (n + V - 2) / V + 1;
  // (an executor for either form of load: where one chose at each round of loads, rows of 24 bf16, 1.1 GB, took 322 us instead of 257)
  if (a.max_span <= 64u && whole) { if (a.stream) red_rows_short_aligned<POL, RIMPL, DT, true>(a); else red_rows_short_aligned<POL, RIMPL, DT, false>(a); }
  else if (a.max_span <= kRedLdsSpan) red_rows_lds<POL, RIMPL, DT>(a);
  else if (a.max_span >= 1024u && row_end - row_begin <= kRedPartialRows) red_rows_quarter<POL, RIMPL, DT>(a);
  else red_rows_stream<POL, RIMPL, DT>(a);
}

// PATH_RED_GENERIC: one wave per output row; outer index decomposed over the
// coalesced outer dims; stride[0][5] walks the reduced dim.
template <int POL, int RIMPL, bool INT>
PATHFN void red_generic(const Record* r_v, uint32_t begin_v, uint32_t end_v, uint32_t tid) {
  const Record* r = lds_arg(r_v);
  const uint32_t row_begin = uni(begin_v), row_end = uni(end_v);
  using M = Mem<POL>;
  const int nd = (int)uni(r->ndim);                   // outer dims
  const uint32_t n = uni(r->red_n), sl = uni(r->stride[0][5]);
  const char* pin = uni_ptr(r->ptr[0]);
  char* po = (char*)uni_ptr(r->ptr[3]);
  const uint32_t idt = uni(r->dtype[0]), odt = uni(r->dtype[3]);
  const uint32_t lane = tid & 63u, wave = tid >> 6;
  for (uint32_t row = row_begin + wave; row < row_end; row += 4) {
    uint32_t rem = row, ioff = 0, ooff = 0;
#pragma unroll
    for (int d = GPUOS_MAX_DIMS - 2; d >= 0; --d) {
      if (d < nd) {
        const uint32_t sz = uni(r->size[d]);
        const uint32_t q = rem / sz, idx = rem - q * sz;
        rem = q;
        ioff += idx * uni(r->stride[0][d]);
        ooff += idx * uni(r->stride[3][d]);
      }
    }
    if (INT) {
      int32_t acc = red_identity<RIMPL, int32_t>();
      for (uint32_t jx = lane; jx < n; jx += 64) acc = red_combine<RIMPL>(acc, (int32_t)M::ld4(pin, ioff + jx * sl));
      acc = wave_reduce<RIMPL>(acc, 64);
      if (lane == 0) M::st4(po, ooff, (uint32_t)acc);
    } else {
      float acc = red_identity<RIMPL, float>();
      for (uint32_t jx = lane; jx < n; jx += 64) acc = red_combine<RIMPL>(acc, load_rt<POL>(pin, ioff + jx * sl, idt));
      acc = wave_reduce<RIMPL>(acc, 64);
      if (lane == 0) red_store<POL>(po, ooff, odt, acc);
    }
  }
}

// ---------------------------------------------------------------------------
// fused row operations (operator library, Section 5.2: softmax, layer normalisation).
// Each row of the last dim is one problem; the output has the input's shape.
//   PATH_ROW_FUSED, PATH_ROW_RAGGED: one dtype, contiguous rows that hold at least a vector; whole aligned
//     vectors, or any length and alignment.
//     A row is cut into 16-byte vectors from its first element on; in a row that is no multiple the
//     last vector covers the row's last V elements, and those the vector before it holds count for
//     nothing (RAGGED: also rows whose base is not 16-byte aligned; accesses need element alignment only).
//     Up to 256 vectors a row is read once into the registers of the P lanes that own it
//     (P = 64 for rows over 64 vectors, else the power of two >= vectors per row, 64 / P rows
//     per wavefront pass), reduced with xor butterflies over those lanes, and written once; longer
//     rows belong to the workgroup (rowop_wg, softmax_held, masked_softmax_long, layernorm_long).
//   PATH_ROW_GENERIC: any strides and dtypes; one wavefront per row, three passes over memory.
// Arithmetic is fp32.  Lanes outside a row feed the identity (-inf to the softmax, 0 to the
// sums).  The softmax maximum ignores NaN; a NaN still poisons its row through the sum.
// ---------------------------------------------------------------------------
DEV float bfly_sum(float v, uint32_t width) { return wave_reduce<GPUOS_IMPL_SUM_LAST>(v, width); }
DEV float bfly_max(float v, uint32_t width) {          // (NaN is left out, the sum of exponentials brings it back)
  float a, b;
  if (width > 32) { butterfly_pair<32>(v, a, b); v = __builtin_fmaxf(a, b); }
  if (width > 16) { butterfly_pair<16>(v, a, b); v = __builtin_fmaxf(a, b); }
  if (width > 8) { butterfly_pair<8>(v, a, b); v = __builtin_fmaxf(a, b); }
  if (width > 4) { butterfly_pair<4>(v, a, b); v = __builtin_fmaxf(a, b); }
  if (width > 2) { butterfly_pair<2>(v, a, b); v = __builtin_fmaxf(a, b); }
  if (width > 1) { butterfly_pair<1>(v, a, b); v = __builtin_fmaxf(a, b); }
  return v;
}

template <int ROP> struct RowOp {
  static constexpr int NIN = ROP == GPUOS_IMPL_SOFTMAX_LAST ? 1 : (ROP == GPUOS_IMPL_MASKED_SOFTMAX_LAST ? 2 : 3);
  static constexpr bool SOFTMAX = ROP != GPUOS_IMPL_LAYERNORM_LAST;
};

// gamma / beta of a layer norm for the V elements of one vector position: of x's dtype (one
// 16-byte vector), or fp32 under 16-bit x (P32: two vectors), as frameworks keep them.
template <int POL, int DT, bool P32> struct RowParam {
  v4i q[P32 ? 2 : 1];
  DEV void load(rsrc_t rs, uint32_t col) {             // from element `col` of the row on
    if (P32) { q[0] = Mem<POL>::ld16(rs, col * 4u); q[P32 ? 1 : 0] = Mem<POL>::ld16(rs, col * 4u + 16u); }
    else q[0] = Mem<POL>::ld16(rs, col * (uint32_t)Elem<DT>::ES);
  }
  // What is kept over rows stays as it was loaded: without this its conversion moves in front of the first
  // row's loads, behind a wait for memory.
  DEV void keep() {
    if (P32) asm volatile("" : "+v"(q[0]), "+v"(q[P32 ? 1 : 0]));
    else asm volatile("" : "+v"(q[0]));
  }
  DEV float get(int e) const {
    if (P32) return Elem<GPUOS_F32>::get(q[(e >> 2) & (P32 ? 1 : 0)], e & 3);
    return Elem<DT>::get(q[0], e);
  }
};

// The vectors of a row of n elements: vector `vec` begins at element begin(vec), and its elements from
// first(vec) on are its own.
template <int V, bool RAGGED> struct RowCut {
  uint32_t n, vpr, tail;                               // vectors per row; elements of the last one that are its own (0: all)
  DEV explicit RowCut(uint32_t n_) : n(n_), vpr((n_ + V - 1) / V), tail(n_ % V) {}
  DEV bool last(uint32_t vec) const { return RAGGED && tail != 0 && vec == vpr - 1; }
  DEV uint32_t begin(uint32_t vec) const { return last(vec) ? n - V : vec * V; }
  DEV int first(uint32_t vec) const { return last(vec) ? V - (int)tail : 0; }
};
// One vector of the output, its own elements only.  STRAIGHT: no branch round the store.  Where several rows'
// loads are in flight, a store that may not have been issued makes the wait for the next row's loads
// one for stores too; where a pass is requested ahead, or the workgroup owns the row, the branch costs less
// (softmax of 65,536 x 24 fp32: 28.7 us with the branch, 25.6 without; layer norm of 1,024 x 2,048 bf16 19.5 and 26.5).
template <int POL, int DT, bool RAGGED, bool STRAIGHT = false> DEV void row_store(rsrc_t ro, uint32_t off, const v4i& q, bool act, int first) {
  using E = Elem<DT>;
  using M = Mem<POL, false, true>;
  if (!RAGGED && STRAIGHT) { M::st16(ro, act ? off : kNoLoad, q); return; }
  if (!RAGGED) { if (act) M::st16(ro, off, q); return; }
  M::st16(ro, act && first == 0 ? off : kNoLoad, q);
  if (act && first != 0) {
#pragma unroll
    for (int e = 1; e < (int)E::V; ++e)
      if (e >= first) {
        if (E::ES == 4) M::stb4(ro, off + e * 4u, (uint32_t)q[e & 3]);
        else M::stb2(ro, off + e * 2u, (uint32_t)q[e / 2] >> ((e & 1) * 16));
      }
  }
}

// Bound by memory for fp32, by memory and conversions together for 16-bit rows.  A pass (UP rows per lane
// group) is a chain load -> reduce -> reduce -> store; layer norm over 16-bit rows, whose chunks are
// several passes, requests the next pass before it computes this one.  (Softmax rows are not: the registers for it
// make the function save its caller's, a memory round trip per chunk.)
template <int POL, int ROP, int DT, int KW, int UP, bool P32, bool RAGGED>
DEV void rowop_fused(const Record* r, uint32_t row_begin, uint32_t row_end, float* s_v, uint32_t tid) {
  using E = Elem<DT>;
  using M = Mem<POL, false, true>;
  using RO = RowOp<ROP>;
  constexpr uint32_t V = E::V;
  constexpr bool MASK = ROP == GPUOS_IMPL_MASKED_SOFTMAX_LAST;
  const uint32_t n = uni(r->red_n);
  const RowCut<V, RAGGED> cut(n);
  const uint32_t vpr = cut.vpr;
  const uint32_t lane = tid & 63u, wave = tid >> 6;
  uint32_t P = 64;
  if (KW == 1) { P = 1; while (P < vpr) P <<= 1; }
  const uint32_t rpw = 64u / P, sub = lane / P, j = lane & (P - 1u);
  const float alpha = r->alpha;
  const uint32_t nrows = row_end - row_begin;
  const uint32_t chunk_bytes = nrows * n * E::ES;
  const uint64_t chunk_off = (uint64_t)row_begin * n * E::ES;
  const rsrc_t rx = make_rsrc(uni_ptr(r->ptr[0]) + chunk_off, chunk_bytes);
  const rsrc_t ro = make_rsrc(uni_ptr(r->ptr[3]) + chunk_off, chunk_bytes);
  // second / third input: laid out like x (K_FULL) or a [period, n] block reused every period rows;
  // layer norm: gamma and beta are always one row
  rsrc_t rs[2];
  uint32_t period = 0;
#pragma unroll
  for (int k = 1; k < RO::NIN; ++k) {
    if (!RO::SOFTMAX) {
      rs[k - 1] = make_rsrc(uni_ptr(r->ptr[k]), n * (P32 ? 4u : (uint32_t)E::ES));
    } else if (uni(r->okind[k]) == K_FULL) {
      rs[k - 1] = make_rsrc(uni_ptr(r->ptr[k]) + chunk_off, chunk_bytes);
    } else {
      period = uni(r->stride[k][0]);
      rs[k - 1] = make_rsrc(uni_ptr(r->ptr[k]), period * n * E::ES);
    }
  }
  // this lane's vectors are the same in every row
  uint32_t at[KW];                                     // byte offset in a row
  int first[KW];
#pragma unroll
  for (int k = 0; k < KW; ++k) {
    const uint32_t vec = j + 64u * k;
    at[k] = cut.begin(vec) * E::ES;
    first[k] = cut.first(vec);
  }
  const uint32_t step = 4u * rpw * UP;
  struct Pass { v4i q[UP][KW], mq[MASK ? UP : 1][MASK ? KW : 1]; };
  auto load = [&](Pass& p, uint32_t base) {            // a row past the chunk is not fetched
#pragma unroll
    for (int u = 0; u < UP; ++u) {
      const uint32_t row = base + u * rpw + sub, lr = row - row_begin;
      uint32_t mr = lr;
      if (MASK && period) mr = row % period;
#pragma unroll
      for (int k = 0; k < KW; ++k) {
        const bool act = row < row_end && j + 64u * k < vpr;
        p.q[u][k] = M::ld16(rx, act ? lr * n * E::ES + at[k] : kNoLoad);
        if (MASK) p.mq[u][k] = M::ld16(rs[0], act ? mr * n * E::ES + at[k] : kNoLoad);
      }
    }
  };
  uint32_t base = row_begin + wave * rpw * UP;
  constexpr bool AHEAD = !RO::SOFTMAX && DT != GPUOS_F32;
  Pass cur, nxt;
  if (AHEAD) load(cur, base);
  // layer norm: gamma and beta lie in LDS, vector by vector (each wavefront loading its own to registers
  // fetched them four times a chunk, as many bytes as the chunk's rows, and left none for the next pass)
  v4i* const params = (v4i*)s_v;                       // [2][vpr][PQ]
  // Not for fp32 rows, which are short of neither registers nor arithmetic: there the staging, its
  // barrier and the registers of the next pass cost 3 us of 22 on 2M elements.
  constexpr uint32_t PQ = P32 ? 2 : 1;
  constexpr int KP = AHEAD || RO::SOFTMAX ? 1 : KW;
  RowParam<POL, DT, P32> gk[KP], bk[KP];
  if (!RO::SOFTMAX && !AHEAD) {
#pragma unroll
    for (int k = 0; k < KP; ++k) {
      const uint32_t col = j + 64u * k < vpr ? cut.begin(j + 64u * k) : 0u;
      gk[k].load(rs[0], col);
      bk[k].load(rs[1], col);
    }
  }
  static_assert(2 * 256 * 2 * 4 <= kScratchFloats, "two rows of 256 vectors of fp32 parameters under 16-bit elements");
  if (AHEAD) {
    for (uint32_t vec = tid; vec < vpr; vec += kThreads) {
      RowParam<POL, DT, P32> g, b;
      g.load(rs[0], cut.begin(vec));
      b.load(rs[1], cut.begin(vec));
#pragma unroll
      for (uint32_t i = 0; i < PQ; ++i) { params[vec * PQ + i] = g.q[i]; params[(vpr + vec) * PQ + i] = b.q[i]; }
    }
    __syncthreads();
  }
  for (; base < row_end; base += step) {
    if (AHEAD) load(nxt, base + step);
    else load(cur, base);
#pragma unroll
    for (int u = 0; u < UP; ++u) {
      const uint32_t row = base + u * rpw + sub, lr = row - row_begin;
      float t[KW][V];
      bool act[KW];
#pragma unroll
      for (int k = 0; k < KW; ++k) act[k] = row < row_end && j + 64u * k < vpr;
      if (RO::SOFTMAX) {
        float m = -__builtin_inff();
#pragma unroll
        for (int k = 0; k < KW; ++k)
#pragma unroll
          for (int e = 0; e < (int)V; ++e) {
            float x = E::get(cur.q[u][k], e);
            if (MASK) x = alpha * x + E::get(cur.mq[MASK ? u : 0][MASK ? k : 0], e);
            t[k][e] = act[k] && (!RAGGED || e >= first[k]) ? x : -__builtin_inff();
            m = __builtin_fmaxf(m, t[k][e]);
          }
        m = bfly_max(m, P);
        float s = 0.0f;
#pragma unroll
        for (int k = 0; k < KW; ++k)
#pragma unroll
          for (int e = 0; e < (int)V; ++e) { t[k][e] = __expf(t[k][e] - m); s += t[k][e]; }
        s = bfly_sum(s, P);
        const float inv = 1.0f / s;
#pragma unroll
        for (int k = 0; k < KW; ++k) {
          v4i oq;
#pragma unroll
          for (int e = 0; e < (int)V; ++e) E::put(oq, e, t[k][e] * inv);
          row_store<POL, DT, RAGGED, !AHEAD>(ro, lr * n * E::ES + at[k], oq, act[k], first[k]);
        }
      } else {
        float s = 0.0f;
#pragma unroll
        for (int k = 0; k < KW; ++k)
#pragma unroll
          for (int e = 0; e < (int)V; ++e) { t[k][e] = E::get(cur.q[u][k], e); s += act[k] && (!RAGGED || e >= first[k]) ? t[k][e] : 0.0f; }
        const float mean = bfly_sum(s, P) / (float)n;
        float ss = 0.0f;
#pragma unroll
        for (int k = 0; k < KW; ++k)
#pragma unroll
          for (int e = 0; e < (int)V; ++e) { t[k][e] -= mean; ss += act[k] && (!RAGGED || e >= first[k]) ? t[k][e] * t[k][e] : 0.0f; }
        const float var = bfly_sum(ss, P) / (float)n;
        const float rstd = 1.0f / __builtin_sqrtf(var + alpha);
#pragma unroll
        for (int k = 0; k < KW; ++k) {
          v4i oq;
          RowParam<POL, DT, P32> g, b;
          if (AHEAD) {
            const uint32_t vec = j + 64u * k < vpr ? j + 64u * k : 0u;
#pragma unroll
            for (uint32_t i = 0; i < PQ; ++i) { g.q[i] = params[vec * PQ + i]; b.q[i] = params[(vpr + vec) * PQ + i]; }
          } else {
            g = gk[k < KP ? k : 0];
            b = bk[k < KP ? k : 0];
          }
#pragma unroll
          for (int e = 0; e < (int)V; ++e) E::put(oq, e, t[k][e] * rstd * g.get(e) + b.get(e));
          row_store<POL, DT, RAGGED, !AHEAD>(ro, lr * n * E::ES + at[k], oq, act[k], first[k]);
        }
      }
    }
    if (AHEAD) cur = nxt;
  }
  if (AHEAD) __syncthreads();                          // the LDS belongs to the next chunk after this
}

template <int POL, int ROP>
PATHFN void rowop_generic(const Record* r_v, uint32_t begin_v, uint32_t end_v, uint32_t tid) {
  const Record* r = lds_arg(r_v);
  const uint32_t row_begin = uni(begin_v), row_end = uni(end_v);
  using RO = RowOp<ROP>;
  const int nd = (int)uni(r->ndim);                   // outer dims
  const uint32_t n = uni(r->red_n);
  const float alpha = r->alpha;
  const char* p[3];
  uint32_t dt[3], sl[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int kk = k < RO::NIN ? k : 0;
    p[k] = uni_ptr(r->ptr[kk]); dt[k] = uni(r->dtype[kk]); sl[k] = uni(r->stride[kk][5]);
  }
  char* po = (char*)uni_ptr(r->ptr[3]);
  const uint32_t odt = uni(r->dtype[3]), slo = uni(r->stride[3][5]);
  const uint32_t lane = tid & 63u, wave = tid >> 6;
  for (uint32_t row = row_begin + wave; row < row_end; row += 4) {
    uint32_t rem = row, off[3] = {0, 0, 0}, ooff = 0;
#pragma unroll
    for (int d = GPUOS_MAX_DIMS - 2; d >= 0; --d) {
      if (d < nd) {
        const uint32_t sz = uni(r->size[d]);
        const uint32_t qd = rem / sz, idx = rem - qd * sz;
        rem = qd;
#pragma unroll
        for (int k = 0; k < RO::NIN; ++k) off[k] += idx * uni(r->stride[k][d]);
        ooff += idx * uni(r->stride[3][d]);
      }
    }
    if (RO::SOFTMAX) {
      auto arg = [&](uint32_t jx) {
        float x = load_rt<POL>(p[0], off[0] + jx * sl[0], dt[0]);
        if (ROP == GPUOS_IMPL_MASKED_SOFTMAX_LAST) x = alpha * x + load_rt<POL>(p[1], off[1] + jx * sl[1], dt[1]);
        return x;
      };
      float m = -__builtin_inff();
      for (uint32_t jx = lane; jx < n; jx += 64) m = __builtin_fmaxf(m, arg(jx));
      m = bfly_max(m, 64);
      float s = 0.0f;
      for (uint32_t jx = lane; jx < n; jx += 64) s += __expf(arg(jx) - m);
      s = bfly_sum(s, 64);
      const float inv = 1.0f / s;
      for (uint32_t jx = lane; jx < n; jx += 64) store_rt<POL>(po, ooff + jx * slo, odt, __expf(arg(jx) - m) * inv);
    } else {
      float s = 0.0f;
      for (uint32_t jx = lane; jx < n; jx += 64) s += load_rt<POL>(p[0], off[0] + jx * sl[0], dt[0]);
      const float mean = bfly_sum(s, 64) / (float)n;
      float ss = 0.0f;
      for (uint32_t jx = lane; jx < n; jx += 64) {
        const float d = load_rt<POL>(p[0], off[0] + jx * sl[0], dt[0]) - mean;
        ss += d * d;
      }
      const float var = bfly_sum(ss, 64) / (float)n;
      const float rstd = 1.0f / __builtin_sqrtf(var + alpha);
      for (uint32_t jx = lane; jx < n; jx += 64) {
        const float d = load_rt<POL>(p[0], off[0] + jx * sl[0], dt[0]) - mean;
        store_rt<POL>(po, ooff + jx * slo, odt,
                      d * rstd * load_rt<POL>(p[1], off[1] + jx * sl[1], dt[1]) + load_rt<POL>(p[2], off[2] + jx * sl[2], dt[2]));
      }
    }
  }
}

// Sum / maximum over the workgroup, through four rotating LDS slots: one barrier per reduction.
struct WgReduce {
  float* slots;                                        // 16 floats
  uint32_t turn, tid;
  DEV float* next() { float* p = slots + (turn & 3u) * 4u; ++turn; return p; }
  DEV float sum(float v) {
    v = bfly_sum(v, 64);
    float* slot = next();
    if ((tid & 63u) == 0) slot[tid >> 6] = v;
    __syncthreads();
    return (slot[0] + slot[1]) + (slot[2] + slot[3]);
  }
  DEV float max(float v) {
    v = bfly_max(v, 64);
    float* slot = next();
    if ((tid & 63u) == 0) slot[tid >> 6] = v;
    __syncthreads();
    return __builtin_fmaxf(__builtin_fmaxf(slot[0], slot[1]), __builtin_fmaxf(slot[2], slot[3]));
  }
};

// Rows longer than one wavefront's registers: the whole workgroup owns a row and holds it in
// registers, 256 lanes x KW vectors, read once and written once.
template <int POL, int ROP, int DT, int KW, bool P32, bool RAGGED>
DEV void rowop_wg(const Record* r, uint32_t row_begin, uint32_t row_end, float* s_red, uint32_t tid) {
  using E = Elem<DT>;
  using M = Mem<POL, false, true>;
  using RO = RowOp<ROP>;
  constexpr uint32_t V = E::V;
  constexpr bool MASK = ROP == GPUOS_IMPL_MASKED_SOFTMAX_LAST;
  const uint32_t n = uni(r->red_n);
  const RowCut<V, RAGGED> cut(n);
  const uint32_t vpr = cut.vpr;
  const float alpha = r->alpha;
  const uint32_t nrows = row_end - row_begin;
  const uint32_t chunk_bytes = nrows * n * E::ES;
  const uint64_t chunk_off = (uint64_t)row_begin * n * E::ES;
  const rsrc_t rx = make_rsrc(uni_ptr(r->ptr[0]) + chunk_off, chunk_bytes);
  const rsrc_t ro = make_rsrc(uni_ptr(r->ptr[3]) + chunk_off, chunk_bytes);
  rsrc_t rs[2];
  uint32_t period = 0;
#pragma unroll
  for (int k = 1; k < RO::NIN; ++k) {
    if (!RO::SOFTMAX) {
      rs[k - 1] = make_rsrc(uni_ptr(r->ptr[k]), n * (P32 ? 4u : (uint32_t)E::ES));      // gamma, beta: one row
    } else if (uni(r->okind[k]) == K_FULL) {
      rs[k - 1] = make_rsrc(uni_ptr(r->ptr[k]) + chunk_off, chunk_bytes);
    } else {
      period = uni(r->stride[k][0]);
      rs[k - 1] = make_rsrc(uni_ptr(r->ptr[k]), period * n * E::ES);
    }
  }
  // layer norm: up to four vectors a lane, this lane's gamma and beta stay in registers; longer rows
  // fill them, and fetch the two again
  constexpr int KP = !RO::SOFTMAX && KW <= 4 ? KW : 1;
  RowParam<POL, DT, P32> gk[KP], bk[KP];
  if (!RO::SOFTMAX && KW <= 4) {
#pragma unroll
    for (int k = 0; k < KP; ++k) {
      const uint32_t vec = tid + kThreads * k;
      gk[k].load(rs[0], vec < vpr ? cut.begin(vec) : 0u);
      bk[k].load(rs[1], vec < vpr ? cut.begin(vec) : 0u);
    }
  }
  WgReduce wg = {s_red, 0, tid};
  for (uint32_t row = row_begin; row < row_end; ++row) {
    const uint32_t lr = row - row_begin;
    uint32_t mr = lr;
    if (MASK && period) mr = row % period;
    v4i q[KW], mq[MASK ? KW : 1];
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      const uint32_t vec = tid + kThreads * k;
      const uint32_t at = cut.begin(vec) * E::ES;
      q[k] = M::ld16(rx, vec < vpr ? lr * n * E::ES + at : kNoLoad);
      if (MASK) mq[k] = M::ld16(rs[0], vec < vpr ? mr * n * E::ES + at : kNoLoad);
    }
    float t[KW][V];
    auto own = [&](int k, int e) { const uint32_t vec = tid + kThreads * k; return vec < vpr && (!RAGGED || e >= cut.first(vec)); };
    if (RO::SOFTMAX) {
      float m = -__builtin_inff();
#pragma unroll
      for (int k = 0; k < KW; ++k)
#pragma unroll
        for (int e = 0; e < (int)V; ++e) {
          float x = E::get(q[k], e);
          if (MASK) x = alpha * x + E::get(mq[MASK ? k : 0], e);
          t[k][e] = own(k, e) ? x : -__builtin_inff();
          m = __builtin_fmaxf(m, t[k][e]);
        }
      m = wg.max(m);
      float sum = 0.0f;
#pragma unroll
      for (int k = 0; k < KW; ++k)
#pragma unroll
        for (int e = 0; e < (int)V; ++e) { t[k][e] = __expf(t[k][e] - m); sum += t[k][e]; }
      const float inv = 1.0f / wg.sum(sum);
#pragma unroll
      for (int k = 0; k < KW; ++k) {
        const uint32_t vec = tid + kThreads * k;
        v4i oq;
#pragma unroll
        for (int e = 0; e < (int)V; ++e) E::put(oq, e, t[k][e] * inv);
        row_store<POL, DT, RAGGED>(ro, lr * n * E::ES + cut.begin(vec) * E::ES, oq, vec < vpr, cut.first(vec));
      }
    } else {
      float sum = 0.0f;
#pragma unroll
      for (int k = 0; k < KW; ++k)
#pragma unroll
        for (int e = 0; e < (int)V; ++e) { t[k][e] = E::get(q[k], e); sum += own(k, e) ? t[k][e] : 0.0f; }
      const float mean = wg.sum(sum) / (float)n;
      float ss = 0.0f;
#pragma unroll
      for (int k = 0; k < KW; ++k)
#pragma unroll
        for (int e = 0; e < (int)V; ++e) { t[k][e] -= mean; ss += own(k, e) ? t[k][e] * t[k][e] : 0.0f; }
      const float rstd = 1.0f / __builtin_sqrtf(wg.sum(ss) / (float)n + alpha);
#pragma unroll
      for (int k = 0; k < KW; ++k) {
        const uint32_t vec = tid + kThreads * k;
        RowParam<POL, DT, P32> g, b;
        if (KW <= 4) {
          gk[k < KP ? k : 0].keep(); bk[k < KP ? k : 0].keep();
          g = gk[k < KP ? k : 0]; b = bk[k < KP ? k : 0];
        } else {
          g.load(rs[0], vec < vpr ? cut.begin(vec) : 0u);
          b.load(rs[1], vec < vpr ? cut.begin(vec) : 0u);
        }
        v4i oq;
#pragma unroll
        for (int e = 0; e < (int)V; ++e) E::put(oq, e, t[k][e] * rstd * g.get(e) + b.get(e));
        row_store<POL, DT, RAGGED>(ro, lr * n * E::ES + cut.begin(vec) * E::ES, oq, vec < vpr, cut.first(vec));
      }
    }
  }
  __syncthreads();                                     // the LDS slots belong to the next chunk after this
}

// Softmax rows too long for the workgroup's registers (over 16,384 elements): two passes over the row.
// The first keeps a running maximum and a sum relative to it per lane, rescaled once per
// batch of vectors; the second writes.
// A lane's first NB batches of three vectors stay in registers (up to eighteen, 72 of the 128: with twenty some went through scratch
// memory) and the next six in LDS; the second pass reads only what is left, of a row of 32,003 fp32 elements eight of 32.  Bound
// by memory: 2 x 1,024 such rows took 175 us with twelve in registers, and as many of a caller's saved and restored (525 MB
// read, 392 MB written, of 262 each); 134 so, of which the plain loads are 5.
// A row has more vectors a lane than stay in registers: those are whole and need no look at the row's end.
// Ragged rows are cut where memory's 16-byte blocks begin, if x and the output lie alike in them: a block at
// either end of a row is shared with its neighbour, every other access is a whole aligned one.  (The block
// that holds a tensor's first or last element may hold bytes outside it, in the same page.)  Cut from a row's
// first element on, each store is written in two parts: 2 x 1,024 rows of 32,003 fp32 wrote 1.7 times and
// read 2.2 times their bytes, 204 us; 181 cut at blocks.
template <int POL, int DT, int NB, bool RAGGED>
DEV void softmax_held(const Record* r, uint32_t row_begin, uint32_t row_end, float* s_v, uint32_t tid) {
  using E = Elem<DT>;
  using M = Mem<POL, false, true>;
  constexpr uint32_t V = E::V, U = 3, NR = NB * U, NL = 6;
  const uint32_t n = uni(r->red_n);
  const uint32_t chunk_bytes = (row_end - row_begin) * n * E::ES;
  const uint64_t chunk_off = (uint64_t)row_begin * n * E::ES;
  const char* const px = uni_ptr(r->ptr[0]) + chunk_off;
  const char* const po = uni_ptr(r->ptr[3]) + chunk_off;
  const BlockCut bc = RAGGED ? block_cut((__UINTPTR_TYPE__)px, (__UINTPTR_TYPE__)po, chunk_bytes) : BlockCut{false, 0u, chunk_bytes};
  const bool blocks = bc.blocks;
  const uint32_t front = bc.front, window = bc.window;
  const rsrc_t rx = make_rsrc(px - front, window);
  const rsrc_t ro = make_rsrc(po - front, window);
  WgReduce wg = {s_v, 0, tid};
  v4i* const kept = (v4i*)(s_v + 16) + tid;            // vector NR + i of this lane lies at kept[i * kThreads]
  static_assert(16 + NL * kThreads * 4 <= kScratchFloats, "six vectors per lane");
  // (A vector's index anew wherever it is asked for: kept for every vector, as the compiler would have it, the indices
  // and what follows from them go through scratch memory.)
  auto vector = [&](uint32_t i) {
    uint32_t v = tid;
    asm volatile("" : "+v"(v));
    return v + kThreads * i;
  };
  for (uint32_t row = row_begin; row < row_end; ++row) {
    // vector `vec` begins at element vec * V - lead of the row (or, its last where rows are not cut at blocks, at n - V)
    const uint32_t start = front + (row - row_begin) * n * E::ES, lead = blocks ? (start & 15u) / E::ES : 0u;
    const uint32_t vpr = (lead + n + V - 1) / V;
    const uint32_t x0 = start - lead * E::ES, mine = x0 + tid * 16u;       // the first vector's first byte, this lane's first
    const uint32_t T = (vpr + kThreads - 1) / kThreads;        // vectors per lane, the last partly filled
    const uint32_t back = RAGGED && !blocks ? vpr * V - n : 0u;          // elements the last vector is shifted back by
    constexpr uint32_t kStep = kThreads * 16u;
    auto at_of = [&](uint32_t vec) { return x0 + vec * 16u - (RAGGED && vec == vpr - 1 ? back * (uint32_t)E::ES : 0u); };    // (past NR)
    auto fetch = [&](uint32_t i) {
      const uint32_t vec = vector(i);
      return M::ld16(rx, vec < vpr ? at_of(vec) : kNoLoad);
    };
    // Elements that are not the row's become -inf, once: they then count for nothing in the maximum and the sum.
    auto settle = [&](uint32_t i, v4i& q) {
      const uint32_t vec = vector(i);
      const bool tail = vec + 1u == vpr;
      const int lo = tail ? (int)back : 0;
      const int hi = vec < vpr ? (RAGGED && blocks && tail ? (int)(lead + n - vec * V) : (int)V) : 0;
#pragma unroll
      for (int e = 0; e < (int)V; ++e) E::put(q, e, e >= lo && e < hi ? E::get(q, e) : -__builtin_inff());
    };
    float m = -__builtin_inff(), sum = 0.0f;
    auto take = [&](const v4i (&q)[U]) {
      float mb = m;
#pragma unroll
      for (uint32_t u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < (int)V; ++e) mb = __builtin_fmaxf(mb, E::get(q[u], e));
      const float ref = mb == -__builtin_inff() ? 0.0f : mb;       // (nothing but -inf so far: relative to 0, every term is 0)
      float part[U];                                   // (added in pairs: a shorter chain, and a smaller error)
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        float t[V];
#pragma unroll
        for (int e = 0; e < (int)V; ++e) t[e] = __expf(E::get(q[u], e) - ref);
#pragma unroll
        for (int w = (int)V / 2; w > 0; w /= 2)
#pragma unroll
          for (int e = 0; e < w; ++e) t[e] += t[e + w];
        part[u] = t[0];
        __builtin_amdgcn_sched_barrier(0);             // (a vector at a time: interleaved they need more registers than there are)
      }
      sum = __builtin_fmaf(sum, __expf(m - ref), (part[0] + part[1]) + part[2]);
      m = mb;
      __builtin_amdgcn_sched_barrier(0);
    };
    v4i keep[NB][U], q[U];
    auto fetch_batch = [&](uint32_t i0) {
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) q[u] = fetch(i0 + u);
    };
    auto take_batch = [&](uint32_t i0) {
#pragma unroll
      for (uint32_t u = 0; u < U; ++u)
        if (i0 + u < NR + NL) kept[(i0 + u - NR) * kThreads] = q[u];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) { settle(i0 + u, q[u]); __builtin_amdgcn_sched_barrier(0); }
      take(q);
    };
    // The first batch of those that do not stay in registers, then all that do, are requested in one go; the second of the
    // former while the latter are looked at.
    fetch_batch(NR);
#pragma unroll
    for (uint32_t i = 0; i < NR; ++i) keep[i / U][i % U] = M::ld16(rx, mine, i * kStep);
    take_batch(NR);
    if (T > NR + U) fetch_batch(NR + U);
    if (RAGGED) {                                      // (the first lane's first vector begins before the row)
#pragma unroll
      for (uint32_t e = 0; e < V; ++e) E::put(keep[0][0], (int)e, tid != 0 || e >= lead ? E::get(keep[0][0], (int)e) : -__builtin_inff());
    }
#pragma unroll
    for (uint32_t c = 0; c < NB; ++c) {
      take(keep[c]);
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) asm volatile("" : "+v"(keep[c][u]));      // (its fp32 values are not kept, they are made again)
    }
    for (uint32_t i0 = NR + U; i0 < T; i0 += U) {
      if (i0 != NR + U) fetch_batch(i0);
      take_batch(i0);
    }
    if (T > NR + NL) fetch_batch(NR + NL);             // (what is read again: ahead of the row's stores, which later loads wait for)
    const float M_ = wg.max(m);
    const float inv = 1.0f / wg.sum(sum * __expf(m - M_));
    auto result = [&](const v4i& x) {
      v4i oq;
#pragma unroll
      for (int e = 0; e < (int)V; ++e) E::put(oq, e, __expf(E::get(x, e) - M_) * inv);
      return oq;
    };
    auto put = [&](uint32_t i, const v4i& x) {         // vector 0, and those past NR
      const uint32_t vec = vector(i);
      const v4i oq = result(x);
      const bool act = vec < vpr;
      const uint32_t off = i == 0 ? mine : at_of(vec);
      // (partly owned: the last vector where it is shifted or ends the row in a block, the first where the row begins in one)
      const bool part = RAGGED && ((vec == 0 && lead != 0) || (vec == vpr - 1 && (vpr * V != lead + n)));
      M::st16(ro, act && !part ? off : kNoLoad, oq);
      if (RAGGED && act && part) {
#pragma unroll
        for (int e = 0; e < (int)V; ++e) {
          const uint32_t at = vec * V + e;             // (counted from the first vector's first element)
          if (blocks ? at - lead < n : (uint32_t)e >= back) {
            if (E::ES == 4) M::stb4(ro, off + e * 4u, (uint32_t)oq[e & 3]);
            else M::stb2(ro, off + e * 2u, (uint32_t)oq[e / 2] >> ((e & 1) * 16));
          }
        }
      }
    };
    if (RAGGED) put(0, keep[0][0]);
    else M::st16(ro, mine, result(keep[0][0]));
#pragma unroll
    for (uint32_t i = 1; i < NR; ++i) {
      M::st16(ro, x0 + vector(i) * 16u, result(keep[i / U][i % U]));
      __builtin_amdgcn_sched_barrier(0);
    }
    for (uint32_t i = NR; i < NR + NL && i < T; ++i) put(i, kept[(i - NR) * kThreads]);
    for (uint32_t i0 = NR + NL; i0 < T; i0 += U) {
      if (i0 != NR + NL) fetch_batch(i0);
#pragma unroll
      for (uint32_t u = 0; u < U; ++u)
        if (i0 + u < T) put(i0 + u, q[u]);
    }
  }
  __syncthreads();                                     // the LDS belongs to the next chunk after this
}

// Masked softmax rows too long for the workgroup's registers: two passes over row and mask, nothing kept between them.
template <int POL, int DT, bool RAGGED>
DEV void masked_softmax_long(const Record* r, uint32_t row_begin, uint32_t row_end, float* s_v, uint32_t tid) {
  using E = Elem<DT>;
  using M = Mem<POL, false, true>;
  constexpr uint32_t V = E::V, U = 4;
  const uint32_t n = uni(r->red_n);
  const RowCut<V, RAGGED> cut(n);
  const uint32_t vpr = cut.vpr;
  const float alpha = r->alpha;
  const uint32_t chunk_bytes = (row_end - row_begin) * n * E::ES;
  const uint64_t chunk_off = (uint64_t)row_begin * n * E::ES;
  const rsrc_t rx = make_rsrc(uni_ptr(r->ptr[0]) + chunk_off, chunk_bytes);
  const rsrc_t ro = make_rsrc(uni_ptr(r->ptr[3]) + chunk_off, chunk_bytes);
  rsrc_t rm = rx;
  uint32_t period = 0;
  if (uni(r->okind[1]) == K_FULL) rm = make_rsrc(uni_ptr(r->ptr[1]) + chunk_off, chunk_bytes);
  else { period = uni(r->stride[1][0]); rm = make_rsrc(uni_ptr(r->ptr[1]), period * n * E::ES); }
  WgReduce wg = {s_v, 0, tid};
  for (uint32_t row = row_begin; row < row_end; ++row) {
    const uint32_t x0 = (row - row_begin) * n * E::ES, m0 = (period ? row % period : row - row_begin) * n * E::ES;
    v4i q[U], mq[U];
    auto fetch_batch = [&](uint32_t v0) {
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t vec = v0 + u * kThreads, at = cut.begin(vec) * E::ES;
        q[u] = M::ld16(rx, vec < vpr ? x0 + at : kNoLoad);
        mq[u] = M::ld16(rm, vec < vpr ? m0 + at : kNoLoad);
      }
    };
    float m = -__builtin_inff(), sum = 0.0f;
    for (uint32_t v0 = tid; v0 < vpr + tid; v0 += U * kThreads) {          // (whole rounds: every lane, the last ones with nothing)
      fetch_batch(v0);
      float x[U][V], mb = m;
#pragma unroll
      for (uint32_t u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < (int)V; ++e) {
          const uint32_t vec = v0 + u * kThreads;
          const float a = alpha * E::get(q[u], e) + E::get(mq[u], e);
          x[u][e] = vec < vpr && (!RAGGED || e >= cut.first(vec)) ? a : -__builtin_inff();
          mb = __builtin_fmaxf(mb, x[u][e]);
        }
      const float ref = mb == -__builtin_inff() ? 0.0f : mb;       // (nothing but -inf so far: relative to 0, every term is 0)
      float part[U];                                   // (added in pairs: a shorter chain, and a smaller error)
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
#pragma unroll
        for (int e = 0; e < (int)V; ++e) x[u][e] = __expf(x[u][e] - ref);
#pragma unroll
        for (int w = (int)V / 2; w > 0; w /= 2)
#pragma unroll
          for (int e = 0; e < w; ++e) x[u][e] += x[u][e + w];
        part[u] = x[u][0];
      }
      sum = sum * __expf(m - ref) + ((part[0] + part[1]) + (part[2] + part[3]));
      m = mb;
    }
    const float M_ = wg.max(m);
    const float inv = 1.0f / wg.sum(sum * __expf(m - M_));
    for (uint32_t v0 = tid; v0 < vpr + tid; v0 += U * kThreads) {
      fetch_batch(v0);
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t vec = v0 + u * kThreads;
        v4i oq;
#pragma unroll
        for (int e = 0; e < (int)V; ++e) E::put(oq, e, __expf(alpha * E::get(q[u], e) + E::get(mq[u], e) - M_) * inv);
        row_store<POL, DT, RAGGED>(ro, x0 + cut.begin(vec) * E::ES, oq, vec < vpr, cut.first(vec));
      }
    }
  }
  __syncthreads();                                     // the LDS slots belong to the next chunk after this
}

// Layer norm rows too long for the workgroup's registers: three passes of vector loads over the row.
template <int POL, int DT, bool P32, bool RAGGED>
DEV void layernorm_long(const Record* r, uint32_t row_begin, uint32_t row_end, float* s_v, uint32_t tid) {
  using E = Elem<DT>;
  using M = Mem<POL, false, true>;
  constexpr uint32_t V = E::V;
  const uint32_t n = uni(r->red_n);
  const RowCut<V, RAGGED> cut(n);
  const uint32_t vpr = cut.vpr;
  const float alpha = r->alpha;
  const uint32_t chunk_bytes = (row_end - row_begin) * n * E::ES;
  const uint64_t chunk_off = (uint64_t)row_begin * n * E::ES;
  const rsrc_t rx = make_rsrc(uni_ptr(r->ptr[0]) + chunk_off, chunk_bytes);
  const rsrc_t ro = make_rsrc(uni_ptr(r->ptr[3]) + chunk_off, chunk_bytes);
  const rsrc_t rg = make_rsrc(uni_ptr(r->ptr[1]), n * (P32 ? 4u : (uint32_t)E::ES)), rb = make_rsrc(uni_ptr(r->ptr[2]), n * (P32 ? 4u : (uint32_t)E::ES));
  WgReduce wg = {s_v, 0, tid};
  for (uint32_t row = row_begin; row < row_end; ++row) {
    const uint32_t x0 = (row - row_begin) * n * E::ES;
    float sum = 0.0f;
    for (uint32_t vec = tid; vec < vpr; vec += kThreads) {
      const v4i q = M::ld16(rx, x0 + cut.begin(vec) * E::ES);
#pragma unroll
      for (int e = 0; e < (int)V; ++e) sum += !RAGGED || e >= cut.first(vec) ? E::get(q, e) : 0.0f;
    }
    const float mean = wg.sum(sum) / (float)n;
    float ss = 0.0f;
    for (uint32_t vec = tid; vec < vpr; vec += kThreads) {
      const v4i q = M::ld16(rx, x0 + cut.begin(vec) * E::ES);
#pragma unroll
      for (int e = 0; e < (int)V; ++e) { const float d = E::get(q, e) - mean; ss += !RAGGED || e >= cut.first(vec) ? d * d : 0.0f; }
    }
    const float rstd = 1.0f / __builtin_sqrtf(wg.sum(ss) / (float)n + alpha);
    for (uint32_t vec = tid; vec < vpr; vec += kThreads) {
      const v4i q = M::ld16(rx, x0 + cut.begin(vec) * E::ES);
      RowParam<POL, DT, P32> g, b;
      g.load(rg, cut.begin(vec));
      b.load(rb, cut.begin(vec));
      v4i oq;
#pragma unroll
      for (int e = 0; e < (int)V; ++e) E::put(oq, e, (E::get(q, e) - mean) * rstd * g.get(e) + b.get(e));
      row_store<POL, DT, RAGGED>(ro, x0 + cut.begin(vec) * E::ES, oq, true, cut.first(vec));
    }
  }
  __syncthreads();                                     // the LDS slots belong to the next chunk after this
}

// The executors of PATH_ROW_FUSED and PATH_ROW_RAGGED.  Aligned rows of up to 1,024 vectors have one per dtype, called from
// the worker loop; ragged and longer rows are reached through rowop_other, one call site for all of
// them.  (Every call site in the worker loop costs every unit: the loop's scalars are put out of the
// call's way round each, and with forty sites more the compiler kept those in a register that it
// stored to scratch memory and fetched from there at every decision, 1.5 us a unit.)
template <int POL, int ROP, int DT, bool P32, bool RAGGED>
DEV void rowop_short(const Record* r, uint32_t begin, uint32_t end, float* s, uint32_t tid) {      // <= 256 vectors
  const uint32_t vpr = (uni(r->red_n) + Elem<DT>::V - 1) / Elem<DT>::V;
  if (vpr <= 64u) rowop_fused<POL, ROP, DT, 1, 4, P32, RAGGED>(r, begin, end, s, tid);
  else if (vpr <= 128u) rowop_fused<POL, ROP, DT, 2, 2, P32, RAGGED>(r, begin, end, s, tid);
  else rowop_fused<POL, ROP, DT, 4, 1, P32, RAGGED>(r, begin, end, s, tid);
}
template <int POL, int ROP, int DT, bool P32, bool RAGGED>
DEV void rowop_mid(const Record* r, uint32_t begin, uint32_t end, float* s, uint32_t tid) {        // <= 1,024 vectors
  const uint32_t vpr = (uni(r->red_n) + Elem<DT>::V - 1) / Elem<DT>::V;
  if (vpr <= 512u) rowop_wg<POL, ROP, DT, 2, P32, RAGGED>(r, begin, end, s, tid);
  else rowop_wg<POL, ROP, DT, 4, P32, RAGGED>(r, begin, end, s, tid);
}
// How many batches stay in registers: the most that every row of the length has whole, while LDS and they hold the row, or four
// and five.
template <int POL, int DT, bool RAGGED>
DEV void softmax_held_rows(const Record* r, uint32_t begin, uint32_t end, float* s, uint32_t tid) {      // rows of over 4,096 vectors, 2,048 of 16-bit elements
  constexpr uint32_t kMore = (DT == GPUOS_F32 ? 21u : 15u) * kThreads;
  constexpr int FEW = DT == GPUOS_F32 ? 5 : 2, MORE = DT == GPUOS_F32 ? 6 : 5;
  static_assert(FEW * 3 <= (DT == GPUOS_F32 ? 16 : 8) && MORE * 3u * kThreads <= kMore, "the rows are longer than what they keep");
  const uint32_t vpr = (uni(r->red_n) + Elem<DT>::V - 1) / Elem<DT>::V;
  if (vpr <= kMore) softmax_held<POL, DT, FEW, RAGGED>(r, begin, end, s, tid);
  else softmax_held<POL, DT, MORE, RAGGED>(r, begin, end, s, tid);
}
template <int POL, int ROP, int DT, bool P32, bool RAGGED>
DEV void rowop_long(const Record* r, uint32_t begin, uint32_t end, float* s, uint32_t tid) {
  const uint32_t vpr = (uni(r->red_n) + Elem<DT>::V - 1) / Elem<DT>::V;
  constexpr bool MASK = ROP == GPUOS_IMPL_MASKED_SOFTMAX_LAST;       // (twice the registers per vector)
  if constexpr (!MASK || DT == GPUOS_F32) {
    if (vpr <= 2048u) return rowop_wg<POL, ROP, DT, 8, P32, RAGGED>(r, begin, end, s, tid);
  }
  if constexpr (!MASK && DT == GPUOS_F32) {
    if (vpr <= 4096u) return rowop_wg<POL, ROP, DT, 16, P32, RAGGED>(r, begin, end, s, tid);
  }
  if constexpr (MASK) masked_softmax_long<POL, DT, RAGGED>(r, begin, end, s, tid);
  else if constexpr (RowOp<ROP>::SOFTMAX) { if constexpr (POL == POL_PLAIN) softmax_held_rows<POL, DT, RAGGED>(r, begin, end, s, tid); }      // (the worker: exec_away)
  else layernorm_long<POL, DT, P32, RAGGED>(r, begin, end, s, tid);
}
enum { kRowShort, kRowMid, kRowLong };
template <int POL, int ROP, int DT, int LEN, bool RAGGED>
PATHFN void rowop_dt(const Record* r_v, uint32_t begin_v, uint32_t end_v, float* s_v, uint32_t tid) {
  const Record* r = lds_arg(r_v);
  float* s = lds_arg(s_v);
  const uint32_t begin = uni(begin_v), end = uni(end_v);
  constexpr bool LN16 = ROP == GPUOS_IMPL_LAYERNORM_LAST && DT != GPUOS_F32;
  if (LN16 && uni(r->dtype[1]) == GPUOS_F32) {                       // fp32 gamma / beta under 16-bit x
    if constexpr (LEN == kRowShort) rowop_short<POL, ROP, DT, LN16, RAGGED>(r, begin, end, s, tid);
    else if constexpr (LEN == kRowMid) rowop_mid<POL, ROP, DT, LN16, RAGGED>(r, begin, end, s, tid);
    else rowop_long<POL, ROP, DT, LN16, RAGGED>(r, begin, end, s, tid);
    return;
  }
  if constexpr (LEN == kRowShort) rowop_short<POL, ROP, DT, false, RAGGED>(r, begin, end, s, tid);
  else if constexpr (LEN == kRowMid) rowop_mid<POL, ROP, DT, false, RAGGED>(r, begin, end, s, tid);
  else rowop_long<POL, ROP, DT, false, RAGGED>(r, begin, end, s, tid);
}
template <int POL, int ROP, int DT>
DEV void rowop_other_dt(const Record* r, uint32_t begin, uint32_t end, float* s, uint32_t tid) {
  const uint32_t vpr = (uni(r->red_n) + Elem<DT>::V - 1) / Elem<DT>::V;
  if (uni(r->path) == PATH_ROW_FUSED) rowop_dt<POL, ROP, DT, kRowLong, false>(r, begin, end, s, tid);
  else if (vpr <= 256u) rowop_dt<POL, ROP, DT, kRowShort, true>(r, begin, end, s, tid);
  else if (vpr <= 1024u) rowop_dt<POL, ROP, DT, kRowMid, true>(r, begin, end, s, tid);
  else rowop_dt<POL, ROP, DT, kRowLong, true>(r, begin, end, s, tid);
}
template <int POL, int ROP>
DEV void rowop_other_op(const Record* r, uint32_t begin, uint32_t end, float* s, uint32_t tid) {
  const uint32_t dt = uni(r->dtype[3]);
  if (dt == GPUOS_F32) rowop_other_dt<POL, ROP, GPUOS_F32>(r, begin, end, s, tid);
  else if (dt == GPUOS_F16) rowop_other_dt<POL, ROP, GPUOS_F16>(r, begin, end, s, tid);
  else rowop_other_dt<POL, ROP, GPUOS_BF16>(r, begin, end, s, tid);
}
template <int POL>
PATHFN void rowop_other(const Record* r_v, uint32_t impl_v, uint32_t begin_v, uint32_t end_v, float* s_v, uint32_t tid) {
  const Record* r = lds_arg(r_v);
  float* s = lds_arg(s_v);
  const uint32_t impl = uni(impl_v), begin = uni(begin_v), end = uni(end_v);
  if (impl == GPUOS_IMPL_SOFTMAX_LAST) rowop_other_op<POL, GPUOS_IMPL_SOFTMAX_LAST>(r, begin, end, s, tid);
  else if (impl == GPUOS_IMPL_MASKED_SOFTMAX_LAST) rowop_other_op<POL, GPUOS_IMPL_MASKED_SOFTMAX_LAST>(r, begin, end, s, tid);
  else rowop_other_op<POL, GPUOS_IMPL_LAYERNORM_LAST>(r, begin, end, s, tid);
}

// What the choice of an executor asks of a record, in registers: the worker reads it with the rest of the
// record's head, in one go (field by field it was two more LDS latencies in a row on every unit).
struct RecHead {
  uint32_t op[3], dims[3];                             // words 0-2 and 8-10 of the record
  static DEV RecHead of(const Record* r) {
    const v4i* h = (const v4i*)r;
    return of(h[0], h[2]);
  }
  static DEV RecHead of(const v4i& q0, const v4i& q2) {
    return {{uni((uint32_t)q0[0]), uni((uint32_t)q0[1]), uni((uint32_t)q0[2])}, {uni((uint32_t)q2[0]), uni((uint32_t)q2[1]), uni((uint32_t)q2[2])}};
  }
  DEV uint32_t path() const { return (op[0] >> 16) & 0xffu; }
  DEV uint32_t dtype_in0() const { return (op[1] >> 8) & 0xffu; }
  DEV uint32_t dtype_out() const { return op[2] & 0xffu; }
  DEV uint32_t rflags() const { return (op[2] >> 8) & 0xffu; }
  DEV uint32_t chunk() const { return dims[0]; }
  DEV uint32_t numel() const { return dims[1]; }
  DEV uint32_t red_n() const { return dims[2]; }
};
static_assert(__builtin_offsetof(Record, path) == 2 && __builtin_offsetof(Record, dtype) == 5 && __builtin_offsetof(Record, rflags) == 9 &&
              __builtin_offsetof(Record, chunk) == 32 && __builtin_offsetof(Record, numel) == 36 && __builtin_offsetof(Record, red_n) == 40, "the words of RecHead");

// the rows that rowop_other takes
DEV bool rowop_is_other(const RecHead& h) {
  const uint32_t path = h.path();
  return path == PATH_ROW_RAGGED || (path == PATH_ROW_FUSED && h.red_n() > (h.dtype_out() == GPUOS_F32 ? 4096u : 8192u));
}
// ... and those of them that the worker runs by exec_away: softmax rows that do not fit the registers
DEV bool rowop_is_away(const RecHead& h, uint32_t impl) {
  const uint32_t path = h.path();
  return impl == GPUOS_IMPL_SOFTMAX_LAST && (path == PATH_ROW_RAGGED || path == PATH_ROW_FUSED) && h.red_n() > 16384u;
}
template <int POL, int ROP>
DEV void run_rowop(const Record* r, const RecHead& h, uint32_t chunk, float* s_red, uint32_t tid) {
  const uint32_t per = h.chunk(), rows = h.numel();
  const uint32_t begin = chunk * per;
  const uint32_t end = (rows - begin < per) ? rows : begin + per;
  if (h.path() == PATH_ROW_FUSED) {
    const uint32_t dt = h.dtype_out();
    const bool wide = h.red_n() * (dt == GPUOS_F32 ? 4u : 2u) > 256u * 16u;     // more than 256 vectors per row
    if (!wide) {
      if (dt == GPUOS_F32) rowop_dt<POL, ROP, GPUOS_F32, kRowShort, false>(r, begin, end, s_red, tid);
      else if (dt == GPUOS_F16) rowop_dt<POL, ROP, GPUOS_F16, kRowShort, false>(r, begin, end, s_red, tid);
      else rowop_dt<POL, ROP, GPUOS_BF16, kRowShort, false>(r, begin, end, s_red, tid);
    } else {
      if (dt == GPUOS_F32) rowop_dt<POL, ROP, GPUOS_F32, kRowMid, false>(r, begin, end, s_red, tid);
      else if (dt == GPUOS_F16) rowop_dt<POL, ROP, GPUOS_F16, kRowMid, false>(r, begin, end, s_red, tid);
      else rowop_dt<POL, ROP, GPUOS_BF16, kRowMid, false>(r, begin, end, s_red, tid);
    }
  } else {
    rowop_generic<POL, ROP>(r, begin, end, tid);
  }
}

// ---------------------------------------------------------------------------
// chunk executor: operator dispatch by implementation id (the role of the
// paper's function-pointer table call, Section 4.1; here a switch over
// precompiled implementations selected by the table entry).
// ---------------------------------------------------------------------------
// The executors of PATH_ROWS: by arity without (groups of three: fp32, fp16, bf16) and with per-row
// scalars, the operators of many instructions, casts, I32.
enum : uint32_t { kClsUnary = 0, kClsBinary = 1, kClsTernary = 2, kClsErf = 3, kClsTanh = 4, kClsNone = 15 };
constexpr int kRowsScalar = 15, kRowsCast = 21, kRowsInt = 27, kRowsPairs = 30, kRowsCount = 31;      // (pairs: PATH_STAGED under RF_PAIRS)
template <int CLS> struct OperOf;
template <> struct OperOf<kClsUnary> { typedef ByArity<1> T; };
template <> struct OperOf<kClsBinary> { typedef ByArity<2> T; };
template <> struct OperOf<kClsTernary> { typedef ByArity<3> T; };
template <> struct OperOf<kClsErf> { typedef FixedOp<GPUOS_IMPL_GELU_ERF> T; };
template <> struct OperOf<kClsTanh> { typedef FixedOp<GPUOS_IMPL_GELU_TANH> T; };
static_assert(GPUOS_F32 == 0 && GPUOS_F16 == 1 && GPUOS_BF16 == 2, "the float dtypes count the members of a group");
// class by implementation, a nibble each: ADD SUB MUL DIV binary, RELU EXP unary, both GELUs, SCALE unary, FMA, SUB_EXP binary, COPY unary
DEV uint32_t op_class(uint32_t impl) { return impl < 16u ? (uint32_t)(0xfff012043001111full >> (4u * impl)) & 15u : (uint32_t)kClsNone; }
// The executors of pairs (RF_PAIRS), behind one call that ends in jumps.
template <int POL> struct PairsExec {
  template <int K> static DEV void run(const Record* r, uint32_t begin, uint32_t end, uint32_t tid) { ew_pairs<POL, typename OperOf<K / 3>::T, K % 3>(r, begin, end, tid); }
};
template <int POL>
PATHFN void run_pairs(const Record* r_v, uint32_t begin_v, uint32_t end_v, uint32_t tid) {
  const Record* r = lds_arg(r_v);
  pick<0, 15, PairsExec<POL>>(op_class(uni(r->impl)) * 3u + uni(r->dtype[3]), r, uni(begin_v), uni(end_v), tid);
}
template <int POL> struct RowsExec {
  template <int K> static DEV void run(const Record* r, uint32_t begin, uint32_t end, uint32_t tid) {
    if constexpr (K < kRowsScalar) ew_rows<POL, typename OperOf<K / 3>::T, K % 3, K % 3, false>(r, begin, end, tid);
    else if constexpr (K < kRowsCast) ew_rows<POL, ByArity<2 + (K - kRowsScalar) / 3>, (K - kRowsScalar) % 3, (K - kRowsScalar) % 3, true>(r, begin, end, tid);
    else if constexpr (K < kRowsInt) {
      // (from, to): 0 1, 0 2, 1 0, 1 2, 2 0, 2 1
      constexpr int FROM = (K - kRowsCast) / 2, TO = (K - kRowsCast) % 2 + ((K - kRowsCast) % 2 >= FROM ? 1 : 0);
      ew_rows<POL, ByArity<1>, FROM, TO, false>(r, begin, end, tid);
    }
    else if constexpr (K < kRowsPairs - 1) ew_rows<POL, ByArity<K - kRowsInt + 1>, GPUOS_I32, GPUOS_I32, false>(r, begin, end, tid);
    else if constexpr (K < kRowsPairs) ew_rows<POL, ByArity<2>, GPUOS_I32, GPUOS_I32, true>(r, begin, end, tid);
    else run_pairs<POL>(r, begin, end, tid);
  }
};

// the executor of a PATH_ROWS task, kRowsCount if it has none
DEV uint32_t rows_variant(const Record* r, uint32_t impl) {
  const uint32_t cls = op_class(impl);
  const uint32_t dt = uni(r->dtype[3]), dti = uni(r->vdtype);
  const bool scalars = uni((uint32_t)r->okind[0] | (uint32_t)r->okind[1] | (uint32_t)r->okind[2]) != 0;
  if (uni(r->rflags) & RF_INT) {
    const bool takes = impl == GPUOS_IMPL_ADD || impl == GPUOS_IMPL_SUB || impl == GPUOS_IMPL_MUL || impl == GPUOS_IMPL_COPY;
    return takes ? kRowsInt + (impl == GPUOS_IMPL_COPY ? 0u : 1u) + (scalars ? 1u : 0u) : (uint32_t)kRowsCount;
  }
  if (dti != dt) return impl == GPUOS_IMPL_COPY ? kRowsCast + 2u * dti + dt - (dt > dti ? 1u : 0u) : (uint32_t)kRowsCount;
  if (!scalars) return cls <= kClsTanh ? cls * 3u + dt : (uint32_t)kRowsCount;
  return cls == kClsBinary || cls == kClsTernary ? kRowsScalar + (cls - 1u) * 3u + dt : (uint32_t)kRowsCount;
}

// Elements [begin, end) of a PATH_ROWS task, whose numbers count vectors, as the element range that the
// general executor walks: for an operator that was swapped in between submission and claim and has
// no executor for the task's combination (another unary operator where a COPY converts).
DEV void rows_elements(const Record* r, uint32_t& begin, uint32_t& end) {
  const uint32_t C = uni(r->size[3]), V = uni(r->vwidth), VR = (C + V - 1) / V;
  const uint32_t b = begin / VR, e = end / VR;
  begin = b * C + (begin - b * VR) * V;
  end = e * C + (end - e * VR) * V;                  // (vector 0 of the next row begins where this row ends)
}

template <int POL, int IMPL>
DEV void run_elementwise(const Record* r, const RecHead& h, uint32_t chunk, float* s_scratch, uint32_t tid) {
  const uint32_t per = h.chunk(), numel = h.numel();
  uint32_t begin = chunk * per, end = (numel - begin < per) ? numel : begin + per;
  const uint32_t path = h.path(), dt = h.dtype_out();
  constexpr bool int_ok = IMPL == GPUOS_IMPL_ADD || IMPL == GPUOS_IMPL_SUB || IMPL == GPUOS_IMPL_MUL || IMPL == GPUOS_IMPL_COPY;
  if (h.rflags() & RF_INT) {
    if (int_ok) {
      if (path == PATH_CONTIG) ew_contig<POL, int_ok ? IMPL : GPUOS_IMPL_COPY, GPUOS_I32>(r, begin, end, tid);
      else ew_generic<POL, int_ok ? IMPL : GPUOS_IMPL_COPY, true>(r, begin, end, tid);
    }
    return;
  }
  if (path == PATH_CONTIG) {
    if (dt == GPUOS_F32) ew_contig<POL, IMPL, GPUOS_F32>(r, begin, end, tid);
    else if (dt == GPUOS_F16) ew_contig<POL, IMPL, GPUOS_F16>(r, begin, end, tid);
    else if constexpr (IMPL == GPUOS_IMPL_GELU_ERF) {
      // (Batches in fp32 need registers that callers keep, 128 bytes a lane to save and restore: with both in one
      // function four tasks of 2,048 elements took 13.0 us, 12.1 so.)
      if (end - begin >= 4u * kThreads * 8u) ew_contig<POL, IMPL, GPUOS_BF16>(r, begin, end, tid);
      else ew_contig<POL, IMPL, GPUOS_BF16, 1>(r, begin, end, tid);
    } else ew_contig<POL, IMPL, GPUOS_BF16>(r, begin, end, tid);
  } else if (path == PATH_ROW2D && Op<IMPL>::N >= 2) {
    constexpr int I2 = Op<IMPL>::N >= 2 ? IMPL : GPUOS_IMPL_ADD;
    const uint32_t k0 = uni(r->okind[0]), k1 = uni(r->okind[1]);
    const int spec = (Op<I2>::N == 2 && k0 == K_FULL) ? (k1 == K_ROWSCALAR ? 1 : (k1 == K_ROWVEC ? 2 : 0)) : 0;
    if (dt == GPUOS_F32) {
      if (spec == 1) ew_row2d<POL, I2, GPUOS_F32, K_ROWSCALAR>(r, begin, end, s_scratch, tid);
      else if (spec == 2) ew_row2d<POL, I2, GPUOS_F32, K_ROWVEC>(r, begin, end, s_scratch, tid);
      else ew_row2d<POL, I2, GPUOS_F32, -1>(r, begin, end, s_scratch, tid);
    } else if (dt == GPUOS_F16) {
      if (spec == 1) ew_row2d<POL, I2, GPUOS_F16, K_ROWSCALAR>(r, begin, end, s_scratch, tid);
      else if (spec == 2) ew_row2d<POL, I2, GPUOS_F16, K_ROWVEC>(r, begin, end, s_scratch, tid);
      else ew_row2d<POL, I2, GPUOS_F16, -1>(r, begin, end, s_scratch, tid);
    } else {
      if (spec == 1) ew_row2d<POL, I2, GPUOS_BF16, K_ROWSCALAR>(r, begin, end, s_scratch, tid);
      else if (spec == 2) ew_row2d<POL, I2, GPUOS_BF16, K_ROWVEC>(r, begin, end, s_scratch, tid);
      else ew_row2d<POL, I2, GPUOS_BF16, -1>(r, begin, end, s_scratch, tid);
    }
  } else if (path == PATH_TILE2D) {
    ew_tile2d<POL, IMPL>(r, begin, end, s_scratch, tid);      // begin / end count tiles here
  } else if (path == PATH_STAGED) {
    ew_staged<POL, IMPL>(r, begin, end, s_scratch, tid);
  } else {
    if constexpr (IMPL >= kImplProg1) {                  // programs, interpreted and native; built-in operators: RowsExec
      const uint32_t k0 = uni((uint32_t)r->okind[0] | (uint32_t)r->okind[1] | (uint32_t)r->okind[2]);
      if (path == PATH_ROWS && uni(r->vdtype) == dt && (k0 == 0 || Op<IMPL>::N >= 2)) {
        constexpr bool S = Op<IMPL>::N >= 2;
        if (dt == GPUOS_F32) { if (k0) ew_rows<POL, FixedOp<IMPL>, GPUOS_F32, GPUOS_F32, S>(r, begin, end, tid); else ew_rows<POL, FixedOp<IMPL>, GPUOS_F32, GPUOS_F32, false>(r, begin, end, tid); }
        else if (dt == GPUOS_F16) { if (k0) ew_rows<POL, FixedOp<IMPL>, GPUOS_F16, GPUOS_F16, S>(r, begin, end, tid); else ew_rows<POL, FixedOp<IMPL>, GPUOS_F16, GPUOS_F16, false>(r, begin, end, tid); }
        else { if (k0) ew_rows<POL, FixedOp<IMPL>, GPUOS_BF16, GPUOS_BF16, S>(r, begin, end, tid); else ew_rows<POL, FixedOp<IMPL>, GPUOS_BF16, GPUOS_BF16, false>(r, begin, end, tid); }
        return;
      }
    }
    if (path == PATH_ROWS) rows_elements(r, begin, end);
    ew_generic<POL, IMPL, false>(r, begin, end, tid);
  }
}

// The executors of reductions, behind one call as well (it ends in jumps): they were 60 call sites of the worker's loop, which
// with other executors in their place fetched 102 of its values from scratch memory, a lone addition 8.8 us instead of 8.2.
template <int POL, int RIMPL>
DEV void run_reduction(const Record* r, const RecHead& h, uint32_t chunk, float* s_red, uint32_t tid) {
  const uint32_t per = h.chunk(), rows = h.numel();
  const uint32_t begin = chunk * per;
  const uint32_t end = (rows - begin < per) ? rows : begin + per;
  const uint32_t path = h.path(), dt = h.dtype_in0();
  if (path == PATH_RED_CONTIG) {
    if (h.rflags() & RF_INT) red_contig<POL, RIMPL, GPUOS_I32>(r, begin, end, s_red, tid);
    else if (dt == GPUOS_F32) red_contig<POL, RIMPL, GPUOS_F32>(r, begin, end, s_red, tid);
    else if (dt == GPUOS_F16) red_contig<POL, RIMPL, GPUOS_F16>(r, begin, end, s_red, tid);
    else red_contig<POL, RIMPL, GPUOS_BF16>(r, begin, end, s_red, tid);
  } else {
    if (h.rflags() & RF_INT) red_generic<POL, RIMPL, true>(r, begin, end, tid);
    else red_generic<POL, RIMPL, false>(r, begin, end, tid);
  }
}
template <int POL>
PATHFN void run_reductions(const Record* r_v, uint32_t impl_v, uint32_t chunk_v, float* s_v, uint32_t tid) {
  const Record* r = lds_arg(r_v);
  float* s = lds_arg(s_v);
  const RecHead h = RecHead::of(r);
  const uint32_t impl = uni(impl_v), chunk = uni(chunk_v);
  if (impl == GPUOS_IMPL_SUM_LAST) run_reduction<POL, GPUOS_IMPL_SUM_LAST>(r, h, chunk, s, tid);
  else if (impl == GPUOS_IMPL_MAX_LAST) run_reduction<POL, GPUOS_IMPL_MAX_LAST>(r, h, chunk, s, tid);
  else run_reduction<POL, GPUOS_IMPL_MIN_LAST>(r, h, chunk, s, tid);
}

// The interpreter's executors, behind one call: in the worker's loop itself they were 44 of its 293 call sites, which cost
// other operations' registers (softmax over rows of 32,003 fp32 elements, then in that loop too: 180.4 us with them there, 175.9
// so).  It ends in
// jumps: where it made calls it had to keep for its caller all that its callees use, 376 bytes a lane, and
// x / (1 + e^-x) over four tensors of 2,048 fp32 elements took 35.7 us instead of 16.0.
template <int POL>
PATHFN void run_program_chunk(const Record* r_v, uint32_t n_in_v, uint32_t chunk_v, float* s_v, uint32_t tid) {
  const Record* r = lds_arg(r_v);
  float* s = lds_arg(s_v);
  const RecHead h = RecHead::of(r);
  const uint32_t n_in = uni(n_in_v), chunk = uni(chunk_v);
  if (n_in == 1) run_elementwise<POL, kImplProg1>(r, h, chunk, s, tid);
  else if (n_in == 2) run_elementwise<POL, kImplProg2>(r, h, chunk, s, tid);
  else run_elementwise<POL, kImplProg3>(r, h, chunk, s, tid);
}

// A task whose operator is a program: fetch the program into LDS (17 lanes x 16 bytes), then run
// the ordinary elementwise paths with the interpreter as their functor.
template <int POL>
DEV int32_t exec_program(const Record* r, const RecHead& h, uint32_t impl, uint32_t chunk, float* s_red, const ProgramImage* progs, uint32_t tid) {
  const uint32_t k = impl - GPUOS_IMPL_PROGRAM_BASE;
  if (progs == nullptr || k >= GPUOS_MAX_PROGRAMS) return GPUOS_E_BADOP;
  const rsrc_t rp = make_rsrc(progs + k, (uint32_t)sizeof(ProgramImage));
  if (tid < sizeof(ProgramImage) / 16) ((v4i*)&g_prog)[tid] = Mem<POL_COHERENT>::ld16(rp, tid * 16u);
  __syncthreads();
  int32_t status = GPUOS_OK;
  const uint32_t n_in = uni(g_prog.n_inputs), n_instr = uni(g_prog.n_instr);
  if (uni(g_prog.ready) != kProgramReady || n_instr < 1 || n_instr > GPUOS_PROGRAM_MAX_INSTR || n_in != uni(r->n_inputs))
    status = GPUOS_E_INVAL;                            // never defined (or not what the task was packed for)
  else run_program_chunk<POL>(r, n_in, chunk, s_red, tid);
  __syncthreads();                                     // the next chunk may bring another program
  return status;
}

// returns the task status contribution of this chunk (0 or an error)
template <int POL>
DEV int32_t exec_chunk(const Record* r, const RecHead& h, uint32_t impl, uint32_t chunk, float* s_red, const ProgramImage* progs, uint32_t tid) {
  if (h.path() == PATH_NOP) return impl == GPUOS_IMPL_FAIL ? GPUOS_E_BADOP : GPUOS_OK;
  if (__builtin_expect(impl >= GPUOS_IMPL_PROGRAM_BASE, 0)) return exec_program<POL>(r, h, impl, chunk, s_red, progs, tid);
  // (beside the switch, not a case in every implementation's paths: see ByArity)
  if (impl >= GPUOS_IMPL_SOFTMAX_LAST && impl <= GPUOS_IMPL_LAYERNORM_LAST && rowop_is_other(h)) {
    const uint32_t per = h.chunk(), rows = h.numel(), begin = chunk * per;
    rowop_other<POL>(r, impl, begin, (rows - begin < per) ? rows : begin + per, s_red, tid);
    return GPUOS_OK;
  }
  const uint32_t k = h.path() == PATH_ROWS ? rows_variant(r, impl) : ((h.rflags() & RF_PAIRS) != 0 && op_class(impl) <= kClsTanh ? (uint32_t)kRowsPairs : (uint32_t)kRowsCount);
  if (k < (uint32_t)kRowsCount) {
    const uint32_t per = h.chunk(), numel = h.numel(), begin = chunk * per;
    pick<0, kRowsCount, RowsExec<POL>>(k, r, begin, (numel - begin < per) ? numel : begin + per, tid);
    return GPUOS_OK;
  }
  switch (impl) {
    case GPUOS_IMPL_ADD: run_elementwise<POL, GPUOS_IMPL_ADD>(r, h, chunk, s_red, tid); break;
    case GPUOS_IMPL_SUB: run_elementwise<POL, GPUOS_IMPL_SUB>(r, h, chunk, s_red, tid); break;
    case GPUOS_IMPL_MUL: run_elementwise<POL, GPUOS_IMPL_MUL>(r, h, chunk, s_red, tid); break;
    case GPUOS_IMPL_DIV: run_elementwise<POL, GPUOS_IMPL_DIV>(r, h, chunk, s_red, tid); break;
    case GPUOS_IMPL_RELU: run_elementwise<POL, GPUOS_IMPL_RELU>(r, h, chunk, s_red, tid); break;
    case GPUOS_IMPL_EXP: run_elementwise<POL, GPUOS_IMPL_EXP>(r, h, chunk, s_red, tid); break;
    case GPUOS_IMPL_GELU_ERF: run_elementwise<POL, GPUOS_IMPL_GELU_ERF>(r, h, chunk, s_red, tid); break;
    case GPUOS_IMPL_GELU_TANH: run_elementwise<POL, GPUOS_IMPL_GELU_TANH>(r, h, chunk, s_red, tid); break;
    case GPUOS_IMPL_SCALE: run_elementwise<POL, GPUOS_IMPL_SCALE>(r, h, chunk, s_red, tid); break;
    case GPUOS_IMPL_FMA: run_elementwise<POL, GPUOS_IMPL_FMA>(r, h, chunk, s_red, tid); break;
    case GPUOS_IMPL_SUB_EXP: run_elementwise<POL, GPUOS_IMPL_SUB_EXP>(r, h, chunk, s_red, tid); break;
    case GPUOS_IMPL_COPY: run_elementwise<POL, GPUOS_IMPL_COPY>(r, h, chunk, s_red, tid); break;
    case GPUOS_IMPL_SUM_LAST: case GPUOS_IMPL_MAX_LAST: case GPUOS_IMPL_MIN_LAST: run_reductions<POL>(r, impl, chunk, s_red, tid); break;
    case GPUOS_IMPL_SOFTMAX_LAST: run_rowop<POL, GPUOS_IMPL_SOFTMAX_LAST>(r, h, chunk, s_red, tid); break;
    case GPUOS_IMPL_MASKED_SOFTMAX_LAST: run_rowop<POL, GPUOS_IMPL_MASKED_SOFTMAX_LAST>(r, h, chunk, s_red, tid); break;
    case GPUOS_IMPL_LAYERNORM_LAST: run_rowop<POL, GPUOS_IMPL_LAYERNORM_LAST>(r, h, chunk, s_red, tid); break;
    case GPUOS_IMPL_FAIL: return GPUOS_E_BADOP;       // kill-switch stub: fail fast, write nothing
    default: return GPUOS_E_BADOP;
  }
  return GPUOS_OK;
}


// Reading the clock is a memory-like operation: a dozen reads per task are measurable, so the phase
// timers are an option and the clock is read only where something needs the value.
DEV uint64_t clock_if(bool on) { return on ? wall_clock64() : 0ull; }

// The 16 lanes that hold a record's 16-byte pieces: the weighted check sum of the whole record
// (see record_check_weight), in every one of them.

DEV uint32_t record_piece_sum(const v4i& q, uint32_t part) {
  uint32_t x = 0;
#pragma unroll
  for (uint32_t j = 0; j < 4; ++j) x += (uint32_t)q[j] * record_check_weight(4u * part + j);
  // sum over the 16 lanes of the row with DPP rotations (row_ror 8, 4, 2, 1): every lane ends with
  // the whole sum, and unlike a shuffle nothing goes through the LDS crossbar
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xf, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xf, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xf, 0xf, false);
  return x;
}

struct BuiltinExec {                // what the library's own workers execute a chunk with
  static DEV int32_t run(const Record* r, const RecHead& h, uint32_t impl, uint32_t chunk, float* s_red, const ProgramImage* progs, uint32_t tid) {
    return exec_chunk<POL_COHERENT>(r, h, impl, chunk, s_red, progs, tid);
  }
};

// ---------------------------------------------------------------------------
// worker (every workgroup but 0)
// ---------------------------------------------------------------------------
constexpr uint32_t kMirrorRetries = 1u << 22;       // fetches of a mirror record that does not (yet) verify: seconds
constexpr uint64_t kStopGraceTicks = 10000000ull;   // 100 ms (100 MHz clock): how long a worker still waits for a dependency once the stop flag is up

// A workgroup holds up to kStash descriptors: work units it has claimed that wait for a dependency,
// and the one it runs.  A workgroup whose unit must wait does not sit on it: it claims the next
// unit and runs whatever it holds that is ready (oldest first).  A chain of dependent small tasks
// then occupies one descriptor slot per link in flight instead of one whole workgroup, so eight
// times as many chains are in flight (Section 6.1's sequences issued one after the other: 1.7 M ->
// see the benchmark).  Progress: units are claimed in publication order and what a waiting unit names
// was published before it, so the unfinished unit with the lowest number is always held by some
// workgroup with nothing left to wait for, and every workgroup looks at everything it holds on every
// poll.
constexpr uint32_t kStash = 8;
constexpr uint32_t kStashFull = (1u << kStash) - 1u;
enum : uint32_t { kActRun = 0, kActFetch = 1, kActExit = 2 };
constexpr uint32_t kHaveClaim = 1u << kStash, kDraining = 2u << kStash;

struct WorkShared {
  Record rec[kStash];              // descriptors held
  uint64_t unit[kStash];           // their work-unit entries
  uint64_t entry[kStash];          // the operator-table slot each one claimed
  uint64_t since[kStash];          // when each began to wait (device clock)
  // The first wavefront's decision, read by all: what to do (kAct*: run the unit in descriptor slot `slot`,
  // fetch the newly claimed unit's descriptor into it, or leave), the slot (<< 8) and whether units
  // were held meanwhile (<< 16); the status of a task whose dependency wait ran out, or 0; the unit.
  alignas(16) uint32_t dec[4];
  // The first wavefront's state from one unit to the next: descriptor slots whose units wait (a bit each),
  // kHaveClaim (a unit number is claimed and its entry has not arrived yet), kDraining (the stop flag
  // was seen: claim nothing more, finish what is held, leave); polls since the claim; the claimed number.
  // Here and not in registers, most of which the call of an executor does not preserve, and in one
  // vector each: a unit costs one read and one write of either.
  alignas(16) uint32_t state[4];
  // where a task's completion goes (the kernel's arguments, which a call does not leave in registers)
  SlotState* st;
  uint64_t* hcomp;
  uint64_t* done_count;
  uint64_t cap_shift;
  const Record* dring;             // (a run's other descriptors)
  const OpSlots* dtable;
  uint32_t cap_mask;
  uint32_t rec_sum;                // weighted check sum of the record as fetched
  uint64_t begun, started;         // clocks of the unit that runs: performance counters, tracing
  uint64_t entered;                // ... and of the worker's start
  uint64_t n_units;                // (ST_WORK_UNITS, and the counters after it)
  uint64_t ticks[ST_WORK_TICKS_TOTAL - ST_WORK_TICKS_WAIT];
  alignas(16) float red[kScratchFloats];   // (16-byte LDS vectors are written into it)
};

// A pointer known to address device or host memory, read from LDS: accessed as such, not with flat instructions.
template <class T> DEV T* global_ptr(T* p) { return (T*)(__attribute__((address_space(1))) T*)p; }

DEV uint64_t uni64(uint64_t v) {
  return ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32)) << 32) | __builtin_amdgcn_readfirstlane((uint32_t)v);
}
DEV uint64_t lane64(uint64_t v, uint32_t lane) {     // `lane` the same in every lane
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), (int)lane) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, (int)lane);
}

// First wavefront: fetch the descriptor that work unit `unit` names (16 lanes x 16 bytes) and the
// operator-table slot it claimed into descriptor slot f, with the record's weighted check sum.
DEV void fetch_descriptor(const WorkerArgs& a, WorkShared* s, rsrc_t rd, uint64_t unit, uint32_t f, uint32_t lane) {
  const uint32_t slot = (uint32_t)((unit >> 20) & 0xffffu);
  const uint32_t op = (uint32_t)((unit >> 36) & 0xffu), sel = (uint32_t)((unit >> 44) & 1u);
  const bool op_valid = ((unit >> 45) & 1u) != 0;
  v4i q = {0, 0, 0, 0};
  uint64_t ent = 0;
  if (lane < 16) q = Mem<POL_COHERENT>::ld16(rd, slot * (uint32_t)sizeof(Record) + lane * 16u);
  if (lane == 16 && op_valid) ent = __hip_atomic_load(&a.dtable[op].slot[sel], __ATOMIC_RELAXED, SC_SYSTEM);
  const uint32_t x = record_piece_sum(q, lane & 15u);
  if (lane < 16) ((v4i*)&s->rec[f])[lane] = q;
  if (lane == 16) s->entry[f] = ent;
  if (lane == 0) s->rec_sum = x;
}

// ---------------------------------------------------------------------------
// runs: a chain of tasks over buffers of one shape, each reading what the one before it wrote.  Its units
// stand for all of its tasks: the workgroup that has run a chunk of one runs the same chunk of the
// next, and what it wrote is still in its registers.  What a link costs when every task has units of
// its own is five memory latencies in a row (done word, poll, operands, stores, their acknowledgement),
// 5.5 us; in a run it costs its arithmetic and the issue of its stores, which nothing waits for before the
// run ends, and the bytes it would have read again.
// The host vouches (LinkRun) that any two operands of the run begin at the same address or do not
// overlap, so a lane meets only its own elements, and a row's lanes only their own row.
// ---------------------------------------------------------------------------
template <int DT, int K> struct EitherArg {              // vectors of one of two sets of registers
  const v4i (&p)[K], (&q)[K];
  bool second;
  DEV v4i raw(int u) const { return second ? q[u] : p[u]; }
  DEV float get(int u, int k) const { return Elem<DT>::get(raw(u), k); }
};
template <int K> struct RowArg {                         // one scalar per vector (of its row)
  const float (&w)[K];
  DEV v4i raw(int) const { return v4i{0, 0, 0, 0}; }
  DEV float get(int u, int) const { return w[u]; }
};
template <int RIMPL, int DT, int K> DEV void link_reduce(const EitherArg<DT, K>& q, bool act, uint32_t width, float (&out)[K]) {
#pragma unroll
  for (int u = 0; u < K; ++u) {
    float acc = red_identity<RIMPL, float>();
    if (act) acc = red_vector<RIMPL, DT>(q.raw(u), 0, 0, 0, false, acc);
    out[u] = wave_reduce<RIMPL>(red_finish<RIMPL>(acc), width);
  }
}

// The chunk of every task of a run, block by block: U vectors a lane, all tasks of the run on one block before
// the next.  ROWS false: elements [begin, end) of flat buffers, a lane per vector, the ragged end an
// element per lane (kept as vector U).  ROWS true: rows [begin, end) of n elements, whole vectors, P lanes a row as in
// rowop_fused; then reductions take part and leave their results in registers as one scalar per row.
template <int POL, int DT, bool ROWS>
__attribute__((not_tail_called)) PATHFN void run_links(const Record* recs_v, uint32_t n_links_v, uint64_t skip_v, uint32_t begin_v, uint32_t end_v, uint32_t n_v, uint32_t tid) {
  const Record* recs = lds_arg(recs_v);
  const uint64_t skip = uni64(skip_v);
  const uint32_t n_links = uni(n_links_v), begin = uni(begin_v), end = uni(end_v), n = uni(n_v);
  using E = Elem<DT>;
  using M = Mem<POL>;
  constexpr uint32_t V = E::V, U = 4, K = ROWS ? U : U + 1;
  const uint32_t len = ROWS ? n : 1u;                    // elements per counted unit
  const uint32_t bytes = (end - begin) * len * E::ES, nvec = bytes / 16u, tail = ROWS ? 0u : (end - begin) % V;
  const uint64_t boff = (uint64_t)begin * len * E::ES;
  const uint32_t lane = tid & 63u, wave = tid >> 6;
  uint32_t P = 1;
  if (ROWS) while (P < n / V) P <<= 1;
  const uint32_t rpw = 64u / P, sub = lane / P, j = lane & (P - 1u);
  const bool col = !ROWS || j < n / V;                   // (a row's lanes past its last vector)
  auto ld1 = [](rsrc_t r, uint32_t off) { return E::ES == 4 ? M::ldb4(r, off) : M::ldb2(r, off); };
  // What a task asks for, in lane k for task k: a read of a lane costs a link less than reads of LDS, whose latency
  // nothing hides.  (Not for rows, whose links are longer, and short of registers.)
  uint32_t h_ptr[3][2] = {}, h_what = 0, h_alpha = 0, h_C = 0;
  if (!ROWS && lane < n_links) {
    const Record* r = recs + lane;
    const v4i p01 = ((const v4i*)r->ptr)[0], p23 = ((const v4i*)r->ptr)[1];
    h_ptr[0][0] = (uint32_t)p01[0]; h_ptr[0][1] = (uint32_t)p01[1]; h_ptr[1][0] = (uint32_t)p01[2]; h_ptr[1][1] = (uint32_t)p01[3];
    h_ptr[2][0] = (uint32_t)p23[2]; h_ptr[2][1] = (uint32_t)p23[3];
    const uint32_t path = r->path, kinds = path == PATH_ROW2D ? (uint32_t)r->okind[0] | ((uint32_t)r->okind[1] << 4) : 0u;
    static_assert(K_FULL == 0, "operands of the other paths are whole");
    h_what = r->impl | (path << 8) | ((uint32_t)r->n_inputs << 12) | (kinds << 16) | ((uint32_t)r->dtype[1] << 24) | ((uint32_t)r->dtype[3] << 28);
    h_alpha = __builtin_bit_cast(uint32_t, r->alpha);
    h_C = r->size[1];
  }
  auto at_lane = [](uint32_t v, uint32_t k) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)k); };
  auto ptr_of = [&](uint32_t k, int i) {                 // input 0 or 1, or (2) the output
    if (ROWS) return (uint64_t)(__UINTPTR_TYPE__)uni_ptr(recs[k].ptr[i == 2 ? 3 : i]);
    return ((uint64_t)at_lane(h_ptr[i][1], k) << 32) | at_lane(h_ptr[i][0], k);
  };
  auto what_of = [&](uint32_t k) {
    if (!ROWS) return at_lane(h_what, k);
    const RecHead h = RecHead::of(recs + k);             // (bytes 0-15: inputs 4, dtypes 6 and 8, kinds 10 and 11)
    const uint32_t path = h.path(), w1 = h.op[1], w2 = h.op[2];
    const uint32_t kinds = path == PATH_ROW2D ? ((w2 >> 16) & 15u) | (((w2 >> 24) & 15u) << 4) : 0u;
    return uni(recs[k].impl) | (path << 8) | ((w1 & 15u) << 12) | (kinds << 16) | (((w1 >> 16) & 15u) << 24) | ((w2 & 15u) << 28);
  };
  static_assert(__builtin_offsetof(Record, n_inputs) == 4 && __builtin_offsetof(Record, okind) == 10, "the words of what_of");
  auto C_of = [&](uint32_t k) { return ROWS ? uni(recs[k].size[1]) : at_lane(h_C, k); };
  auto alpha_of = [&](uint32_t k) { return __builtin_bit_cast(float, ROWS ? uni(__builtin_bit_cast(uint32_t, recs[k].alpha)) : at_lane(h_alpha, k)); };
  // The first tasks' operands from outside the run (a mask, the other operand of an update): one of them is
  // requested with the head's first operand.  (A load behind the first stores is waited for behind them.)
  const uint64_t head_p = ptr_of(0, 0);
  const uint32_t head_kind = (what_of(0) >> 16) & 15u, head_C = C_of(0);
  uint64_t ext_p = 0;
  uint32_t ext_kind = 0, ext_C = 0;
#pragma unroll 1
  for (uint32_t k = 0; k < n_links && k < 3u && ext_p == 0; ++k) {
    const uint32_t what = what_of(k);
    auto outside = [&](uint64_t p, uint32_t kind) {
      if (ext_p != 0 || kind == K_ROWSCALAR || p == head_p || (k > 0 && p == ptr_of(0, 2)) || (k > 1 && p == ptr_of(1, 2))) return;
      ext_p = p; ext_kind = kind; ext_C = C_of(k);
    };
    if (k > 0) outside(ptr_of(k, 0), (what >> 16) & 15u);
    if (((what >> 12) & 15u) == 2u) outside(ptr_of(k, 1), (what >> 20) & 15u);
  }
  for (uint32_t b0 = ROWS ? begin : 0u;;) {
    const bool last = ROWS ? b0 + 4u * rpw * U >= end : b0 + U * kThreads >= nvec;
    uint32_t off[U], row[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      if (ROWS) {
        row[u] = b0 + (u * 4u + wave) * rpw + sub;
        off[u] = col && row[u] < end ? ((row[u] - begin) * (n / V) + j) * 16u : kNoLoad;
      } else {
        off[u] = b0 + tid + u * kThreads < nvec ? (b0 + tid + u * kThreads) * 16u : kNoLoad;
      }
    }
    const uint32_t off1 = !ROWS && last && tid < tail ? (nvec * V + tid) * E::ES : kNoLoad;
    // what the registers hold: the buffer that `cur`, `oth` and `sc` were read from or written to
    v4i cur[K], oth[K];
    float sc[U];
    uint64_t cur_p = 0, oth_p = 0, sc_p = 0;
    auto load = [&](v4i (&q)[K], uint64_t p, uint32_t kind, uint32_t C) {
      if (kind == K_ROWVEC) {                            // C elements over and over
        const rsrc_t rs = make_rsrc((const void*)(__UINTPTR_TYPE__)p, C * E::ES);
        const uint32_t cv = C / V, first = (uint32_t)(boff / 16u);         // (a task has less than 2^31 elements)
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) q[u] = M::ld16(rs, off[u] != kNoLoad ? (first + off[u] / 16u) % cv * 16u : kNoLoad);
        if constexpr (!ROWS) q[U] = v4i{0, 0, 0, 0};     // (whole vectors: no ragged end)
        return;
      }
      const rsrc_t rs = make_rsrc((const char*)(__UINTPTR_TYPE__)p + boff, bytes);
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) q[u] = M::ld16(rs, off[u]);
      if constexpr (!ROWS) q[U] = v4i{(int)ld1(rs, off1), 0, 0, 0};
    };
    // Loaded vectors are waited for where they are loaded.  Left to the compiler, which does not see on which way
    // round the loop it came to a use, every link waited for the stores of the one before.
    auto arrive = [&](v4i (&q)[K]) {
#pragma unroll
      for (uint32_t u = 0; u < K; ++u) asm volatile("" : "+v"(q[u]));
    };
    load(cur, head_p, head_kind, head_C);
    cur_p = head_p;
    if (ext_p != 0) { load(oth, ext_p, ext_kind, ext_C); oth_p = ext_p; arrive(oth); }
    arrive(cur);
    for (uint32_t k = 0; k < n_links; ++k) {
      const uint64_t p0 = ptr_of(k, 0), p1 = ptr_of(k, 1), po = ptr_of(k, 2);
      const uint32_t what = what_of(k), impl = what & 0xffu, path = (what >> 8) & 15u, C = C_of(k);
      const float alpha = alpha_of(k);
      const bool two = ((what >> 12) & 15u) == 2u;
      const uint32_t kind0 = (what >> 16) & 15u, kind1 = (what >> 20) & 15u;
      const bool scalar = ROWS && two && kind1 == K_ROWSCALAR, pair = two && !scalar;
      if ((skip >> k) & 1u) continue;                    // (completes with an error, writes nothing)
      const bool b_cur = pair && p1 == cur_p;
      bool a_cur = p0 == cur_p;
      if (!a_cur && p0 != oth_p) {
        if (b_cur) { load(oth, p0, kind0, C); oth_p = p0; arrive(oth); }
        else { load(cur, p0, kind0, C); cur_p = p0; a_cur = true; arrive(cur); }
      }
      bool b_oth = false;
      if (pair && p1 != cur_p) {
        if (p1 == oth_p) b_oth = true;
        else if (a_cur) { load(oth, p1, kind1, C); oth_p = p1; b_oth = true; arrive(oth); }
        else { load(cur, p1, kind1, C); cur_p = p1; arrive(cur); }
      }
      typedef EitherArg<DT, K> Arg;
      const Arg qa = {cur, oth, !a_cur}, qb = {cur, oth, b_oth};
      if constexpr (ROWS) {
        if (path == PATH_RED_CONTIG) {
          if (impl == GPUOS_IMPL_SUM_LAST) link_reduce<GPUOS_IMPL_SUM_LAST, DT>(qa, col, P, sc);
          else if (impl == GPUOS_IMPL_MAX_LAST) link_reduce<GPUOS_IMPL_MAX_LAST, DT>(qa, col, P, sc);
          else link_reduce<GPUOS_IMPL_MIN_LAST, DT>(qa, col, P, sc);
          const uint32_t odt = what >> 28;
#pragma unroll
          for (uint32_t u = 0; u < U; ++u) {
            const bool mine = j == 0 && row[u] < end;
            const uint32_t at = row[u] - begin;
            if (odt == GPUOS_F32) {
              M::stb4(make_rsrc((const char*)(__UINTPTR_TYPE__)po + (uint64_t)begin * 4u, (end - begin) * 4u), mine ? at * 4u : kNoLoad, __builtin_bit_cast(uint32_t, sc[u]));
            } else {
              const uint32_t h = odt == GPUOS_F16 ? f2h(sc[u]) : f2b(sc[u]);
              M::stb2(make_rsrc((const char*)(__UINTPTR_TYPE__)po + (uint64_t)begin * 2u, (end - begin) * 2u), mine ? at * 2u : kNoLoad, h);
              sc[u] = odt == GPUOS_F16 ? h2f(h) : b2f(h);
            }
          }
          sc_p = po;
          continue;
        }
        if (scalar && p1 != sc_p) {                      // a scalar per row from memory
          const uint32_t sdt = (what >> 24) & 15u;
#pragma unroll
          for (uint32_t u = 0; u < U; ++u) sc[u] = row[u] < end ? load_rt<POL>((const void*)(__UINTPTR_TYPE__)p1, row[u], sdt) : 0.0f;
#pragma unroll
          for (uint32_t u = 0; u < U; ++u) asm volatile("" : "+v"(sc[u]));
          sc_p = p1;
        }
      }
      const rsrc_t ro = make_rsrc((const char*)(__UINTPTR_TYPE__)po + boff, bytes);
      auto sink = [&](int u, const v4i& q) {
        if (u < (int)U) M::st16(ro, off[u < (int)U ? u : 0], q);
        else if (E::ES == 4) M::stb4(ro, off1, (uint32_t)q[0]);
        else M::stb2(ro, off1, (uint32_t)q[0]);
        cur[u] = q;
        __builtin_amdgcn_sched_barrier(0);               // (a vector at a time: interleaved they need registers that callers keep)
      };
      if (!two) ByArity<1>::template vectors<DT, K>(impl, qa, qa, qa, alpha, sink);
      else if (pair) ByArity<2>::template vectors<DT, K>(impl, qa, qb, qa, alpha, sink);
      else if constexpr (ROWS) ByArity<2>::template vectors<DT, K>(impl, qa, RowArg<K>{sc}, qa, alpha, sink);
      cur_p = po;
      if (oth_p == po) oth_p = 0;
    }
    if (last) break;
    b0 += ROWS ? 4u * rpw * U : U * kThreads;
  }
}

// One unit of a run, from the head's descriptor (slot f) to the completion of its tasks.
// Neither this nor run_links keeps a register for its caller (both are called, never jumped to, and the compiler sees
// every call): a chunk of 8K elements, 82 KB of a chain's memory traffic, saved and restored another 66 KB of them.
// The worker, which would have to keep its own registers instead, calls it where it holds none (see run_worker).
// Chains of six over fp16 rows, 24 in flight: 675 K tasks/s with the registers saved, 785 without, 855 with the call there.
__attribute__((not_tail_called, disable_tail_calls)) PATHFN void exec_run(WorkShared* s_v, uint32_t f_v, uint32_t chunk_v, int32_t status_v, uint32_t tid) {
  WorkShared* s = lds_arg(s_v);
  const uint32_t f = uni(f_v), chunk = uni(chunk_v), lane = tid & 63u;
  const Record* head = &s->rec[f];
  const uint32_t n = uni(head->run), cap_mask = uni(s->cap_mask), cap_shift = uni((uint32_t)s->cap_shift);
  const uint64_t ticket = uni64(head->ticket);
  // the descriptors, through the mirror like the head's: each proves itself (see mirror_record_valid)
  Record* const recs = (Record*)s->red;
  uint32_t* const ok = (uint32_t*)s->red + kRunMax * sizeof(Record) / 4;       // per task: seen whole; then the status it completes with
  static_assert((kRunMax * sizeof(Record) + kRunMax * 4) <= kScratchFloats * 4 && kRunMax <= 64, "a run's descriptors fit the scratch");
  const rsrc_t rd = make_rsrc(uni_ptr((uint64_t)(__UINTPTR_TYPE__)s->dring), (cap_mask + 1u) * (uint32_t)sizeof(Record));
  const OpSlots* const table = (const OpSlots*)uni_ptr((uint64_t)(__UINTPTR_TYPE__)s->dtable);
  bool whole = true;
  for (uint32_t attempt = 0;; ++attempt) {
    constexpr uint32_t kPieces = kRunMax * 16u / kThreads;
    v4i q[kPieces];
#pragma unroll
    for (uint32_t j = 0; j < kPieces; ++j) {
      const uint32_t k = (tid + j * kThreads) >> 4, slot = (uint32_t)((ticket + k) & cap_mask);
      q[j] = Mem<POL_COHERENT>::ld16(rd, k < n ? slot * (uint32_t)sizeof(Record) + (tid & 15u) * 16u : kNoLoad);
    }
    uint64_t ent[kPieces];
#pragma unroll
    for (uint32_t j = 0; j < kPieces; ++j) {
      // the table slot it claimed, from the lane that holds the words that name it
      const uint32_t k = (tid + j * kThreads) >> 4, op = (uint32_t)q[j][0] & 0xffu, sel = ((uint32_t)q[j][3] >> 8) & 1u;
      ent[j] = 0;
      if ((tid & 15u) == 0 && k < n) ent[j] = __hip_atomic_load(&table[op].slot[sel], __ATOMIC_RELAXED, SC_SYSTEM);
    }
#pragma unroll
    for (uint32_t j = 0; j < kPieces; ++j) {
      const uint32_t k = (tid + j * kThreads) >> 4;
      ((v4i*)recs)[tid + j * kThreads] = q[j];
      const uint32_t x = record_piece_sum(q[j], tid & 15u);
      // its ticket and version, in lanes 3 and 1 of the sixteen
      const uint32_t t_lo = (uint32_t)__shfl((int)q[j][2], (int)((lane & 48u) + 3u)), t_hi = (uint32_t)__shfl((int)q[j][3], (int)((lane & 48u) + 3u));
      const uint32_t version = (uint32_t)__shfl((int)q[j][1], (int)((lane & 48u) + 1u));
      const uint64_t t = ticket + k;
      const bool valid = x == record_check_seed(t) && t_lo == (uint32_t)t && t_hi == (uint32_t)(t >> 32);
      if ((tid & 15u) == 0 && k < n) ok[k] = !valid ? 1u : ((uint32_t)(ent[j] >> 32) != version ? (uint32_t)GPUOS_E_VERSION : 0u);
    }
    __syncthreads();
    whole = __ballot(lane < n && ok[lane] == 1u) == 0;
    if (whole || attempt >= kMirrorRetries) break;
    __syncthreads();                                     // everyone has looked at this attempt's copies
    __builtin_amdgcn_s_sleep(2);
  }
  if (!whole) { __syncthreads(); return; }               // (dropped, as a lone descriptor that is never seen whole)
  if (tid == 0 && status_v != GPUOS_OK) ok[0] = (uint32_t)status_v;
  __syncthreads();
  const uint64_t skip = __ballot(lane < n && ok[lane] != 0);
  // rows, if one of the tasks reduces rows or has a scalar per row: their length, and the head's chunk in rows
  uint32_t row_n = 0;
  if (lane < n) {
    const Record* r = recs + lane;
    if (r->path == PATH_RED_CONTIG) row_n = r->red_n;
    else if (r->path == PATH_ROW2D && r->okind[1] == K_ROWSCALAR) row_n = r->size[1];
  }
  const uint64_t m_rows = __ballot(row_n != 0);
  const uint32_t len = m_rows != 0 ? (uint32_t)__builtin_amdgcn_readlane((int)row_n, (int)__builtin_ctzll(m_rows)) : 0u;
  const bool counts_rows = uni(head->path) == PATH_RED_CONTIG;
  uint32_t per = uni(head->chunk), numel = uni(head->numel);
  if (len != 0 && !counts_rows) { per /= len; numel /= len; }
  const uint32_t begin = chunk * per, end = numel - begin < per ? numel : begin + per;
  const uint32_t dt = uni(head->dtype[0]);
  if (len == 0) {
    if (dt == GPUOS_F32) run_links<POL_COHERENT, GPUOS_F32, false>(recs, n, skip, begin, end, 0, tid);
    else if (dt == GPUOS_F16) run_links<POL_COHERENT, GPUOS_F16, false>(recs, n, skip, begin, end, 0, tid);
    else run_links<POL_COHERENT, GPUOS_BF16, false>(recs, n, skip, begin, end, 0, tid);
  } else {
    if (dt == GPUOS_F32) run_links<POL_COHERENT, GPUOS_F32, true>(recs, n, skip, begin, end, len, tid);
    else if (dt == GPUOS_F16) run_links<POL_COHERENT, GPUOS_F16, true>(recs, n, skip, begin, end, len, tid);
    else run_links<POL_COHERENT, GPUOS_BF16, true>(recs, n, skip, begin, end, len, tid);
  }
  drain_stores();
  __syncthreads();                                       // every wave's stores of every task have reached memory
  if (tid < 64) {
    SlotState* const st = global_ptr(s->st);
    uint64_t* const comp = global_ptr(s->hcomp);
    const bool mine = lane < n;
    const Record* r = recs + (mine ? lane : 0u);
    const uint32_t nchunks = uni(head->nchunks);
    const uint64_t t = ticket + lane, target = done_target(t, cap_shift);
    const uint32_t slot = (uint32_t)(t & cap_mask);
    bool last = mine;
    if (mine && nchunks > 1) {
      const uint64_t share = chunk + 1 == nchunks ? kDoneTask - (nchunks - 1) : 1ull;
      last = __hip_atomic_fetch_add(&st[slot].done_seq, share, __ATOMIC_RELAXED, SC_AGENT) + share == target;
    }
    if (mine && nchunks <= 1) __hip_atomic_store(&st[slot].done_seq, target, __ATOMIC_RELAXED, SC_SYSTEM);
    if (last) __hip_atomic_store(&comp[slot], pack_completion(t, (int32_t)ok[lane], r->version), __ATOMIC_RELAXED, SC_SYSTEM);
    const uint64_t m = __ballot(last);
    if (lane == 0 && m != 0) __hip_atomic_fetch_add(global_ptr(s->done_count), (uint64_t)__popcll(m), __ATOMIC_RELAXED, SC_AGENT);
  }
  __syncthreads();                                       // the descriptors and the scratch may be overwritten after this
}

// What the worker runs away from its choice of executors: one that would use most of the registers that a function keeps for
// its caller, and keeps none (it is called and never jumped to, and the compiler sees every call).  Kept, they were 63 KiB written and
// read back for a row of 125 KiB.  All it goes by lies in LDS: what is live where the choice below is
// made goes through scratch memory, a trip to memory under load for each level of choices.
template <int DT, bool RAGGED>
__attribute__((not_tail_called)) PATHFN void softmax_away(WorkShared* s_v, uint32_t tid) {
  WorkShared* s = lds_arg(s_v);
  const v4i dec = *(const v4i*)s->dec;
  const Record* r = &s->rec[(uni((uint32_t)dec[0]) >> 8) & 0xffu];
  const uint32_t per = uni(r->chunk), rows = uni(r->numel), begin = (uni((uint32_t)dec[2]) & 0x3ffu) * per;
  softmax_held_rows<POL_COHERENT, DT, RAGGED>(r, begin, rows - begin < per ? rows : begin + per, s->red, tid);
}
__attribute__((not_tail_called)) PATHFN void exec_away(WorkShared* s_v, uint32_t wave_v) {
  WorkShared* s = lds_arg(s_v);
  const uint32_t wave = uni(wave_v);
  const Record* r = &s->rec[(uni(s->dec[0]) >> 8) & 0xffu];
  const uint32_t k = 2u * uni(r->dtype[3]) + (uni(r->path) == PATH_ROW_RAGGED ? 1u : 0u);
  if (k < 2u) { if (k == 0) softmax_away<GPUOS_F32, false>(s, thread_index(wave)); else softmax_away<GPUOS_F32, true>(s, thread_index(wave)); }
  else if (k < 4u) { if (k == 2) softmax_away<GPUOS_F16, false>(s, thread_index(wave)); else softmax_away<GPUOS_F16, true>(s, thread_index(wave)); }
  else { if (k == 4) softmax_away<GPUOS_BF16, false>(s, thread_index(wave)); else softmax_away<GPUOS_BF16, true>(s, thread_index(wave)); }
}

// RING 0: the library's own workers, on the main unit ring, executing through EXEC = the built-in
// chunk executor.  RING 1: the workers of a kernel compiled at run time, on the second unit ring
// (the dispatcher routes the tasks of natively compiled operator programs there), executing through
// the EXEC that kernel brings; `gen` is the generation of that kernel: its workers leave when the
// host asks for a later one.
//
// next_unit: the next unit that can run (its descriptor and what it needs of it: `u`), or false: the worker leaves.
struct Unit {
  RecHead head;
  uint32_t f, chunk, impl, run;                       // descriptor slot, chunk, implementation; tasks that it stands for
  int32_t status;
};
template <int RING>
DEV bool next_unit(const WorkerArgs& a, WorkShared* s, uint32_t gen, uint32_t wave, Unit& out) {
  const uint32_t lane = thread_index(0);              // (anew, and all that follows from it: nothing is kept over a run)
  const bool leader = wave == 0 && lane == 0;
  uint64_t* const claim_ctr = RING == 0 ? &a.d->claim : &a.d->claim_j;
  const uint64_t* const unit_ring = RING == 0 ? a.units : a.units_j;
  const rsrc_t rd = make_rsrc(a.dring, (a.cap_mask + 1u) * (uint32_t)sizeof(Record));
  const bool timing = a.timing != 0, tracing = a.trace != nullptr;
  auto count = [&](uint32_t which, uint64_t add) { if (leader) s->ticks[which - ST_WORK_TICKS_WAIT] += add; };
  while (true) {
    const uint64_t c0 = clock_if(timing);
    // ---- decide what to do next (first wavefront): one round of loads per poll ----
    // Lane 32 polls the claimed entry itself (its stamp is the ready flag: every waiting workgroup
    // polls a different address); lane k < kStash looks at the done words that descriptor slot k waits for.
    if (wave == 0) {
      uint32_t action = kActExit, f = 0;
      int32_t dep_status = 0;
      uint64_t u_new = 0;
      const v4i st = *(const v4i*)s->state;
      uint32_t waiting = uni((uint32_t)st[0]) & kStashFull, polls = uni((uint32_t)st[1]), yield_every = 0;
      bool have_claim = (uni((uint32_t)st[0]) & kHaveClaim) != 0, draining = (uni((uint32_t)st[0]) & kDraining) != 0;
      uint64_t g = ((uint64_t)uni((uint32_t)st[3]) << 32) | uni((uint32_t)st[2]);
      const bool held_any = waiting != 0;
      if (!have_claim && !draining && waiting != kStashFull) {
        uint64_t gg = 0;
        if (leader) gg = __hip_atomic_fetch_add(claim_ctr, 1ull, __ATOMIC_RELAXED, SC_AGENT);
        g = uni64(gg);
        have_claim = true;
        polls = 0;
      }
      const uint64_t* up = &unit_ring[g & a.unit_mask];
      const uint64_t want = unit_stamp(g, a.unit_shift);
      // What is awaited was published before the unit that waits (the dispatcher sees to that), so the
      // wait ends when resident workgroups finish work they hold.  It is bounded all the same (the
      // context's wait limit; a short grace once the stop flag is up): a task that runs into the
      // bound completes with GPUOS_E_TIMEOUT without executing, and the kernel always leaves.
      const bool mine = lane < kStash && ((waiting >> lane) & 1u);
      uint64_t need[3] = {0ull, 0ull, 0ull};
      const uint64_t* done_word[3] = {nullptr, nullptr, nullptr};
      if (mine) {
        const Record* r = &s->rec[lane];
        const uint64_t ticket = r->ticket;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const uint32_t back = r->dep[k];
          if (back != 0 && back <= ticket) {
            need[k] = done_target(ticket - back, a.cap_shift);
            done_word[k] = &a.st[(ticket - back) & a.cap_mask].done_seq;
          }
        }
      }
      // One round of loads per poll.  (Keeping a second round in flight, to sample twice per memory
      // round trip, was measured: with 767 workgroups polling, the doubled traffic cost a lone task
      // more than the earlier sample gained, 7.7 against 6.5 us.)
      struct Poll { uint64_t u, seen[3]; };
      // While something is held, every lane issues all four loads, the lanes with nothing to look at from
      // the unit-ring entry that lane 32 polls anyway (one request for the whole wavefront): loads under
      // conditions that differ between lanes are waited for one after the other (a poll would take up
      // to four memory round trips instead of one).
      const uint64_t* const anyword = up;
      auto request = [&]() {
        Poll p;
        if (waiting == 0) {
          p.u = 0;
          if (lane == 32 && have_claim) p.u = __hip_atomic_load(up, __ATOMIC_RELAXED, SC_SYSTEM);
          p.seen[0] = p.seen[1] = p.seen[2] = ~0ull;
        } else {
          p.u = __hip_atomic_load(up, __ATOMIC_RELAXED, SC_SYSTEM);
#pragma unroll
          for (int k = 0; k < 3; ++k) p.seen[k] = __hip_atomic_load(done_word[k] ? done_word[k] : anyword, __ATOMIC_RELAXED, SC_SYSTEM);
        }
        return p;
      };
      while (true) {
        const Poll cur = request();
        bool ready = mine && cur.seen[0] >= need[0] && cur.seen[1] >= need[1] && cur.seen[2] >= need[2];
        int32_t gave_up = 0;
        if (mine && !ready && (polls & 31u) == 31u) {
          uint64_t limit = a.dep_wait_ticks;
          if (limit > kStopGraceTicks && __hip_atomic_load(&a.d->stop_dev, __ATOMIC_RELAXED, SC_SYSTEM)) limit = kStopGraceTicks;
          if (wall_clock64() - s->since[lane] > limit) { gave_up = GPUOS_E_TIMEOUT; ready = true; }
        }
        order_loads();
        const uint64_t m_ready = __ballot(ready);
        u_new = lane64(cur.u, 32u);
        if (m_ready != 0) {                                   // the first descriptor slot whose unit can run (any ready
          f = (uint32_t)__builtin_ctzll(m_ready);             // one makes progress)
          dep_status = __builtin_amdgcn_readlane(gave_up, (int)f);
          waiting &= ~(1u << f);
          u_new = s->unit[f];
          action = kActRun;
          break;
        }
        if (have_claim && (u_new >> 46) == want) {
          f = (uint32_t)__builtin_ctz(~waiting);              // a free descriptor slot (claims are made only while one exists)
          have_claim = false;
          action = kActFetch;
          fetch_descriptor(a, s, rd, u_new, f, lane);  // requested at once: the other wavefronts need not hear of the unit first
          break;
        }
        ++polls;
        if ((polls & 31u) == 0) {
          // (a run-time kernel also leaves when a later generation is wanted: the host asks for that
          // only once nothing is routed to this ring any more and everything routed has completed)
          const bool stop = __hip_atomic_load(&a.d->stop_dev, __ATOMIC_RELAXED, SC_SYSTEM) != 0 ||
                            (RING == 1 && __hip_atomic_load(&a.d->jit_gen, __ATOMIC_RELAXED, SC_SYSTEM) > gen);
          if (stop && !draining) {
            order_loads();                                    // every unit was stored before the stop flag
            if (have_claim) {
              u_new = uni64(__hip_atomic_load(up, __ATOMIC_RELAXED, SC_SYSTEM));
              order_loads();
              if ((u_new >> 46) == want) {
                f = (uint32_t)__builtin_ctz(~waiting);
                have_claim = false;
                action = kActFetch;
                fetch_descriptor(a, s, rd, u_new, f, lane);
                break;
              }
              // The number claimed will never be served.  The second ring stays in use across
              // generations of run-time kernels while the dispatcher runs on: give the number back
              // (nothing is being published to that ring at this time, so the count ends exact).
              if (RING == 1 && leader) __hip_atomic_fetch_add(claim_ctr, ~0ull, __ATOMIC_RELAXED, SC_AGENT);
              have_claim = false;
            }
            draining = true;
          }
          yield_every = __hip_atomic_load(&a.d->yield_every, __ATOMIC_RELAXED, SC_SYSTEM);
        }
        if (draining && !have_claim && waiting == 0) { action = kActExit; break; }
        // polling policy (paper Section 4.1): short back-off while spinning, longer pauses every
        // yield_every-th empty poll when the host asked for them and nothing is held
        if (yield_every != 0 && waiting == 0 && (polls % yield_every) == 0) { for (int k = 0; k < 16; ++k) __builtin_amdgcn_s_sleep(127); }
        else if (polls < 64 || waiting != 0) __builtin_amdgcn_s_sleep(1);
        else __builtin_amdgcn_s_sleep(8);
      }
      if (leader) {
        const v4i next = {(int)(waiting | (have_claim ? kHaveClaim : 0u) | (draining ? kDraining : 0u)), (int)polls, (int)(uint32_t)g, (int)(uint32_t)(g >> 32)};
        const v4i dec = {(int)(action | (f << 8) | (held_any ? 1u << 16 : 0u)), dep_status, (int)(uint32_t)u_new, (int)(uint32_t)(u_new >> 32)};
        *(v4i*)s->state = next;
        *(v4i*)s->dec = dec;
      }
    }
    __syncthreads();
    const v4i dec = *(const v4i*)s->dec;
    const uint32_t action = uni((uint32_t)dec[0]) & 0xffu, f = (uni((uint32_t)dec[0]) >> 8) & 0xffu;
    if (action == kActExit) {
      if (leader) {
        uint64_t* st = a.d->stat;
        __hip_atomic_fetch_add(&st[ST_WORK_UNITS], s->n_units, __ATOMIC_RELAXED, SC_AGENT);
        for (uint32_t k = ST_WORK_TICKS_WAIT; k < ST_WORK_TICKS_TOTAL; ++k)
          __hip_atomic_fetch_add(&st[k], s->ticks[k - ST_WORK_TICKS_WAIT], __ATOMIC_RELAXED, SC_AGENT);
        __hip_atomic_fetch_add(&st[ST_WORK_TICKS_TOTAL], c0 - s->entered, __ATOMIC_RELAXED, SC_AGENT);
      }
      return false;
    }
    const uint64_t c1 = clock_if(timing || tracing);
    if (timing) count(uni((uint32_t)dec[0]) >> 16 ? ST_WORK_TICKS_DEP : ST_WORK_TICKS_WAIT, c1 - c0);
    // the unit is the same for the whole workgroup: keep its fields in scalar registers
    const uint32_t unit_lo = uni((uint32_t)dec[2]), unit_hi = uni((uint32_t)dec[3]);
    const uint64_t unit = ((uint64_t)unit_hi << 32) | unit_lo;
    const uint32_t chunk = (uint32_t)(unit & 0x3ffu), lap10 = (uint32_t)((unit >> 10) & 0x3ffu);
    const uint32_t slot = (uint32_t)((unit >> 20) & 0xffffu);
    const Record* r = &s->rec[f];
    // What the rest of this unit's handling asks of the record, read in one go (field by field, where each
    // is wanted, was eight LDS latencies in a row before the executor is reached).
    struct { v4i op, impl, dims, links; uint64_t entry; uint32_t sum; } head;
    auto read_head = [&]() {
      const v4i* h = (const v4i*)r;
      head.op = h[0]; head.impl = h[1]; head.dims = h[2]; head.links = h[3];
      head.entry = s->entry[f];
      head.sum = s->rec_sum;
      asm volatile("" : "+v"(head.op), "+v"(head.impl), "+v"(head.dims), "+v"(head.links), "+v"(head.entry), "+v"(head.sum));
    };
    static_assert(__builtin_offsetof(Record, impl) == 16 && __builtin_offsetof(Record, version) == 20 && __builtin_offsetof(Record, status) == 24 &&
                  __builtin_offsetof(Record, nchunks) == 28 && __builtin_offsetof(Record, dep) == 48 && __builtin_offsetof(Record, ticket) == 56, "the words that are read as vectors");
    read_head();
    const auto word = [](const v4i& q, int k) { return uni((uint32_t)q[k]); };
    const auto pair = [](const v4i& q, int k) { return ((uint64_t)uni((uint32_t)q[k + 1]) << 32) | uni((uint32_t)q[k]); };
    if (action == kActFetch) {
      // ---- fetch the descriptor (16 lanes x 16 bytes) and the claimed table slot ----
      // The dispatcher does not wait for its mirror stores before it publishes a unit: the record is
      // taken only once its check word holds for the ticket the unit names (else its pieces are still
      // landing, or belong to the slot's previous lap) and fetched again otherwise.  The stores are on
      // their way, so this ends; it is bounded like every wait here (a workgroup that runs out leaves
      // the task to the host's time limit).
      // (the first wavefront has fetched it once already, when it saw the unit)
      bool valid = false;
      for (uint32_t attempt = 0;; ++attempt) {
        valid = mirror_record_valid(uni(head.sum), pair(head.links, 2), slot, lap10, a.cap_mask, a.cap_shift);
        if (valid || attempt >= kMirrorRetries) break;
        __syncthreads();                                  // everyone has looked at this attempt's copy
        __builtin_amdgcn_s_sleep(2);
        if (wave == 0) fetch_descriptor(a, s, rd, unit, f, thread_index(0));
        __syncthreads();
        read_head();
      }
      const uint64_t c2 = clock_if(timing);
      if (timing) count(ST_WORK_TICKS_FETCH, c2 - c1);
      if (!valid) {
        // never seen whole: nothing in it can be trusted, not even the ticket it would complete.  The
        // unit is dropped; the host's wait for the ticket runs into its time limit.
        __syncthreads();
        continue;
      }
      if ((pair(head.links, 0) & 0xffffffffffffull) != 0 &&    /* (dep[3]; the halfword behind them is `run`) */ (((uint32_t)word(head.op, 2) >> 8) & RF_DEPS_RESOLVED) == 0) {
        // It names earlier tasks: it joins the units held, and the first wavefront looks at its done
        // words with the next poll (and runs it at once if they are all there).
        if (leader) {
          s->unit[f] = unit;
          s->state[0] |= 1u << f;
          s->since[f] = wall_clock64();
        }
        if (wave == 0) lds_wave_sync();
        continue;
      }
    }
    int32_t status = (int32_t)word(head.impl, 2);
    const uint32_t impl = word(head.impl, 0), nchunks = word(head.impl, 3);
    if (status == GPUOS_OK && uni((uint32_t)(head.entry >> 32)) != word(head.impl, 1)) status = GPUOS_E_VERSION;
    if (status == GPUOS_OK) status = (int32_t)word(dec, 1);
    out = Unit{RecHead::of(head.op, head.dims), f, chunk, impl, word(head.links, 1) >> 16, status};
    if (timing || tracing) {
      // a task's start in the trace is the moment a workgroup took its descriptor (a unit that waited: when it began to)
      const uint64_t c_start = (tracing && action == kActRun) ? s->since[f] : c1;
      if (leader) {
        s->begun = clock_if(timing);
        s->started = c_start;
        if (tracing && chunk == 0 && nchunks > 1)
          __hip_atomic_store(&a.st[slot].t_first, c_start, __ATOMIC_RELAXED, SC_SYSTEM);   // in memory before this chunk is counted
      }
    }
    return true;
  }
}

// A chunk that has been executed, to the completion of its task.  It goes by what lies in LDS and by the kernel's arguments.
template <int RING>
DEV void complete_unit(const WorkerArgs& a, WorkShared* s, int32_t status, uint32_t tid) {
  const bool leader = tid == 0;
  const bool timing = a.timing != 0, tracing = a.trace != nullptr;
  const v4i dec = *(const v4i*)s->dec;
  const uint32_t f = (uni((uint32_t)dec[0]) >> 8) & 0xffu, unit_lo = uni((uint32_t)dec[2]), unit_hi = uni((uint32_t)dec[3]);
  const uint64_t unit = ((uint64_t)unit_hi << 32) | unit_lo;
  const uint32_t chunk = (uint32_t)(unit & 0x3ffu), slot = (uint32_t)((unit >> 20) & 0xffffu);
  const Record* r = &s->rec[f];
  if (RING == 1 && leader) __hip_atomic_fetch_add(&a.d->jit_units, 1ull, __ATOMIC_RELAXED, SC_AGENT);
  // (read while the stores are still on their way)
  const v4i impl_w = ((const v4i*)r)[1];
  const uint64_t ticket = r->ticket;
  SlotState* const st = a.st;
  uint64_t *const comp = a.hcomp, *const done_count = &a.d->done_count;
  const uint32_t cap_shift = a.cap_shift;
  drain_stores();                   // this wave's (write-through) stores have reached memory
  __syncthreads();                  // ... and so have the other three waves'
  const uint64_t c4 = clock_if(timing || tracing);
  // ---- complete ----
  if (leader) {
    const uint32_t nchunks = (uint32_t)impl_w[3], version = (uint32_t)impl_w[1];
    const uint64_t target = done_target(ticket, cap_shift);
    bool last = true;
    if (nchunks > 1) {
      const uint64_t share = chunk + 1 == nchunks ? kDoneTask - (nchunks - 1) : 1ull;
      last = __hip_atomic_fetch_add(&st[slot].done_seq, share, __ATOMIC_RELAXED, SC_AGENT) + share == target;
    }
    if (last) {
      if (tracing) {
        // the tracepoint lands before the completion word that lets the host read it
        const uint64_t origin = __hip_atomic_load(&a.h->clock_origin, __ATOMIC_RELAXED, SC_SYSTEM);
        const uint64_t t_start = nchunks > 1 ? __hip_atomic_load(&st[slot].t_first, __ATOMIC_RELAXED, SC_SYSTEM) : s->started;
        TraceRec* tr = &a.trace[ticket & a.trace_mask];
        const uint64_t tdq = ((uint64_t)r->t_dequeue[1] << 32) | r->t_dequeue[0];
        __hip_atomic_store(&tr->t_dequeue, tdq - origin, __ATOMIC_RELAXED, SC_SYSTEM);
        __hip_atomic_store(&tr->t_start, t_start - origin, __ATOMIC_RELAXED, SC_SYSTEM);
        // The clock is read here, once this workgroup knows it finished the task: the time taken
        // right after its own chunk (c4) can lie before the start of chunk 0 when this workgroup's
        // count arrives late (seen once in a few thousand multi-chunk tasks).
        const uint64_t t_done = nchunks > 1 ? wall_clock64() : c4;
        __hip_atomic_store(&tr->t_done, t_done - origin, __ATOMIC_RELAXED, SC_SYSTEM);
        const uint64_t w4 = (uint64_t)version | ((uint64_t)r->op_id << 32) | ((uint64_t)(uint8_t)(int8_t)status << 48);
        __hip_atomic_store((uint64_t*)&tr->op_version, w4, __ATOMIC_RELAXED, SC_SYSTEM);
        const uint64_t w5 = (uint64_t)nchunks | ((uint64_t)blockIdx.x << 32);
        __hip_atomic_store((uint64_t*)&tr->nchunks, w5, __ATOMIC_RELAXED, SC_SYSTEM);
        __hip_atomic_store(&tr->ticket, ticket, __ATOMIC_RELAXED, SC_SYSTEM);
        drain_stores();
      }
      if (nchunks <= 1) __hip_atomic_store(&st[slot].done_seq, target, __ATOMIC_RELAXED, SC_SYSTEM);
      __hip_atomic_store(&comp[slot], pack_completion(ticket, status, version), __ATOMIC_RELAXED, SC_SYSTEM);
      __hip_atomic_fetch_add(done_count, 1ull, __ATOMIC_RELAXED, SC_AGENT);
    }
  }
  __syncthreads();                  // the descriptor in LDS may be overwritten after this
  const uint64_t c5 = clock_if(timing);
  if (leader) {
    s->n_units += 1;
    if (timing) { s->ticks[ST_WORK_TICKS_EXEC - ST_WORK_TICKS_WAIT] += c4 - s->begun; s->ticks[ST_WORK_TICKS_COMPLETE - ST_WORK_TICKS_WAIT] += c5 - c4; }
  }
}

// The kernel's arguments (its first parameter), apart from the dispatcher's: with values that both read kept over both,
// either held the other's in registers (1,000 small additions 95.7 us instead of 85.0).
DEV const WorkerArgs& worker_args() {
  typedef const __attribute__((address_space(4))) WorkerArgs* args_t;
  args_t p = (args_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const WorkerArgs*)p;
}

template <int RING, class EXEC>
DEV void run_worker(WorkShared* s, uint32_t gen = 0) {
  const WorkerArgs& a = worker_args();
  const uint32_t my_wave = uni(threadIdx.x >> 6);     // (this thread's place as the wavefront's index, a scalar, and the lane; see thread_index)
  if (my_wave == 0 && lane_id() == 0) {
    s->state[0] = s->state[1] = s->state[2] = s->state[3] = 0;
    s->n_units = 0;
    s->st = a.st; s->hcomp = a.hcomp; s->done_count = &a.d->done_count; s->cap_shift = a.cap_shift;
    s->dring = a.dring; s->dtable = a.dtable; s->cap_mask = a.cap_mask;
    for (uint32_t k = 0; k < ST_WORK_TICKS_TOTAL - ST_WORK_TICKS_WAIT; ++k) s->ticks[k] = 0;
    s->entered = clock_if(a.timing != 0);
  }
  lds_wave_sync();                                    // (only the first wavefront reads them)
  while (true) {
    uint32_t wave = my_wave;
    asm volatile("" : "+s"(wave));                    // (nothing that follows from it is kept from one unit to the next)
    Unit u;
    if (!next_unit<RING>(a, s, gen, wave, u)) return;
    if (RING == 0 && __builtin_expect(u.run > 1u, 0)) {                  // a run of two or more tasks
      exec_run(s, u.f, u.chunk, u.status, thread_index(wave));
      if (thread_index(wave) == 0) {
        s->n_units += 1;
        if (a.timing != 0) s->ticks[ST_WORK_TICKS_EXEC - ST_WORK_TICKS_WAIT] += wall_clock64() - s->begun;
      }
      continue;
    }
    int32_t status = u.status;
    if (RING == 0 && __builtin_expect(status == GPUOS_OK && rowop_is_away(u.head, u.impl), 0)) exec_away(s, wave);
    else if (status == GPUOS_OK) status = EXEC::run(&s->rec[u.f], u.head, u.impl, u.chunk, s->red, a.progs, thread_index(wave));
    complete_unit<RING>(a, s, status, thread_index(wave));
  }
}

}  // namespace gpuos

// lbm_device.h -- device functions shared by the gfx950 kernels of the
// plane-strain LBM: storage codecs, finite differences, Hooke's law, load
// amplitudes and the displacement update.
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "../../include/lbm.h"
#include "lbm_types.h"

namespace lbm {

// ------------------------------------------------------------------ codecs
//
// A codec maps the stored representation of one field's five populations
// to populations in the collision precision C and back.  eq_pops gives the
// populations of f_eq(rho, J) (eq. feq, lattice units c = 1, b = 1) exactly
// as load() returns them after store_eq().

// 16-bit conversions for the stored non-equilibrium moments.
//
// x to BF16 by truncation after adding r (0 <= r < 2^16) below its last
// significand bit: with r uniform, x rounds away from zero with probability
// equal to its distance from the truncated value in ulps (the magnitude
// bits are linear in the value within a binade; a carry moves to the next
// binade as it should).  NaN stays NaN.
__device__ __forceinline__ uint16_t f32_to_bf16_sr(float x, uint32_t r) {
  const uint32_t u = __float_as_uint(x);
  if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0x007fffffu) ? 0x40 : 0));
  return (uint16_t)((u + r) >> 16);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

__device__ __forceinline__ uint16_t f32_to_f16_rne(float x) {
  return __half_as_ushort(__float2half_rn(x));
}
__device__ __forceinline__ float f16_to_f32(uint16_t h) { return __half2float(__ushort_as_half(h)); }
// x to FP16 by adding r (0 <= r < 2^13) below the last significand bit of
// an FP16 normal number and clearing the FP32 bits below it: in the FP16
// normal range the result converts exactly, so x rounds away from zero
// with probability equal to its fraction of an ulp.  Below that range
// (|x| < 2^-14) the conversion rounds to nearest once more; infinity and
// NaN convert as they are.
__device__ __forceinline__ uint16_t f32_to_f16_sr(float x, uint32_t r) {
  const uint32_t u = __float_as_uint(x);
  if ((u & 0x7f800000u) == 0x7f800000u) return f32_to_f16_rne(x);
  return f32_to_f16_rne(__uint_as_float((u + r) & 0xffffe000u));
}

// 32 well-mixed bits from three words and a small tag: each word enters
// through a multiply by an odd constant, then the lowbias32 finalizer
// (C. Wellons, "Prospecting for hash functions", 2018).
__device__ __forceinline__ uint32_t rand_bits(uint32_t a, uint32_t b, uint32_t c, uint32_t tag) {
  uint32_t h = a * 0x9e3779b1u + b * 0x85ebca77u + c * 0xc2b2ae3du + tag * 0x27d4eb2fu;
  h ^= h >> 16;
  h *= 0x7feb352du;
  h ^= h >> 15;
  h *= 0x846ca68bu;
  h ^= h >> 16;
  return h;
}

template <class T>
__device__ __forceinline__ T ldg(const void *p, int64_t k) {
  return static_cast<const T *>(p)[k];
}
// Store; NT: a nontemporal store (data written once and not read again in
// the launch: the final state of a two-step pass).
template <class T, bool NT = false>
__device__ __forceinline__ void stg(void *p, int64_t k, T v) {
  if constexpr (NT)
    __builtin_nontemporal_store(v, static_cast<T *>(p) + k);
  else
    static_cast<T *>(p)[k] = v;
}

// One rounding for x y + z.  Used only where x is a power of two: the product is
// then exact and the result that of the separate operations, but for products of
// 0.25 and 0.5 in the denormal range, where those round twice.  Fields below 1e-37
// (FP32; 1e-307 in FP64) then end in other last bits than separately rounded sums,
// and the far field of a pulse carries that on: after 20 to 50 steps results differ
// by 1e-20 of the field in BF16DEV, whose rounding hash reads those bits, by 3e-32
// or less in the other FP32 storages.  Errors against FP64 are as before: over 40
// runs of plates with a hole (14 seeds, 1024^2 to 8192^2, 1000 to 4000 steps), fused
// over separate, geometric means BF16DEV 0.996 (single runs 0.93 to 1.09), FP32,
// F32DEV and F16DEV 0.999 to 1.000.  (Separate: 16-bit storages 1.4 to 2.7 % slower, the
// others 0 to 1.4.)  Every launch uses the same forms, so block passes and tile
// launches agree in all bits.
__device__ __forceinline__ double fma1(double x, double y, double z) { return __builtin_fma(x, y, z); }
__device__ __forceinline__ float fma1(float x, float y, float z) { return __builtin_fmaf(x, y, z); }

template <class C>
__device__ __forceinline__ void eq_populations(C a0, C a, C rho, C jx, C jy, C f[5]) {
  const C ar = a * rho;
  f[0] = a0 * rho;
  f[1] = fma1(C(0.5), jx, ar);
  f[2] = fma1(C(0.5), jy, ar);
  f[3] = fma1(C(-0.5), jx, ar);
  f[4] = fma1(C(-0.5), jy, ar);
}

// Post-collision populations f* = f - 2 (f - f_eq(f)) and zeroth moment of
// one field (eq. LBE with dt/tau = 2).
template <class C>
__device__ __forceinline__ void collide_populations(C a0, C a, const C f[5], C &rho, C fs[5]) {
  const C r = f[0] + ((f[1] + f[3]) + (f[2] + f[4]));
  const C jx = f[1] - f[3], jy = f[2] - f[4];
  C e[5];
  eq_populations<C>(a0, a, r, jx, jy, e);
#pragma unroll
  for (int q = 0; q < 5; q++) fs[q] = fma1(C(-2.0), f[q] - e[q], f[q]);
  rho = r;
}

// Plain populations, FP64 or FP32.
template <class T>
struct PopCodec {
  using C = T;
  using U = T;
  using Slot = T;  // raw stored word of one slot
  __device__ static void load_raw(const DevState &s, int b, int fl, int64_t k, Slot r[5]) {
#pragma unroll
    for (int q = 0; q < 5; q++) r[q] = ldg<T>(s.pop[b][fl][q], k);
  }
  __device__ static void raw_to_pops(const PlateDev &, int, const Slot r[5], C f[5]) {
#pragma unroll
    for (int q = 0; q < 5; q++) f[q] = r[q];
  }
  __device__ static void raw_flux(const Slot r[5], C &jx, C &jy) {
    jx = r[1] - r[3];
    jy = r[2] - r[4];
  }
  __device__ static C raw_rho(const Slot r[5]) { return r[0] + ((r[1] + r[3]) + (r[2] + r[4])); }
  // (a select of the two fields' values, not an index: fl may differ between
  // lanes, and an indexed plate record would have to live in scratch memory)
  __device__ static C aw(const PlateDev &P, int fl) { return (C)(fl ? P.a[1] : P.a[0]); }
  __device__ static C a0w(const PlateDev &P, int fl) { return (C)(fl ? P.a0[1] : P.a0[0]); }
  __device__ static void load(const DevState &s, int b, int fl, int64_t k, const PlateDev &,
                              C f[5]) {
#pragma unroll
    for (int q = 0; q < 5; q++) f[q] = ldg<T>(s.pop[b][fl][q], k);
  }
  template <bool NT = false>
  __device__ static void store(const DevState &s, int b, int fl, int64_t k, const PlateDev &,
                               const C f[5]) {
#pragma unroll
    for (int q = 0; q < 5; q++) stg<T, NT>(s.pop[b][fl][q], k, f[q]);
  }
  __device__ static void flux(const DevState &s, int b, int fl, int64_t k, const PlateDev &,
                              C &jx, C &jy) {
    jx = ldg<T>(s.pop[b][fl][1], k) - ldg<T>(s.pop[b][fl][3], k);
    jy = ldg<T>(s.pop[b][fl][2], k) - ldg<T>(s.pop[b][fl][4], k);
  }
  __device__ static void eq_pops(const PlateDev &P, int fl, C rho, C jx, C jy, C f[5]) {
    eq_populations<C>(a0w(P, fl), aw(P, fl), rho, jx, jy, f);
  }
  __device__ static void store_eq(const DevState &s, int b, int fl, int64_t k, const PlateDev &P,
                                  C rho, C jx, C jy) {
    C f[5];
    eq_pops(P, fl, rho, jx, jy, f);
    store(s, b, fl, k, P, f);
  }
  __device__ static double field(const DevState &s, int b, int fl, int64_t k, const PlateDev &P) {
    C f[5];
    load(s, b, fl, k, P, f);
    return (double)(f[0] + ((f[1] + f[3]) + (f[2] + f[4])));
  }
  // populations f as the words a store would leave in memory
  __device__ static void encode(const PlateDev &, int, const C f[5], Slot r[5]) {
#pragma unroll
    for (int q = 0; q < 5; q++) r[q] = f[q];
  }
  // the stored words of f_eq(rho, J = 0)
  __device__ static void eq_raw(const PlateDev &P, int fl, C rho, Slot r[5]) {
    eq_pops(P, fl, rho, C(0), C(0), r);
  }
  // the same with flux J
  __device__ static void eq_raw(const PlateDev &P, int fl, C rho, C jx, C jy, Slot r[5]) {
    eq_pops(P, fl, rho, jx, jy, r);
  }
  __device__ static void store_raw(const DevState &s, int b, int fl, int64_t k, const Slot r[5]) {
#pragma unroll
    for (int q = 0; q < 5; q++) stg<T>(s.pop[b][fl][q], k, r[q]);
  }
  // rho and f* of the stored populations r (eq. LBE)
  __device__ static void collide_raw(const PlateDev &P, int fl, const Slot r[5], C &rho,
                                     C fs[5]) {
    collide_populations<C>(a0w(P, fl), aw(P, fl), r, rho, fs);
  }
  // rho and f* of populations f as a store and a load would return them
  // (plain storage keeps them exactly)
  __device__ static void collide_stored(const PlateDev &P, int fl, const C f[5], C &rho,
                                        C fs[5]) {
    collide_populations<C>(a0w(P, fl), aw(P, fl), f, rho, fs);
  }
};

// Deviation from the local rest equilibrium in a moment basis:
// rho, J_x = f1 - f3, J_y = f2 - f4 in FP32; N = (f1 + f3) - (f2 + f4) and
// D = (f1 + f2 + f3 + f4) - 4 a rho in FP32 (H = 0) or in a 16-bit type
// (H = 1 FP16, H = 2 BF16) scaled by a power of two and packed in one word.
template <int H>
struct DevCodec {
  using C = float;
  using U = double;
  using Slot = uint32_t;  // raw stored word of one slot
  __device__ static C aw(const PlateDev &P, int fl) { return fl ? P.af[1] : P.af[0]; }
  __device__ static C a0w(const PlateDev &P, int fl) { return fl ? P.a0f[1] : P.a0f[0]; }
  __device__ static float scale(const PlateDev &P, int fl) { return fl ? P.scale[1] : P.scale[0]; }
  __device__ static float iscale(const PlateDev &P, int fl) {
    return fl ? P.iscale[1] : P.iscale[0];
  }
  __device__ static void unpack(uint32_t w, const PlateDev &P, int fl, float &n, float &d) {
    const uint16_t lo = (uint16_t)(w & 0xffffu), hi = (uint16_t)(w >> 16);
    if (H == 1) {
      n = f16_to_f32(lo) * iscale(P, fl);
      d = f16_to_f32(hi) * iscale(P, fl);
    } else {
      n = bf16_to_f32(lo) * iscale(P, fl);
      d = bf16_to_f32(hi) * iscale(P, fl);
    }
  }
  // N = m[3] and D = m[4] in the 16-bit type, rounded stochastically:
  // each value rounds away from zero with probability equal to its fraction
  // of an ulp, so the rounding errors are unbiased and uncorrelated from
  // step to step (round-to-nearest leaves nearly the same error on a slowly
  // varying moment step after step, and those errors add up).  The random
  // bits are a hash of the node's stored rho and J, whose low bits change
  // from step to step, so the stored state stays a function of the state
  // it comes from (every tiling and launch shape gives the same bits).
  __device__ static uint32_t pack(const float m[5], const PlateDev &P, int fl) {
    const float sn = m[3] * scale(P, fl), sd = m[4] * scale(P, fl);
    uint16_t lo, hi;
    const uint32_t r = rand_bits(__float_as_uint(m[0]), __float_as_uint(m[1]),
                                 __float_as_uint(m[2]), (uint32_t)fl);
    if (H == 1) {
      lo = f32_to_f16_sr(sn, r & 0x1fffu);
      hi = f32_to_f16_sr(sd, (r >> 16) & 0x1fffu);
    } else {
      lo = f32_to_bf16_sr(sn, r & 0xffffu);
      hi = f32_to_bf16_sr(sd, r >> 16);
    }
    return (uint32_t)lo | ((uint32_t)hi << 16);
  }
  __device__ static void load_moments(const DevState &s, int b, int fl, int64_t k,
                                      const PlateDev &P, float m[5]) {
    m[0] = ldg<float>(s.pop[b][fl][0], k);
    m[1] = ldg<float>(s.pop[b][fl][1], k);
    m[2] = ldg<float>(s.pop[b][fl][2], k);
    if (H == 0) {
      m[3] = ldg<float>(s.pop[b][fl][3], k);
      m[4] = ldg<float>(s.pop[b][fl][4], k);
    } else {
      unpack(ldg<uint32_t>(s.pop[b][fl][3], k), P, fl, m[3], m[4]);
    }
  }
  __device__ static void load_raw(const DevState &s, int b, int fl, int64_t k, Slot r[5]) {
    r[0] = ldg<uint32_t>(s.pop[b][fl][0], k);
    r[1] = ldg<uint32_t>(s.pop[b][fl][1], k);
    r[2] = ldg<uint32_t>(s.pop[b][fl][2], k);
    r[3] = ldg<uint32_t>(s.pop[b][fl][3], k);
    r[4] = H == 0 ? ldg<uint32_t>(s.pop[b][fl][4], k) : 0u;
  }
  __device__ static void raw_flux(const Slot r[5], C &jx, C &jy) {
    jx = __uint_as_float(r[1]);
    jy = __uint_as_float(r[2]);
  }
  __device__ static C raw_rho(const Slot r[5]) { return __uint_as_float(r[0]); }
  __device__ static void raw_to_pops(const PlateDev &P, int fl, const Slot r[5], C f[5]) {
    float m[5];
    m[0] = __uint_as_float(r[0]);
    m[1] = __uint_as_float(r[1]);
    m[2] = __uint_as_float(r[2]);
    if (H == 0) {
      m[3] = __uint_as_float(r[3]);
      m[4] = __uint_as_float(r[4]);
    } else {
      unpack(r[3], P, fl, m[3], m[4]);
    }
    moments_to_pops(P, fl, m, f);
  }
  __device__ static void moments_to_pops(const PlateDev &P, int fl, const float m[5], C f[5]) {
    const float q = m[4] + 4.0f * aw(P, fl) * m[0];
    // f1 = ((q + N) / 2 + J_x) / 2 and so on (the halves are exact)
    const float t13 = q + m[3], t24 = q - m[3];
    const float hx = 0.5f * m[1], hy = 0.5f * m[2];
    f[0] = m[0] - q;
    f[1] = fma1(0.25f, t13, hx);
    f[3] = fma1(0.25f, t13, -hx);
    f[2] = fma1(0.25f, t24, hy);
    f[4] = fma1(0.25f, t24, -hy);
  }
  __device__ static void load(const DevState &s, int b, int fl, int64_t k, const PlateDev &P,
                              C f[5]) {
    float m[5];
    load_moments(s, b, fl, k, P, m);
    moments_to_pops(P, fl, m, f);
  }
  template <bool NT = false>
  __device__ static void store_moments(const DevState &s, int b, int fl, int64_t k,
                                       const PlateDev &P, const float m[5]) {
    stg<float, NT>(s.pop[b][fl][0], k, m[0]);
    stg<float, NT>(s.pop[b][fl][1], k, m[1]);
    stg<float, NT>(s.pop[b][fl][2], k, m[2]);
    if (H == 0) {
      stg<float, NT>(s.pop[b][fl][3], k, m[3]);
      stg<float, NT>(s.pop[b][fl][4], k, m[4]);
    } else {
      stg<uint32_t, NT>(s.pop[b][fl][3], k, pack(m, P, fl));
    }
  }
  template <bool NT = false>
  __device__ static void store(const DevState &s, int b, int fl, int64_t k, const PlateDev &P,
                               const C f[5]) {
    const float s13 = f[1] + f[3], s24 = f[2] + f[4];
    const float q = s13 + s24;
    float m[5];
    m[0] = f[0] + q;
    m[1] = f[1] - f[3];
    m[2] = f[2] - f[4];
    m[3] = s13 - s24;
    m[4] = q - 4.0f * aw(P, fl) * m[0];
    store_moments<NT>(s, b, fl, k, P, m);
  }
  __device__ static void flux(const DevState &s, int b, int fl, int64_t k, const PlateDev &,
                              C &jx, C &jy) {
    jx = ldg<float>(s.pop[b][fl][1], k);
    jy = ldg<float>(s.pop[b][fl][2], k);
  }
  __device__ static void eq_pops(const PlateDev &P, int fl, C rho, C jx, C jy, C f[5]) {
    const float m[5] = {rho, jx, jy, 0.0f, 0.0f};
    moments_to_pops(P, fl, m, f);
  }
  __device__ static void store_eq(const DevState &s, int b, int fl, int64_t k, const PlateDev &P,
                                  C rho, C jx, C jy) {
    const float m[5] = {rho, jx, jy, 0.0f, 0.0f};
    store_moments(s, b, fl, k, P, m);
  }
  __device__ static double field(const DevState &s, int b, int fl, int64_t k, const PlateDev &) {
    return (double)ldg<float>(s.pop[b][fl][0], k);
  }
  // The collision in the moment basis: rho and J are kept and the two
  // non-equilibrium moments N and D change sign (f* = 2 f_eq - f with
  // f_eq of rho and J, eq. LBE with dt/tau = 2), so rho is conserved
  // exactly whatever the rounding of the weights.
  __device__ static void post_collision(const PlateDev &P, int fl, const float m[5], C &rho,
                                        C fs[5]) {
    const float mc[5] = {m[0], m[1], m[2], -m[3], -m[4]};
    moments_to_pops(P, fl, mc, fs);
    rho = m[0];
  }
  // populations f as the words a store would leave in memory
  __device__ static void encode(const PlateDev &P, int fl, const C f[5], Slot r[5]) {
    const float s13 = f[1] + f[3], s24 = f[2] + f[4];
    const float q = s13 + s24;
    float m[5];
    m[0] = f[0] + q;
    m[1] = f[1] - f[3];
    m[2] = f[2] - f[4];
    m[3] = s13 - s24;
    m[4] = q - 4.0f * aw(P, fl) * m[0];
    r[0] = __float_as_uint(m[0]);
    r[1] = __float_as_uint(m[1]);
    r[2] = __float_as_uint(m[2]);
    r[3] = H == 0 ? __float_as_uint(m[3]) : pack(m, P, fl);
    r[4] = H == 0 ? __float_as_uint(m[4]) : 0u;
  }
  // the stored words of f_eq(rho, J = 0) (both deviation moments are 0)
  __device__ static void eq_raw(const PlateDev &, int, C rho, Slot r[5]) {
    r[0] = __float_as_uint(rho);
    r[1] = r[2] = r[3] = r[4] = 0u;
  }
  __device__ static void eq_raw(const PlateDev &, int, C rho, C jx, C jy, Slot r[5]) {
    r[0] = __float_as_uint(rho);
    r[1] = __float_as_uint(jx);
    r[2] = __float_as_uint(jy);
    r[3] = r[4] = 0u;
  }
  __device__ static void store_raw(const DevState &s, int b, int fl, int64_t k, const Slot r[5]) {
#pragma unroll
    for (int q = 0; q < (H == 0 ? 5 : 4); q++) stg<uint32_t>(s.pop[b][fl][q], k, r[q]);
  }
  // rho and f* of the stored moments r
  __device__ static void collide_raw(const PlateDev &P, int fl, const Slot r[5], C &rho,
                                     C fs[5]) {
    float m[5];
    m[0] = __uint_as_float(r[0]);
    m[1] = __uint_as_float(r[1]);
    m[2] = __uint_as_float(r[2]);
    if (H == 0) {
      m[3] = __uint_as_float(r[3]);
      m[4] = __uint_as_float(r[4]);
    } else {
      unpack(r[3], P, fl, m[3], m[4]);
    }
    post_collision(P, fl, m, rho, fs);
  }
  // rho and f* of populations f as store() followed by a load returns them:
  // the same moments and rounding, without the memory
  __device__ static void collide_stored(const PlateDev &P, int fl, const C f[5], C &rho,
                                        C fs[5]) {
    const float s13 = f[1] + f[3], s24 = f[2] + f[4];
    const float q = s13 + s24;
    float m[5];
    m[0] = f[0] + q;
    m[1] = f[1] - f[3];
    m[2] = f[2] - f[4];
    m[3] = s13 - s24;
    m[4] = q - 4.0f * aw(P, fl) * m[0];
    if (H != 0) unpack(pack(m, P, fl), P, fl, m[3], m[4]);
    post_collision(P, fl, m, rho, fs);
  }
};

template <int ST>
struct CodecOf;
template <>
struct CodecOf<LBM_STORE_F64> {
  using type = PopCodec<double>;
};
template <>
struct CodecOf<LBM_STORE_F32> {
  using type = PopCodec<float>;
};
template <>
struct CodecOf<LBM_STORE_F32DEV> {
  using type = DevCodec<0>;
};
template <>
struct CodecOf<LBM_STORE_F16DEV> {
  using type = DevCodec<1>;
};
template <>
struct CodecOf<LBM_STORE_BF16DEV> {
  using type = DevCodec<2>;
};

// --------------------------------------------------------- node geometry

__device__ __forceinline__ int64_t node_of(const PlateDev &P, int i, int j) {
  return P.off + (int64_t)j * P.pitch + i;
}
__device__ __forceinline__ int wrapc(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// Finite-difference derivative of q along axis ax at body node (i, j), per
// axis: central if both neighbours are in the body, else the one-sided
// 3-point second-order formula, else 2-point first order, else 0.  The
// neighbour bits of the class byte already account for periodic wrapping.
template <class U>
__device__ U fd_axis(const DevState &s, const U *q, const PlateDev &P, int i, int j, int ax) {
  const int64_t k0 = node_of(P, i, j);
  const uint8_t c0 = s.cls[k0];
  const uint8_t bp = ax == 0 ? NB_E : NB_N, bm = ax == 0 ? NB_W : NB_S;
  const int di = ax == 0 ? 1 : 0, dj = ax == 0 ? 0 : 1;
  const U h = (U)P.dh;
  const bool hp = (c0 & bp) != 0, hm = (c0 & bm) != 0;
  if (hp && hm) {
    const int64_t kp = node_of(P, wrapc(i + di, P.nx), wrapc(j + dj, P.ny));
    const int64_t km = node_of(P, wrapc(i - di, P.nx), wrapc(j - dj, P.ny));
    return (q[kp] - q[km]) / (U(2.0) * h);
  }
  if (hp) {
    const int ip = wrapc(i + di, P.nx), jp = wrapc(j + dj, P.ny);
    const int64_t kp = node_of(P, ip, jp);
    if (s.cls[kp] & bp) {
      const int64_t kpp = node_of(P, wrapc(ip + di, P.nx), wrapc(jp + dj, P.ny));
      return ((U(-3.0) * q[k0] + U(4.0) * q[kp]) - q[kpp]) / (U(2.0) * h);
    }
    return (q[kp] - q[k0]) / h;
  }
  if (hm) {
    const int im = wrapc(i - di, P.nx), jm = wrapc(j - dj, P.ny);
    const int64_t km = node_of(P, im, jm);
    if (s.cls[km] & bm) {
      const int64_t kmm = node_of(P, wrapc(im - di, P.nx), wrapc(jm - dj, P.ny));
      return ((U(3.0) * q[k0] - U(4.0) * q[km]) + q[kmm]) / (U(2.0) * h);
    }
    return (q[k0] - q[km]) / h;
  }
  return U(0.0);
}

// div u and (curl u).e_z (Sec. 2, eq. phi-psi) by finite differences.
template <class U>
__device__ void div_curl(const DevState &s, int b, const PlateDev &P, int i, int j, U &dv, U &cu) {
  const U *ux = static_cast<const U *>(s.u[b][0]);
  const U *uy = static_cast<const U *>(s.u[b][1]);
  const U dxux = fd_axis<U>(s, ux, P, i, j, 0), dyuy = fd_axis<U>(s, uy, P, i, j, 1);
  const U dxuy = fd_axis<U>(s, uy, P, i, j, 0), dyux = fd_axis<U>(s, ux, P, i, j, 1);
  dv = dxux + dyuy;
  cu = dxuy - dyux;
}

__device__ inline double load_amp(const DevState &s, int li, double t) {
  if (li < 0) return 1.0;
  const LoadTable &L = s.loads[li];
  const int n = L.n;
  if (n <= 0) return 1.0;
  if (t <= L.t[0]) return L.g[0];
  if (t >= L.t[n - 1]) return L.g[n - 1];
  for (int m = 0; m + 1 < n; m++) {
    if (t <= L.t[m + 1]) {
      const double w = (t - L.t[m]) / (L.t[m + 1] - L.t[m]);
      return L.g[m] + w * (L.g[m + 1] - L.g[m]);
    }
  }
  return L.g[n - 1];
}

// Collision of populations that are not a stored state (the averaged
// populations of the second-row rule).
template <class CD>
__device__ __forceinline__ void collide_pops(const PlateDev &P, int fl, const typename CD::C f[5],
                                             typename CD::C &rho, typename CD::C fs[5]) {
  collide_populations<typename CD::C>(CD::a0w(P, fl), CD::aw(P, fl), f, rho, fs);
}

// ------------------------------------------- boundary / second-row work

// Finite difference with a precomputed stencil code from the node's value
// q0 and the values qa, qb of the further stencil nodes, branch-free:
// ((c0 q0 + ca qa) + cb qb) * scale with the coefficients of the code
// (central: qa - qb, one-sided 3-point: (-3 q0 + 4 qa) - qb and its mirror,
// 2-point: qa - q0 and q0 - qa; these sums round exactly as the written-out
// formulas); scale is 1/(2 dh) or 1/dh.
template <class U>
__device__ __forceinline__ U fd_vals(int code, U q0, U qa, U qb, const PlateDev &P) {
  const bool cen = code == FD_CENTRAL, f3 = code == FD_FWD3, b3 = code == FD_BWD3;
  const bool f2 = code == FD_FWD2, b2 = code == FD_BWD2;
  const U c0 = f3 ? U(-3.0) : b3 ? U(3.0) : f2 ? U(-1.0) : b2 ? U(1.0) : U(0.0);
  const U ca = (cen || f2) ? U(1.0) : f3 ? U(4.0) : b3 ? U(-4.0) : b2 ? U(-1.0) : U(0.0);
  const U cb = (cen || f3) ? U(-1.0) : b3 ? U(1.0) : U(0.0);
  const U sc = (f2 || b2) ? (U)P.inv_h : (cen || f3 || b3) ? (U)P.inv_2h : U(0.0);
  return ((c0 * q0 + ca * qa) + cb * qb) * sc;
}

// Further stencil nodes a and b of a finite difference with code `code`
// along axis ax at node (i, j) (the node k0 itself where the stencil has no
// such node).  Every index touched lies in the body (the code was built from
// the mask).
__device__ __forceinline__ void fd_nodes(const PlateDev &P, int i, int j, int ax, int code,
                                         int64_t k0, int64_t &ka, int64_t &kb) {
  const int di = ax == 0 ? 1 : 0, dj = ax == 0 ? 0 : 1;
  ka = k0;
  kb = k0;
  if (code == FD_CENTRAL || code == FD_FWD3 || code == FD_FWD2) {
    const int ip = wrapc(i + di, P.nx), jp = wrapc(j + dj, P.ny);
    ka = node_of(P, ip, jp);
    if (code == FD_CENTRAL) kb = node_of(P, wrapc(i - di, P.nx), wrapc(j - dj, P.ny));
    if (code == FD_FWD3) kb = node_of(P, wrapc(ip + di, P.nx), wrapc(jp + dj, P.ny));
  } else if (code == FD_BWD3 || code == FD_BWD2) {
    const int im = wrapc(i - di, P.nx), jm = wrapc(j - dj, P.ny);
    ka = node_of(P, im, jm);
    if (code == FD_BWD3) kb = node_of(P, wrapc(im - di, P.nx), wrapc(jm - dj, P.ny));
  }
}

// The values of q that the finite differences along x (code cx) and y
// (code cy) at node (i, j) combine, read straight from q: v[0] at the node,
// v[1], v[2] the x stencil's nodes a, b, v[3], v[4] the y stencil's (fd_vals
// of (v[0], v[1], v[2]) is d/dx, of (v[0], v[3], v[4]) d/dy).
template <class U>
__device__ __forceinline__ void fd_stencil_values(const U *q, const PlateDev &P, int i, int j,
                                                  int cx, int cy, U v[5]) {
  const int64_t k0 = node_of(P, i, j);
  int64_t xa, xb, ya, yb;
  fd_nodes(P, i, j, 0, cx, k0, xa, xb);
  fd_nodes(P, i, j, 1, cy, k0, ya, yb);
  v[0] = q[k0];
  v[1] = q[xa];
  v[2] = q[xb];
  v[3] = q[ya];
  v[4] = q[yb];
}

// Hooke's law (Sec. 2, eq. hooke) from a displacement gradient
// g = (d_x u_x, d_y u_x, d_x u_y, d_y u_y).
template <class U>
__device__ __forceinline__ void hooke(const PlateDev &P, const U *g, U &sxx, U &syy, U &sxy) {
  const U exx = g[0], eyy = g[3];
  const U exy = U(0.5) * (g[1] + g[2]);
  const U tr = exx + eyy;
  const U lam = (U)P.lam, mu = (U)P.mu;
  sxx = lam * tr + U(2.0) * mu * exx;
  syy = lam * tr + U(2.0) * mu * eyy;
  sxy = U(2.0) * mu * exy;
}

// Displacement update of step n from u, v and the acceleration a at t_n,
// as u += dt v + m a, v += k a with step coefficients (k, m):
// integ 0, eq. integration as printed: k = dt, m = dt^2/2.
// integ 1, central difference (Newmark gamma = 1/2, beta = 0) in
// half-step form (v kept at t - dt/2: v += dt a, then u += dt v): k = dt,
// m = dt^2; the first step (n = 0, v given at t = 0) takes half the velocity
// increment, k = dt/2, m = dt^2/2, which gives the same u(t_1) as the
// printed update.  The coefficients are uniform over a launch.
template <class U>
struct Kick {
  U k, m;
};
template <class U>
__device__ __forceinline__ Kick<U> kick_of(const PlateDev &P, bool first) {
  const U dt = (U)P.dt;
  if (P.integ) {
    const U k = first ? U(0.5) * dt : dt;
    return {k, dt * k};
  }
  return {dt, dt * dt / U(2.0)};
}
template <class U>
__device__ __forceinline__ void newmark(const PlateDev &P, const Kick<U> &K, U ax, U ay, U ux,
                                        U uy, U vx, U vy, U &nux, U &nuy, U &nvx, U &nvy) {
  const U dt = (U)P.dt;
  nux = ux + dt * vx + K.m * ax;
  nuy = uy + dt * vy + K.m * ay;
  nvx = vx + K.k * ax;
  nvy = vy + K.k * ay;
}

// Interior acceleration of eq. navier, c_d^2 grad phi - c_s^2 curl(psi e_z)
// with curl(psi e_z) = (d_y psi, -d_x psi) and central differences of the
// neighbours' zeroth moments (E, W, N, S; field 0 = phi, 1 = psi), followed
// by the displacement update with coefficients K.  Shared by the interior kernel
// and the boundary kernel's recomputation so both give identical values.
// Differences are scaled by the precomputed 1/(2 dh) (exact for dh = 1).
template <class U>
__device__ __forceinline__ void interior_update(const PlateDev &P, const Kick<U> &K, U e0, U w0,
                                                U n0, U s0, U e1, U w1, U n1, U s1, U ux, U uy,
                                                U vx, U vy, U &nux, U &nuy, U &nvx, U &nvy) {
  const U i2h = (U)P.inv_2h;
  const U cd2 = (U)P.cd2, cs2 = (U)P.cs2;
  const U dphix = (e0 - w0) * i2h;
  const U dphiy = (n0 - s0) * i2h;
  const U dpsix = (e1 - w1) * i2h;
  const U dpsiy = (n1 - s1) * i2h;
  const U ax = cd2 * dphix - cs2 * dpsiy;
  const U ay = cd2 * dphiy - cs2 * (-dpsix);
  newmark<U>(P, K, ax, ay, ux, uy, vx, vy, nux, nuy, nvx, nvy);
}

// Boundary acceleration of eq. acc_neumann: own stress s (xx, yy, xy), the
// stresses r of the body neighbours E, N, W, S (has: the neighbour is in the
// body), external force (Fx, Fy), cell lengths l and volume V.  sigma_kr is
// the mean of the two nodal stresses.
template <class U>
__device__ __forceinline__ void neumann_accel(const PlateDev &P, const U s[3], const bool has[4],
                                              const U r[4][3], U V, const U l[4], U Fx, U Fy,
                                              U &ax, U &ay) {
  U tEx = 0, tEy = 0, tWx = 0, tWy = 0, tNx = 0, tNy = 0, tSx = 0, tSy = 0;
  if (has[0]) {
    tEx = U(0.5) * (s[0] + r[0][0]) * l[0];
    tEy = U(0.5) * (s[2] + r[0][2]) * l[0];
  }
  if (has[2]) {
    tWx = -(U(0.5) * (s[0] + r[2][0])) * l[2];
    tWy = -(U(0.5) * (s[2] + r[2][2])) * l[2];
  }
  if (has[1]) {
    tNx = U(0.5) * (s[2] + r[1][2]) * l[1];
    tNy = U(0.5) * (s[1] + r[1][1]) * l[1];
  }
  if (has[3]) {
    tSx = -(U(0.5) * (s[2] + r[3][2])) * l[3];
    tSy = -(U(0.5) * (s[1] + r[3][1])) * l[3];
  }
  const U m = (U)P.rho_m * V;
  ax = (((tEx + tWx) + (tNx + tSx)) + Fx) / m;
  ay = (((tEy + tWy) + (tNy + tSy)) + Fy) / m;
}

// Boundary acceleration of eq. acc_dirichlet: the one that makes u(t + dt) =
// u* under the update in use (n: the step).
template <class U>
__device__ __forceinline__ void dirichlet_accel(const PlateDev &P, unsigned long long n, U usx,
                                                U usy, U ux, U uy, U vx, U vy, U &ax, U &ay) {
  const U dt = (U)P.dt;
  if (P.integ && n != 0) {
    ax = (usx - ux) / (dt * dt) - vx / dt;
    ay = (usy - uy) / (dt * dt) - vy / dt;
  } else {
    ax = U(2.0) / (dt * dt) * (usx - ux) - U(2.0) / dt * vx;
    ay = U(2.0) / (dt * dt) * (usy - uy) - U(2.0) / dt * vy;
  }
}

__device__ __forceinline__ int tile_index(int b, int q) { return (b & 7) * q + (b >> 3); }

}  // namespace lbm

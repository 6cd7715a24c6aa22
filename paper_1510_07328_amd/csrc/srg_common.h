// Shared device code of the surrogate's kernels: operand types, GELU and its
// table, the input features.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <type_traits>

#include "lds_limit.h"

namespace srg {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

constexpr int CH = 64;
constexpr int KT = 5;
constexpr float FS = 0.25f;       // feature scale
constexpr float TAU_C = 0.75f;    // tau centre

// erf by Abramowitz & Stegun, Handbook of Mathematical Functions (1964), formula
// 7.1.26 (Hastings' approximation): for x >= 0,
//   erf(x) = 1 - t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) exp(-x^2),  t = 1 / (1 + p x),
// with an absolute error of at most 1.5e-7 (far below the bfloat16 rounding the
// activations then take); odd extension for x < 0.  exp(-x^2) is shared with GELU'.
struct ErfExp {
    float erf, e;  // erf(x) and exp(-x^2)
};
__device__ __forceinline__ ErfExp erf_exp(float x) {
    const float ax = __builtin_fabsf(x);
    const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.3275911f, ax, 1.0f));
    float p = __builtin_fmaf(1.061405429f, t, -1.453152027f);
    p = __builtin_fmaf(p, t, 1.421413741f);
    p = __builtin_fmaf(p, t, -0.284496736f);
    p = __builtin_fmaf(p, t, 0.254829592f);
    const float e = __builtin_amdgcn_exp2f(-ax * ax * 1.4426950408889634f);
    const float r = __builtin_fmaf(-p * t, e, 1.0f);
    return {__builtin_copysignf(r, x), e};
}
// GELU(z) = z Phi(z) = z (1 + erf(z / sqrt 2)) / 2
__device__ __forceinline__ float gelu(float z) {
    return 0.5f * z * (1.0f + erf_exp(z * 0.70710678118654752f).erf);
}
__device__ __forceinline__ __bf16 to_bf(float v) { return (__bf16)v; }
__device__ __forceinline__ float to_f(__bf16 v) { return (float)v; }

// bf16(GELU(z)) for a bfloat16 z by table: the forward rounds z to bfloat16
// before the GELU, so the result is a function of 16 bits.  A table covers the
// NE biased exponents E0 .. E0 + NE - 1 of both signs (2 NE 128 entries) and is
// written by gelu() itself, so a lookup gives the bits the computation gives;
// values outside it (smaller or larger magnitudes, zero, non-finite) are
// computed.  GeluT16: |z| in [2^-12, 16), 4096 entries, 8 KB of LDS (the layer-1
// kernel); GeluT32: |z| in [2^-24, 128), 8192 entries, 16 KB (the fused kernel,
// where a wavefront takes the computed path for all its values as soon as one
// lane holds a value outside the table: with the trained weights about 1 % of
// the pre-activations of layers 1-2 lie below 2^-12, and on strong shocks up to
// 17 % of layer 3's reach 16 and beyond (up to 62), so that with the smaller
// table nearly every wavefront took that path).
template <int E0, int NE>
struct GeluTable {
    static constexpr int HALF = NE * 128, N = 2 * HALF, BIAS = E0 << 7;
    static_assert(HALF == 0x800 || HALF == 0x1000, "the index's sign bit is bit 11 or 12");
    // writes the table with all threads of the workgroup; the two signs of a
    // magnitude share its error function
    static __device__ __forceinline__ void fill(unsigned short *tab) {
        for (int i = threadIdx.x; i < HALF; i += blockDim.x) {
            const float z = to_f(__builtin_bit_cast(__bf16, (unsigned short)((E0 << 7) + i)));
            const float e = erf_exp(z * 0.70710678118654752f).erf;
            tab[i] = __builtin_bit_cast(unsigned short, to_bf(0.5f * z * (1.0f + e)));
            tab[HALF + i] = __builtin_bit_cast(unsigned short, to_bf(0.5f * -z * (1.0f - e)));
        }
    }
    static __device__ __forceinline__ bool lookup(__bf16 z, unsigned *index) {
        const unsigned bits = __builtin_bit_cast(unsigned short, z);
        const unsigned t = (bits & 0x7fffu) - (unsigned)(E0 << 7);
        *index = t + (bits >> 15) * HALF;
        return t < (unsigned)HALF;
    }
};
using GeluT16 = GeluTable<115, 16>;
using GeluT32 = GeluTable<103, 32>;

// GELU of bfloat16 pairs (32-bit words, low half first) by table, the index
// formed by 16-bit packed operations: per half t = (z & 0x7fff) - (E0 << 7), in
// the table when t < HALF, entry t + HALF sign.
typedef unsigned short us2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned pack_bf2(float x, float y) {
    const bf16x2 v = {to_bf(x), to_bf(y)};
    return __builtin_bit_cast(unsigned, v);
}
// t of both halves
template <class Tab>
__device__ __forceinline__ unsigned gelu_bf2_t(unsigned z) {
    return __builtin_bit_cast(unsigned, __builtin_bit_cast(us2, z & 0x7fff7fffu) - (us2)((unsigned short)Tab::BIAS));
}
// v[i] from the table for every value, every read issued before any result is
// used; the index is taken within the table, so a value outside it reads some
// entry and must be replaced (gelu_bf2_outside, gelu_bf2_word)
template <class Tab, int N>
__device__ __forceinline__ void gelu_bf2_table(const unsigned (&z)[N], unsigned (&v)[N], const unsigned short *tab) {
    constexpr unsigned H = Tab::HALF;
    constexpr unsigned LOW = (H - 1u) * 0x10001u;  // t within the table
    constexpr unsigned SIGN = H * 0x10001u;        // the index's sign bit
    constexpr unsigned SH = H == 0x800 ? 4u : 3u;  // bit 15 -> that bit
    const char *tb = reinterpret_cast<const char *>(tab);
    us2 e[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const unsigned idx = (gelu_bf2_t<Tab>(z[i]) & LOW) | ((z[i] >> SH) & SIGN);
        const unsigned off = __builtin_bit_cast(unsigned, __builtin_bit_cast(us2, idx) << (us2)(1));
        e[i].x = *reinterpret_cast<const unsigned short *>(tb + (off & 0xffffu));
        e[i].y = *reinterpret_cast<const unsigned short *>(tb + (off >> 16));
    }
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = __builtin_bit_cast(unsigned, e[i]);
}
// nonzero when some value of z lies outside the table
template <class Tab, int N>
__device__ __forceinline__ unsigned gelu_bf2_outside(const unsigned (&z)[N]) {
    unsigned any = 0u;
#pragma unroll
    for (int i = 0; i < N; ++i) any |= gelu_bf2_t<Tab>(z[i]);
    return any & ((0x10000u - Tab::HALF) * 0x10001u);
}
// one word, each half from the table or computed
template <class Tab>
__device__ __forceinline__ unsigned gelu_bf2_word(unsigned z, const unsigned short *tab) {
    unsigned short r[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const __bf16 zh = __builtin_bit_cast(__bf16, (unsigned short)(z >> (16 * h)));
        unsigned idx;
        r[h] = Tab::lookup(zh, &idx) ? tab[idx] : __builtin_bit_cast(unsigned short, to_bf(gelu(to_f(zh))));
    }
    return r[0] | ((unsigned)r[1] << 16);
}
// v[i] = bf16(GELU(.)) of z[i]: the table when no lane of the wave holds a value
// outside it, else each value from the table or computed
template <class Tab, int N>
__device__ __forceinline__ void gelu_bf2_n(const unsigned (&z)[N], unsigned (&v)[N], const unsigned short *tab) {
    if (__builtin_amdgcn_ballot_w64(gelu_bf2_outside<Tab>(z) != 0u) == 0) {
        gelu_bf2_table<Tab>(z, v, tab);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = gelu_bf2_word<Tab>(z[i], tab);
    }
}

// feature channel ci at position x of sample b (zero outside [0, L))
__device__ __forceinline__ float feature(const float *__restrict__ nu, const float *__restrict__ tau, int b, int L,
                                         int ci, int x) {
    if (x < 0 || x >= L) return 0.0f;
    if (ci == 0) return (nu[(int64_t)b * 2 * L + x] - 1.0f) / FS;
    if (ci == 1) return nu[(int64_t)b * 2 * L + L + x] / FS;
    return (tau[b] - TAU_C) / FS;
}

constexpr int RS = CH + 8;  // LDS row stride of a 64-channel activation row, in elements (144 bytes)

using lbm::kMaxDevices;
using lbm::LdsLimit;

// Compute units of the current device (cached per device).
inline int device_cus() {
    static std::mutex m;
    static int cus[kMaxDevices] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
    std::lock_guard<std::mutex> lock(m);
    if (cus[dev] == 0 && hipDeviceGetAttribute(&cus[dev], hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus[dev] = 0;
    return cus[dev];
}

}  // namespace srg

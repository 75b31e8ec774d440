// Device-side helpers shared by the kernels of libnsmi (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nsmi {

typedef __attribute__((__vector_size__(8 * sizeof(short)))) short bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef __attribute__((__vector_size__(4 * sizeof(double)))) double f64x4_t;

// round-to-nearest-even float -> bf16 bits
// FP32 -> BF16, round to nearest even (one v_cvt_pk_bf16_f32 on gfx950)
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Low BF16 part of the split v = hi + lo, hi = f2bf(v): lo = f2bf(v - hi) with
// the subtraction kept apart from whatever product produced v (a fused
// multiply-subtract would see the unrounded product instead of v).
__device__ __forceinline__ uint16_t bf16_lo(float v, uint16_t hi) {
#pragma clang fp contract(off)
    return f2bf(v - bf2f(hi));
}

// a b + c with the constant c taken from scalar registers: left to itself the
// compiler copies each constant of a polynomial to vector registers first, two
// moves per fused multiply-add
__device__ __forceinline__ double fma_const(double a, double b, double c) {
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
}

// 2^(x c), c = c_hi + c_lo, as 2^n p with p in [0.7, 1.42]: n = round(x c), the
// rest f by two fused multiply-adds, 2^f = 1 + f q(f) with q of degree 10
// interpolating (2^f - 1) / f at the Chebyshev nodes of [-1/2, 1/2] (error
// 2e-17).  |x c| < 2^31.
__device__ __forceinline__ double exp2_scaled(double x, double c_hi, double c_lo, int& n) {
    const double t = fma(x, c_hi, 0x1.8p52);
    const double m = t - 0x1.8p52;
    const double f = fma(x, c_lo, fma(x, c_hi, -m));
    n = __double2loint(t);
    double q = fma_const(f, 0x1.e9d40bd1335b2p-32, 0x1.e6064f626db12p-28);
    q = fma_const(q, f, 0x1.b524fadf5b6e0p-24);
    q = fma_const(q, f, 0x1.62bfd46f7ae0cp-20);
    q = fma_const(q, f, 0x1.ffcbfc6710084p-17);
    q = fma_const(q, f, 0x1.4309130972778p-13);
    q = fma_const(q, f, 0x1.5d87fe78a5272p-10);
    q = fma_const(q, f, 0x1.3b2ab6fba1dd0p-7);
    q = fma_const(q, f, 0x1.c6b08d704a0c2p-5);
    q = fma_const(q, f, 0x1.ebfbdff82c598p-3);
    q = fma_const(q, f, 0x1.62e42fefa39efp-1);
    return fma(q, f, 1.0);
}

// e^x (FP64) as 2^n p with p in [0.7, 1.42]: x = n ln 2 + r, r = rh - rl with
// rh exact, e^r = 1 + rh + (r^2 q(r) - rl) with q of degree 9 interpolating at
// the Chebyshev nodes of |r| <= ln(2)/2 (error 2e-17), what 1 + rh leaves over
// added to the small terms.  Error against 80-bit values, in 2^-53: rms 0.438, at
// most 1.09 (the library's 0.446 and 1.22; as 2^(x log2 e) in one polynomial
// 0.452 and 1.42).  |x| < 2^31.  exp_of takes 34 vector instructions, the
// library's exp 41.
__device__ __forceinline__ double exp_parts(double x, int& n) {
    const double t = fma(x, 0x1.71547652b82fep+0, 0x1.8p52);
    const double m = t - 0x1.8p52;
    const double rh = fma(m, -0x1.62e42fefa38p-1, x), rl = m * 0x1.ef35793c7673p-45;
    const double r = rh - rl;
    n = __double2loint(t);
    double q = fma_const(r, 0x1.af38a9b0ec855p-26, 0x1.289185613a3d6p-22);
    q = fma_const(q, r, 0x1.71de0dae63bb3p-19);
    q = fma_const(q, r, 0x1.a019b90d2ae7ap-16);
    q = fma_const(q, r, 0x1.a01a01a7c41d5p-13);
    q = fma_const(q, r, 0x1.6c16c1788bd90p-10);
    q = fma_const(q, r, 0x1.11111111109b3p-7);
    q = fma_const(q, r, 0x1.5555555553d63p-5);
    q = fma_const(q, r, 0x1.5555555555556p-3);
    q = fma(q, r, 0.5);
    const double one = 1.0 + rh, left = (1.0 - one) + rh;
    return one + (fma(r * r, q, -rl) + left);
}
__device__ __forceinline__ double exp_of(double x) {
    x = x > 800.0 ? 800.0 : x;                  // beyond, inf or 0 as well
    x = x < -800.0 ? -800.0 : x;
    int n;
    const double p = exp_parts(x, n);
    return ldexp(p, n);
}

// 1 / (1 + exp(-u)).  FP64: in 40 vector instructions instead of 53 with the
// library's exp and division, which are what bounds the layers' epilogues; u is
// held to [-700, 700] (outside, the sigmoid is 0 or 1 to 1e-304), a NaN stays
// one.  Error for normal arguments of scale 1 (0.1 to 30), in 2^-53: rms 0.665
// (0.585 to 0.739), at most 2.07 (2.42); with the library's exp and division
// 0.670 (0.589 to 0.740), 2.14 (2.42).
template <class T> __device__ __forceinline__ T sigmoid(T u);
template <> __device__ __forceinline__ double sigmoid<double>(double u) {
    u = u > 700.0 ? 700.0 : u;
    u = u < -700.0 ? -700.0 : u;
    int n;
    const double p = exp_parts(-u, n);
    const double d = 1.0 + __hiloint2double(__double2hiint(p) + (n << 20), __double2loint(p));
    // reciprocal: the hardware's estimate and two Newton steps
    double y = __builtin_amdgcn_rcp(d);
    y = fma(y, fma(-d, y, 1.0), y);
    return fma(y, fma(-d, y, 1.0), y);
}
// FP32: hardware exp2 and reciprocal (about 1 ulp each)
template <> __device__ __forceinline__ float sigmoid<float>(float u) {
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(u * -1.44269504088896341f));
}
// 10^y (output transform of log10-emulated spectra)
template <class T> __device__ __forceinline__ T exp10_of(T y);
// FP64: 2^(y log2 10), 28 instead of 42 vector instructions, and without the rounding
// of y ln 10; beyond the range of a double it overflows and underflows alike
template <> __device__ __forceinline__ double exp10_of<double>(double y) {
    y = y > 400.0 ? 400.0 : y;
    y = y < -400.0 ? -400.0 : y;
    int n;
    const double p = exp2_scaled(y, 0x1.a934f0979a371p+1, 0x1.7f2495fb7fa6dp-53, n);
    return ldexp(p, n);
}
// FP32: 10^y = 2^(p_hi + p_lo) with p_hi = fl(y log2 10) and p_lo its rounding
// residual (plus the residual of log2 10 itself), so that the argument
// rounding (up to |y log2 10| 2^-24) does not reach the result; then
// 2^p_lo = 1 + p_lo ln 2 to first order (|p_lo| < 1e-5)
template <> __device__ __forceinline__ float exp10_of<float>(float y) {
    const float c_hi = 3.321928024291992f, c_lo = 7.059536955011936e-08f;
    const float p_hi = y * c_hi;
    const float p_lo = fmaf(y, c_hi, -p_hi) + y * c_lo;
    return __builtin_amdgcn_exp2f(p_hi) * fmaf(p_lo, 0.6931471824645996f, 1.0f);
}

// gated activation (gamma + (1 - gamma) sigmoid(beta t)) t
template <class T> __device__ __forceinline__ T gated(T t, T beta, T gamma) {
    return (gamma + (T(1) - gamma) * sigmoid<T>(beta * t)) * t;
}

// ----------------------------------------------------------- reductions
template <class T> __device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
template <class T> __device__ __forceinline__ T wave_max(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// v of the lane that DPP control CTRL names, 0 where there is none or the row
// is not in ROWS
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_get(double v) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false));
}
// inclusive prefix sum over the wave: within rows of 16 lanes, then row totals
// (data-parallel moves: three instructions a step, no trip through the LDS unit)
__device__ __forceinline__ double wave_scan(double v) {
    v += dpp_get<0x111, 0xf>(v);
    v += dpp_get<0x112, 0xf>(v);
    v += dpp_get<0x114, 0xf>(v);
    v += dpp_get<0x118, 0xf>(v);
    v += dpp_get<0x142, 0xa>(v);
    v += dpp_get<0x143, 0xc>(v);
    return v;
}
__device__ __forceinline__ int wave_total(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return __builtin_amdgcn_readlane(v, 63);
}
// sum over the wave, the same in every lane
__device__ __forceinline__ double wave_total(double v) {
    v = wave_scan(v);
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                            __builtin_amdgcn_readlane(__double2loint(v), 63));
}

// block-wide sum; `red` is LDS scratch of >= blockDim.x/64 elements
template <class T> __device__ T block_sum(T v, T* red) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    v = wave_sum(v);
    __syncthreads();
    if (lane == 0) red[wid] = v;
    __syncthreads();
    T s = T(0);
    for (int i = 0; i < nw; ++i) s += red[i];
    return s;
}

// ---------------------------------------------------------- Philox4x64-10
struct u64x4 { uint64_t x[4]; };

__device__ __forceinline__ u64x4 philox4x64(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3,
                                            uint64_t k0, uint64_t k1) {
    const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
    const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        uint64_t hi0 = __umul64hi(M0, c0), lo0 = M0 * c0;
        uint64_t hi1 = __umul64hi(M1, c2), lo1 = M1 * c2;
        uint64_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
        k0 += W0; k1 += W1;
    }
    u64x4 o;
    o.x[0] = c0; o.x[1] = c1; o.x[2] = c2; o.x[3] = c3;
    return o;
}

__device__ __forceinline__ double u01(uint64_t w) { return (double)(w >> 11) * 0x1.0p-53; }

// draw q of the sequence (c1, c2, c3) under key (seed, stream): word q mod 4
// of Philox block q / 4 (picked by selects, not by a run-time array index,
// which would put the block in scratch memory)
__device__ __forceinline__ double philox_uniform(uint64_t seed, uint64_t stream, uint64_t c1,
                                                 uint64_t c2, uint64_t c3, uint64_t q) {
    const u64x4 b = philox4x64(q >> 2, c1, c2, c3, seed, stream);
    const int r = (int)(q & 3);
    return u01(r == 0 ? b.x[0] : r == 1 ? b.x[1] : r == 2 ? b.x[2] : b.x[3]);
}

// draws q and q + 1 (q even) of the sequence: one Philox block
__device__ __forceinline__ void philox_uniform_pair(uint64_t seed, uint64_t stream, uint64_t c1, uint64_t c2,
                                                    uint64_t c3, uint64_t q, double& a, double& b) {
    const u64x4 x = philox4x64(q >> 2, c1, c2, c3, seed, stream);
    const bool hi = (q & 2) != 0;
    a = u01(hi ? x.x[2] : x.x[0]);
    b = u01(hi ? x.x[3] : x.x[1]);
}

}  // namespace nsmi

// FP64 products on the int8 matrix cores (gfx950), for the wide emulator
// layers in the NS_FP64 form.
//
// Each operand row is scaled by a power of two over blocks of DG_K = 512
// inputs and rounded to a 55-bit integer v, |v| < 127 2^48, written as seven
// balanced base-256 digits (v = sum_i d_i 256^(6-i), d_i a signed byte).  The
// digit products d_i e_j with i + j <= 6 (28 of the 49) are summed by
// v_mfma_i32_32x32x32_i8 in one int32 accumulator per i + j, exactly: at most
// 7 x 512 products of 2^14 stay below 2^26.  The accumulators form
//   T = 2^24 (a0 2^24 + a1 2^16 + a2 2^8 + a3) + (a4 2^16 + a5 2^8 + a6)
// with one rounding, and the result is T times the two scales.  The dropped
// digit products are below 2^-54 of the operands' largest entries, less than
// the roundings of 512 FP64 multiply-adds: over the emulators' layers the
// error against extended precision is half that of the FP64 product.  Integer
// sums have no order, so a row's result does not depend on the batch, the
// tile or the launch shape.
//
// Why: v_mfma_f64_16x16x4f64 peaks at 73 TFLOP/s on this chip; the int8 pipe
// sustains 3400 TOPS on random digits (power bound), 121 TFLOP/s of 28-fold
// products.
#pragma once

#include "devutil.h"
#include "gemm_bf16.h"

#include <type_traits>

namespace nsmi {

typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i32x4_t;
typedef __attribute__((__vector_size__(16 * sizeof(int)))) int i32x16_t;

constexpr int DG_N = 7;                         // digits
constexpr int DG_K = 512;                       // inputs that share a scale
constexpr int DG_ROWS = 32;                     // rows of a workgroup
constexpr int DG_LDS = DG_K + 16;               // bytes per row of a digit plane in LDS (16-byte reads, conflict free)
constexpr int DG_PLANE = DG_ROWS * DG_LDS;      // bytes per digit plane

// v is computed here: the compiler otherwise moves the last steps of an
// activation behind the next tile's loop, to its use, and keeps the several
// values they start from in scratch memory meanwhile.
__device__ __forceinline__ void pin(double& v) { asm volatile("" : "+v"(v)); }

// Scale of a row from the high word of its largest magnitude: exponent e with
// max < 127/128 2^(e+1).  to_int: multiplier to the integer v; back: the
// factor of T (half of the 2^48 that T's integer weights leave out).
struct DigitScale {
    double to_int, back;
};
__device__ __forceinline__ DigitScale digit_scale(int max_hi) {
    const int ef = (max_hi + 0x4000) >> 20;                       // biased exponent
    const int e = max(ef, 64) - 1023;                             // below 2^-959: digits keep fewer bits
    DigitScale s;
    s.to_int = __longlong_as_double((long long)(54 - e + 1023) << 52);
    s.back = max_hi == 0 ? 0.0 : __longlong_as_double((long long)(e - 30 + 1023) << 52);
    if (ef >= 0x7ff) {                                            // infinity or NaN in the row
        s.to_int = 0.0;
        s.back = __longlong_as_double(0x7ff8000000000000ll);
    }
    return s;
}

// Seven balanced digits of x * to_int, least significant in byte 0.  The
// integer is taken in two parts, 2^24 H + L with |L| <= 2^23, each read from
// the low word of a sum with 1.5 2^52 (no conversions); 0x808080 added to both
// makes every byte but the top one unsigned, and the exclusive or signed.
__device__ __forceinline__ uint2 digits_of(double x, double to_int) {
    constexpr double MAGIC = 0x1.8p52 + 0x808080;
    const double v = x * to_int;
    const double y = fma(v, 0x1p-24, MAGIC);
    const double z = fma(y - MAGIC, -0x1p24, v) + MAGIC;
    const int h = __double2loint(y);
    const unsigned long long q = ((unsigned long long)(long long)h << 24) + (uint32_t)__double2loint(z);
    return make_uint2((uint32_t)q ^ 0x80808080u, (uint32_t)(q >> 32) ^ 0x00008080u);
}

// Bytes 0..3 of four words -> word b holds byte b of each (a 4 x 4 transpose).
__device__ __forceinline__ void byte_transpose(const uint32_t (&a)[4], uint32_t (&o)[4]) {
    const uint32_t p01 = __builtin_amdgcn_perm(a[1], a[0], 0x05010400u);   // a0.0 a1.0 a0.1 a1.1
    const uint32_t q01 = __builtin_amdgcn_perm(a[1], a[0], 0x07030602u);   // a0.2 a1.2 a0.3 a1.3
    const uint32_t p23 = __builtin_amdgcn_perm(a[3], a[2], 0x05010400u);
    const uint32_t q23 = __builtin_amdgcn_perm(a[3], a[2], 0x07030602u);
    o[0] = __builtin_amdgcn_perm(p23, p01, 0x05040100u);
    o[1] = __builtin_amdgcn_perm(p23, p01, 0x07060302u);
    o[2] = __builtin_amdgcn_perm(q23, q01, 0x05040100u);
    o[3] = __builtin_amdgcn_perm(q23, q01, 0x07060302u);
}

// Byte of digit 0 of input k (of K, a multiple of 32) of row r in fragment
// tiles [rows / 32][K / 32][7][lane][16 bytes]: K step k / 32, lane
// r % 32 + 32 (k % 32 / 16), byte k % 16; digit i is 1024 i further.
__device__ __forceinline__ int64_t digit_offset(int64_t r, int k, int K) {
    return ((r >> 5) * (K >> 5) + (k >> 5)) * (DG_N * 1024) + ((r & 31) + 32 * ((k & 31) >> 4)) * 16 + (k & 15);
}

// Digit words of four consecutive inputs of a row: o[i] holds digit i (0 most
// significant) of the four.
__device__ __forceinline__ void pack4(const double (&x)[4], double to_int, uint32_t (&o)[DG_N]) {
    uint32_t lo[4], hi[4], tl[4], th[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint2 d = digits_of(x[k], to_int);
        lo[k] = d.x;
        hi[k] = d.y;
    }
    byte_transpose(lo, tl);
    byte_transpose(hi, th);
    o[0] = th[2]; o[1] = th[1]; o[2] = th[0];
    o[3] = tl[3]; o[4] = tl[2]; o[5] = tl[1]; o[6] = tl[0];
}

// One K step of 32: the 28 digit products of the row fragments x and the unit
// fragments w.  A fragment is free after its last product and is refilled at
// once with the next step's (w from wn, x from xn, whose digits are XD bytes
// apart; digit i of w after its products, digit 6 - i of x with it), so the
// loads have most of a step to arrive and take no registers of their own.
// SWAP: the accumulator holds [unit][row] instead of [row][unit].
template <bool SWAP, int XD>
__device__ __forceinline__ void digit_step(i32x16_t (&acc)[DG_N], i32x4_t (&w)[DG_N], i32x4_t (&x)[DG_N],
                                           const i32x4_t* __restrict__ wn, const char* xn) {
#pragma unroll
    for (int i = 0; i < DG_N; ++i) {
#pragma unroll
        for (int j = DG_N - 1 - i; j >= 0; --j)
            acc[i + j] = SWAP ? __builtin_amdgcn_mfma_i32_32x32x32_i8(w[i], x[j], acc[i + j], 0, 0, 0)
                              : __builtin_amdgcn_mfma_i32_32x32x32_i8(x[j], w[i], acc[i + j], 0, 0, 0);
        w[i] = wn[i * 64];
        x[DG_N - 1 - i] = *reinterpret_cast<const i32x4_t*>(xn + (DG_N - 1 - i) * XD);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The two exact integer parts of T (hi < 2^51, lo < 2^43 in magnitude).
__device__ __forceinline__ long long digit_hi(const i32x16_t (&acc)[DG_N], int r) {
    return ((long long)acc[0][r] << 24) + ((long long)acc[1][r] << 16) + ((long long)acc[2][r] << 8) + acc[3][r];
}
__device__ __forceinline__ long long digit_lo(const i32x16_t (&acc)[DG_N], int r) {
    return ((long long)acc[4][r] << 16) + ((long long)acc[5][r] << 8) + acc[6][r];
}
// T from its parts: the conversions are exact, the sum rounds once.
__device__ __forceinline__ double digit_value(long long hi, long long lo) {
    return fma((double)hi, 0x1p24, (double)lo);
}
// The same from the accumulators without 64-bit integers.
__device__ __forceinline__ double digit_value(const i32x16_t (&acc)[DG_N], int r) {
    const double h = fma(fma(fma((double)acc[0][r], 256.0, (double)acc[1][r]), 256.0, (double)acc[2][r]), 256.0,
                         (double)acc[3][r]);
    const double l = fma(fma((double)acc[4][r], 256.0, (double)acc[5][r]), 256.0, (double)acc[6][r]);
    return fma(h, 0x1p24, l);
}

// The 32 x kc values (kc <= DG_K) of rows [m0, m0 + 32) of A (FP64, row stride
// lda) from input k0 on, to digit planes in LDS by a workgroup of eight waves,
// and each row's factor; rows past M are zero.  Wave w takes rows 4 w .. + 3, a
// lane four consecutive inputs of each half of a row: the row loads are whole
// cache lines (a lane's own 128 bytes at a time touched a line per lane and
// took 6 us of a launch's 12 at 32 rows) and all in flight together.
struct PlaneRows {
    double x[4][2][4];
    __device__ __forceinline__ void load(const double* __restrict__ A, int64_t lda, int64_t m0, int64_t M, int k0,
                                         int kc, int wave, int lane) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int64_t r = m0 + 4 * wave + q;
                const bool in = r < M && 256 * s + 4 * lane < kc;
                const double2* src = reinterpret_cast<const double2*>(A + (in ? r * lda + k0 + 256 * s + 4 * lane : 0));
                const double2 a = in ? src[0] : make_double2(0.0, 0.0), b = in ? src[1] : make_double2(0.0, 0.0);
                x[q][s][0] = a.x; x[q][s][1] = a.y; x[q][s][2] = b.x; x[q][s][3] = b.y;
            }
    }
    __device__ __forceinline__ void store(char* planes, double* back, int kc, int wave, int lane) const {
        int mx[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            mx[q] = 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) mx[q] = max(mx[q], __double2hiint(x[q][e >> 2][e & 3]) & 0x7fffffff);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int q = 0; q < 4; ++q) mx[q] = max(mx[q], __shfl_xor(mx[q], o, 64));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const DigitScale sc = digit_scale(mx[q]);
            if (lane == 0) back[4 * wave + q] = sc.back;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                if (256 * s + 4 * lane >= kc) continue;
                uint32_t d[DG_N];
                pack4(x[q][s], sc.to_int, d);
                char* dst = planes + (4 * wave + q) * DG_LDS + 256 * s + 4 * lane;
#pragma unroll
                for (int i = 0; i < DG_N; ++i) *reinterpret_cast<uint32_t*>(dst + i * DG_PLANE) = d[i];
            }
        }
    }
};

// Digit fragments of A [M x K] (FP64, row stride lda): tiles
// [M / 32][K / 32][7][lane][16 bytes], and the rows' factors [block of DG_K
// inputs][M rounded up to 32].  One wave per (row, block).  A launch of its
// own: every tile of a layer reads the same fragments, and converting a row
// block's 16 384 values in each of a layer's 16 or more workgroups took 3 us
// of each one's 7.
struct DigitRows {
    const double* A[4];
    char* tiles[4];
    double* back[4];
};
template <int>
__global__ __launch_bounds__(256) void digit_rows_kernel(DigitRows P, int64_t lda, int64_t M, int K, int64_t m32,
                                                         const int* __restrict__ count, int rows_per_count) {
    const int g = blockIdx.z, blk = blockIdx.y, lane = threadIdx.x & 63;
    if (count) M = min<int64_t>(M, (int64_t)(*count) * rows_per_count);
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= M) return;
    const int k = blk * DG_K + lane * 4;                 // and + 256
    const double* src = P.A[g] + r * lda + k;
    double x[2][4];
    int h = 0;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const bool in = k + 256 * s < min(K, (blk + 1) * DG_K);
        const double2* q = reinterpret_cast<const double2*>(in ? src + 256 * s : P.A[g]);
        const double2 a = in ? q[0] : make_double2(0.0, 0.0), b = in ? q[1] : make_double2(0.0, 0.0);
        x[s][0] = a.x; x[s][1] = a.y; x[s][2] = b.x; x[s][3] = b.y;
#pragma unroll
        for (int e = 0; e < 4; ++e) h = max(h, __double2hiint(x[s][e]) & 0x7fffffff);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) h = max(h, __shfl_xor(h, o, 64));
    const DigitScale sc = digit_scale(h);
    if (lane == 0) P.back[g][(int64_t)blk * m32 + r] = sc.back;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int ks = k + 256 * s;
        if (ks >= K) break;
        uint32_t d[DG_N];
        pack4(x[s], sc.to_int, d);
        char* t = P.tiles[g] + digit_offset(r, ks, K);
#pragma unroll
        for (int i = 0; i < DG_N; ++i) *reinterpret_cast<uint32_t*>(t + i * 1024) = d[i];
    }
}

// Y[M x N] = epi(X[M x K] W^T), one layer, for batches too small for the
// one-kernel forward: a workgroup of eight waves takes 32 rows and `tpw` tiles
// of 32 units.  Wave w takes K steps w and w + 8 of a block of DG_K inputs and
// keeps its row fragments in registers for all tiles.  Per tile the waves' two
// integer parts of T add up in LDS, exactly, and all 512 threads finish the
// 1024 outputs.  MULTI: more than DG_K inputs, in blocks whose contributions
// are added in order (tpw <= GI_TPW).  A, W: digit fragments of the rows and of
// the units; Al, Wl: their factors [block][m32 or N rounded up to 32].
constexpr int GI_TPW = 4;

template <class Epi> struct DigitGroup {
    const void* A[4];
    const double* Al[4];
    const void* W[4];
    const double* Wl[4];
    Epi epi[4];
};

template <class Epi, bool MULTI>
__global__ __launch_bounds__(512) void gemm_i8_kernel(DigitGroup<Epi> G, int64_t m32, int64_t M, int N, int K, int tpw,
                                                      const int* __restrict__ count, int rows_per_count) {
    __shared__ unsigned long long sums[2][2][1024];      // [buffer][hi, lo][32 x 32]
    const int g = blockIdx.z;
    if (count) M = min<int64_t>(M, (int64_t)(*count) * rows_per_count);
    const int64_t m0 = (int64_t)blockIdx.y * DG_ROWS;
    if (m0 >= M) return;
    const double* wback = G.Wl[g];
    const double* xback = G.Al[g] + m0;
    const Epi& epi = G.epi[g];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KB = K / 32, NB = (N + 31) / 32, n32 = NB * 32;
    const int t0 = blockIdx.x * tpw, nt = min(tpw, NB - t0);
    const i32x4_t* X = static_cast<const i32x4_t*>(G.A[g]) + ((int64_t)blockIdx.y * KB + wave) * (DG_N * 64) + lane;
    const i32x4_t* W = static_cast<const i32x4_t*>(G.W[g]) + ((int64_t)t0 * KB + wave) * (DG_N * 64) + lane;
    const int ec = tid & 31, er = tid >> 5;              // epilogue: column, rows er and er + 16
    double tot[MULTI ? GI_TPW : 1][2];
    int zr[2] = {0, 0};
    if (const int per = epi.period()) {
        const int z0 = (int)(m0 % per);
        zr[0] = (z0 + er) % per;
        zr[1] = (z0 + er + 16) % per;
    }
    int buf = 0;
#pragma unroll 1
    for (int k0 = 0; k0 < K; k0 += DG_K) {
        const int nkb = min(DG_K, K - k0) >> 5, blk = k0 / DG_K;
        const i32x4_t* wt = W + (int64_t)(k0 >> 5) * (DG_N * 64);
        const i32x4_t* xt = X + (int64_t)(k0 >> 5) * (DG_N * 64);
        const bool two = wave + 8 < nkb;                 // the wave has a second K step in the block
        i32x4_t w[DG_N], x[2][DG_N];
        if (wave < nkb) {
#pragma unroll
            for (int i = 0; i < DG_N; ++i) {
                x[0][DG_N - 1 - i] = xt[(DG_N - 1 - i) * 64];
                w[i] = wt[i * 64];
            }
        }
        if (two) {
#pragma unroll
            for (int i = DG_N - 1; i >= 0; --i) x[1][i] = xt[(8 * DG_N + i) * 64];
        }
        const double xb[2] = {xback[blk * m32 + er], xback[blk * m32 + er + 16]};
        if (k0 == 0) {
            unsigned long long* z = &sums[0][0][0];
#pragma unroll
            for (int e = 0; e < 8; ++e) z[tid + 512 * e] = 0;
            __syncthreads();
        }
        auto tile = [&](int t, auto last) {
            // the epilogue's operands arrive under the products
            const int c = (t0 + t) * 32 + ec, cc = min(c, N - 1);
            const double wb = wback[(int64_t)blk * n32 + c];
            typename Epi::Col col{};
            typename Epi::Pre pre[2]{};
            if (last) {
                col = epi.col(cc);
#pragma unroll
                for (int i = 0; i < 2; ++i) pre[i] = epi.pre(min(m0 + er + 16 * i, M - 1), cc, zr[i]);
            }
            i32x16_t acc[DG_N];
#pragma unroll
            for (int i = 0; i < DG_N; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][r] = 0;
            // a unit fragment is refilled as its last product is issued: with
            // the second K step's, then the next tile's
            const i32x4_t* w1 = wt + ((int64_t)t * KB + 8) * (DG_N * 64);
            const i32x4_t* wn = wt + (int64_t)min(t + 1, nt - 1) * KB * (DG_N * 64);
            auto step = [&](const i32x4_t (&xs)[DG_N], const i32x4_t* nxt, bool refill) {
#pragma unroll
                for (int i = 0; i < DG_N; ++i) {
#pragma unroll
                    for (int j = DG_N - 1 - i; j >= 0; --j)
                        acc[i + j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xs[j], w[i], acc[i + j], 0, 0, 0);
                    if (refill) w[i] = nxt[i * 64];
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            if (wave < nkb) step(x[0], two ? w1 : wn, two || nt > 1);
            if (two) step(x[1], wn, nt > 1);
            if (wave < nkb) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int e = ((lane >> 5) * 4 + (r >> 2) * 8 + (r & 3)) * 32 + (lane & 31);
                    atomicAdd(&sums[buf][0][e], (unsigned long long)digit_hi(acc, r));
                    atomicAdd(&sums[buf][1][e], (unsigned long long)digit_lo(acc, r));
                }
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int e = (er + 16 * i) * 32 + ec;
                const double T = digit_value((long long)sums[buf][0][e], (long long)sums[buf][1][e]);
                sums[buf][0][e] = 0;
                sums[buf][1][e] = 0;
                double y = (T * xb[i]) * wb;
                if (MULTI) {
                    if (k0) y = tot[t][i] + y;
                    tot[t][i] = y;
                }
                const int64_t r = m0 + er + 16 * i;
                if (last && r < M && c < N) epi.store(r, c, col, y, pre[i]);
            }
            buf ^= 1;
        };
        if (MULTI) {
            const bool last = k0 + DG_K >= K;
#pragma unroll
            for (int t = 0; t < GI_TPW; ++t) {
                if (t >= nt) break;
                tile(t, last);
            }
        } else {
            for (int t = 0; t < nt; ++t) tile(t, std::true_type{});
        }
    }
}

// The same layer for more tiles: a workgroup of WAVES waves copies its 32
// rows' fragments of a block of inputs to LDS, and each wave runs whole tiles
// (tiles wave, wave + WAVES, ... of the workgroup's `tpw`), so that nothing is
// added up between waves and nothing waits per tile.  MULTI: one tile per wave.
constexpr int GW_ZR = (DG_K / 32) * DG_N * 1024;           // LDS: fragments, then the rows' places in the epilogue's period
constexpr int GW_LDS_BYTES = GW_ZR + DG_ROWS * 4;

template <class Epi, int WAVES, bool MULTI>
__global__ __launch_bounds__(64 * WAVES) void gemm_i8_wide_kernel(DigitGroup<Epi> G, int64_t m32, int64_t M, int N,
                                                                  int K, int tpw, const int* __restrict__ count,
                                                                  int rows_per_count) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int g = blockIdx.z;
    if (count) M = min<int64_t>(M, (int64_t)(*count) * rows_per_count);
    const int64_t m0 = (int64_t)blockIdx.y * DG_ROWS;
    if (m0 >= M) return;
    const double* wback = G.Wl[g];
    const Epi& epi = G.epi[g];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KB = K / 32, NB = (N + 31) / 32, n32 = NB * 32;
    const int t0 = blockIdx.x * tpw, nt = min(tpw, NB - t0);
    const i32x4_t* X = static_cast<const i32x4_t*>(G.A[g]) + (int64_t)blockIdx.y * KB * (DG_N * 64);
    const i32x4_t* W = static_cast<const i32x4_t*>(G.W[g]) + (int64_t)t0 * KB * (DG_N * 64) + lane;
    const double* xback = G.Al[g] + m0 + (lane >> 5) * 4;        // + 8 (r / 4) + r % 4
    const char* xa = lds + lane * 16;
    int* zrow = reinterpret_cast<int*>(lds + GW_ZR);
    const int per = epi.period();
    if (per && tid < DG_ROWS) zrow[tid] = (int)((m0 + tid) % per);
    double tot[16];
#pragma unroll 1
    for (int k0 = 0; k0 < K; k0 += DG_K) {
        const int nkb = min(DG_K, K - k0) >> 5, blk = k0 / DG_K;
        const i32x4_t* wt = W + (int64_t)(k0 >> 5) * (DG_N * 64);
        const i32x4_t* xt = X + (int64_t)(k0 >> 5) * (DG_N * 64);
        i32x4_t w[DG_N], x[DG_N];
        const i32x4_t* wp = wt + (int64_t)min(wave, nt - 1) * KB * (DG_N * 64);
#pragma unroll
        for (int i = 0; i < DG_N; ++i) w[i] = wp[i * 64];
        if (k0) __syncthreads();                         // every wave past its reads of the last block
        constexpr int CP = GW_ZR / 16 / (64 * WAVES);
        i32x4_t c[CP];
#pragma unroll
        for (int e = 0; e < CP; ++e) c[e] = xt[min(tid + e * 64 * WAVES, nkb * DG_N * 64 - 1)];
#pragma unroll
        for (int e = 0; e < CP; ++e) *reinterpret_cast<i32x4_t*>(lds + (tid + e * 64 * WAVES) * 16) = c[e];
        __syncthreads();
#pragma unroll 1
        for (int t = wave; t < nt; t += WAVES) {
            const int col = (t0 + t) * 32 + (lane & 31), cc = min(col, N - 1);
            const bool last = !MULTI || k0 + DG_K >= K;
            const double wb = wback[(int64_t)blk * n32 + col];
            typename Epi::Col q = epi.col(cc);
            typename Epi::Pre pre[16];
            if (sizeof(typename Epi::Pre) > 1 && last) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int lr = (lane >> 5) * 4 + (r >> 2) * 8 + (r & 3);
                    pre[r] = epi.pre(min(m0 + lr, M - 1), cc, per ? zrow[lr] : 0);
                }
            }
            i32x16_t acc[DG_N];
#pragma unroll
            for (int i = 0; i < DG_N; ++i) {
                x[i] = *reinterpret_cast<const i32x4_t*>(xa + i * 1024);
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][r] = 0;
            }
            const i32x4_t* next = wt + (int64_t)(t + WAVES < nt ? t + WAVES : t) * KB * (DG_N * 64);
            wp = wt + (int64_t)t * KB * (DG_N * 64);
#pragma unroll 1
            for (int kb = 1; kb < nkb; ++kb)
                digit_step<false, 1024>(acc, w, x, wp + kb * (DG_N * 64), xa + kb * (DG_N * 1024));
            digit_step<false, 1024>(acc, w, x, next, xa);
            double y[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                y[r] = (digit_value(acc, r) * xback[blk * m32 + (r >> 2) * 8 + (r & 3)]) * wb;
                if (MULTI) {
                    if (k0) y[r] = tot[r] + y[r];
                    tot[r] = y[r];
                }
                pin(y[r]);
                if (r & 1) __builtin_amdgcn_sched_barrier(0);
            }
            if (!last || col >= N) continue;
            const int64_t row0 = m0 + (lane >> 5) * 4;
            const bool whole = m0 + DG_ROWS <= M;
#pragma unroll
            for (int h = 0; h < 16; h += 4) {
                if (whole)
#pragma unroll
                    for (int r = h; r < h + 4; ++r) epi.store(row0 + (r >> 2) * 8 + (r & 3), col, q, y[r], pre[r]);
                else
#pragma unroll
                    for (int r = h; r < h + 4; ++r)
                        if (row0 + (r >> 2) * 8 + (r & 3) < M)
                            epi.store(row0 + (r >> 2) * 8 + (r & 3), col, q, y[r], pre[r]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}

}  // namespace nsmi

// FP64 products on the int8 matrix cores (gfx950), for the wide emulator
// layers in the NS_FP64 form: Ozaki-type splitting (Ozaki et al. 2012, on
// integer matrix units Ootomo et al. 2024) with one scale per row and block.
//
// Over blocks of DG_K = 512 inputs, a row's entries are rounded to multiples of
// 2^(e-54), 2^e <= the largest entry, and a unit's weights to multiples of a
// step of eight significant bits just above their largest / (127 2^48): 55-bit
// integers v, |v| <= 127 2^48, written as seven balanced base-256 digits
// (v = sum_i d_i 256^(6-i), d_i a signed byte).  The digit products d_i e_j
// with i + j <= 6 (28 of the 49) are summed by v_mfma_i32_32x32x32_i8 in one
// int32 accumulator per i + j, exactly: at most 7 x 512 products of 2^14 stay
// below 2^26.  The accumulators form
//   T = 2^24 (a0 2^24 + a1 2^16 + a2 2^8 + a3) + (a4 2^16 + a5 2^8 + a6)
// with one rounding, and the result is T times the two steps.  Integer sums
// have no order, so a row's result does not depend on the batch, the tile or
// the launch shape.
//
// Error of one product, relative to the product of the blocks' largest
// entries: the six dropped pairs of i + j = 7 are at most 6 2^14 2^40 of at
// least 2^108.9, 2^-52.3 (rms over random digits about 2^-56); the operands'
// rounding is below 2^-54 of each block's largest entry.  An FP64 product is
// relative to its own size instead, so digits are the better of the two only
// where a row's entries, and a unit's weights, are of similar size.  Both are
// checked: the weights on the host (digit_rule.cpp), and every row where it is
// converted, from the sum of its leading digits' magnitudes; a row that fails,
// or holds infinities, NaN or values beyond 2^(+-900), takes FP64 products in
// the same kernels (fp64_rows below).  On rows that pass, the error against
// extended precision is below an FP64 chain's (a third of it for normal draws).
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

constexpr double DG_FP64 = -1.0;                // factor of a row that takes FP64 products in any case

// Scale of a row from the high word of its largest magnitude: exponent e with
// max < 127/128 2^(e+1).  to_int: multiplier to the integer v; back: the
// factor of T (half of the 2^48 that T's integer weights leave out), 0 for a
// row of zeros; both 0 for a row outside 2^(+-900), infinities and NaN too.
struct DigitScale {
    double to_int, back;
};
__device__ __forceinline__ DigitScale digit_scale(int max_hi) {
    const int ef = (max_hi + 0x4000) >> 20;                       // biased exponent
    const bool in = ef > 1023 - 900 && ef < 1023 + 900;
    DigitScale s;
    s.to_int = in ? __longlong_as_double((long long)(54 + 1023 + 1023 - ef) << 52) : 0.0;
    s.back = in ? __longlong_as_double((long long)(ef - 30) << 52) : 0.0;
    return s;
}
// Whether digits serve a row of one block: its largest magnitude's high word,
// and the sum of its leading digits' magnitudes against the layer's minimum.
__device__ __forceinline__ bool digit_row(int max_hi, int sum, int minimum) { return sum >= minimum || max_hi == 0; }
// A row's factor, marked where no digits can hold it.
__device__ __forceinline__ double row_factor(int max_hi) {
    const double back = digit_scale(max_hi).back;
    return back == 0.0 && max_hi != 0 ? DG_FP64 : back;
}
// The same over several blocks of K inputs: the blocks' sums weigh with their
// factors, and the factor that the whole is held against is their root mean square.
__device__ __forceinline__ bool digit_row(const double* factors, const int* sums, int stride, int K, int minimum) {
    const int blocks = (K + DG_K - 1) / DG_K;
    double most = 0.0;
    bool held = true;
    for (int b = 0; b < blocks; ++b) {
        const double f = factors[b * stride];
        held &= f >= 0.0;
        most = fmax(most, f);
    }
    double have = 0.0, need = 0.0;
    for (int b = 0; b < blocks && most > 0.0; ++b) {
        const double q = factors[b * stride] / most;
        have += sums[b * stride] * q;
        need += min(DG_K, K - b * DG_K) * q * q;
    }
    return held && have * have * K >= (double)minimum * minimum * need;
}
// Magnitudes of the four leading digits in a word, added to s.
__device__ __forceinline__ uint32_t digit_sum(uint32_t d0, uint32_t s) {
    return __builtin_amdgcn_sad_u8(d0 ^ 0x80808080u, 0x80808080u, s);
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

// The same of v + dv, |dv| <= 2^4.
__device__ __forceinline__ uint2 digits_of_sum(double v, double dv) {
    constexpr double MAGIC = 0x1.8p52 + 0x808080;
    const double y = fma(v, 0x1p-24, MAGIC);
    const double z = (fma(y - MAGIC, -0x1p24, v) + dv) + MAGIC;
    const int h = __double2loint(y);
    const unsigned long long q = ((unsigned long long)(long long)h << 24) + (uint32_t)__double2loint(z);
    return make_uint2((uint32_t)q ^ 0x80808080u, (uint32_t)(q >> 32) ^ 0x00008080u);
}

// Step of a unit's weights of which mx > 0 is the largest: eight significant
// bits, so that w / step rounds exactly, and no more than 1/128 wide of the mark.
__device__ __forceinline__ double weight_step(double mx) {
    return __hiloint2double((__double2hiint(mx * (0x1p-48 / 127.0)) + 0x1000) & ~0xfff, 0);
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
__device__ __forceinline__ void pack4(const uint2 (&d)[4], uint32_t (&o)[DG_N]) {
    uint32_t lo[4], hi[4], tl[4], th[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        lo[k] = d[k].x;
        hi[k] = d[k].y;
    }
    byte_transpose(lo, tl);
    byte_transpose(hi, th);
    o[0] = th[2]; o[1] = th[1]; o[2] = th[0];
    o[3] = tl[3]; o[4] = tl[2]; o[5] = tl[1]; o[6] = tl[0];
}

__device__ __forceinline__ void pack4(const double (&x)[4], double to_int, uint32_t (&o)[DG_N]) {
    const uint2 d[4] = {digits_of(x[0], to_int), digits_of(x[1], to_int), digits_of(x[2], to_int),
                        digits_of(x[3], to_int)};
    pack4(d, o);
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

// T times the row's and the unit's factors.  The second product rounds: it is
// not to be fused with what a kernel adds to it, so that all kernels agree.
__device__ __forceinline__ double digit_product(double T, double row, double unit) {
#pragma clang fp contract(off)
    return (T * row) * unit;
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
    __device__ __forceinline__ void store(char* planes, double* back, int* sums, int kc, int wave, int lane) const {
        int mx[4];
        uint32_t sq[4];
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
            sq[q] = 0;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                if (256 * s + 4 * lane >= kc) continue;
                uint32_t d[DG_N];
                pack4(x[q][s], sc.to_int, d);
                sq[q] = digit_sum(d[0], sq[q]);
                char* dst = planes + (4 * wave + q) * DG_LDS + 256 * s + 4 * lane;
#pragma unroll
                for (int i = 0; i < DG_N; ++i) *reinterpret_cast<uint32_t*>(dst + i * DG_PLANE) = d[i];
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int sum = wave_total((int)sq[q]);
            if (lane == 0) {
                back[4 * wave + q] = row_factor(mx[q]);
                sums[4 * wave + q] = sum;
            }
        }
    }
};

// Digit fragments of A [M x K] (FP64, row stride lda): tiles
// [M / 32][K / 32][7][lane][16 bytes], and the rows' factors [block of DG_K
// inputs][M rounded up to 32], all DG_FP64 for a row that digits do not serve.
// One wave per (row, block).  A launch of its own: every tile of a layer reads the same fragments, and converting a row
// block's 16 384 values in each of a layer's 16 or more workgroups took 3 us
// of each one's 7.
struct DigitRows {
    const double* A[4];
    char* tiles[4];
    double* back[4];
    int minimum[4];                                      // digit_row
};
constexpr int DR_WAVES = 8;
// MULTI: a workgroup has one row, a wave every DR_WAVES'th block of it.
template <bool MULTI>
__global__ __launch_bounds__(MULTI ? 64 * DR_WAVES : 256) void digit_rows_kernel(DigitRows P, int64_t lda, int64_t row0, int64_t M, int K, int64_t m32,
                                                         const int* __restrict__ count, int rows_per_count) {
    const int g = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (count) M = min<int64_t>(M, (int64_t)(*count) * rows_per_count);
    const int64_t r = MULTI ? blockIdx.x : (int64_t)blockIdx.x * 4 + wave;   // of this part, from row0 on
    if (row0 + r >= M) return;
    extern __shared__ __attribute__((aligned(16))) char dr_lds[];
    const int blocks = MULTI ? (K + DG_K - 1) / DG_K : 1;
    double* factors = reinterpret_cast<double*>(dr_lds);
    int* sums = reinterpret_cast<int*>(factors + blocks);
    for (int blk = MULTI ? wave : 0; blk < blocks; blk += DR_WAVES) {
        const int k = blk * DG_K + lane * 4;             // and + 256
        const double* src = P.A[g] + (row0 + r) * lda + k;
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
        uint32_t sq = 0;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int ks = k + 256 * s;
            if (ks >= K) break;
            uint32_t d[DG_N];
            pack4(x[s], sc.to_int, d);
            sq = digit_sum(d[0], sq);
            char* t = P.tiles[g] + digit_offset(r, ks, K);
#pragma unroll
            for (int i = 0; i < DG_N; ++i) *reinterpret_cast<uint32_t*>(t + i * 1024) = d[i];
        }
        const int sum = wave_total((int)sq);
        if (lane > 0) continue;
        if (MULTI) {
            factors[blk] = row_factor(h);
            sums[blk] = sum;
        } else {
            P.back[g][r] = digit_row(h, sum, P.minimum[g]) ? row_factor(h) : DG_FP64;
        }
    }
    if (!MULTI) return;
    __syncthreads();
    const bool served = digit_row(factors, sums, 1, K, P.minimum[g]);
    for (int b = threadIdx.x; b < blocks; b += 64 * DR_WAVES) P.back[g][b * m32 + r] = served ? factors[b] : DG_FP64;
}

// The rows of a tile that take FP64 products.  The sum over a block of inputs
// is the same in every kernel: fused multiply-adds in order over its first 256
// inputs and over the rest, then the two added.
//
// One wave, up to four rows (x[j], inputs k of the block), 32 units of which
// the lane has one (w: its weights, `ldw` apart per input): lanes 0 .. 31 take
// the first 256 inputs, the others the rest; all get the sums.  Inputs from
// `present` on have no weights (they are zeros), the block has kc of them (a
// multiple of 32).
__device__ __forceinline__ void fp64_rows(const double* const (&x)[4], const double* __restrict__ w, int64_t ldw, int kc,
                                          int present, int lane, double (&y)[4]) {
    const int k0 = (lane >> 5) * 256, k1 = min(kc, k0 + 256);
#pragma unroll
    for (int j = 0; j < 4; ++j) y[j] = 0.0;
#pragma unroll 1
    for (int k = k0; k < k1; k += 8) {
        double b[8], a[4][8];
#pragma unroll
        for (int e = 0; e < 8; ++e) b[e] = w[min(k + e, present - 1) * ldw];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) a[j][e] = x[j][k + e];
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int j = 0; j < 4; ++j) y[j] = fma(a[j][e], b[e], y[j]);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) y[j] = y[j] + __shfl_xor(y[j], 32, 64);
}
// The next four rows of the set `rem`, taken out of it (the last one again
// where fewer are left).
__device__ __forceinline__ void next_rows(uint32_t& rem, int (&r)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        r[j] = rem ? __builtin_ctz(rem) : r[j > 0 ? j - 1 : 0];
        rem &= rem - 1;
    }
}

// Y[M x N] = epi(X[M x K] W^T), one layer, for batches too small for the
// one-kernel forward: a workgroup of eight waves takes 32 rows and `tpw` tiles
// of 32 units.  Wave w takes K steps w and w + 8 of a block of DG_K inputs and
// keeps its row fragments in registers for all tiles.  Per tile the waves' two
// integer parts of T add up in LDS, exactly, and all 512 threads finish the
// 1024 outputs.  MULTI: more than DG_K inputs, in blocks whose contributions
// are added in order (tpw <= GI_TPW).  A, W: digit fragments of the rows and of
// the units; Al, Wl: their factors [block][m32 or N rounded up to 32].  Rows
// The launch takes the rows of a part, from row0 on (A and Al are the part's).  Rows
// that digits do not serve (factor DG_FP64) are left out and formed at the end, from
// A64 (row stride lda) and the weights Wk, input by input (stride ldw,
// `present` inputs): there nothing else holds registers, and a launch without
// such rows does not fetch the code.
constexpr int GI_TPW = 4;

template <class Epi> struct DigitGroup {
    const void* A[4];
    const double* Al[4];
    const void* W[4];
    const double* Wl[4];
    const double* A64[4];
    const double* Wk[4];
    int64_t lda, ldw;
    int present;
    Epi epi[4];
};

// Rows `odd` of the row block at m0 in tiles [t0, t0 + nt): four rows of a tile
// per wave at a time, their blocks' sums added in order.
template <class Epi>
__device__ __forceinline__ void fp64_tiles(const DigitGroup<Epi>& G, int g, uint32_t odd, int64_t m0, int N, int K,
                                           int t0, int nt, int wave, int waves, int lane) {
    const Epi& epi = G.epi[g];
    const int sets = (__popc(odd) + 3) / 4, per = epi.period();
    for (int e = wave; e < sets * nt; e += waves) {
        uint32_t rem = odd;
        int rr[4] = {};
        for (int q = 0; q <= e % sets; ++q) next_rows(rem, rr);
        const int c = (t0 + e / sets) * 32 + (lane & 31), cc = min(c, N - 1);
        double y[4] = {};
        for (int k0 = 0; k0 < K; k0 += DG_K) {
            const double* x[4];
            double v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = G.A64[g] + (m0 + rr[j]) * G.lda + k0;
            fp64_rows(x, G.Wk[g] + k0 * G.ldw + cc, G.ldw, min(DG_K, K - k0), G.present - k0, lane, v);
#pragma unroll
            for (int j = 0; j < 4; ++j) y[j] = k0 ? y[j] + v[j] : v[j];
        }
        if (lane >= 32 || c >= N) continue;
        const auto col = epi.col(c);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            epi.store(m0 + rr[j], c, col, y[j], epi.pre(m0 + rr[j], c, per ? (int)((m0 + rr[j]) % per) : 0));
    }
}

template <class Epi, bool MULTI>
__global__ __launch_bounds__(512) void gemm_i8_kernel(DigitGroup<Epi> G, int64_t m32, int64_t row0, int64_t M, int N, int K, int tpw,
                                                      const int* __restrict__ count, int rows_per_count) {
    __shared__ unsigned long long sums[2][2][1024];      // [buffer][hi, lo][32 x 32]
    const int g = blockIdx.z;
    if (count) M = min<int64_t>(M, (int64_t)(*count) * rows_per_count);
    const int64_t part = (int64_t)blockIdx.y * DG_ROWS, m0 = row0 + part;
    if (m0 >= M) return;
    const double* wback = G.Wl[g];
    const double* xback = G.Al[g] + part;
    const Epi& epi = G.epi[g];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KB = K / 32, NB = (N + 31) / 32, n32 = NB * 32;
    const int t0 = blockIdx.x * tpw, nt = min(tpw, NB - t0);
    const i32x4_t* X = static_cast<const i32x4_t*>(G.A[g]) + ((int64_t)blockIdx.y * KB + wave) * (DG_N * 64) + lane;
    const i32x4_t* W = static_cast<const i32x4_t*>(G.W[g]) + ((int64_t)t0 * KB + wave) * (DG_N * 64) + lane;
    const int ec = tid & 31, er = tid >> 5;              // epilogue: column, rows er and er + 16
    uint32_t odd = 0;                                    // the wave's epilogue rows with the factor DG_FP64
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
                double y = digit_product(T, xb[i], wb);
                if (MULTI) {
                    if (k0) y = tot[t][i] + y;
                    tot[t][i] = y;
                }
                const int64_t r = m0 + er + 16 * i;
                if (last && r < M && c < N && xb[i] >= 0.0) epi.store(r, c, col, y, pre[i]);
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
        if (k0 + DG_K >= K)                              // (asked at the start, the factors' loads took 0.8 us of a launch)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const unsigned long long marked = __ballot(m0 + er + 16 * i < M && xb[i] < 0.0);
                odd |= (uint32_t)((marked & 1) | (marked >> 32 & 1) << 1) << (2 * wave + 16 * i);
            }
    }
    if (__builtin_expect(odd != 0, 0)) fp64_tiles(G, g, odd, m0, N, K, t0, nt, 0, 1, lane);
}

// The same layer for more tiles: a workgroup of WAVES waves copies its 32
// rows' fragments of a block of inputs to LDS, and each wave runs whole tiles
// (tiles wave, wave + WAVES, ... of the workgroup's `tpw`), so that nothing is
// added up between waves and nothing waits per tile.  MULTI: one tile per wave.
constexpr int GW_ZR = (DG_K / 32) * DG_N * 1024;           // LDS: fragments, then the rows' places in the epilogue's period
constexpr int GW_LDS_BYTES = GW_ZR + DG_ROWS * 4;

template <class Epi, int WAVES, bool MULTI>
__global__ __launch_bounds__(64 * WAVES) void gemm_i8_wide_kernel(DigitGroup<Epi> G, int64_t m32, int64_t row0, int64_t M, int N,
                                                                  int K, int tpw, const int* __restrict__ count,
                                                                  int rows_per_count) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int g = blockIdx.z;
    if (count) M = min<int64_t>(M, (int64_t)(*count) * rows_per_count);
    const int64_t part = (int64_t)blockIdx.y * DG_ROWS, m0 = row0 + part;
    if (m0 >= M) return;
    const double* wback = G.Wl[g];
    const Epi& epi = G.epi[g];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KB = K / 32, NB = (N + 31) / 32, n32 = NB * 32;
    const int t0 = blockIdx.x * tpw, nt = min(tpw, NB - t0);
    const i32x4_t* X = static_cast<const i32x4_t*>(G.A[g]) + (int64_t)blockIdx.y * KB * (DG_N * 64);
    const i32x4_t* W = static_cast<const i32x4_t*>(G.W[g]) + (int64_t)t0 * KB * (DG_N * 64) + lane;
    const double* xback = G.Al[g] + part + (lane >> 5) * 4;        // + 8 (r / 4) + r % 4
    const uint32_t odd = (uint32_t)__ballot(m0 + (lane & 31) < M && G.Al[g][part + (lane & 31)] < 0.0);   // DG_FP64
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
                y[r] = digit_product(digit_value(acc, r), xback[blk * m32 + (r >> 2) * 8 + (r & 3)], wb);
                if (MULTI) {
                    if (k0) y[r] = tot[r] + y[r];
                    tot[r] = y[r];
                }
                pin(y[r]);
                if (r & 1) __builtin_amdgcn_sched_barrier(0);
            }
            if (!last || col >= N) continue;
            const int64_t row0 = m0 + (lane >> 5) * 4;
            const bool whole = m0 + DG_ROWS <= M && odd == 0;
#pragma unroll
            for (int h = 0; h < 16; h += 4) {
                if (whole)
#pragma unroll
                    for (int r = h; r < h + 4; ++r) epi.store(row0 + (r >> 2) * 8 + (r & 3), col, q, y[r], pre[r]);
                else
#pragma unroll
                    for (int r = h; r < h + 4; ++r)
                        if (row0 + (r >> 2) * 8 + (r & 3) < M &&
                            !(odd >> ((lane >> 5) * 4 + (r >> 2) * 8 + (r & 3)) & 1))
                            epi.store(row0 + (r >> 2) * 8 + (r & 3), col, q, y[r], pre[r]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    if (__builtin_expect(odd != 0, 0)) fp64_tiles(G, g, odd, m0, N, K, t0, nt, wave, WAVES, lane);
}

}  // namespace nsmi

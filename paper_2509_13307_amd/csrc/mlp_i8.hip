// Whole-network FP64 forward and adjoint on the int8 matrix cores for large
// batches of networks whose hidden layers are all 512 wide (digit products:
// gemm_i8.h).
//
// One workgroup of eight waves owns 32 rows of one network.  The rows'
// activations live in LDS as seven digit planes (118 KB) from the first layer
// to the last; the weights' digit tiles stream from L2 in fragment order
// straight into registers.  Wave w owns unit tiles w and w + 8 of a hidden
// layer: the accumulator holds [unit][row], so a lane has 16 units of one row
// per tile and its row's scale in a register, and packs the digits of four
// consecutive units into one LDS word per plane.  The row's scale is the
// maximum over the layer, so a layer ends with an LDS maximum, a barrier, the
// digits, and a second barrier.  The output layer holds [row][unit], whose
// stores are coalesced, and has no barriers.
//
// Bound by the chip's power: at 4 096 rows of four 6-512^4-2500 networks the
// launch takes 830 us with the matrix cores busy 910 k cycles per SIMD at
// about 1.7 GHz; the digit products alone, on operands that stay in registers,
// take 600 us at that clock, with the weight and LDS streams 750 us, and the
// rest is FP64 activations and digits.  Wave priorities make no difference
// (the older of two waves on a SIMD goes first by itself, so that one's
// activations run under the other's products).  The FP64 MFMA layers that this
// replaced took 1 380 us (50 TFLOP/s), and the adjoint of 32 768 rows of one
// 8-512^4-420 network 1 460 us against 1 070 us now (713 us here for the hidden
// layers; its output layer's rows mostly fail the check and stay on FP64
// products, 353 us).
//
// A layer's rows that digits do not serve (gemm_i8.h) take FP64 products: the
// workgroup forms their next layer from the values themselves, four rows at a
// time through LDS, before it goes on with the digits of the others.  4 096
// rows of a 6-512^4-2500 network with one such layer for every row: 580 us
// (even rows 347, FP64 products throughout 435); 500 rows, layer by layer, 156
// (107, 142).
//
// Every value is that of the layer-by-layer kernels (exact integer sums, the
// same scales, rows on FP64 products and epilogue expressions), so a row's
// result does not depend on which of the two a batch takes.
#include "gemm_i8.h"
#include "nsmi.h"

namespace nsmi {

constexpr int DM_H = 512, DM_MAXHID = 6, DM_WAVES = 8;
constexpr int DM_STEP = DG_N * 64;                  // 16-byte units of one K step of a tile
// LDS: the small arrays first, within the reach of an LDS instruction's 16-bit
// offset from one base register (behind the planes each address would take a
// register of its own)
constexpr int DM_MAX = 4 * DM_H * 8;                // after the layer parameters [4][512]: row maxima [2][32]
constexpr int DM_SUM = DM_MAX + 2 * DG_ROWS * 4;     // rows' sums of leading digits [2][32]
constexpr int DM_BACK = DM_SUM + 2 * DG_ROWS * 4;    // row factors [32]
constexpr int DM_ZROW = DM_BACK + DG_ROWS * 8;      // rows' redshift nodes [32]
constexpr int DM_PLANES = DM_ZROW + DG_ROWS * 4;    // digit planes
constexpr int DM_ROWS64 = DM_PLANES + DG_N * DG_PLANE;   // four rows of values [4][512]
constexpr int DM_MAXBLOCKS = 4 * DM_H * 8 / (DG_ROWS * 12);   // blocks whose factors and sums fit there
constexpr int DM_LDS_BYTES = DM_ROWS64 + 4 * DM_H * 8;

struct DigitLayer {
    const i32x4_t* W;                   // digit tiles
    const double* back;                 // unit factors
    const double* Wk;                   // weights input by input (FP64 rows)
    const double *b, *beta, *gamma;
    int minimum;                        // digit_row of the layer's input rows
    double* t;                          // pre-activations [rows x 512]: written by the forward when wanted, read by the adjoint
};
struct DigitNet {
    const double *W1, *b1, *be1, *ga1, *shift, *scale;
    double* t1;
    DigitLayer hid[DM_MAXHID];
    DigitLayer out;                     // output layer (forward: W, back, b; adjoint: W^T's tiles, none: its adjoint is done)
    double* y64;                        // scratch [rows x 512]: products of the rows on FP64
    const double *mu, *sigma;
    double* y;                          // forward: outputs; adjoint: delta of the first layer
    const double* delta;                // adjoint: output deltas [rows x n_pad]
    int is_log;
};
struct DigitArgs {
    DigitNet net[4];
    int n_hidden, n_in, N_out, n_pad, mu_rows, nrb;
    int64_t ldo;
};

// Workgroup -> (network, row block): each XCD (workgroups i, i + 8, ...) takes
// a contiguous run, so that its L2 streams one network's weights.
__device__ __forceinline__ int digit_block() {
    const int n = gridDim.x, i = blockIdx.x;
    return (n & 7) ? i : (i & 7) * (n >> 3) + (i >> 3);
}

struct DigitWave {
    char* lds;
    int lane, wave, row, u0;            // u0: lane's first unit within a tile
    uint32_t hoff;                      // byte offset of the lane's first value in a [32 x 512] block of doubles
    const char* xa;
    i32x4_t w[DG_N], x[DG_N];
    i32x16_t acc[DG_N];
    double back;                        // factor of the lane's row
    uint32_t odd;                       // rows that take FP64 products in the coming layer

    __device__ __forceinline__ double* prm(int i) const { return reinterpret_cast<double*>(lds) + i * DM_H; }
    __device__ __forceinline__ int* rmax(int p) const { return reinterpret_cast<int*>(lds + DM_MAX) + p * DG_ROWS; }
    __device__ __forceinline__ int* rsum(int p) const { return reinterpret_cast<int*>(lds + DM_SUM) + p * DG_ROWS; }
    __device__ __forceinline__ double* rows64() const { return reinterpret_cast<double*>(lds + DM_ROWS64); }
    __device__ __forceinline__ double* rback() const { return reinterpret_cast<double*>(lds + DM_BACK); }
    // units 8 q + 256 t (+ 0..3) of the lane's row in such a block: a uniform base, the lane's offset and an immediate
    __device__ __forceinline__ double2* units(double* block, int t, int q) const {
        return reinterpret_cast<double2*>(reinterpret_cast<char*>(block) + hoff + (8 * q + 256 * t) * 8);
    }
    __device__ __forceinline__ void load_w(const i32x4_t* p) {
#pragma unroll
        for (int i = 0; i < DG_N; ++i) w[i] = p[i * 64];
    }
    __device__ __forceinline__ void load_x() {
#pragma unroll
        for (int i = 0; i < DG_N; ++i) x[i] = *reinterpret_cast<const i32x4_t*>(xa + i * DG_PLANE);
    }
    // one tile of nkb K steps; the last step's refill takes the next tile's weights
    template <bool SWAP>
    __device__ __forceinline__ void tile(const i32x4_t* p, const i32x4_t* next, int nkb) {
#pragma unroll
        for (int i = 0; i < DG_N; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][r] = 0;
#pragma unroll 1
        for (int kb = 1; kb < nkb; ++kb) digit_step<SWAP, DG_PLANE>(acc, w, x, p + kb * DM_STEP, xa + kb * 32);
        digit_step<SWAP, DG_PLANE>(acc, w, x, next, xa);
    }
    // v = the tile's sums for the lane's row, done before anything else so that
    // the accumulators' registers are free for it
    __device__ __forceinline__ void sums(double (&v)[16]) const {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            v[r] = digit_value(acc, r);
            pin(v[r]);
            if (r & 1) __builtin_amdgcn_sched_barrier(0);
        }
    }
    // y[row][u] = or += (`add`), for the rows of `odd` and units u < units (whose
    // weights stand in even rows), the sums of fp64_rows over a block of inputs
    // (`present` of them with weights); `put` writes a row's values to its place in LDS, zeros
    // up to 512
    template <class F>
    __device__ __forceinline__ void products64(F put, const double* Wk, int64_t ldw, int present, int units, double* y,
                                               int64_t ldy, bool add) const {
        constexpr int KS = 8;                            // inputs whose weights are in flight together
        double* xs = rows64();
        for (uint32_t rem = odd; rem;) {
            int r[4] = {};
            next_rows(rem, r);
            __syncthreads();                             // the places are free, what `put` reads is there
#pragma unroll
            for (int j = 0; j < 4; ++j) put(r[j], xs + j * DM_H);
            __syncthreads();
            // a lane has two units (a wave 64) and one half of the inputs
            const int half = (lane >> 5) * 256;
#pragma unroll 1
            for (int u = wave * 64 + (lane & 31) * 2; u < units; u += 512) {
                double v[4][2] = {};
#pragma unroll 1
                for (int k = half; k < half + 256; k += KS) {
                    double2 w[KS];
#pragma unroll
                    for (int e = 0; e < KS; ++e)
                        w[e] = *reinterpret_cast<const double2*>(Wk + min(k + e, present - 1) * ldw + u);
#pragma unroll
                    for (int e = 0; e < KS; e += 2)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const double2 x = *reinterpret_cast<const double2*>(xs + j * DM_H + k + e);
                            v[j][0] = fma(x.y, w[e + 1].x, fma(x.x, w[e].x, v[j][0]));
                            v[j][1] = fma(x.y, w[e + 1].y, fma(x.x, w[e].y, v[j][1]));
                        }
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const double sum = v[j][i] + __shfl_xor(v[j][i], 32, 64);
                        double* o = y + r[j] * ldy + u + i;
                        if (lane < 32 && u + i < units && (j == 0 || r[j] != r[j - 1])) *o = add ? *o + sum : sum;
                    }
            }
        }
        __syncthreads();
    }
    // the same from the layer's values h
    __device__ __forceinline__ void products64(const double (&h)[2][16], const double* Wk, int64_t ldw, int units,
                                               double* y, int64_t ldy) const {
        products64([&](int r, double* place) {
            if (row != r) return;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int e = 0; e < 16; ++e) place[(wave + 8 * t) * 32 + u0 + (e >> 2) * 8 + (e & 3)] = h[t][e];
        }, Wk, ldw, DM_H, units, y, ldy, false);
    }
    // v = those sums of tile t for a row of `odd`
    __device__ __forceinline__ void take64(double* block, int t, double (&v)[16]) const {
        if (!(odd >> row & 1)) return;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double2* o = units(block, t, q);
            const double2 a = o[0], b = o[1];
            v[4 * q] = a.x; v[4 * q + 1] = a.y; v[4 * q + 2] = b.x; v[4 * q + 3] = b.y;
        }
    }
    // the layer's values h (tiles wave and wave + 8) become the next layer's
    // digit planes, and `odd` is the set of its rows (of those that count) that
    // digits do not serve; `stage` runs between the barriers
    template <class F>
    __device__ __forceinline__ void to_planes(const double (&h)[2][16], int p, bool counts, int minimum, F stage) {
        int mx = 0;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = max(mx, __double2hiint(h[t][r]) & 0x7fffffff);
        mx = max(mx, __shfl_xor(mx, 32, 64));
        if (lane < 32) atomicMax(&rmax(p)[row], mx);
        __syncthreads();
        const DigitScale sc = digit_scale(rmax(p)[row]);
        back = sc.back;
        if (wave == 0 && lane < 32) {
            rmax(p ^ 1)[row] = 0;
            rsum(p ^ 1)[row] = 0;
            rback()[row] = back;
        }
        uint32_t sq = 0;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double v[4] = {h[t][4 * q], h[t][4 * q + 1], h[t][4 * q + 2], h[t][4 * q + 3]};
                uint32_t d[DG_N];
                pack4(v, sc.to_int, d);
                sq = digit_sum(d[0], sq);
                char* dst = lds + DM_PLANES + row * DG_LDS + (wave + 8 * t) * 32 + u0 + 8 * q;
#pragma unroll
                for (int i = 0; i < DG_N; ++i) *reinterpret_cast<uint32_t*>(dst + i * DG_PLANE) = d[i];
                __builtin_amdgcn_sched_barrier(0);
            }
        sq += __shfl_xor(sq, 32, 64);
        if (lane < 32) atomicAdd(&rsum(p)[row], (int)sq);
        stage();
        __syncthreads();
        // (a row that no digits can hold by its factor: its leading digits may be anything)
        odd = (uint32_t)__ballot(counts && (back == 0.0 ? rmax(p)[row] != 0 : rsum(p)[row] < minimum));
        load_x();
    }
};

// Forward; NI: inputs held per lane; SAVE: the pre-activations are kept for the adjoint.
template <int NI, bool SAVE>
__global__ __launch_bounds__(512) void mlp_i8_kernel(const double* __restrict__ theta, int64_t ld, int64_t rows,
                                                     int rpw, const int* __restrict__ src,
                                                     const double* __restrict__ fix,
                                                     const double* __restrict__ znodes, DigitArgs A,
                                                     const int* __restrict__ count) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int blk = digit_block();
    const int g = blk / A.nrb;
    const DigitNet& N = A.net[g];
    const int64_t M = count ? min<int64_t>(rows, (int64_t)(*count) * rpw) : rows;
    const int64_t m0 = (int64_t)(blk - g * A.nrb) * DG_ROWS;
    if (m0 >= M) return;
    const int tid = threadIdx.x;
    DigitWave S;
    S.lds = lds;
    S.lane = tid & 63;
    S.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    S.row = S.lane & 31;
    S.u0 = (S.lane >> 5) * 4;
    S.hoff = (uint32_t)(S.row * DM_H + S.wave * 32 + S.u0) * 8u;
    S.xa = lds + DM_PLANES + S.row * DG_LDS + (S.lane >> 5) * 16;
    const int wave = S.wave, lane = S.lane;
    const int64_t grow = m0 + S.row;
    const bool valid = grow < M;

    // layer 1 on the VALU: its weights pass through LDS (before the planes are in use)
    double* w1 = reinterpret_cast<double*>(lds + DM_PLANES);
    for (int e = tid; e < DM_H * NI; e += 512) {
        const int u = e / NI, k = e % NI;
        w1[e] = k < A.n_in ? N.W1[u * A.n_in + k] : 0.0;
    }
    S.prm(0)[tid] = N.b1[tid];
    S.prm(1)[tid] = N.be1[tid];
    S.prm(2)[tid] = N.ga1[tid];
    if (tid < 2 * DG_ROWS) S.rmax(0)[tid] = S.rsum(0)[tid] = 0;
    int* zrow = reinterpret_cast<int*>(lds + DM_ZROW);
    if (tid < DG_ROWS) zrow[tid] = A.mu_rows > 1 ? (int)((m0 + tid) % A.mu_rows) * A.N_out : 0;
    double xv[NI];
    {
        const int64_t wk = valid ? grow / rpw : 0;
        const int zi = valid ? (int)(grow % rpw) : 0;
#pragma unroll
        for (int k = 0; k < NI; ++k) {
            xv[k] = 0.0;
            if (k < A.n_in && valid) {
                const int s = src[k];
                const double t = s >= 0 ? theta[wk * ld + s] : (s == SRC_ZNODE ? znodes[zi] : fix[k]);
                xv[k] = (t - N.shift[k]) / N.scale[k];
            }
        }
    }
    __syncthreads();
    double h[2][16];
    auto keep = [&](double* dst, int t) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            double2* ts = S.units(dst + m0 * DM_H, t, q);
            ts[0] = make_double2(h[t][4 * q], h[t][4 * q + 1]);
            ts[1] = make_double2(h[t][4 * q + 2], h[t][4 * q + 3]);
        }
    };
    // four units at a time: more would not fit the registers
    auto activate = [&](int t) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int u = (wave + 8 * t) * 32 + S.u0 + (r >> 2) * 8 + (r & 3);
            h[t][r] = gated<double>(h[t][r], S.prm(1)[u], S.prm(2)[u]);
            pin(h[t][r]);
            if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int u = (wave + 8 * t) * 32 + S.u0 + 8 * q;
            double a[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) a[r] = S.prm(0)[u + r];
#pragma unroll
            for (int k = 0; k < NI; ++k)                 // past n_in: zeros
#pragma unroll
                for (int r = 0; r < 4; ++r) a[r] += w1[(u + r) * NI + k] * xv[k];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                h[t][4 * q + r] = a[r];
                pin(h[t][4 * q + r]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        if (SAVE && valid) keep(N.t1, t);
        activate(t);
    }
    const int nkb = DM_H / 32;
    int p = 0;
    S.load_w(N.hid[0].W + (int64_t)wave * nkb * DM_STEP + lane);
    for (int l = 0; l <= A.n_hidden; ++l) {
        // parameters of this layer, loaded before the barrier that frees their place
        double pr[4] = {0.0, 0.0, 0.0, 0.0};
        if (l < A.n_hidden) {
            const DigitLayer& D = N.hid[l];
            pr[0] = D.b[tid]; pr[1] = D.beta[tid]; pr[2] = D.gamma[tid]; pr[3] = D.back[tid];
        }
        const DigitLayer& D = l < A.n_hidden ? N.hid[l] : N.out;
        S.to_planes(h, p, valid, D.minimum, [&]() {
            if (l < A.n_hidden)
#pragma unroll
                for (int i = 0; i < 4; ++i) S.prm(i)[tid] = pr[i];
        });
        p ^= 1;
        if (__builtin_expect(S.odd != 0, 0)) {                                     // the output layer's go to their place among the outputs
            if (l < A.n_hidden) S.products64(h, D.Wk, DM_H, DM_H, N.y64 + m0 * DM_H, DM_H);
            else S.products64(h, D.Wk, A.n_pad, A.N_out, N.y + m0 * A.ldo, A.ldo);
        }
        if (l == A.n_hidden) break;
        const i32x4_t* wt = D.W + (int64_t)wave * nkb * DM_STEP + lane;
        const i32x4_t* wl = (l + 1 < A.n_hidden ? N.hid[l + 1].W : N.out.W) +
                            (l + 1 < A.n_hidden || wave * 32 < A.N_out ? (int64_t)wave * nkb * DM_STEP : 0) + lane;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const i32x4_t* wp = wt + (int64_t)t * 8 * nkb * DM_STEP;
            S.tile<true>(wp, t == 0 ? wt + (int64_t)8 * nkb * DM_STEP : wl, nkb);
            S.sums(h[t]);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int u = (wave + 8 * t) * 32 + S.u0 + (r >> 2) * 8 + (r & 3);
                h[t][r] = digit_product(h[t][r], S.back, S.prm(3)[u]) + S.prm(0)[u];
                pin(h[t][r]);
                if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            }
            if (__builtin_expect(S.odd != 0, 0)) {
                S.take64(N.y64 + m0 * DM_H, t, h[t]);
                if (S.odd >> S.row & 1)
#pragma unroll
                    for (int r = 0; r < 16; ++r) h[t][r] += S.prm(0)[(wave + 8 * t) * 32 + S.u0 + (r >> 2) * 8 + (r & 3)];
            }
            if (SAVE && valid) keep(D.t, t);
            activate(t);
        }
    }
    // output layer: accumulator rows 4 (lane / 32) + 8 (r / 4) + r % 4, unit lane % 32
    const int nb = (A.N_out + 31) / 32;
    for (int t = wave; t < nb; t += DM_WAVES) {
        const i32x4_t* wp = N.out.W + (int64_t)t * nkb * DM_STEP + lane;
        // the epilogue's operands arrive under the products
        const int c = t * 32 + S.row, cc = min(c, A.N_out - 1);
        const double wb = N.out.back[cc], b = N.out.b[cc], sg = N.sigma[cc];
        double mu[16];
        mu[0] = N.mu[zrow[S.u0] + cc];
        if (A.mu_rows > 1) {
#pragma unroll
            for (int r = 1; r < 16; ++r) mu[r] = N.mu[zrow[S.u0 + (r >> 2) * 8 + (r & 3)] + cc];
        } else {
#pragma unroll
            for (int r = 1; r < 16; ++r) mu[r] = mu[0];
        }
        S.tile<false>(wp, t + DM_WAVES < nb ? wp + (int64_t)DM_WAVES * nkb * DM_STEP : wp, nkb);
        if (c >= A.N_out) continue;
        // rows through wave-uniform addresses, the lane's part in one 32-bit offset
        const uint32_t off = (uint32_t)(S.u0 * A.ldo + c) * 8u;
        char* y0 = reinterpret_cast<char*>(N.y + m0 * A.ldo);
        const bool whole = m0 + DG_ROWS <= M;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            double y[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double a = digit_product(digit_value(S.acc, 4 * q + r), S.rback()[8 * q + r + S.u0], wb);
                y[r] = mu[4 * q + r] + sg * (a + b);
                pin(y[r]);
            }
            if (__builtin_expect(S.odd != 0, 0))
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (S.odd >> (8 * q + r + S.u0) & 1)
                        y[r] = mu[4 * q + r] + sg * (*reinterpret_cast<const double*>(y0 + (int64_t)(8 * q + r) * A.ldo * 8 + off) + b);
            if (N.is_log)
#pragma unroll
                for (int r = 0; r < 4; ++r) y[r] = exp10_of<double>(y[r]);
            if (whole)
#pragma unroll
                for (int r = 0; r < 4; ++r) *reinterpret_cast<double*>(y0 + (int64_t)(8 * q + r) * A.ldo * 8 + off) = y[r];
            else
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (m0 + 8 * q + r + S.u0 < M)
                        *reinterpret_cast<double*>(y0 + (int64_t)(8 * q + r) * A.ldo * 8 + off) = y[r];
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// Adjoint: output deltas back to the first layer's.
__global__ __launch_bounds__(512) void mlp_i8_back_kernel(int64_t rows, int n_pad, DigitArgs A) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int blk = digit_block();
    const int g = blk / A.nrb;
    const DigitNet& N = A.net[g];
    const int64_t m0 = (int64_t)(blk - g * A.nrb) * DG_ROWS;
    const int tid = threadIdx.x;
    DigitWave S;
    S.lds = lds;
    S.lane = tid & 63;
    S.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    S.row = S.lane & 31;
    S.u0 = (S.lane >> 5) * 4;
    S.hoff = (uint32_t)(S.row * DM_H + S.wave * 32 + S.u0) * 8u;
    S.xa = lds + DM_PLANES + S.row * DG_LDS + (S.lane >> 5) * 16;
    const int wave = S.wave, lane = S.lane;
    const int64_t grow = m0 + S.row;
    const bool valid = grow < rows;
    if (tid < 2 * DG_ROWS) S.rmax(0)[tid] = S.rsum(0)[tid] = 0;

    double h[2][16];
    // delta_l W_l, times f'(t) of the layer below (rows past the end: t = 0)
    auto through = [&](double* tsave, int t) {
        double tv[16] = {};
        if (valid) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double2* ts = S.units(tsave + m0 * DM_H, t, q);
                const double2 a = ts[0], b = ts[1];
                tv[4 * q] = a.x; tv[4 * q + 1] = a.y; tv[4 * q + 2] = b.x; tv[4 * q + 3] = b.y;
            }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int u = (wave + 8 * t) * 32 + S.u0 + (r >> 2) * 8 + (r & 3);
            const double be = S.prm(1)[u], ga = S.prm(2)[u];
            const double s = sigmoid<double>(be * tv[r]);
            h[t][r] *= ga + (1.0 - ga) * (s + be * tv[r] * s * (1.0 - s));
            pin(h[t][r]);
            if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);
        }
    };
    // the output layer: n_pad inputs in blocks of 512
    const int KB = n_pad / 32;
    if (N.out.W) {
        const DigitLayer& B = N.hid[A.n_hidden - 1];
        S.prm(1)[tid] = B.beta[tid];
        S.prm(2)[tid] = B.gamma[tid];
    }
    const i32x4_t* wt = N.out.W + (int64_t)wave * KB * DM_STEP + lane;
    int* sums = reinterpret_cast<int*>(S.rows64() + DM_MAXBLOCKS * DG_ROWS);
    S.load_w(N.out.W ? wt : N.hid[A.n_hidden - 1].W + (int64_t)wave * 16 * DM_STEP + lane);
    if (!N.out.W) __syncthreads();                       // the row maxima are cleared
    for (int k0 = 0; k0 < n_pad && N.out.W; k0 += DG_K) {
        const int kc = min(DG_K, n_pad - k0), nkb = kc / 32;
        PlaneRows R;
        R.load(N.delta, n_pad, m0, rows, k0, kc, wave, lane);
        if (k0) __syncthreads();                         // every wave past its reads of the planes
        double* factors = S.rows64() + k0 / DG_K * DG_ROWS;
        R.store(lds + DM_PLANES, factors, sums + k0 / DG_K * DG_ROWS, kc, wave, lane);
        S.prm(3)[tid] = N.out.back[(int64_t)(k0 / DG_K) * DM_H + tid];
        __syncthreads();
        S.back = factors[S.row];
        S.load_x();
        const i32x4_t* wk = wt + (int64_t)(k0 / 32) * DM_STEP;
        const i32x4_t* wn = k0 + DG_K < n_pad ? wk + 16 * DM_STEP
                                              : N.hid[A.n_hidden - 1].W + (int64_t)wave * 16 * DM_STEP + lane;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const i32x4_t* wp = wk + (int64_t)t * 8 * KB * DM_STEP;
            S.tile<true>(wp, t == 0 ? wk + (int64_t)8 * KB * DM_STEP : wn, nkb);
            // the running sums of the blocks wait in the output's place (the
            // lane's own elements): 64 registers of them would spill the loops
            double v[16];
            S.sums(v);
#pragma unroll
            for (int r = 0; r < 16; ++r)
                v[r] = digit_product(v[r], S.back, S.prm(3)[(wave + 8 * t) * 32 + S.u0 + (r >> 2) * 8 + (r & 3)]);
            if (!valid) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                double2* o = S.units(N.y + m0 * DM_H, t, q);
                double2 a = make_double2(0.0, 0.0), b = a;
                if (k0) { a = o[0]; b = o[1]; }
                o[0] = make_double2(a.x + v[4 * q], a.y + v[4 * q + 1]);
                o[1] = make_double2(b.x + v[4 * q + 2], b.y + v[4 * q + 3]);
            }
        }
    }
    // rows that digits do not serve, all their blocks
    if (N.out.W) {
        const double* factors = S.rows64() + S.row;
        const bool served = n_pad > DG_K ? digit_row(factors, sums + S.row, DG_ROWS, n_pad, N.out.minimum)
                                         : factors[0] == 0.0 || (factors[0] > 0.0 && sums[S.row] >= N.out.minimum);
        S.odd = (uint32_t)__ballot(valid && !served);
        for (int k0 = 0; k0 < n_pad && __builtin_expect(S.odd != 0, 0); k0 += DG_K)
            S.products64([&](int r, double* place) {
                place[tid] = k0 + tid < n_pad ? N.delta[(m0 + r) * n_pad + k0 + tid] : 0.0;
            }, N.out.Wk + (int64_t)k0 * DM_H, DM_H, A.N_out - k0, DM_H, N.y + m0 * DM_H, DM_H, k0 > 0);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            double2 a = make_double2(0.0, 0.0), b = a;
            if (valid) {
                const double2* o = S.units(N.y + m0 * DM_H, t, q);
                a = o[0];
                b = o[1];
            }
            h[t][4 * q] = a.x; h[t][4 * q + 1] = a.y; h[t][4 * q + 2] = b.x; h[t][4 * q + 3] = b.y;
        }
        if (N.out.W) through(N.hid[A.n_hidden - 1].t, t);
    }
    // the hidden layers: l's W^T takes delta of hidden GEMM layer l to the layer below (l - 1, or the first layer)
    const int nkb = DM_H / 32;
    int p = 0;
    for (int l = A.n_hidden - 1; l >= 0; --l) {
        const DigitLayer& D = N.hid[l];
        const double be = l > 0 ? N.hid[l - 1].beta[tid] : N.be1[tid], ga = l > 0 ? N.hid[l - 1].gamma[tid] : N.ga1[tid];
        const double wb = D.back[tid];
        S.to_planes(h, p, valid, D.minimum, [&]() {
            S.prm(1)[tid] = be;
            S.prm(2)[tid] = ga;
            S.prm(3)[tid] = wb;
        });
        p ^= 1;
        if (__builtin_expect(S.odd != 0, 0)) S.products64(h, D.Wk, DM_H, DM_H, N.y64 + m0 * DM_H, DM_H);
        const i32x4_t* wk = D.W + (int64_t)wave * nkb * DM_STEP + lane;
        const i32x4_t* wn = (l > 0 ? N.hid[l - 1].W : D.W) + (int64_t)wave * nkb * DM_STEP + lane;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            S.tile<true>(wk + (int64_t)t * 8 * nkb * DM_STEP, t == 0 ? wk + (int64_t)8 * nkb * DM_STEP : wn, nkb);
            S.sums(h[t]);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int u = (wave + 8 * t) * 32 + S.u0 + (r >> 2) * 8 + (r & 3);
                h[t][r] = digit_product(h[t][r], S.back, S.prm(3)[u]);
            }
            if (__builtin_expect(S.odd != 0, 0)) S.take64(N.y64 + m0 * DM_H, t, h[t]);
            through(l > 0 ? N.hid[l - 1].t : N.t1, t);
        }
    }
    if (!valid) return;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            double2* o = S.units(N.y + m0 * DM_H, t, q);
            o[0] = make_double2(h[t][4 * q], h[t][4 * q + 1]);
            o[1] = make_double2(h[t][4 * q + 2], h[t][4 * q + 3]);
        }
}

// Networks the one-kernel forms take: every hidden width 512, at most six
// hidden GEMM layers; batches whose row blocks fill 13/32 of the CUs (the
// adjoint: 5/16).  A network takes one workgroup the same time whatever the
// batch, and the layer-by-layer launches, which split each layer over all CUs,
// grow with it.  One network, layered against one kernel, us: 2 500 outputs
// forward 301 / 318 at 2 880 rows, 313 / 319 at 3 520, 509 / 333 at 4 160, and
// adjoint 307 / 340 at 2 240, 345 / 342 at 2 880, 390 / 345 at 3 520; 200
// outputs forward 188 / 186 at 2 880, 208 / 187 at 3 520, and adjoint
// 116 / 176 at 1 600, 197 / 176 at 2 240, 213 / 176 at 2 880.
static bool digit_one_kernel(const ns_model* m, const Net& n0, int G, int64_t rows, bool back) {
    if (!(back ? n0.digits_back : n0.digits) || n0.n_layers < 3 || n0.n_layers - 2 > DM_MAXHID) return false;
    for (int l = 1; l < n0.n_layers; ++l)
        if (n0.dims[l] != DM_H) return false;
    if (back && n0.layers[n0.n_layers - 1]->n_pad > DM_MAXBLOCKS * DG_K) return false;
    return (rows + DG_ROWS - 1) / DG_ROWS * G * 32 >= (back ? 10 : 13) * (int64_t)device_cus(m->device);
}

bool emulator_forward_digits(ns_model* m, const int* nets, int G, const double* theta, int64_t ld, int64_t B,
                             void* const* outs, int64_t ldo, const int* is_log, double* tsave, size_t net_stride,
                             size_t slot_stride, const int* count, hipStream_t s) {
    const Net& n0 = *m->nets[nets[0]];
    const int L = n0.n_layers, rpw = n0.out_mu_rows;
    const int64_t rows = B * rpw;
    if (!digit_one_kernel(m, n0, G, rows, false)) return false;
    DigitArgs A{};
    A.n_hidden = L - 2;
    A.n_in = n0.dims[0];
    A.N_out = n0.dims[L];
    A.n_pad = n0.layers[L - 1]->n_pad;
    A.mu_rows = rpw;
    A.nrb = (int)((rows + DG_ROWS - 1) / DG_ROWS);
    A.ldo = ldo;
    m->ws_act[0].ensure((size_t)G * rows * DM_H * sizeof(double));
    for (int g = 0; g < G; ++g) {
        const Net& net = *m->nets[nets[g]];
        DigitNet& N = A.net[g];
        N.y64 = m->ws_act[0].as<double>() + (size_t)g * rows * DM_H;
        const Layer& l1 = *net.layers[0];
        N.W1 = l1.W64.as<double>(); N.b1 = l1.b64.as<double>();
        N.be1 = l1.beta64.as<double>(); N.ga1 = l1.gamma64.as<double>();
        N.shift = net.in_shift.as<double>();
        N.scale = net.in_scale.as<double>();
        N.t1 = tsave ? tsave + g * net_stride : nullptr;
        for (int l = 1; l < L; ++l) {
            const Layer& ly = *net.layers[l];
            DigitLayer& D = l < L - 1 ? N.hid[l - 1] : N.out;
            D.W = ly.Wd.as<i32x4_t>();
            D.back = ly.wback.as<double>();
            NS_CHECK(D.W && D.back, NS_E_UNSUPPORTED, "network without digit tiles");
            D.Wk = ly.WT64.as<double>();
            D.minimum = ly.dmin;
            D.b = ly.b64.as<double>();
            D.beta = ly.beta64.as<double>();
            D.gamma = ly.gamma64.as<double>();
            D.t = tsave && l < L - 1 ? tsave + g * net_stride + l * slot_stride : nullptr;
        }
        N.mu = net.out_mu64.as<double>();
        N.sigma = net.out_sigma64.as<double>();
        N.y = static_cast<double*>(outs[g]);
        N.is_log = is_log[g];
    }
    TraceScope ts(m, s, "mlp_i8_f64");
    const dim3 grid((unsigned)(A.nrb * G));
    auto go = [&](auto kern) {
        if (m->lds_attr_set.insert((const void*)kern).second)
            NS_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, DM_LDS_BYTES));
        hipLaunchKernelGGL(kern, grid, dim3(512), DM_LDS_BYTES, s, theta, ld, rows, rpw, m->emu_src_d.as<int>(),
                           m->emu_fix_d.as<double>(), m->znodes_d.as<double>(), A, count);
    };
    if (A.n_in <= 8) tsave ? go(mlp_i8_kernel<8, true>) : go(mlp_i8_kernel<8, false>);
    else tsave ? go(mlp_i8_kernel<16, true>) : go(mlp_i8_kernel<16, false>);
    NS_HIP(hipGetLastError());
    return true;
}

bool emulator_backward_digits(ns_model* m, const int* nets, int G, int64_t B, const double* delta, double* delta1,
                              size_t dstride, const double* tsave, size_t net_stride, size_t slot_stride,
                              hipStream_t s) {
    const Net& n0 = *m->nets[nets[0]];
    const int L = n0.n_layers, rpw = n0.out_mu_rows;
    const int64_t rows = B * rpw;
    if (!digit_one_kernel(m, n0, G, rows, true)) return false;
    DigitArgs A{};
    A.n_hidden = L - 2;
    A.N_out = n0.dims[L];
    A.nrb = (int)((rows + DG_ROWS - 1) / DG_ROWS);
    m->ws_act[0].ensure((size_t)G * rows * DM_H * sizeof(double));
    for (int g = 0; g < G; ++g) {
        const Net& net = *m->nets[nets[g]];
        DigitNet& N = A.net[g];
        N.y64 = m->ws_act[0].as<double>() + (size_t)g * rows * DM_H;
        const Layer& l1 = *net.layers[0];
        N.be1 = l1.beta64.as<double>(); N.ga1 = l1.gamma64.as<double>();
        double* t = const_cast<double*>(tsave) + g * net_stride;
        N.t1 = t;
        for (int l = 1; l < L; ++l) {
            const Layer& ly = *net.layers[l];
            DigitLayer& D = l < L - 1 ? N.hid[l - 1] : N.out;
            D.W = ly.WTd.as<i32x4_t>();
            D.back = ly.wtback.as<double>();
            NS_CHECK((D.W && D.back) || (l == L - 1 && !n0.digits_out), NS_E_UNSUPPORTED, "network without digit tiles");
            D.Wk = ly.W64.as<double>();
            D.minimum = ly.dtmin;
            D.beta = ly.beta64.as<double>();
            D.gamma = ly.gamma64.as<double>();
            D.t = l < L - 1 ? t + l * slot_stride : nullptr;
        }
        N.delta = delta + g * dstride;
        N.y = delta1 + g * dstride;
    }
    TraceScope ts(m, s, "mlp_i8_f64_adjoint");
    const auto kern = mlp_i8_back_kernel;
    if (m->lds_attr_set.insert((const void*)kern).second)
        NS_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, DM_LDS_BYTES));
    hipLaunchKernelGGL(kern, dim3((unsigned)(A.nrb * G)), dim3(512), DM_LDS_BYTES, s, rows, n0.layers[L - 1]->n_pad, A);
    NS_HIP(hipGetLastError());
    return true;
}

}  // namespace nsmi

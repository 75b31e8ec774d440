// Which FP64 layers run as int8 digit products (gemm_i8.h), and which of their
// input rows: the host's part of the decision, from the weights alone.
//
// Digits hold every entry of a row (or of a unit's weights) to one absolute
// step, 2^-55 of a bound B just above the block's largest entry (the next power
// of two for rows; for weights at most 1/60 above the entry itself), and the
// dropped digit products are of that size too.  The error of one output is so
// proportional to the product of two bounds, while an FP64 chain's is
// proportional to the products present, |x w| in the 2-norm.  With
//   f = rms over units of (B sqrt(inputs) / |w|)
//       / rms weight of the faintest inputs (units scaled to rms 1)
// (the faintest thirty-second of the inputs: a row whose large entries all meet
// those) and s = f B 0.8 sqrt(inputs) / sum |x| for the row (for normal entries
// f B / |x|; the sum, because rows of few or a few large entries also make FP64
// sums of few roundings), digits' error is up to 0.37 s of that of an FP64 chain
// over 256 to 512 inputs and 0.4 s over 128, on average 0.3 s: measured against
// extended precision over normal, rectified, exponential, log-normal,
// Student-t, sparse, bump-shaped and decaying rows, rows of 1 to 48 entries and
// of one entry 6 to 40 times the others, against normal, uniform, Laplace and
// Student-t weights (with |x| in the place of the sum, rows of two entries reach
// hundreds).  Rows with s above DG_ROW_LIMIT = 2.5 therefore take FP64 products,
// row by row, in the kernels (sum |x| from the leading digits' magnitudes, whose
// unit is B / 128).  A normal row of 512 has s of 0.6 to 1.3 against normal
// weights; of 60 000 rows of activations and of hidden and CMB output deltas of
// the emulators none exceeded 2.1, of the shear's output deltas 95% did.
//
// A layer whose weights leave most rows to FP64, or whose units hold mostly
// zeros (an error bound by the largest entries would then exceed an FP64
// sum's, which has few terms), runs on FP64 products altogether.
#include <algorithm>
#include <cmath>
#include <vector>

#include "nsmi.h"

namespace nsmi {

constexpr int BLOCK = 512;              // inputs that share a scale (DG_K)
constexpr double DG_ROW_LIMIT = 2.5;

// Bound of a block of weights of which mx is the largest magnitude: 128 times
// the step of the leading digit, as the weights' kernel chooses it.
static double bound_of(double mx) {
    int e;
    const double m = std::frexp(mx / 127.0, &e);
    return 128.0 * std::ldexp(std::ceil(256.0 * m) / 256.0, e);
}

int digit_row_minimum(const double* W, int units, int inputs) {
    if (inputs < 128) return 0;                           // short sums: FP64's errors are the smaller (up to 0.7 s)
    std::vector<double> faint(inputs, 0.0);               // sum over units of (w / norm of the unit)^2
    std::vector<double> worst((inputs + BLOCK - 1) / BLOCK, 0.0);   // per block: sum of (B sqrt(n) / |w|)^2
    std::vector<int> live(worst.size(), 0);
    int units_live = 0;
    for (int u = 0; u < units; ++u) {
        const double* w = W + (int64_t)u * inputs;
        double total = 0.0;
        for (int k0 = 0, b = 0; k0 < inputs; k0 += BLOCK, ++b) {
            const int n = std::min(BLOCK, inputs - k0);
            // four sums side by side: one would wait for itself at each weight
            double mx4[4] = {}, ss4[4] = {};
            for (int k = 0; k + 4 <= n; k += 4)
                for (int e = 0; e < 4; ++e) {
                    const double v = std::fabs(w[k0 + k + e]);
                    mx4[e] = mx4[e] < v ? v : mx4[e];
                    ss4[e] += v * v;
                }
            for (int k = n & ~3; k < n; ++k) {
                mx4[0] = std::max(mx4[0], std::fabs(w[k0 + k]));
                ss4[0] += w[k0 + k] * w[k0 + k];
            }
            const double mx = std::max(std::max(mx4[0], mx4[1]), std::max(mx4[2], mx4[3]));
            const double ss = (ss4[0] + ss4[1]) + (ss4[2] + ss4[3]);
            if (ss == 0.0 && mx == 0.0) continue;         // exact in digits
            // (not finite: the sum is not)
            if (!(ss < INFINITY) || !(mx > 1e-140 && mx < 1e140) || mx * mx * n > 64.0 * ss) return 0;
            total += ss;
            const double tiny = std::sqrt(ss / n) / 32.0;
            int present = 0;
            for (int k = k0; k < k0 + n; ++k) present += std::fabs(w[k]) >= tiny;
            if (2 * present < n) return 0;
            const double q = bound_of(mx);
            worst[b] += q * q * n / ss;
            ++live[b];
        }
        if (total == 0.0) continue;
        ++units_live;
        const double per = 1.0 / total;
        for (int k = 0; k < inputs; ++k) faint[k] += w[k] * w[k] * per;
    }
    if (units_live == 0) return 1;                        // no weights at all: exact zeros
    double most = 0.0;
    for (size_t b = 0; b < worst.size(); ++b)
        if (live[b]) most = std::max(most, worst[b] / live[b]);
    std::sort(faint.begin(), faint.end());
    const int nf = std::max(1, inputs / 32);
    double low = 0.0;
    for (int k = 0; k < nf; ++k) low += faint[k] * inputs / nf / units_live;
    if (!(low > 0.0)) return 0;
    const double f2 = most / low;
    // rows of which the largest entry is four times the rms should pass, at
    // the middle of the powers of two: f 1.5 4 / sqrt(inputs) <= limit, with some room
    if (f2 > 0.36 * std::min(inputs, BLOCK)) return 0;
    return (int)std::ceil(128.0 * 0.8 * std::sqrt(f2 * inputs) / DG_ROW_LIMIT);
}

// W^T [K x N] of W [N x K] into T, in squares that stay in cache.
static const double* transposed(const double* W, int N, int K, std::vector<double>& T) {
    if (T.size() < (size_t)N * K) T.resize((size_t)N * K);
    for (int n0 = 0; n0 < N; n0 += 32)
        for (int k0 = 0; k0 < K; k0 += 32)
            for (int k = k0; k < std::min(K, k0 + 32); ++k)
                for (int n = n0; n < std::min(N, n0 + 32); ++n) T[(size_t)k * N + n] = W[(size_t)n * K + k];
    return T.data();
}

bool digit_shape(const std::vector<int>& dims) {
    const int L = (int)dims.size() - 1;
    if (L < 2) return false;
    for (int l = 1; l < L; ++l)
        if (dims[l] < 256) return false;
    return true;
}

DigitPlan digit_plan(const ns_model_desc* D) {
    DigitPlan p;
    if (!D->nets || D->n_nets < 1) return p;
    p.forward = p.back = p.out = true;
    p.nets.resize(D->n_nets);
    std::vector<double> turned;
    for (int i = 0; i < D->n_nets && p.forward; ++i) {
        const ns_net_desc& nd = D->nets[i];
        DigitPlan::Rows& r = p.nets[i];
        if (nd.n_layers < 2 || !nd.dims || !nd.W) return DigitPlan{};
        const std::vector<int> dims(nd.dims, nd.dims + nd.n_layers + 1);
        for (int v : dims)
            if (v < 1) return DigitPlan{};
        for (int l = 0; l < nd.n_layers; ++l)
            if (!nd.W[l]) return DigitPlan{};
        if (!digit_shape(dims)) return DigitPlan{};
        r.forward.assign(nd.n_layers, 0);
        r.back.assign(nd.n_layers, 0);
        for (int l = 1; l < nd.n_layers; ++l) {
            const int K = dims[l], N = dims[l + 1];
            const bool last = l == nd.n_layers - 1;
            r.forward[l] = digit_row_minimum(nd.W[l], N, K);
            if (!r.forward[l]) return DigitPlan{};
            if (last && D->kind == NS_MODEL_SHEAR) p.out = false;
            if (last ? !p.out : !p.back) continue;
            r.back[l] = digit_row_minimum(transposed(nd.W[l], N, K, turned), K, N);
            if (!r.back[l]) (last ? p.out : p.back) = false;
        }
    }
    return p;
}

}  // namespace nsmi

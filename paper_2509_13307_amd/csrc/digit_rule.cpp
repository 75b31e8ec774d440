// Which FP64 layers run as int8 digit products (gemm_i8.h), and which of their
// input rows: the host's part of the decision, from the weights alone.
//
// Digits hold every entry of a row (or of a unit's weights) to one absolute
// step, 2^-55 of a bound B just above the block's largest entry (the next power
// of two for rows; for weights 1/127 to 1/128 above the entry itself), and the
// dropped digit products are of that size too.  The error of one output is so
// proportional to the product of two bounds, while an FP64 chain's is
// proportional to the products present, |x w| in the 2-norm.  With
//   f = rms over units of (B sqrt(inputs) / |w|)
//       / rms weight of the faintest inputs (units scaled to rms 1)
// (the faintest thirty-second of the inputs: a row whose large entries all meet
// those) and s = f B / |x| for the row, digits have 0.28 to 0.37 s of the error
// of an FP64 chain over 256 to 512 inputs: measured against extended precision
// over normal, rectified, exponential, log-normal, Student-t, bump-shaped and
// decaying rows (sparse ones up to 0.5 s) against normal, uniform, Laplace and
// Student-t weights.  Rows with s above DG_ROW_LIMIT = 2.75 therefore take FP64
// products, row by row, in the kernels (|x|^2 from the sum of squares of the
// leading digits, whose unit is B / 128).  A normal row of 512 has s of 0.6 to
// 1.3 against normal weights; of 50 000 activation rows of the emulators none
// reached 2.4.
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
constexpr double DG_ROW_LIMIT = 2.75;

// Bound of a block of weights of which mx is the largest magnitude: 128 times
// the step of the leading digit, as the weights' kernel chooses it.
static double bound_of(double mx) {
    int e;
    const double m = std::frexp(mx / 127.0, &e);
    return 128.0 * std::ldexp(std::ceil(256.0 * m) / 256.0, e);
}

int digit_row_minimum(const double* W, int units, int inputs, int64_t su, int64_t si) {
    std::vector<double> faint(inputs, 0.0);               // sum over units of (w / rms of the unit)^2
    double worst = 0.0;                                   // largest of the blocks' mean (B sqrt(n) / |w|)^2
    std::vector<double> sq(units, 0.0);
    for (int k0 = 0; k0 < inputs; k0 += BLOCK) {
        const int n = std::min(BLOCK, inputs - k0);
        double sum = 0.0;
        int live = 0;
        for (int u = 0; u < units; ++u) {
            const double* w = W + u * su + k0 * si;
            double mx = 0.0, ss = 0.0;
            for (int k = 0; k < n; ++k) {
                const double v = std::fabs(w[k * si]);
                if (!std::isfinite(v)) return 0;
                mx = std::max(mx, v);
                ss += v * v;
            }
            sq[u] += ss;
            if (mx == 0.0) continue;                      // exact in digits
            if (!(mx > 1e-140 && mx < 1e140) || mx * mx * n > 64.0 * ss) return 0;
            const double tiny = std::sqrt(ss / n) / 32.0;
            int present = 0;
            for (int k = 0; k < n; ++k) present += std::fabs(w[k * si]) >= tiny;
            if (2 * present < n) return 0;
            const double q = bound_of(mx);
            sum += q * q * n / ss;
            ++live;
        }
        if (live) worst = std::max(worst, sum / live);
    }
    if (worst == 0.0) return 1;                           // no weights at all: exact zeros
    int live = 0;
    for (int u = 0; u < units; ++u) {
        if (sq[u] == 0.0) continue;
        ++live;
        for (int k = 0; k < inputs; ++k) {
            const double v = W[u * su + k * si];
            faint[k] += v * v * inputs / sq[u];
        }
    }
    std::sort(faint.begin(), faint.end());
    const int nf = std::max(1, inputs / 32);
    double low = 0.0;
    for (int k = 0; k < nf; ++k) low += faint[k] / nf / live;
    if (!(low > 0.0)) return 0;
    const double f2 = worst / low;
    // rows of which the largest entry is four times the rms should pass, at
    // the middle of the powers of two: f 1.5 4 / sqrt(inputs) <= limit, with some room
    if (f2 > 0.36 * std::min(inputs, BLOCK)) return 0;
    return (int)std::ceil(128.0 * 128.0 * f2 / (DG_ROW_LIMIT * DG_ROW_LIMIT));
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
            r.forward[l] = digit_row_minimum(nd.W[l], N, K, K, 1);
            if (!r.forward[l]) return DigitPlan{};
            if (last && D->kind == NS_MODEL_SHEAR) p.out = false;
            if (last ? !p.out : !p.back) continue;
            r.back[l] = digit_row_minimum(nd.W[l], K, N, 1, K);
            if (!r.back[l]) (last ? p.out : p.back) = false;
        }
    }
    return p;
}

}  // namespace nsmi

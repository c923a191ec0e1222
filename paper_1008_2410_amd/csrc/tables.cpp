// Radius-scaled translation operators for p-term expansions (host generation, FP64,
// uploaded once per p as FP64 and FP32 copies).
//
// With multipoles scaled as a_m / w^m and locals as b_l w^(l+1) (w = cell width of
// the level), the textbook translations become level independent:
//   M2M (stage 5): A_m = sum_{k<=m} C(m,k) d^(m-k) 2^-k a_k,           d = (c_child - c_parent)/w_parent
//   M2L (stage 6): b_l = sum_m (-1)^l C(l+m,m) delta^-(l+m+1) a_m,     delta = (c_T - c_S)/w
//   L2L (stage 7): b_k = sum_{l>=k} C(l,k) d^(l-k) 2^-(k+1) b_l
// derived from the multipole coefficients of section "Complexity Estimates" and the
// expansion 1/(D + u - v) = sum_{l,m} (-1)^l C(l+m,l) u^l v^m / D^(l+m+1).
#include <complex>
#include <map>
#include <mutex>
#include <vector>

#include "fmm_internal.h"
#include "translate.h"

namespace fmm {

namespace {

using cd = std::complex<double>;

std::vector<double> binomials(int nmax)
{
    std::vector<double> c((size_t)(nmax + 1) * (nmax + 1), 0.0);
    for (int n = 0; n <= nmax; ++n) {
        c[(size_t)n * (nmax + 1)] = 1.0;
        for (int k = 1; k <= n; ++k)
            c[(size_t)n * (nmax + 1) + k] = c[(size_t)(n - 1) * (nmax + 1) + k - 1] + c[(size_t)(n - 1) * (nmax + 1) + k];
    }
    return c;
}

cd child_offset(int q) { return cd(((q & 1) - 0.5) * 0.5, ((q >> 1) - 0.5) * 0.5); }

}  // namespace

void free_tables(Tables &tb)
{
    hipFree(tb.mfma_f);
    hipFree(tb.mfma_d);
    hipFree(tb.mfma_entries);
    hipFree(tb.zero_row);
    tb = Tables{};
}

int upload_tables(Tables &tb, int p, std::string &err)
{
    if (tb.p == p) return 0;
    free_tables(tb);
    const int nb = 2 * p;
    const std::vector<double> C = binomials(nb);
    auto binom = [&](int n, int k) { return C[(size_t)n * (nb + 1) + k]; };

    // Real 2p x 2p embedding: y = x R with x, y interleaved (re, im),
    // R[2m][2l] = Re T_lm, R[2m+1][2l] = -Im T_lm, R[2m][2l+1] = Im T_lm, R[2m+1][2l+1] = Re T_lm.
    const size_t ks = trans_ks(p), nc = trans_cols64(p), kf = trans_kf(p), nf = trans_cols32(p);
    std::vector<double> md((size_t)57 * 4 * nc * ks, 0.0);
    std::vector<float> mf((size_t)57 * 2 * nf * kf, 0.0f);
    auto put = [&](int slot, int m, int l, cd v) {  // input coefficient m, output coefficient l
        const size_t k[2] = {(size_t)(2 * m), (size_t)(2 * m + 1)}, c[2] = {(size_t)(2 * l), (size_t)(2 * l + 1)};
        const double r[2][2] = {{v.real(), v.imag()}, {-v.imag(), v.real()}};
        for (int i = 0; i < 2; ++i)
            for (int j = 0; j < 2; ++j) {
                // lane and step of the element, and its place among the lane's vector loads
                const size_t ld = k[i] / ks * 16 + c[j] % 16, sd = k[i] % ks;
                const size_t lf = k[i] / kf * 32 + c[j] % 32, sf = k[i] % kf;
                md[((((size_t)slot * (nc / 16) + c[j] / 16) * (ks / 2) + sd / 2) * 64 + ld) * 2 + sd % 2] = r[i][j];
                mf[((((size_t)slot * (nf / 32) + c[j] / 32) * (kf / 4) + sf / 4) * 64 + lf) * 4 + sf % 4] =
                    (float)r[i][j];
            }
    };
    for (int q = 0; q < 4; ++q) {
        const cd d = child_offset(q);
        for (int m = 0; m < p; ++m)  // M2M: parent coefficient m from child q's coefficient k
            for (int k = 0; k <= m; ++k)
                put(53 + q, k, m, binom(m, k) * std::pow(d, m - k) * std::ldexp(1.0, -k));
        for (int k = 0; k < p; ++k)  // L2L: child q's coefficient k from parent coefficient l
            for (int l = k; l < p; ++l)
                put(49 + q, l, k, binom(l, k) * std::pow(d, l - k) * std::ldexp(1.0, -(k + 1)));
    }
    for (int dx = -3; dx <= 3; ++dx)
        for (int dy = -3; dy <= 3; ++dy) {
            if (dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1) continue;
            const cd inv = 1.0 / cd(dx, dy);
            // powers inv^n, n = 1 .. 2p-1, by repeated multiplication
            std::vector<cd> pw(2 * p + 1);
            pw[0] = 1.0;
            for (int n = 1; n <= 2 * p; ++n) pw[n] = pw[n - 1] * inv;
            for (int m = 0; m < p; ++m)
                for (int l = 0; l < p; ++l)
                    put((dx + 3) * 7 + (dy + 3), m, l, ((l & 1) ? -1.0 : 1.0) * binom(l + m, m) * pw[l + m + 1]);
        }
    // Entry lists of the MFMA kernel: per parity class (qx, qy) the 27 interaction-list
    // source offsets (dx in [-2-qx, 3-qx], dy in [-2-qy, 3-qy] outside the 3x3 block) and
    // the L2L entry; then the four M2M children.  delta = (c_T - c_S)/w = (-dx, -dy).
    std::vector<int4> ent;
    for (int q = 0; q < 4; ++q) {
        const int qx = q & 1, qy = q >> 1;
        for (int dy = -2 - qy; dy <= 3 - qy; ++dy)
            for (int dx = -2 - qx; dx <= 3 - qx; ++dx) {
                if (dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1) continue;
                ent.push_back(make_int4(dx, dy, (3 - dx) * 7 + (3 - dy), 0));
            }
        ent.push_back(make_int4(0, 0, 49 + q, 1));
    }
    for (int q = 0; q < 4; ++q) ent.push_back(make_int4(q, 0, 53 + q, 2));
    int rc = 0;
    {
        if (device_malloc((void **)&tb.mfma_f, mf.size() * sizeof(float)) != hipSuccess ||
            device_malloc((void **)&tb.mfma_d, md.size() * sizeof(double)) != hipSuccess) {
            err = "device allocation failed: operator tables";
            rc = -2;
        } else if (hipMemcpy(tb.mfma_f, mf.data(), mf.size() * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
                   hipMemcpy(tb.mfma_d, md.data(), md.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess) {
            err = "hipMemcpy failed for operator tables";
            rc = -3;
        }
    }
    if (!rc) {
        if (device_malloc((void **)&tb.mfma_entries, ent.size() * sizeof(int4)) != hipSuccess) {
            err = "device allocation failed: operator tables";
            rc = -2;
        } else if (hipMemcpy(tb.mfma_entries, ent.data(), ent.size() * sizeof(int4), hipMemcpyHostToDevice) !=
                   hipSuccess) {
            err = "hipMemcpy failed for operator tables";
            rc = -3;
        }
    }
    if (!rc) {
        if (device_malloc((void **)&tb.zero_row, 128 * sizeof(double)) != hipSuccess ||
            hipMemset(tb.zero_row, 0, 128 * sizeof(double)) != hipSuccess) {
            err = "allocation of the zero row failed";
            rc = -2;
        }
    }
    if (rc) {
        free_tables(tb);
        return rc;
    }
    tb.p = p;
    return 0;
}

int shared_tables(int device, int p, const Tables **out, std::string &err, bool create)
{
    static std::mutex mu;
    static std::map<std::pair<int, int>, Tables> cache;  // node addresses stay valid
    std::lock_guard<std::mutex> lock(mu);
    auto it = cache.find({device, p});
    if (it == cache.end()) {
        if (!create) {
            err = "the expansion tables of p = " + std::to_string(p) + " are not on this device yet";
            return -5;
        }
        Tables tb;
        if (int rc = upload_tables(tb, p, err)) return rc;
        it = cache.emplace(std::make_pair(device, p), tb).first;
    }
    *out = &it->second;
    return 0;
}

}  // namespace fmm

// Exact solvers (the references of Sec. VII, extended past 2x2): the
// Hamiltonian of Eq. (effi) applied to a state, its ground energy by the
// Lanczos recurrence, and stepwise exact evolution exp(-i dt H(s_k)) by a
// Krylov (Lanczos) basis per step.  Every vector operation runs on the
// device; the host only sequences launches and works on the small
// tridiagonal matrices.
#include <string.h>

#include <algorithm>
#include <cmath>
#include <complex>
#include <vector>

#include "z2h_runtime.h"
#include "z2h_solvers.h"

using namespace z2h;
using namespace z2h::rt;

namespace {

constexpr int kCheckEvery = 8;   // Lanczos iterations between convergence checks
static_assert(kHamWorkersMax <= kVecBlocks, "the |w|^2 partials of a fused pass fit the vector-kernel slots");

size_t state_bytes(const Plan &P) { return P.esize << P.n; }

int ham_workers(const GroupGeom &g) {
    const uint64_t tiles = 1ull << g.tiles_log2;
    return (int)std::min<uint64_t>(tiles, (uint64_t)kHamWorkersMax);
}

// Groups of qubits a Hamiltonian pass is made for, and the workgroups (one
// partial each) of the passes over a group.
bool ham_wave(const Plan &P) { return ham_wave_blocks(P.c128, P.n, false) > 0; }
int ham_groups(const Plan &P) { return ham_wave(P) ? 2 : P.K; }
int ham_workers(const Plan &P, int group) {
    return ham_wave(P) ? ham_wave_blocks(P.c128, P.n, group > 0) : ham_workers(P.geom[group]);
}

unsigned vec_blocks(const Plan &P) {
    const uint64_t need = ((1ull << P.n) + 255) / 256;
    return (unsigned)std::min<uint64_t>(need, (uint64_t)kVecBlocks);
}

// XCD-major order for the passes over the groups the plan selects, on
// grids of eight or more workers per CU (as the Trotter pass kernels).
static int ham_xcd(const Plan &P, int group, int workers) {
    return ((P.xcd >> group) & 1) && workers >= 8 * 256 ? 1 : 0;
}

// Pass i, over group gi.
hipError_t launch_pass(const Plan &P, HamArgs &a, int gi, int i, hipStream_t s) {
    if (ham_wave(P)) return launch_ham_wave(i < 2 ? i : !a.lz ? 3 : a.g ? 4 : 2, a, s);
    const int w = ham_workers(P, gi);
    a.geom = P.geom[gi];
    a.xcd = ham_xcd(P, gi, w);
    return launch_ham(P.c128, a.geom.R, a, (unsigned)w, obs_lds_bytes(P, a.geom, a.geom.R), s);
}

// y = H x: passes over groups 0, 1, .., K-1, .., 1, 0 (one pass when K = 1).
// The last pass writes Re<x, y> partials to apart (if not null).
z2h_status ham_passes(const Plan &P, const void *x, void *y, const z2h_couplings &H, double *apart,
                      int *napart, hipStream_t s) {
    HamArgs a;
    memset(&a, 0, sizeof a);
    a.lat = P.lat;
    a.JA = H.JA;
    a.JB = H.JB;
    a.hx = H.hx;
    a.hz = H.hz;
    a.xscale = std::ldexp(1.0, -P.n);
    const int K = ham_groups(P), npass = 2 * K - 1;
    for (int i = 0; i < npass; ++i) {
        const int gi = i < K ? i : 2 * K - 2 - i;
        a.src = i == 0 ? x : y;
        a.dst = y;
        a.top = gi == K - 1;
        a.final_pass = i == npass - 1;
        a.x = a.final_pass ? x : nullptr;
        a.part = a.final_pass ? apart : nullptr;
        if (a.final_pass && napart) *napart = ham_workers(P, gi);
        hipError_t e = launch_pass(P, a, gi, i, s);
        if (e != hipSuccess) return fail(Z2H_ERR_HIP, "Hamiltonian pass failed: %s", hipGetErrorString(e));
    }
    return Z2H_OK;
}

// Scratch of the Lanczos recurrence inside a workspace.
struct LanczosWs {
    void *vec[kKrylovMax + 1];   // state-sized buffers
    double *apart, *apart_x, *wpart;
    LanczosCoef *coef;
};

size_t lanczos_carve(const Plan &P, int nvec, int ncoef, char *base, LanczosWs *L) {
    Carver c{base, 0};
    LanczosWs tmp;
    memset(&tmp, 0, sizeof tmp);
    for (int i = 0; i < nvec; ++i) tmp.vec[i] = c.take(state_bytes(P));
    tmp.apart = (double *)c.take(sizeof(double) * 2 * kVecBlocks);  // also the dot kernel's (Re, Im) pairs
    tmp.apart_x = (double *)c.take(sizeof(double) * kHamWorkersMax);
    tmp.wpart = (double *)c.take(sizeof(double) * kVecBlocks);
    tmp.coef = (LanczosCoef *)c.take(sizeof(LanczosCoef) * (size_t)ncoef);
    if (L) *L = tmp;
    return align256(c.off);
}

z2h_status norm_start(const Plan &P, const void *u, const LanczosWs &L, hipStream_t s) {
    VecArgs v;
    memset(&v, 0, sizeof v);
    v.u = u;
    v.nelem = 1ull << P.n;
    v.mode = 1;
    v.part = L.wpart;
    const unsigned nb = vec_blocks(P);
    hipError_t e = launch_vec(P.c128, v, nb, s);
    if (e == hipSuccess) {
        ScalarArgs sa;
        memset(&sa, 0, sizeof sa);
        sa.wpart = L.wpart;
        sa.nwpart = (int)nb;
        sa.mode = 1;
        sa.coef = L.coef;
        e = launch_scalar(sa, s);
    }
    if (e != hipSuccess) return fail(Z2H_ERR_HIP, "Lanczos start norm failed: %s", hipGetErrorString(e));
    return Z2H_OK;
}

z2h_status launch_scalar_k(const LanczosWs &L, const double *wpart, int k, int napart, int napart2, int nwpart, hipStream_t s) {
    ScalarArgs sa;
    memset(&sa, 0, sizeof sa);
    sa.apart = L.apart;
    sa.napart = napart;
    sa.apart2 = napart2 ? L.apart_x : nullptr;
    sa.napart2 = napart2;
    sa.wpart = wpart;
    sa.nwpart = nwpart;
    sa.k = k;
    sa.mode = 0;
    sa.coef = L.coef;
    hipError_t e = launch_scalar(sa, s);
    if (e != hipSuccess) return fail(Z2H_ERR_HIP, "Lanczos coefficient kernel failed: %s", hipGetErrorString(e));
    return Z2H_OK;
}

// Iterations whose last pass takes the coefficients from the partials
// themselves: the |w|^2 partials of two iterations fit the vector-kernel
// slots side by side (one half is read while the other is written).
bool coefs_inline(const Plan &P) { return ham_groups(P) > 1 && ham_workers(P, 0) <= kVecBlocks / 2; }

// One Lanczos iteration k: w = sigma_k (H u - alpha_k u) - beta_k sigma_{k-1} p
// written to w; coef[k].alpha and coef[k+1] (beta, sigma), the latter by the
// next iteration, or now if last.  With several
// groups the update is fused into the Hamiltonian's passes (alpha from the
// first and the top pass, w written by the last one); a one-group plan
// forms y = H u and updates in an elementwise kernel.
// acc (passes of two groups, k > 0): the Ritz vector takes u and p on the way.
struct RitzAcc {
    void *g;
    double sp, su;
    int first;
};
z2h_status lanczos_iter(const Plan &P, const z2h_couplings &H, int k, const void *u, const void *p, void *w,
                        void *y, const LanczosWs &L, bool last, hipStream_t s, const RitzAcc *acc = nullptr) {
    if (ham_groups(P) > 1) {
        const bool inl = coefs_inline(P);
        double *wpart = L.wpart + (inl && (k & 1) ? kVecBlocks / 2 : 0);
        HamArgs a;
        memset(&a, 0, sizeof a);
        a.lat = P.lat;
        a.JA = H.JA;
        a.JB = H.JB;
        a.hx = H.hx;
        a.hz = H.hz;
        a.xscale = std::ldexp(1.0, -P.n);
        const int K = ham_groups(P), npass = 2 * K - 1;
        const int nz = ham_workers(P, 0), nx = ham_workers(P, K - 1);
        for (int i = 0; i < npass; ++i) {
            const int gi = i < K ? i : 2 * K - 2 - i;
            a.src = i == 0 ? u : y;
            a.dst = y;
            a.top = gi == K - 1;
            a.final_pass = i == npass - 1;
            a.part_z = i == 0 ? L.apart : nullptr;
            a.part_x = gi == K - 1 ? L.apart_x : nullptr;
            if (a.final_pass) {
                a.x = u;
                a.lz = 1;
                a.p = k > 0 ? p : nullptr;
                a.use_prev = k > 0;
                a.w = w;
                a.part_w = wpart;
                a.record = inl;
                if (inl && k > 0) {
                    a.prev_w = L.wpart + (k & 1 ? 0 : kVecBlocks / 2);
                    a.nprev_w = nz;
                }
                a.apart_z = L.apart;
                a.napart_z = nz;
                a.apart_x = L.apart_x;
                a.napart_x = nx;
                a.coef = L.coef;
                a.k = k;
                if (acc) {
                    a.g = acc->g;
                    a.g_first = acc->first;
                    a.gs[0] = acc->sp;
                    a.gs[1] = acc->su;
                }
            }
            hipError_t e = launch_pass(P, a, gi, i, s);
            if (e != hipSuccess) return fail(Z2H_ERR_HIP, "Lanczos pass failed: %s", hipGetErrorString(e));
        }
        return inl && !last ? Z2H_OK : launch_scalar_k(L, wpart, k, nz, nx, nz, s);
    }
    int napart = 0;
    z2h_status st = ham_passes(P, u, y, H, L.apart, &napart, s);
    if (st) return st;
    VecArgs v;
    memset(&v, 0, sizeof v);
    v.y = y;
    v.u = u;
    v.p = k > 0 ? p : nullptr;
    v.w = w;
    v.nelem = 1ull << P.n;
    v.apart = L.apart;
    v.napart = napart;
    v.k = k;
    v.use_prev = k > 0;
    v.mode = 0;
    v.coef = L.coef;
    v.part = L.wpart;
    const unsigned nb = vec_blocks(P);
    hipError_t e = launch_vec(P.c128, v, nb, s);
    if (e != hipSuccess) return fail(Z2H_ERR_HIP, "Lanczos update failed: %s", hipGetErrorString(e));
    return launch_scalar_k(L, L.wpart, k, napart, 0, (int)nb, s);
}

// Both pointers valid and the byte ranges [a, a + na) and [b, b + nb) disjoint.
z2h_status check_pair(const void *a, size_t sa, const void *b, size_t sb, const char *na, const char *nb) {
    z2h_status st = validate_state_ptr(a, na);
    if (!st) st = validate_state_ptr(b, nb);
    if (st) return st;
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    if (x < y + sb && y < x + sa) return fail(Z2H_ERR_INVALID, "%s and %s overlap", na, nb);
    return Z2H_OK;
}

bool finite4(const z2h_couplings &c) {
    return std::isfinite(c.JA) && std::isfinite(c.JB) && std::isfinite(c.hx) && std::isfinite(c.hz);
}

// Number of eigenvalues below x of the symmetric tridiagonal matrix with
// diagonal a[0..m) and off-diagonal b[1..m) (Sturm count from the pivots of
// the LDL^T factorisation of T - x I).
int sturm_count(const double *a, const double *b, int m, double x) {
    int cnt = 0;
    double q = 1.0;
    for (int i = 0; i < m; ++i) {
        const double off = i > 0 ? b[i] * b[i] / q : 0.0;
        q = a[i] - x - off;
        if (q == 0.0) q = -1e-300;
        if (q < 0) ++cnt;
    }
    return cnt;
}

// Lowest eigenvalue by bisection inside the Gershgorin interval.
double tridiag_lowest(const double *a, const double *b, int m) {
    double lo = a[0], hi = a[0];
    for (int i = 0; i < m; ++i) {
        const double r = (i > 0 ? std::fabs(b[i]) : 0.0) + (i + 1 < m ? std::fabs(b[i + 1]) : 0.0);
        lo = std::min(lo, a[i] - r);
        hi = std::max(hi, a[i] + r);
    }
    for (int it = 0; it < 200 && hi - lo > 0.0; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (mid <= lo || mid >= hi) break;
        if (sturm_count(a, b, m, mid) >= 1)
            hi = mid;
        else
            lo = mid;
    }
    return 0.5 * (lo + hi);
}

// Eigen-decomposition of the symmetric tridiagonal T (diagonal a[0..m),
// off-diagonal b[1..m)) by implicit QR steps with Wilkinson's shift (Golub
// and Van Loan, Matrix Computations, sec. 8.3): T = Q diag(lam) Q^T, Q
// row-major (column l is the eigenvector of lam[l]).  The host waits for it
// between two steps of the exact evolution: cyclic Jacobi sweeps over the
// full matrix took 0.5 ms of each step at m = 16, with the GPU idle (3x3: 20
// steps 21.9 -> 11.4 ms).
void tridiag_eigs(const double *a, const double *b, int m, std::vector<double> &lam, std::vector<double> &Q) {
    lam.assign(a, a + m);
    std::vector<double> e((size_t)m, 0.0);  // e[i] couples i and i + 1
    for (int i = 0; i + 1 < m; ++i) e[i] = b[i + 1];
    Q.assign((size_t)m * m, 0.0);  // transposed while it is built: row l is column l
    for (int i = 0; i < m; ++i) Q[(size_t)i * m + i] = 1.0;
    double *d = lam.data();
    const double eps = 1.1e-16;
    int hi = m - 1;
    for (int step = 0; hi > 0 && step < 60 * m; ++step) {
        int lo = hi;
        while (lo > 0 && std::fabs(e[lo - 1]) > eps * (std::fabs(d[lo - 1]) + std::fabs(d[lo]))) --lo;
        if (lo == hi) {
            --hi;
            continue;
        }
        const double h = 0.5 * (d[hi - 1] - d[hi]), f = e[hi - 1];
        const double mu = d[hi] - f * f / (h + std::copysign(std::hypot(h, f), h));
        double x = d[lo] - mu, z = e[lo];
        for (int k = lo; k < hi; ++k) {
            const double r = std::hypot(x, z), c = r > 0.0 ? x / r : 1.0, s = r > 0.0 ? z / r : 0.0;
            if (k > lo) e[k - 1] = r;
            const double d1 = d[k], d2 = d[k + 1], ek = e[k], t = 2.0 * c * s * ek;
            d[k] = c * c * d1 + t + s * s * d2;
            d[k + 1] = s * s * d1 - t + c * c * d2;
            e[k] = c * s * (d2 - d1) + (c * c - s * s) * ek;
            if (k + 1 < hi) {
                x = e[k];
                z = s * e[k + 1];
                e[k + 1] *= c;
            }
            double *q0 = &Q[(size_t)k * m], *q1 = q0 + m;
            for (int i = 0; i < m; ++i) {
                const double u = q0[i], v = q1[i];
                q0[i] = c * u + s * v;
                q1[i] = c * v - s * u;
            }
        }
    }
    for (int i = 0; i < m; ++i)
        for (int j = i + 1; j < m; ++j) std::swap(Q[(size_t)i * m + j], Q[(size_t)j * m + i]);
}

// Eigenvector of the lowest eigenvalue theta of T (diagonal a[0..m),
// off-diagonal b[1..m)) by inverse iteration: with the shift theta - delta
// just below the spectrum, T - shift is positive definite, so each solve is
// a stable LDL^T (Thomas) elimination.  The result has unit norm.
void tridiag_lowest_vector(const double *a, const double *b, int m, double theta, std::vector<double> &x) {
    double scale = 0.0;
    for (int i = 0; i < m; ++i) scale = std::max(scale, std::fabs(a[i]) + (i > 0 ? std::fabs(b[i]) : 0.0));
    const double shift = theta - 1e-10 * std::max(1.0, scale);
    x.assign((size_t)m, 1.0 / std::sqrt((double)m));
    std::vector<double> d((size_t)m), l((size_t)m), z((size_t)m);
    for (int it = 0; it < 4; ++it) {
        // factor (T - shift) = L D L^T and solve L D L^T x' = x
        d[0] = a[0] - shift;
        z[0] = x[0];
        for (int i = 1; i < m; ++i) {
            l[i] = b[i] / d[i - 1];
            d[i] = a[i] - shift - l[i] * b[i];
            z[i] = x[i] - l[i] * z[i - 1];
        }
        x[m - 1] = z[m - 1] / d[m - 1];
        for (int i = m - 2; i >= 0; --i) x[i] = z[i] / d[i] - l[i + 1] * x[i + 1];
        double nrm = 0.0;
        for (int i = 0; i < m; ++i) nrm += x[i] * x[i];
        nrm = std::sqrt(nrm);
        for (int i = 0; i < m; ++i) x[i] /= nrm;
    }
}

// exp(-i tau T) e_1 = Q diag(exp(-i tau lam)) Q^T e_1 (m <= kKrylovMax).
void tridiag_expv(const double *a, const double *b, int m, double tau, std::complex<double> *out) {
    std::vector<double> lam, Q;
    tridiag_eigs(a, b, m, lam, Q);
    for (int j = 0; j < m; ++j) out[j] = 0.0;
    for (int l = 0; l < m; ++l) {
        const std::complex<double> ph(std::cos(tau * lam[l]), -std::sin(tau * lam[l]));
        const double w = Q[(size_t)0 * m + l];
        for (int j = 0; j < m; ++j) out[j] += Q[(size_t)j * m + l] * w * ph;
    }
}

// Sum of the dot kernel's per-block partials (fixed order): (Re, Im) in
// mode 0, the squared norm in mode 1.
z2h_status dot_host(const Plan &P, const void *x, const void *y, double theta, int mode, double *part, double out[2],
                    hipStream_t s) {
    DotArgs d;
    memset(&d, 0, sizeof d);
    d.a = x;
    d.b = y;
    d.theta = theta;
    d.mode = mode;
    d.nelem = 1ull << P.n;
    d.part = part;
    const unsigned nb = vec_blocks(P);
    hipError_t e = launch_dot(P.c128, d, nb, s);
    if (e != hipSuccess) return fail(Z2H_ERR_HIP, "dot kernel failed: %s", hipGetErrorString(e));
    std::vector<double> h(2 * (size_t)nb);
    HIP_TRY(hipMemcpyAsync(h.data(), part, sizeof(double) * h.size(), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    out[0] = out[1] = 0.0;
    for (unsigned i = 0; i < nb; ++i) {
        out[0] += h[2 * i];
        out[1] += h[2 * i + 1];
    }
    return Z2H_OK;
}

double sched_s_host(const z2h_schedule &S, int64_t k) {
    return S.sampling ? (double)(k + 1) / (double)S.steps : ((double)k + 0.5) / (double)S.steps;
}

}  // namespace

extern "C" {

z2h_status z2h_hamiltonian_apply(const z2h_plan *plan, const void *d_x, void *d_y, const z2h_couplings *H,
                                 void *stream) {
    try {
        if (!plan) return fail(Z2H_ERR_INVALID, "plan is NULL");
        const Plan &P = plan->P;
        if (!H || !finite4(*H)) return fail(Z2H_ERR_INVALID, "couplings NULL or not finite");
        z2h_status st = check_pair(d_x, state_bytes(P), d_y, state_bytes(P), "d_x", "d_y");
        if (st) return st;
        if ((st = check_device_(P))) return st;
        return ham_passes(P, d_x, d_y, *H, nullptr, nullptr, (hipStream_t)stream);
    } catch (...) {
        return fail(Z2H_ERR_OOM, "exception in z2h_hamiltonian_apply");
    }
}

z2h_status z2h_lanczos_sizes(const z2h_plan *plan, int32_t max_iter, size_t *ws_bytes) {
    if (!plan || !ws_bytes) return fail(Z2H_ERR_INVALID, "plan or ws_bytes is NULL");
    if (max_iter < 1 || max_iter > 100000) return fail(Z2H_ERR_INVALID, "max_iter %d out of [1, 100000]", max_iter);
    *ws_bytes = lanczos_carve(plan->P, 2, max_iter + 2, nullptr, nullptr);
    return Z2H_OK;
}

z2h_status z2h_lanczos_ground(const z2h_plan *plan, void *d_v, void *d_ws, size_t ws_bytes, const z2h_couplings *H,
                              int32_t max_iter, double tol, double *h_alpha, double *h_beta, int32_t *iters,
                              double *e0, void *stream) {
    try {
        if (!plan) return fail(Z2H_ERR_INVALID, "plan is NULL");
        const Plan &P = plan->P;
        if (!H || !finite4(*H)) return fail(Z2H_ERR_INVALID, "couplings NULL or not finite");
        if (!e0 || !iters) return fail(Z2H_ERR_INVALID, "e0 or iters is NULL");
        if (max_iter < 1 || max_iter > 100000) return fail(Z2H_ERR_INVALID, "max_iter %d out of [1, 100000]", max_iter);
        if (!(tol >= 0.0)) return fail(Z2H_ERR_INVALID, "tol must be >= 0");
        z2h_status st = validate_state_ptr(d_v, "d_v");
        if (st) return st;
        if (!d_ws || ((uintptr_t)d_ws & 255)) return fail(Z2H_ERR_INVALID, "d_ws NULL or not 256-byte aligned");
        const size_t need = lanczos_carve(P, 2, max_iter + 2, nullptr, nullptr);
        if (ws_bytes < need) return fail(Z2H_ERR_WORKSPACE, "workspace of %zu bytes, %zu needed", ws_bytes, need);
        if ((st = check_pair(d_v, state_bytes(P), d_ws, ws_bytes, "d_v", "d_ws"))) return st;
        if ((st = check_device_(P))) return st;
        hipStream_t s = (hipStream_t)stream;
        LanczosWs L;
        lanczos_carve(P, 2, max_iter + 2, (char *)d_ws, &L);
        void *u = d_v, *p = L.vec[0], *y = L.vec[1];
        if ((st = norm_start(P, u, L, s))) return st;
        std::vector<LanczosCoef> hc((size_t)max_iter + 2);
        std::vector<double> a, b;
        double theta = 0.0, prev = NAN;
        int done = 0;
        for (int k = 0; k < max_iter; ++k) {
            done = k + 1;
            const bool check = done % kCheckEvery == 0 || done == max_iter;
            if ((st = lanczos_iter(P, *H, k, u, p, p, y, L, check, s))) return st;
            std::swap(u, p);  // the new vector was written over the previous one
            if (!check) continue;
            HIP_TRY(hipMemcpyAsync(hc.data(), L.coef, sizeof(LanczosCoef) * (size_t)(done + 1), hipMemcpyDeviceToHost, s));
            HIP_TRY(hipStreamSynchronize(s));
            if (!(hc[0].beta > 0.0)) return fail(Z2H_ERR_NUMERIC, "start vector has zero norm");
            a.assign((size_t)done, 0.0);
            b.assign((size_t)done + 1, 0.0);
            for (int i = 0; i < done; ++i) {
                a[i] = hc[i].alpha;
                b[i] = i > 0 ? hc[i].beta : 0.0;
                if (!std::isfinite(a[i]) || !std::isfinite(b[i])) return fail(Z2H_ERR_NUMERIC, "non-finite Lanczos coefficient");
            }
            b[done] = hc[done].beta;
            // An invariant subspace (beta ~ 0) ends the recurrence: T is cut
            // there, and the vectors after it are not used.
            double scale = 0.0;
            for (int i = 0; i < done; ++i) scale = std::max(scale, std::fabs(a[i]) + b[i]);
            int cut = 0;
            for (int i = 1; i <= done && !cut; ++i)
                if (b[i] <= 1e-13 * std::max(scale, 1e-300)) cut = i;
            if (cut) {
                done = cut;
                theta = tridiag_lowest(a.data(), b.data(), done);
                break;
            }
            theta = tridiag_lowest(a.data(), b.data(), done);
            if (std::fabs(theta - prev) <= tol * std::max(1.0, std::fabs(theta))) break;
            prev = theta;
        }
        *iters = done;
        *e0 = theta;
        for (int i = 0; i < done; ++i) {
            if (h_alpha) h_alpha[i] = a[i];
            if (h_beta) h_beta[i] = b[i + 1];
        }
        return Z2H_OK;
    } catch (...) {
        return fail(Z2H_ERR_OOM, "exception in z2h_lanczos_ground");
    }
}

z2h_status z2h_exact_sizes(const z2h_plan *plan, int32_t krylov_dim, size_t *ws_bytes) {
    if (!plan || !ws_bytes) return fail(Z2H_ERR_INVALID, "plan or ws_bytes is NULL");
    if (krylov_dim < 1 || krylov_dim > kKrylovMax)
        return fail(Z2H_ERR_INVALID, "krylov_dim %d out of [1, %d]", krylov_dim, kKrylovMax);
    *ws_bytes = lanczos_carve(plan->P, krylov_dim + 1, krylov_dim + 2, nullptr, nullptr);
    return Z2H_OK;
}

z2h_status z2h_exact_evolve(const z2h_plan *plan, void *d_state, void *d_ws, size_t ws_bytes,
                            const z2h_schedule *sched, int32_t krylov_dim, double *err_est, void *stream) {
    try {
        if (!plan) return fail(Z2H_ERR_INVALID, "plan is NULL");
        const Plan &P = plan->P;
        z2h_status st = validate_schedule(P, sched);
        if (st) return st;
        if (krylov_dim < 1 || krylov_dim > kKrylovMax)
            return fail(Z2H_ERR_INVALID, "krylov_dim %d out of [1, %d]", krylov_dim, kKrylovMax);
        const int m = krylov_dim;
        if ((st = validate_state_ptr(d_state, "d_state"))) return st;
        if (!d_ws || ((uintptr_t)d_ws & 255)) return fail(Z2H_ERR_INVALID, "d_ws NULL or not 256-byte aligned");
        const size_t need = lanczos_carve(P, m + 1, m + 2, nullptr, nullptr);
        if (ws_bytes < need) return fail(Z2H_ERR_WORKSPACE, "workspace of %zu bytes, %zu needed", ws_bytes, need);
        if ((st = check_pair(d_state, state_bytes(P), d_ws, ws_bytes, "d_state", "d_ws"))) return st;
        if ((st = check_device_(P))) return st;
        hipStream_t s = (hipStream_t)stream;
        LanczosWs L;
        lanczos_carve(P, m + 1, m + 2, (char *)d_ws, &L);
        void *y = L.vec[m];
        const void *ub[kKrylovMax + 1];
        ub[0] = d_state;
        for (int j = 1; j <= m; ++j) ub[j] = L.vec[j - 1];
        std::vector<LanczosCoef> hc((size_t)m + 2);
        std::vector<double> a((size_t)m), b((size_t)m + 1);
        std::vector<std::complex<double>> e((size_t)m);
        double err = 0.0;
        const z2h_schedule &S = *sched;
        for (int64_t k = S.k_begin; k < S.k_end; ++k) {
            const double s0 = sched_s_host(S, k);
            const double sz = S.sZ ? S.sZ[k] : s0, sx = S.sX ? S.sX[k] : s0;
            z2h_couplings H;
            H.JA = S.start.JA + sx * (S.end.JA - S.start.JA);
            H.hx = S.start.hx + sx * (S.end.hx - S.start.hx);
            H.JB = S.start.JB + sz * (S.end.JB - S.start.JB);
            H.hz = S.start.hz + sz * (S.end.hz - S.start.hz);
            if (!finite4(H)) return fail(Z2H_ERR_INVALID, "step %lld: couplings not finite", (long long)k);
            if ((st = norm_start(P, d_state, L, s))) return st;
            for (int j = 0; j < m; ++j) {
                if ((st = lanczos_iter(P, H, j, ub[j], j > 0 ? ub[j - 1] : nullptr, (void *)ub[j + 1], y, L, j + 1 == m, s)))
                    return st;
            }
            HIP_TRY(hipMemcpyAsync(hc.data(), L.coef, sizeof(LanczosCoef) * (size_t)(m + 1), hipMemcpyDeviceToHost, s));
            HIP_TRY(hipStreamSynchronize(s));
            const double nrm = hc[0].beta;
            if (!(nrm > 0.0) || !std::isfinite(nrm)) return fail(Z2H_ERR_NUMERIC, "step %lld: state norm %g", (long long)k, nrm);
            for (int j = 0; j < m; ++j) {
                a[j] = hc[j].alpha;
                b[j] = j > 0 ? hc[j].beta : 0.0;
                if (!std::isfinite(a[j]) || !std::isfinite(b[j]))
                    return fail(Z2H_ERR_NUMERIC, "step %lld: non-finite Krylov coefficient", (long long)k);
            }
            b[m] = hc[m].beta;
            tridiag_expv(a.data(), b.data(), m, S.dt, e.data());
            err += nrm * b[m] * std::abs(e[m - 1]);
            CombineArgs c;
            memset(&c, 0, sizeof c);
            c.psi = d_state;
            c.m = m;
            c.nelem = 1ull << P.n;
            for (int j = 0; j < m; ++j) {
                c.u[j] = ub[j];
                const std::complex<double> cj = nrm * hc[j].sigma * e[j];
                c.cre[j] = cj.real();
                c.cim[j] = cj.imag();
            }
            hipError_t he = launch_combine(P.c128, c, vec_blocks(P), s);
            if (he != hipSuccess) return fail(Z2H_ERR_HIP, "Krylov combination failed: %s", hipGetErrorString(he));
        }
        if (err_est) *err_est = err;
        return Z2H_OK;
    } catch (...) {
        return fail(Z2H_ERR_OOM, "exception in z2h_exact_evolve");
    }
}

z2h_status z2h_lanczos_vector_sizes(const z2h_plan *plan, int32_t iters, size_t *ws_bytes) {
    if (!plan || !ws_bytes) return fail(Z2H_ERR_INVALID, "plan or ws_bytes is NULL");
    if (iters < 1 || iters > 4096) return fail(Z2H_ERR_INVALID, "iters %d out of [1, 4096]", iters);
    *ws_bytes = lanczos_carve(plan->P, 3, iters + 2, nullptr, nullptr);
    return Z2H_OK;
}

z2h_status z2h_lanczos_vector(const z2h_plan *plan, void *d_v, void *d_ws, size_t ws_bytes, const z2h_couplings *H,
                              const double *h_alpha, const double *h_beta, int32_t iters, double *energy,
                              double *residual, void *stream) {
    try {
        if (!plan) return fail(Z2H_ERR_INVALID, "plan is NULL");
        const Plan &P = plan->P;
        if (!H || !finite4(*H)) return fail(Z2H_ERR_INVALID, "couplings NULL or not finite");
        if (iters < 1 || iters > 4096) return fail(Z2H_ERR_INVALID, "iters %d out of [1, 4096]", iters);
        if (!h_alpha || (iters > 1 && !h_beta)) return fail(Z2H_ERR_INVALID, "alpha or beta is NULL");
        z2h_status st = validate_state_ptr(d_v, "d_v");
        if (st) return st;
        if (!d_ws || ((uintptr_t)d_ws & 255)) return fail(Z2H_ERR_INVALID, "d_ws NULL or not 256-byte aligned");
        const size_t need = lanczos_carve(P, 3, iters + 2, nullptr, nullptr);
        if (ws_bytes < need) return fail(Z2H_ERR_WORKSPACE, "workspace of %zu bytes, %zu needed", ws_bytes, need);
        if ((st = check_pair(d_v, state_bytes(P), d_ws, ws_bytes, "d_v", "d_ws"))) return st;
        for (int i = 0; i < iters; ++i)
            if (!std::isfinite(h_alpha[i]) || (i + 1 < iters && !std::isfinite(h_beta[i])))
                return fail(Z2H_ERR_INVALID, "coefficient %d not finite", i);
        if ((st = check_device_(P))) return st;
        // lowest eigenpair of T
        std::vector<double> b((size_t)iters + 1, 0.0), sv;
        for (int i = 1; i < iters; ++i) b[i] = h_beta[i - 1];
        const double theta = tridiag_lowest(h_alpha, b.data(), iters);
        tridiag_lowest_vector(h_alpha, b.data(), iters, theta, sv);
        hipStream_t s = (hipStream_t)stream;
        LanczosWs L;
        lanczos_carve(P, 3, iters + 2, (char *)d_ws, &L);
        void *u = d_v, *p = L.vec[0], *y = L.vec[1], *g = L.vec[2];
        // the same recurrence again (same kernels, so the same vectors),
        // accumulating g = sum_k s_k v_k, two vectors at a time; where the
        // update's pass reads both anyway, inside it
        auto fused = [&](int k) { return ham_wave(P) && (k & 1) && k + 1 < iters; };
        if ((st = norm_start(P, u, L, s))) return st;
        const unsigned nb = vec_blocks(P);
        for (int k = 0; k < iters; ++k) {
            if (!fused(k) && ((k & 1) || k + 1 == iters)) {
                AccArgs a;
                memset(&a, 0, sizeof a);
                const int k0 = k & ~1;
                a.g = g;
                a.u = k & 1 ? p : u;
                a.u2 = k & 1 ? u : nullptr;
                a.coef = L.coef;
                a.s = sv[k0];
                a.s2 = k & 1 ? sv[k] : 0.0;
                a.k = k0;
                a.first = k0 == 0;
                a.nelem = 1ull << P.n;
                hipError_t e = launch_acc(P.c128, a, nb, s);
                if (e != hipSuccess) return fail(Z2H_ERR_HIP, "Ritz accumulation failed: %s", hipGetErrorString(e));
            }
            if (k + 1 < iters) {
                // (an accumulation launch for k + 1 reads that vector's coefficient)
                const bool last = !fused(k + 1) && (((k + 1) & 1) || k + 2 == iters);
                const RitzAcc acc{g, k ? sv[k - 1] : 0.0, sv[k], k == 1};
                if ((st = lanczos_iter(P, *H, k, u, p, p, y, L, last, s, fused(k) ? &acc : nullptr))) return st;
                std::swap(u, p);
            }
        }
        double nn[2];
        if ((st = dot_host(P, g, g, 0.0, 0, L.apart, nn, s))) return st;
        if (!(nn[0] > 0.0) || !std::isfinite(nn[0])) return fail(Z2H_ERR_NUMERIC, "Ritz vector norm %g", nn[0]);
        CombineArgs c;
        memset(&c, 0, sizeof c);
        c.psi = d_v;
        c.u[0] = g;
        c.cre[0] = 1.0 / std::sqrt(nn[0]);
        c.m = 1;
        c.nelem = 1ull << P.n;
        hipError_t e = launch_combine(P.c128, c, nb, s);
        if (e != hipSuccess) return fail(Z2H_ERR_HIP, "normalisation failed: %s", hipGetErrorString(e));
        double rq = theta;
        if (energy || residual) {
            if ((st = ham_passes(P, d_v, y, *H, nullptr, nullptr, s))) return st;
            double hv[2], rr[2];
            if ((st = dot_host(P, d_v, y, 0.0, 0, L.apart, hv, s))) return st;
            rq = hv[0];
            if ((st = dot_host(P, y, d_v, rq, 1, L.apart, rr, s))) return st;
            if (residual) *residual = std::sqrt(rr[0]);
        }
        if (energy) *energy = rq;
        return Z2H_OK;
    } catch (...) {
        return fail(Z2H_ERR_OOM, "exception in z2h_lanczos_vector");
    }
}

z2h_status z2h_overlap(const z2h_plan *plan, const void *d_a, const void *d_b, void *d_ws, size_t ws_bytes,
                       double *re, double *im, void *stream) {
    try {
        if (!plan) return fail(Z2H_ERR_INVALID, "plan is NULL");
        if (!re || !im) return fail(Z2H_ERR_INVALID, "re or im is NULL");
        z2h_status st = validate_state_ptr(d_a, "d_a");
        if (!st) st = validate_state_ptr(d_b, "d_b");
        if (st) return st;
        if (!d_ws || ((uintptr_t)d_ws & 255)) return fail(Z2H_ERR_INVALID, "d_ws NULL or not 256-byte aligned");
        if (ws_bytes < sizeof(double) * 2 * kVecBlocks)
            return fail(Z2H_ERR_WORKSPACE, "workspace of %zu bytes, %zu needed", ws_bytes, sizeof(double) * 2 * kVecBlocks);
        if ((st = check_device_(plan->P))) return st;
        double o[2];
        if ((st = dot_host(plan->P, d_a, d_b, 0.0, 0, (double *)d_ws, o, (hipStream_t)stream))) return st;
        *re = o[0];
        *im = o[1];
        return Z2H_OK;
    } catch (...) {
        return fail(Z2H_ERR_OOM, "exception in z2h_overlap");
    }
}

z2h_status z2h_tridiag_lowest(int32_t m, const double *alpha, const double *beta, double *out) {
    if (m < 1 || !alpha || !out || (m > 1 && !beta)) return fail(Z2H_ERR_INVALID, "bad tridiagonal arguments");
    std::vector<double> b((size_t)m + 1, 0.0);
    for (int i = 1; i < m; ++i) b[i] = beta[i - 1];
    *out = tridiag_lowest(alpha, b.data(), m);
    return Z2H_OK;
}

z2h_status z2h_tridiag_expv(int32_t m, const double *alpha, const double *beta, double tau, double *out_re,
                            double *out_im) {
    if (m < 1 || m > kKrylovMax || !alpha || !out_re || !out_im || (m > 1 && !beta))
        return fail(Z2H_ERR_INVALID, "bad tridiagonal arguments");
    std::vector<double> b((size_t)m + 1, 0.0);
    for (int i = 1; i < m; ++i) b[i] = beta[i - 1];
    std::vector<std::complex<double>> e((size_t)m);
    tridiag_expv(alpha, b.data(), m, tau, e.data());
    for (int j = 0; j < m; ++j) {
        out_re[j] = e[j].real();
        out_im[j] = e[j].imag();
    }
    return Z2H_OK;
}

}  // extern "C"

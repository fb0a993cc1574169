// Lanczos propagation (SI "Krylov subspace methods"): e^{zH} psi is replaced by
// ||psi|| V e^{zT} e_1, with V an orthonormal basis of span{psi, H psi, ...}
// (m vectors) and T = V^dag H V the m x m tridiagonal projection.  The basis
// is orthogonalised against all previous vectors with two passes of classical
// Gram-Schmidt; inner products are FP64 on the device, T (tridiagonal QR for
// its eigen-decomposition) and its exponential are FP64 on the host.  Up to 16 basis vectors the first pass's update and
// the second pass's projection share one sweep over the basis (states of at
// most 2048 rows do the whole iteration after the product in one launch, of at
// most 256 rows the whole build).  The
// projections, alpha, beta and the invariant-subspace test stay on the device
// for the whole build (no host round trip per iteration); the last iteration
// writes them to pinned host memory, which the host reads after one
// synchronisation.
#include "krylov.hpp"
#include "timing.hpp"
#include "tridiag_eig.hpp"

#include <algorithm>

#include <cmath>
#include <cstdio>
#include <cstdlib>

namespace syk {

BlockCtx::BlockCtx(syk_terms_s& h_, syk_dtype dt, int nvec_, const int32_t* real, hipStream_t s, int sector)
    : h(h_), dtype(dt), nvec(nvec_), real_of_col(real), stream(s), sector0(sector),
      Hact(sector < 0 ? &h_.H : &sector_ham(h_, sector)), plan(plan_for(h_, Hact->M, nvec_, dt)),
      ops(h_, dt, (int64_t)1 << Hact->M, nvec_, s)
{
}

void BlockCtx::apply_H(const void* in, void* out) { launch_apply_h(*Hact, dtype, nvec, real_of_col, in, out, plan, stream); }

void BlockCtx::at(int s)
{
    if (sector0 >= 0) Hact = &sector_ham(h, s);
}

void BlockCtx::majorana(int a, int s_in, const void* in, void* out)
{
    if (s_in < 0) ops.majorana(a, in, out);
    else ops.majorana_sector(a, Hact->M, s_in, in, out);
}

// Builds the Krylov basis of psi (V, m vectors in the workspace) and the
// tridiagonal projection per column.
LanczosBasis lanczos_build(BlockCtx& c, const void* psi, int m)
{
    const int B = c.nvec;
    VecOps& ops = c.ops;
    const size_t vb = ops.vec_bytes();
    LanczosBasis L;
    L.m = m;
    L.V = (char*)c.h.ws.get("krylov_V", vb * (size_t)m);
    void* w = c.h.ws.get("krylov_w", vb);
    char* V = L.V;

    LanczosScalars z;
    const int n_masks = (int)c.Hact->host_masks->size();
    // (with kernel timing on, every product is a launch of its own)
    const void* table = ops.one_launch_lanczos(m, n_masks) && !timing_enabled()
                            ? coefficient_table(*c.Hact, c.plan, c.dtype, B, c.stream) : nullptr;
    if (table) {
        z = ops.lanczos_build(psi, V, m, table, c.Hact->masks, n_masks, c.real_of_col);
    } else {
        z = ops.lanczos_begin(psi, V, m);
        for (int j = 0; j < m; ++j) {
            c.apply_H(V + (size_t)j * vb, w);
            ops.lanczos_step(w, V, j, m, z);
        }
    }
    ops.synchronize();
    const size_t nB = (size_t)B;
    L.alpha.assign(z.h_alpha, z.h_alpha + m * nB);
    L.beta.assign(z.h_beta, z.h_beta + m * nB);
    L.nrm.assign(z.h_nrm, z.h_nrm + nB);
    L.kdim.assign(z.h_kdim, z.h_kdim + nB);
    for (int b = 0; b < B; ++b)
        if (z.h_flag[b] != 0) throw Error(SYK_EBREAKDOWN, "non-finite norm or Lanczos coefficient in Krylov step");
    return L;
}

void ritz_values(const LanczosBasis& L, int col, int nvec, std::vector<double>& ev, std::vector<double>& S)
{
    const int k = L.kdim[col];
    std::vector<double> d(k), e(k > 1 ? k - 1 : 0);
    for (int i = 0; i < k; ++i) {
        d[i] = L.alpha[(size_t)i * nvec + col];
        if (i + 1 < k) e[i] = L.beta[(size_t)i * nvec + col];
    }
    try {
        tridiag_eig(k, d, e, ev, S);
    } catch (const std::runtime_error& x) {
        throw Error(SYK_EBREAKDOWN, x.what());
    }
}

void krylov_step(BlockCtx& c, void* psi, std::complex<double> z, int m, KrylovStats& st)
{
    const int B = c.nvec;
    LanczosBasis L = lanczos_build(c, psi, m);
    const std::vector<double>& beta = L.beta;
    const std::vector<int>& kdim = L.kdim;
    const std::vector<double>& nrm = L.nrm;
    char* V = L.V;
    VecOps& ops = c.ops;

    // Per column: y = ||psi|| V S e^{z Lambda} S^T e_1.
    std::vector<zd> coef((size_t)m * B, zd(0.0, 0.0));
    if (st.err.size() != (size_t)B) st.err.assign(B, 0.0);
    for (int b = 0; b < B; ++b) {
        const int k = kdim[b];
        std::vector<double> ev, S;
        ritz_values(L, b, B, ev, S);
        std::vector<zd> g(k);
        for (int l = 0; l < k; ++l) g[l] = std::exp(z * ev[l]) * S[(size_t)0 * k + l];
        for (int i = 0; i < k; ++i) {
            zd s(0.0, 0.0);
            for (int l = 0; l < k; ++l) s += S[(size_t)i * k + l] * g[l];
            coef[(size_t)i * B + b] = nrm[b] * s;
        }
        if (k == m) {
            const double e = beta[(size_t)(m - 1) * B + b] * std::abs(coef[(size_t)(m - 1) * B + b]);
            st.err[b] = std::max(st.err[b], e);
        }
    }
    ops.combine(psi, V, m, coef);
    ++st.steps;
}

void lanczos_extremes(BlockCtx& c, const void* psi, int m, double* emin, double* emax)
{
    require(c.nvec == 1, "spectrum bounds: one column");
    LanczosBasis L = lanczos_build(c, psi, m);
    std::vector<double> ev, S;
    ritz_values(L, 0, 1, ev, S);
    *emin = ev[0];
    *emax = ev[0];
    for (double e : ev) {
        *emin = std::min(*emin, e);
        *emax = std::max(*emax, e);
    }
}

int lowest_eigenvalues(BlockCtx& c, const void* psi, int m, int k, double* ev_out, double* res_out)
{
    require(c.nvec == 1, "eigenvalues: one column");
    LanczosBasis L = lanczos_build(c, psi, m);
    std::vector<double> ev, S;
    ritz_values(L, 0, 1, ev, S);
    const int kd = L.kdim[0];
    std::vector<int> ord(kd);
    for (int i = 0; i < kd; ++i) ord[i] = i;
    std::sort(ord.begin(), ord.end(), [&](int a, int b) { return ev[a] < ev[b]; });
    // beta of the step that would extend the basis; 0 when the space is invariant
    const double bl = (kd == m) ? L.beta[(size_t)(m - 1)] : 0.0;
    const int n = std::min(k, kd);
    for (int i = 0; i < n; ++i) {
        ev_out[i] = ev[ord[i]];
        if (res_out) res_out[i] = bl * std::fabs(S[(size_t)(kd - 1) * kd + ord[i]]);
    }
    return n;
}

void krylov_propagate(BlockCtx& c, void* psi, std::complex<double> z, double total, double step, int m,
                      KrylovStats& st)
{
    if (total == 0.0) return;
    require(total > 0 && step > 0, "propagation length and step must be positive");
    const int n = std::max(1, (int)std::ceil(total / step - 1e-9));
    const double h = total / n;
    // With SYK_PROGRESS set in the environment, every finished step is reported
    // on stderr (each step has already read its Lanczos scalars back).
    static const bool report = std::getenv("SYK_PROGRESS") != nullptr;
    for (int i = 0; i < n; ++i) {
        krylov_step(c, psi, z * h, m, st);
        if (report) {
            std::fprintf(stderr, "[syk] Krylov step %d/%d of exp((%g%+gi) H), %d column(s)\n", i + 1, n, h * z.real(),
                         h * z.imag(), c.nvec);
            std::fflush(stderr);
        }
    }
}

}  // namespace syk

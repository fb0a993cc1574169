// Vector kernels on [dim][nvec] blocks: Majorana action, FP64 reductions,
// Gram-Schmidt updates and basis combinations.
#pragma once

#include <complex>
#include <string>
#include <vector>

#include "handle.hpp"

namespace syk {

using zd = std::complex<double>;

// Arrays of one Lanczos build.  Device: alpha and beta [m][nvec], the scale
// estimate and Krylov dimension before each iteration [m + 1][nvec], the start
// norm and an error flag per column.  Pinned host mirrors the last iteration
// writes (read them after synchronising the stream).
struct LanczosScalars {
    double *alpha, *beta, *scale, *nrm;
    int *kdim, *flag;
    double *h_alpha, *h_beta, *h_nrm;
    int *h_kdim, *h_flag;
};

class VecOps {
public:
    VecOps(syk_terms_s& h, syk_dtype dt, int64_t dim, int nvec, hipStream_t s);

    size_t vec_bytes() const { return (size_t)dim_ * nvec_ * elem_bytes(dt_); }
    int64_t dim() const { return dim_; }
    int nvec() const { return nvec_; }
    syk_dtype dtype() const { return dt_; }
    hipStream_t stream() const { return s_; }

    // out = chi_a in (SI Jordan-Wigner map, with the 2^{-1/2}).
    void majorana(int a, const void* in, void* out);
    // chi_a between parity sectors: rows u of a sector-s_in state stand for the
    // full rows u + 2^top (parity(u) ^ s_in); out is in sector 1 - s_in
    void majorana_sector(int a, int top, int s_in, const void* in, void* out);
    // Basis vectors one sweep of a Gram-Schmidt kernel serves.
    static constexpr int kFusedMax = 16;

    // host [K][nvec]: <V_k | w> per column, V_k = V + k * vec_bytes (synchronises the stream).
    std::vector<zd> multidot(const void* V, int K, const void* w);
    // host [nvec]: ||a||^2 per column.
    std::vector<double> norm2(const void* a);
    // V_0 = psi / ||psi|| and the scalars of a Lanczos build of m vectors.
    LanczosScalars lanczos_begin(const void* psi, void* V, int m);
    // A whole build of m vectors in one launch (states of few rows), the product
    // taken from a coefficient table of the handle's realisations.
    bool one_launch_lanczos(int m, int n_masks) const;
    LanczosScalars lanczos_build(const void* psi, void* V, int m, const void* table, const MaskRec* masks, int n_masks,
                                 const int32_t* real_of_col);
    // Iteration j after the product w = H V_j: two passes of classical
    // Gram-Schmidt against V_0 .. V_j, alpha_j, beta_j, the invariant-subspace
    // test and V_{j+1} (zero for a column whose subspace became invariant).
    // Nothing waits for the host; the last iteration (j = m - 1) stores no vector
    // and fills the host mirrors.
    void lanczos_step(void* w, void* V, int j, int m, const LanczosScalars& z);
    void synchronize();
    // y = sum_k coef[k][c] V_k (FP64 accumulation)
    void combine(void* y, const void* V, int K, const std::vector<zd>& coef);
    void copy(void* dst, const void* src);

private:
    syk_terms_s& h_;
    syk_dtype dt_;
    int64_t dim_;
    int nvec_;
    hipStream_t s_;
    // Sums over workgroups not formed yet: G partial sums per column.
    struct Sums {
        const double* p;
        int G;
    };
    bool fused() const;
    double* part_buffer(const std::string& slot, size_t doubles);
    dim3 reduce_grid() const;
    bool small_lanczos(int m) const;
    LanczosScalars lanczos_arrays(int m);
    Sums finished(const double* part, int G, int n, const char* slot);
    Sums partial_dots(const void* V, int k0, int kk, const void* w, const std::string& slot, int most);
    Sums dots(const void* V, int k0, int kk, const void* w, const std::string& slot, int most);
    Sums subtract(void* w, const void* V, int k0, int kk, Sums p, const char* norm_slot);
    Sums subtract_dots(void* w, const void* V, int K, Sums p, const std::string& slot, int most);
};

}  // namespace syk

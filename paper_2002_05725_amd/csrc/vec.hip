// Vector kernels on blocks of nvec states of dimension dim, stored one after
// another (entry (r, c) at c*dim + r).
//
// Grid (gx, nvec): workgroup (bx, c) strides over the rows of column c, so
// loads are coalesced and every column reduces on its own.  Reductions
// accumulate in FP64 per thread, reduce over each wave with a fixed butterfly
// of lane exchanges, over the four waves of the workgroup in wave order, then
// over the fixed number of workgroups in index order: the result does not
// depend on timing.
#include <cmath>
#include <cstring>
#include <type_traits>

#include "sums.hpp"
#include "vec.hpp"

namespace syk {

namespace {

constexpr int RB = 256;    // threads per workgroup
constexpr int KC = 8;      // vectors per pass of a multi-vector kernel
constexpr int kWaves = RB / 64;

struct Shape {
    int64_t D;   // rows per column
    int B;       // columns
};

// Workgroups per column: about 2048 over the whole block (a few per CU, enough
// loads in flight to stream at HBM speed), at most 1024 per column.  For
// reductions this count is a function of the shape only, so the summation
// order, and the result, do not depend on timing.
inline dim3 grid_of(const Shape& S, bool reduction)
{
    const int64_t want = (S.D + RB - 1) / RB;
    int gx = reduction ? std::max(32, std::min(1024, 2048 / std::max(1, S.B)))
                       : (int)std::max<int64_t>(1, 4096 / std::max(1, S.B));
    if (want < gx) gx = (int)want;
    if (gx < 1) gx = 1;
    return dim3(gx, S.B);
}

constexpr int ceil_pow2(int n) { return n <= 1 ? 1 : 2 * ceil_pow2((n + 1) / 2); }

// One halving step of wave_scatter_sum: P values per lane become P / 2, each the
// sum over this lane and the lane that differs in lane bit OFF; lanes with the
// bit clear keep the lower half of the values, the others the upper half.
template <int P, int OFF, int N>
__device__ __forceinline__ void scatter_step(double (&v)[N], int lane)
{
    if constexpr (P > 1) {
        const bool up = (lane & OFF) != 0;
#pragma unroll
        for (int i = 0; i < P / 2; ++i) {
            const double keep = up ? v[i + P / 2] : v[i], give = up ? v[i] : v[i + P / 2];
            v[i] = keep + __shfl_xor(give, OFF, 64);
        }
        scatter_step<P / 2, OFF / 2>(v, lane);
    } else {
        // one value left: the lane bits below pick copies of it
#pragma unroll
        for (int off = OFF; off > 0; off >>= 1) v[0] += __shfl_xor(v[0], off, 64);
    }
}

// Workgroup sums of a[0..N): each wave adds its 64 lanes by halving exchanges
// (P + 5 - log2 P lane exchanges for P = N rounded up to a power of two; a
// butterfly per value takes 6 N and was a third of a sweep over 16 vectors of
// 2^16 rows: 10 us, 7 with it), the lane that holds value i stores it in
// red[wave][i], and after one barrier thread i < N returns red[0][i] + red[1][i]
// + red[2][i] + red[3][i] (others return 0).  red holds kWaves * N doubles.
template <int N>
__device__ __forceinline__ double block_sum(double (&a)[N], double* red)
{
    constexpr int P = ceil_pow2(N);
    static_assert(P <= 64, "block_sum: at most 64 values");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double v[P];
#pragma unroll
    for (int i = 0; i < P; ++i) v[i] = i < N ? a[i] : 0.0;
    scatter_step<P, 32>(v, lane);
    // lane bit 5 chose the top bit of the value's index, and so on down
    const int i = lane / (64 / P);
    if (lane % (64 / P) == 0 && i < N) red[wave * N + i] = v[0];
    __syncthreads();
    double s = 0.0;
    if ((int)threadIdx.x < N)
        for (int w = 0; w < kWaves; ++w) s += red[w * N + threadIdx.x];
    return s;
}

template <typename R>
__global__ void __launch_bounds__(RB) k_majorana(const cplx<R>* __restrict__ in, cplx<R>* __restrict__ out,
                                                 Shape S, int a)
{
    const int64_t col = (int64_t)blockIdx.y * S.D;
    const int k = a >> 1;
    const uint64_t bit = (uint64_t)1 << k;
    const uint64_t below = bit - 1;
    const R amp = (R)0.70710678118654752440;
    const int64_t step = (int64_t)gridDim.x * RB;
    for (int64_t r = (int64_t)blockIdx.x * RB + threadIdx.x; r < S.D; r += step) {
        const uint64_t s = (uint64_t)r ^ bit;   // source row
        const cplx<R> v = in[col + (int64_t)s];
        int neg = __popcll(s & below) & 1;
        cplx<R> o;
        if (a & 1) {             // i (-1)^{s_k} times the Z string
            neg ^= (int)((s >> k) & 1);
            o.re = -amp * v.im;
            o.im = amp * v.re;
        } else {
            o.re = amp * v.re;
            o.im = amp * v.im;
        }
        if (neg) { o.re = -o.re; o.im = -o.im; }
        out[col + r] = o;
    }
}

// chi_a on a parity-sector state (rows u: full row u + 2^top (parity(u) ^ s_in)).
// For k = a/2 < top the map is the full-space one on u; for k = top the flipped
// qubit is the implied one, so u maps to itself and the Z string below it covers
// every bit of u.
template <typename R>
__global__ void __launch_bounds__(RB) k_majorana_sector(const cplx<R>* __restrict__ in, cplx<R>* __restrict__ out,
                                                        Shape S, int a, int top, int s_in)
{
    const int64_t col = (int64_t)blockIdx.y * S.D;
    const int k = a >> 1;
    const bool implied = (k == top);
    const uint64_t bit = implied ? 0u : (uint64_t)1 << k;
    const uint64_t below = implied ? (uint64_t)S.D - 1u : bit - 1u;
    const R amp = (R)0.70710678118654752440;
    const int64_t step = (int64_t)gridDim.x * RB;
    for (int64_t r = (int64_t)blockIdx.x * RB + threadIdx.x; r < S.D; r += step) {
        const uint64_t s = (uint64_t)r ^ bit;   // source row
        const cplx<R> v = in[col + (int64_t)s];
        int neg = __popcll(s & below) & 1;
        cplx<R> o;
        if (a & 1) {             // i (-1)^{s_k} times the Z string
            neg ^= implied ? ((__popcll(s) & 1) ^ s_in) : (int)((s >> k) & 1);
            o.re = -amp * v.im;
            o.im = amp * v.re;
        } else {
            o.re = amp * v.re;
            o.im = amp * v.im;
        }
        if (neg) { o.re = -o.re; o.im = -o.im; }
        out[col + r] = o;
    }
}

// The multi-vector kernels take the number of basis vectors K as a template
// argument: every load of a row is then unconditional and issued before the
// first is used, instead of one branch and one wait per vector.
template <int N, typename F>
void with_count(int k, F&& f)
{
    if constexpr (N > 0) {
        if (k == N) f(std::integral_constant<int, N>{});
        else with_count<N - 1>(k, f);
    } else {
        throw Error(SYK_EINVAL, "vector kernels: unsupported number of basis vectors");
    }
}

// Groups left after n of them are halved until at most 16 remain.
constexpr int folded(int n) { return n <= 16 ? n : folded((n + 1) / 2); }

// tmp[q N + i] += tmp[(q + h) N + i], h the upper half of the n groups, until at
// most 16 remain.
template <int N, int n>
__device__ __forceinline__ void fold_groups(double* tmp, int t)
{
    if constexpr (n > 16) {
        constexpr int h = (n + 1) / 2;
        if (t < (n - h) * N) tmp[t] += tmp[t + h * N];
        __syncthreads();
        fold_groups<N, h>(tmp, t);
    }
}

// Partial sums of a reduction of N doubles per column: [column][workgroup g < G][N].
// Every workgroup of the kernel that uses the sums adds the G entries itself, in
// a fixed order (256 / N strided groups of four running sums each, then the groups
// pairwise: one after another, the 256 of ||w||^2 at 2^16 rows had five times the
// rounding error), or, for large blocks, a finishing kernel has reduced them and G
// is 1 (kFusedRows).  The result is in out[0..N) of LDS for every thread.
template <int N>
__device__ __forceinline__ void sum_partials(const double* __restrict__ partial, int G, double (&tmp)[RB],
                                             double (&out)[N])
{
    constexpr int kGroups = RB / N;
    const double* p = partial + (int64_t)blockIdx.y * G * N;
    const int t = threadIdx.x, i = t % N, q = t / N;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (q < kGroups)
        for (int g = q; g < G; g += 4 * kGroups) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (g + u * kGroups < G) s[u] += p[(int64_t)(g + u * kGroups) * N + i];
        }
    tmp[t] = (s[0] + s[1]) + (s[2] + s[3]);
    __syncthreads();
    // halved in LDS down to at most 16 groups, which one thread per value adds
    fold_groups<N, kGroups>(tmp, t);
    if (t < N) out[t] = pairwise_sum<folded(kGroups)>(tmp + t, N);
    __syncthreads();
}

// partial[c][bx][2k, 2k + 1] = sum over this workgroup's rows of conj(V_k[r,c]) w[r,c]
template <typename R, int K>
__global__ void __launch_bounds__(RB) k_multidot(const cplx<R>* __restrict__ V, int64_t vstride,
                                                 const cplx<R>* __restrict__ w, Shape S,
                                                 double* __restrict__ partial)
{
    __shared__ double red[kWaves * 2 * K];
    const int64_t col = (int64_t)blockIdx.y * S.D;
    double a[2 * K];
#pragma unroll
    for (int k = 0; k < 2 * K; ++k) a[k] = 0.0;
    const int64_t step = (int64_t)gridDim.x * RB;
    for (int64_t r = (int64_t)blockIdx.x * RB + threadIdx.x; r < S.D; r += step) {
        const int64_t e = col + r;
        const cplx<R> b = w[e];
        cplx<R> v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = V[k * vstride + e];
        const double br = b.re, bi = b.im;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double vr = v[k].re, vi = v[k].im;
            a[2 * k] += vr * br + vi * bi;
            a[2 * k + 1] += vr * bi - vi * br;
        }
    }
    const double t = block_sum(a, red);
    // thread i < 2K holds (k, re/im) = (i / 2, i % 2)
    if ((int)threadIdx.x < 2 * K)
        partial[((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * (2 * K) + threadIdx.x] = t;
}

// w -= sum_k c_k V_k with c the sums of proj (G partial sums per column);
// optionally partial[c][bx] = sum |w_new|^2
template <typename R, int K>
__global__ void __launch_bounds__(RB) k_update(cplx<R>* __restrict__ w, const cplx<R>* __restrict__ V,
                                               int64_t vstride, const double* __restrict__ proj, int G,
                                               Shape S, double* __restrict__ partial)
{
    __shared__ double tmp[RB], cs[2 * K];
    const int c = blockIdx.y;
    const int64_t col = (int64_t)c * S.D;
    sum_partials<2 * K>(proj, G, tmp, cs);
    double cr[K], ci[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        cr[k] = cs[2 * k];
        ci[k] = cs[2 * k + 1];
    }
    double nrm = 0.0;
    const int64_t step = (int64_t)gridDim.x * RB;
    for (int64_t r = (int64_t)blockIdx.x * RB + threadIdx.x; r < S.D; r += step) {
        const int64_t e = col + r;
        const cplx<R> b = w[e];
        cplx<R> v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = V[k * vstride + e];
        double xr = b.re, xi = b.im;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            xr -= cr[k] * v[k].re - ci[k] * v[k].im;
            xi -= cr[k] * v[k].im + ci[k] * v[k].re;
        }
        cplx<R> o;
        o.re = (R)xr;
        o.im = (R)xi;
        w[e] = o;
        const double orr = o.re, oi = o.im;
        nrm += orr * orr + oi * oi;
    }
    if (!partial) return;
    double a[1] = {nrm};
    const double t = block_sum(a, tmp);
    if (threadIdx.x == 0) partial[(int64_t)c * gridDim.x + blockIdx.x] = t;
}

// The first Gram-Schmidt update fused with the second projection, for K
// basis vectors: w' = w - sum_k c_k V_k with c the sums of proj (w' rounded to
// the state's precision, as stored), and partial[c][bx][k] = sum over this
// workgroup's rows of conj(V_k[r,c]) w'[r,c].  Each V_k[r] is read once for both
// uses.
template <typename R, int K>
__global__ void __launch_bounds__(RB) k_update_dot(cplx<R>* __restrict__ w, const cplx<R>* __restrict__ V,
                                                   int64_t vstride, const double* __restrict__ proj, int G,
                                                   Shape S, double* __restrict__ partial)
{
    __shared__ double tmp[RB], cs[2 * K], red[kWaves * 2 * K];
    const int c = blockIdx.y;
    const int64_t col = (int64_t)c * S.D;
    sum_partials<2 * K>(proj, G, tmp, cs);
    double cr[K], ci[K], a[2 * K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        cr[k] = cs[2 * k];
        ci[k] = cs[2 * k + 1];
        a[2 * k] = a[2 * k + 1] = 0.0;
    }
    const int64_t step = (int64_t)gridDim.x * RB;
    for (int64_t r = (int64_t)blockIdx.x * RB + threadIdx.x; r < S.D; r += step) {
        const int64_t e = col + r;
        const cplx<R> b = w[e];
        cplx<R> v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = V[k * vstride + e];
        double xr = b.re, xi = b.im;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            xr -= cr[k] * v[k].re - ci[k] * v[k].im;
            xi -= cr[k] * v[k].im + ci[k] * v[k].re;
        }
        cplx<R> o;
        o.re = (R)xr;
        o.im = (R)xi;
        w[e] = o;
        const double orr = o.re, oi = o.im;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double vr = v[k].re, vi = v[k].im;
            a[2 * k] += vr * orr + vi * oi;
            a[2 * k + 1] += vr * oi - vi * orr;
        }
    }
    const double t = block_sum(a, red);
    if ((int)threadIdx.x < 2 * K) partial[((int64_t)c * gridDim.x + blockIdx.x) * (2 * K) + threadIdx.x] = t;
}

// out[c][i] = sum of partial[c][g][i] over g < G, for i < n doubles: one wave
// per output, lane l adding g = l, l + 64, ... in order, then a fixed butterfly
// over the lanes (the same order on every run).  Four outputs per workgroup: one
// each was bound by dispatching them (120,000 outputs: 54 us, 18 with four).
__global__ void __launch_bounds__(RB) k_finish(const double* __restrict__ partial, int G, int n, int64_t outputs,
                                               double* __restrict__ out)
{
    const int64_t o = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (o >= outputs) return;
    const int64_t c = (uint32_t)o / (uint32_t)n;
    const int i = (int)(o - c * n), lane = (int)(threadIdx.x & 63u);
    double s = 0.0;
    for (int g = lane; g < G; g += 64) s += partial[(c * G + g) * n + i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) out[o] = s;
}

void launch_finish(const double* partial, int G, int n, int nvec, double* out, hipStream_t st)
{
    const int64_t outputs = (int64_t)n * nvec;
    hipLaunchKernelGGL(k_finish, dim3((unsigned)((outputs + kWaves - 1) / kWaves)), dim3(RB), 0, st, partial, G, n,
                       outputs, out);
    SYK_HIP(hipGetLastError());
}

// The scalars of one column at Lanczos iteration j, the same on every thread
// that calls it: alpha_j = a (the two projections on the newest basis vector),
// beta_j = sqrt(wn).  While the column is still growing its basis, its scale
// estimate max_i (|alpha_i| + beta_{i-1}) is updated, and unless j is the last
// iteration, beta_j at or below 1e-13 times that scale (or a zero start vector)
// marks the subspace invariant (kdim = j + 1, factor 0); otherwise the factor
// 1 / beta_j scales w into the next basis vector.  Iteration j's scale and kdim
// are read from slot j and written to slot j + 1, so that every workgroup of the
// launch that forms the scalars reads the same values; one thread per column
// (`writer`) stores.
__device__ __forceinline__ double lanczos_scalars(const LanczosScalars& z, double a, double wn, int j, int m, int B,
                                                  int c, bool writer)
{
    const double bt = sqrt(wn);
    const size_t o = (size_t)j * B + c;
    double sc = z.scale[o], f = 0.0;
    int kd = z.kdim[o];
    if (j < kd) {
        sc = fmax(sc, fabs(a) + (j > 0 ? z.beta[o - B] : 0.0));
        if (j < m - 1) {
            if (bt <= 1e-13 * sc || z.nrm[c] == 0.0) kd = j + 1;
            else f = 1.0 / bt;
        }
    }
    if (writer) {
        z.alpha[o] = a;
        z.beta[o] = bt;
        z.scale[o + B] = sc;
        z.kdim[o + B] = kd;
        if (!isfinite(a) || !isfinite(bt)) z.flag[c] = 1;
    }
    return f;
}

// The scalars of one column start from its norm: slot 0, the error flag for a
// norm that is not finite; returns 1 / norm (0 for a zero column).
__device__ __forceinline__ double lanczos_start(const LanczosScalars& z, double n2, int m, int c, bool writer)
{
    const double nrm = sqrt(n2);
    if (writer) {
        z.nrm[c] = nrm;
        z.scale[c] = 0.0;
        z.kdim[c] = m;
        z.flag[c] = isfinite(n2) ? 0 : 1;
    }
    return nrm > 0.0 ? 1.0 / nrm : 0.0;
}

// A column's results to the host mirror (pinned memory the host reads after
// synchronising the stream: no copy in between).  One thread per iteration.
__device__ __forceinline__ void lanczos_publish(const LanczosScalars& z, int m, int B, int c, int t, int nt)
{
    for (int k = t; k < m; k += nt) {
        z.h_alpha[(size_t)k * B + c] = z.alpha[(size_t)k * B + c];
        z.h_beta[(size_t)k * B + c] = z.beta[(size_t)k * B + c];
    }
    if (t == 0) {
        z.h_nrm[c] = z.nrm[c];
        z.h_kdim[c] = z.kdim[(size_t)m * B + c];
        z.h_flag[c] = z.flag[c];
    }
}

// V_0 = psi / ||psi|| and the scalars' start, from the G partial sums of ||psi||^2.
template <typename R>
__global__ void __launch_bounds__(RB) k_lanczos_start(const cplx<R>* __restrict__ psi, cplx<R>* __restrict__ V,
                                                      const double* __restrict__ norm, int G, int m, Shape S,
                                                      LanczosScalars z)
{
    __shared__ double tmp[RB], n2[2];
    const int c = blockIdx.y;
    sum_partials<2>(norm, G, tmp, n2);
    const double f = lanczos_start(z, n2[0], m, c, blockIdx.x == 0 && threadIdx.x == 0);
    const int64_t col = (int64_t)c * S.D, step = (int64_t)gridDim.x * RB;
    for (int64_t r = (int64_t)blockIdx.x * RB + threadIdx.x; r < S.D; r += step) {
        const cplx<R> v = psi[col + r];
        cplx<R> o;
        o.re = (R)(f * (double)v.re);
        o.im = (R)(f * (double)v.im);
        V[col + r] = o;
    }
}

// The end of Lanczos iteration j: alpha_j from the two projections' partial
// sums (entry `at` of n per workgroup), beta_j from those of ||w||^2, and V_{j+1}
// = w / beta_j.  The last iteration only stores the scalars, and everything to
// the host mirror.
template <typename R>
__global__ void __launch_bounds__(RB) k_lanczos_next(const cplx<R>* __restrict__ w, cplx<R>* __restrict__ out,
                                                     const double* __restrict__ p1, int G1,
                                                     const double* __restrict__ p2, int G2, int n, int at,
                                                     const double* __restrict__ norm, int Gn, int j, int m, Shape S,
                                                     LanczosScalars z)
{
    __shared__ double tmp[RB], n2[1], red[kWaves * 2];
    const int c = blockIdx.y;
    sum_partials<1>(norm, Gn, tmp, n2);
    double a[2] = {0.0, 0.0};
    for (int g = threadIdx.x; g < G1; g += RB) a[0] += p1[((int64_t)c * G1 + g) * n + at];
    for (int g = threadIdx.x; g < G2; g += RB) a[1] += p2[((int64_t)c * G2 + g) * n + at];
    const double t = block_sum(a, red);
    __syncthreads();
    if (threadIdx.x < 2) tmp[threadIdx.x] = t;
    __syncthreads();
    const bool writer = blockIdx.x == 0 && threadIdx.x == 0;
    const double f = lanczos_scalars(z, tmp[0] + tmp[1], n2[0], j, m, S.B, c, writer);
    if (j == m - 1) {
        __syncthreads();   // the writer's stores (same workgroup) before they are read back
        if (blockIdx.x == 0) lanczos_publish(z, m, S.B, c, threadIdx.x, RB);
        return;
    }
    const int64_t col = (int64_t)c * S.D, step = (int64_t)gridDim.x * RB;
    for (int64_t r = (int64_t)blockIdx.x * RB + threadIdx.x; r < S.D; r += step) {
        const cplx<R> v = w[col + r];
        cplx<R> o;
        o.re = (R)(f * (double)v.re);
        o.im = (R)(f * (double)v.im);
        out[col + r] = o;
    }
}

// States of at most kSmallRows rows: everything of a Lanczos iteration after
// the product in one launch, one workgroup of 16 waves per column with w in LDS.
// A projection is one wave's work (its lanes over the rows, one butterfly), an
// update one thread per row; both read the basis from L2.  Bound by one CU's
// read rate (four reads of the basis, (j + 1) x 16 KiB each at 1,024 complex128
// rows), against the sweeps' launches (four of ~5 us up to 16 vectors, four more
// per further 16).  us per step, sweeps -> one launch an iteration: 512 rows m=20
// 499 -> 319; 1,024 rows m=20 503 -> 372, m=64 2,620 -> 1,890, m=200 24,900 ->
// 15,600; 2,048 rows m=20 541 -> 502, m=40 1,370 -> 1,350, 64 columns 2,390 ->
// 2,230, and past the line there m=64 2,840 -> 2,930, m=200 25,700-27,200 -> 27,900.
constexpr int kSmallRows = 2048, kSmallThreads = 1024, kSmallMaxM = 512;

template <typename R>
__global__ void __launch_bounds__(kSmallThreads) k_lanczos_small(const cplx<R>* __restrict__ w, cplx<R>* V,
                                                                 int64_t vstride, int j, int m, Shape S,
                                                                 LanczosScalars z)
{
    __shared__ cplx<R> ws[kSmallRows];
    __shared__ double cs[2][2 * kSmallMaxM];   // the projections of the two passes
    __shared__ double red[kSmallThreads / 64];
    const int c = blockIdx.y, K = j + 1, D = (int)S.D;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t col = (int64_t)c * S.D;
    const cplx<R>* Vc = V + col;
    for (int r = t; r < D; r += kSmallThreads) ws[r] = w[col + r];
    __syncthreads();
    double nrm = 0.0;
    for (int pass = 0; pass < 2; ++pass) {
        for (int k = wave; k < K; k += kSmallThreads / 64) {
            const cplx<R>* v = Vc + k * vstride;
            // four running sums per lane and 1,024 rows: chains of at most four
            // additions (of eight, 7% more rounding at 2,048 rows than a reduction
            // over workgroups)
            double ar = 0.0, ai = 0.0;
            for (int h = 0; h < D; h += 1024) {
                double a4[4] = {0.0, 0.0, 0.0, 0.0}, b4[4] = {0.0, 0.0, 0.0, 0.0};
                auto add = [&](int r, int u) {
                    const cplx<R> x = v[r], y = ws[r];
                    const double vr = x.re, vi = x.im, br = y.re, bi = y.im;
                    a4[u] += vr * br + vi * bi;
                    b4[u] += vr * bi - vi * br;
                };
                const int end = min(D, h + 1024);
                if (D >= 256) {   // D is a power of two
#pragma unroll 2
                    for (int r = h + lane; r < end; r += 256) {
#pragma unroll
                        for (int u = 0; u < 4; ++u) add(r + 64 * u, u);
                    }
                } else {
                    for (int r = lane; r < D; r += 64) add(r, 0);
                }
                ar += (a4[0] + a4[1]) + (a4[2] + a4[3]);
                ai += (b4[0] + b4[1]) + (b4[2] + b4[3]);
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                ar += __shfl_xor(ar, off, 64);
                ai += __shfl_xor(ai, off, 64);
            }
            if (lane == 0) {
                cs[pass][2 * k] = ar;
                cs[pass][2 * k + 1] = ai;
            }
        }
        __syncthreads();
        for (int r = t; r < D; r += kSmallThreads) {
            const cplx<R> b = ws[r];
            double xr = b.re, xi = b.im;
#pragma unroll 8
            for (int k = 0; k < K; ++k) {
                const cplx<R> x = Vc[k * vstride + r];
                const double cr = cs[pass][2 * k], ci = cs[pass][2 * k + 1];
                xr -= cr * x.re - ci * x.im;
                xi -= cr * x.im + ci * x.re;
            }
            cplx<R> o;
            o.re = (R)xr;
            o.im = (R)xi;
            ws[r] = o;
            const double orr = o.re, oi = o.im;
            if (pass == 1) nrm += orr * orr + oi * oi;
        }
        __syncthreads();
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) nrm += __shfl_xor(nrm, off, 64);
    if (lane == 0) red[wave] = nrm;
    __syncthreads();
    const double wn = pairwise_sum<kSmallThreads / 64>(red);
    const double f = lanczos_scalars(z, cs[0][2 * j] + cs[1][2 * j], wn, j, m, S.B, c, t == 0);
    if (j == m - 1) {
        __syncthreads();
        lanczos_publish(z, m, S.B, c, t, kSmallThreads);
        return;
    }
    cplx<R>* vn = V + (int64_t)K * vstride + col;
    for (int r = t; r < D; r += kSmallThreads) {
        const cplx<R> x = ws[r];
        cplx<R> o;
        o.re = (R)(f * (double)x.re);
        o.im = (R)(f * (double)x.im);
        vn[r] = o;
    }
}

// States of at most kOneRows rows: a whole Lanczos build in one launch, one
// workgroup of 16 waves per column, with the basis in LDS and the product from the
// handle's coefficient table ([realisation][row block][mask][16], apply_h.hip).
// Two launches per iteration cost ~15 us whatever they did (G(t) at N=16 in one
// sector: 15.2 ms of which the arithmetic is well under one); here an iteration is
// bound by reading the table from L2 by one CU (0.4 MB at 256 rows) and by the
// barriers between its six steps.
constexpr int kOneRows = 256, kOneBasis = 8192, kOneMasks = 512, kOneColumns = 64, kOneMaxM = 128;

struct OneColumns {
    int32_t real[kOneColumns];
};

template <typename R>
__global__ void __launch_bounds__(kSmallThreads) k_lanczos_build(const cplx<R>* __restrict__ psi, cplx<R>* V,
                                                                 int64_t vstride, int m, Shape S,
                                                                 const cplx<R>* __restrict__ table,
                                                                 const MaskRec* __restrict__ masks, int n_masks,
                                                                 OneColumns C, LanczosScalars z)
{
    constexpr int kW = kSmallThreads / 64;
    __shared__ cplx<R> vs[kOneBasis];          // V_k at k * D
    __shared__ cplx<R> ws[kOneRows];
    __shared__ c128 part[kSmallThreads];       // product: partial sums per row
    __shared__ double cs[2][2 * kOneMaxM];     // the projections of the two passes
    __shared__ double red[kW];
    __shared__ uint32_t xs[kOneMasks];
    const int c = blockIdx.x, D = (int)S.D;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t col = (int64_t)c * D;
    const int nblk = (D + 15) / 16;
    // row of this thread in the product, and its group of masks
    const int r = t & (D - 1), group = t / D, groups = kSmallThreads / D;
    const cplx<R>* tab = table + ((int64_t)C.real[c] * nblk + (r >> 4)) * n_masks * 16 + (r & 15);
    for (int i = t; i < n_masks; i += kSmallThreads) xs[i] = masks[i].x;
    // sum of one double per thread over the workgroup, in a fixed order
    auto block_add = [&](double v) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        __syncthreads();
        if (lane == 0) red[wave] = v;
        __syncthreads();
        return pairwise_sum<kW>(red);
    };
    double n2 = 0.0;
    if (t < D) {
        const cplx<R> v = psi[col + t];
        ws[t] = v;
        n2 = (double)v.re * v.re + (double)v.im * v.im;
    }
    double f = lanczos_start(z, block_add(n2), m, c, t == 0);
    for (int j = 0;; ++j) {
        // V_j = f w, in LDS and for the combination
        if (t < D) {
            cplx<R> o;
            o.re = (R)(f * (double)ws[t].re);
            o.im = (R)(f * (double)ws[t].im);
            vs[j * D + t] = o;
            V[j * vstride + col + t] = o;
        }
        __syncthreads();
        double ar = 0.0, ai = 0.0;
#pragma unroll 8
        for (int k = group; k < n_masks; k += groups) {
            const cplx<R> d = tab[(int64_t)k * 16];
            const cplx<R> v = vs[j * D + (r ^ (int)xs[k])];
            const double dr = d.re, di = d.im, vr = v.re, vi = v.im;
            ar = fma(dr, vr, ar);
            ar = fma(-di, vi, ar);
            ai = fma(dr, vi, ai);
            ai = fma(di, vr, ai);
        }
        // lanes of a wave that hold the same row, then the waves in order
        for (int off = D; off < 64; off <<= 1) {
            ar += __shfl_xor(ar, off, 64);
            ai += __shfl_xor(ai, off, 64);
        }
        part[t] = c128{ar, ai};
        __syncthreads();
        if (t < D) {
            const int step = D < 64 ? 64 : D;
            double sr = 0.0, si = 0.0;
            for (int u = t; u < kSmallThreads; u += step) {
                sr += part[u].re;
                si += part[u].im;
            }
            cplx<R> o;
            o.re = (R)sr;
            o.im = (R)si;
            ws[t] = o;
        }
        __syncthreads();
        const int K = j + 1;
        double nrm = 0.0;
        for (int pass = 0; pass < 2; ++pass) {
            for (int k = wave; k < K; k += kW) {
                double br = 0.0, bi = 0.0;
                for (int q = lane; q < D; q += 64) {
                    const cplx<R> x = vs[k * D + q], y = ws[q];
                    const double vr = x.re, vi = x.im, wr = y.re, wi = y.im;
                    br += vr * wr + vi * wi;
                    bi += vr * wi - vi * wr;
                }
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) {
                    br += __shfl_xor(br, off, 64);
                    bi += __shfl_xor(bi, off, 64);
                }
                if (lane == 0) {
                    cs[pass][2 * k] = br;
                    cs[pass][2 * k + 1] = bi;
                }
            }
            __syncthreads();
            if (t < D) {
                const cplx<R> b = ws[t];
                double xr = b.re, xi = b.im;
#pragma unroll 4
                for (int k = 0; k < K; ++k) {
                    const cplx<R> x = vs[k * D + t];
                    const double cr = cs[pass][2 * k], ci = cs[pass][2 * k + 1];
                    xr -= cr * x.re - ci * x.im;
                    xi -= cr * x.im + ci * x.re;
                }
                cplx<R> o;
                o.re = (R)xr;
                o.im = (R)xi;
                ws[t] = o;
                const double orr = o.re, oi = o.im;
                if (pass == 1) nrm = orr * orr + oi * oi;
            }
            __syncthreads();
        }
        f = lanczos_scalars(z, cs[0][2 * j] + cs[1][2 * j], block_add(nrm), j, m, S.B, c, t == 0);
        __syncthreads();   // the scalars stored above are read by the next iteration
        if (j == m - 1) break;
    }
    lanczos_publish(z, m, S.B, c, t, kSmallThreads);
}

// Coefficients of a combination for one column, passed with the launch.
struct CombineArg {
    static constexpr int kMax = 64;
    double c[2 * kMax];
};

// y = sum_k c_k V_k for all K vectors; the coefficients come with the launch
// (one column) or from the device array coef[k][c].
template <typename R, bool ARG>
__global__ void __launch_bounds__(RB) k_combine(cplx<R>* y, const cplx<R>* V, int64_t vstride, int K, CombineArg arg,
                                                const double* __restrict__ coef, Shape S)
{
    const int c = blockIdx.y;
    const int64_t col = (int64_t)c * S.D;
    const int64_t step = (int64_t)gridDim.x * RB;
    auto cf = [&](int k, int i) { return ARG ? arg.c[2 * k + i] : coef[((int64_t)k * S.B + c) * 2 + i]; };
    for (int64_t r = (int64_t)blockIdx.x * RB + threadIdx.x; r < S.D; r += step) {
        const int64_t e = col + r;
        double xr = 0.0, xi = 0.0;
        int k = 0;
        for (; k + KC <= K; k += KC) {   // KC loads in flight, then their FMAs
            cplx<R> v[KC];
#pragma unroll
            for (int u = 0; u < KC; ++u) v[u] = V[(k + u) * vstride + e];
#pragma unroll
            for (int u = 0; u < KC; ++u) {
                const double cr = cf(k + u, 0), ci = cf(k + u, 1);
                xr += cr * v[u].re - ci * v[u].im;
                xi += cr * v[u].im + ci * v[u].re;
            }
        }
        for (; k < K; ++k) {
            const double cr = cf(k, 0), ci = cf(k, 1);
            const cplx<R> v = V[k * vstride + e];
            xr += cr * v.re - ci * v.im;
            xi += cr * v.im + ci * v.re;
        }
        cplx<R> o;
        o.re = (R)xr;
        o.im = (R)xi;
        y[e] = o;
    }
}

}  // namespace

VecOps::VecOps(syk_terms_s& h, syk_dtype dt, int64_t dim, int nvec, hipStream_t s)
    : h_(h), dt_(dt), dim_(dim), nvec_(nvec), s_(s)
{
    require(nvec >= 1 && nvec <= 65535, "nvec must be in [1, 65535]");
}

void VecOps::majorana(int a, const void* in, void* out)
{
    Shape S{dim_, nvec_};
    dim3 g = grid_of(S, false);
    if (dt_ == SYK_C128)
        hipLaunchKernelGGL(k_majorana<double>, g, dim3(RB), 0, s_, (const c128*)in, (c128*)out, S, a);
    else
        hipLaunchKernelGGL(k_majorana<float>, g, dim3(RB), 0, s_, (const c64*)in, (c64*)out, S, a);
    SYK_HIP(hipGetLastError());
}

void VecOps::majorana_sector(int a, int top, int s_in, const void* in, void* out)
{
    if ((a >> 1) > top || top >= 63 || (s_in != 0 && s_in != 1)) throw Error(SYK_EINVAL, "majorana: bad sector arguments");
    Shape S{dim_, nvec_};
    dim3 g = grid_of(S, false);
    if (dt_ == SYK_C128)
        hipLaunchKernelGGL(k_majorana_sector<double>, g, dim3(RB), 0, s_, (const c128*)in, (c128*)out, S, a, top, s_in);
    else
        hipLaunchKernelGGL(k_majorana_sector<float>, g, dim3(RB), 0, s_, (const c64*)in, (c64*)out, S, a, top, s_in);
    SYK_HIP(hipGetLastError());
}

// Workgroups per column of a reduction and, for large blocks, the finishing
// kernel: G partial sums of n doubles per column become 1.  Up to kFusedRows
// rows in all, a column's reduction takes at most kMaxFusedGroups workgroups and
// each kernel that uses the sums adds them itself, three launches of ~5 us less
// per Lanczos iteration (N=32, m=30: 3.63 -> 3.35 ms a step; N=20: 61 -> 26 ms an
// OTOC curve, with the one-launch iteration).  Larger blocks need more workgroups
// to stream at HBM speed and there a finishing launch is less than every
// workgroup's own sum (64 complex64 columns at N=36: 134.4 ms a step without it,
// 133.6 with).
// A handle with a workspace cap runs the finishing kernel at every size: its partial
// sums are used up at once and share one buffer, where the others are kept per 16
// basis vectors (up to 2% of a basis, which a cap may not leave).
constexpr int kMaxFusedGroups = 256;
constexpr int64_t kFusedRows = (int64_t)1 << 18;

bool VecOps::fused() const { return dim_ * nvec_ <= kFusedRows && h_.ws.limit == 0; }

// The buffer of a reduction's partial sums.
double* VecOps::part_buffer(const std::string& slot, size_t doubles)
{
    return (double*)h_.ws.get(fused() ? slot : "gs_part", doubles * sizeof(double));
}

dim3 VecOps::reduce_grid() const
{
    Shape S{dim_, nvec_};
    dim3 g = grid_of(S, true);
    if (fused() && g.x > (unsigned)kMaxFusedGroups) g.x = kMaxFusedGroups;
    return g;
}

VecOps::Sums VecOps::finished(const double* part, int G, int n, const char* slot)
{
    if (fused()) return Sums{part, G};
    double* out = (double*)h_.ws.get(slot, (size_t)2 * kFusedMax * nvec_ * sizeof(double));
    launch_finish(part, G, n, nvec_, out, s_);
    return Sums{out, 1};
}

// <V_k | w> for k in [k0, k0 + kk) as partial sums in `slot` (kk <= kFusedMax),
// which is sized for `most` vectors: no reallocation as a basis grows.
VecOps::Sums VecOps::partial_dots(const void* V, int k0, int kk, const void* w, const std::string& slot, int most)
{
    Shape S{dim_, nvec_};
    const dim3 g = reduce_grid();
    double* part = part_buffer(slot, (size_t)g.x * most * nvec_ * 2);
    const char* v = (const char*)V + (size_t)k0 * vec_bytes();
    const int64_t vs = dim_ * nvec_;
    with_count<kFusedMax>(kk, [&](auto kc) {
        constexpr int K_ = decltype(kc)::value;
        if (dt_ == SYK_C128)
            hipLaunchKernelGGL((k_multidot<double, K_>), g, dim3(RB), 0, s_, (const c128*)v, vs, (const c128*)w, S, part);
        else
            hipLaunchKernelGGL((k_multidot<float, K_>), g, dim3(RB), 0, s_, (const c64*)v, vs, (const c64*)w, S, part);
    });
    SYK_HIP(hipGetLastError());
    return Sums{part, (int)g.x};
}

VecOps::Sums VecOps::dots(const void* V, int k0, int kk, const void* w, const std::string& slot, int most)
{
    const Sums p = partial_dots(V, k0, kk, w, slot, most);
    return finished(p.p, p.G, 2 * kk, (slot + "_f").c_str());
}

// w -= sum_k c_k V_k for k in [k0, k0 + kk), c the sums of p; with norm_slot,
// the partial sums of ||w||^2.
VecOps::Sums VecOps::subtract(void* w, const void* V, int k0, int kk, Sums p, const char* norm_slot)
{
    Shape S{dim_, nvec_};
    const dim3 g = reduce_grid();
    double* part = norm_slot ? part_buffer(norm_slot, (size_t)g.x * nvec_ * 2) : nullptr;
    const char* v = (const char*)V + (size_t)k0 * vec_bytes();
    const int64_t vs = dim_ * nvec_;
    with_count<kFusedMax>(kk, [&](auto kc) {
        constexpr int K_ = decltype(kc)::value;
        if (dt_ == SYK_C128)
            hipLaunchKernelGGL((k_update<double, K_>), g, dim3(RB), 0, s_, (c128*)w, (const c128*)v, vs, p.p, p.G, S, part);
        else
            hipLaunchKernelGGL((k_update<float, K_>), g, dim3(RB), 0, s_, (c64*)w, (const c64*)v, vs, p.p, p.G, S, part);
    });
    SYK_HIP(hipGetLastError());
    if (!norm_slot) return Sums{nullptr, 0};
    return finished(part, (int)g.x, 1, (std::string(norm_slot) + "_f").c_str());
}

// The first update and the second projection in one sweep (K <= kFusedMax).
VecOps::Sums VecOps::subtract_dots(void* w, const void* V, int K, Sums p, const std::string& slot, int most)
{
    Shape S{dim_, nvec_};
    const dim3 g = reduce_grid();
    double* part = part_buffer(slot, (size_t)g.x * most * nvec_ * 2);
    const int64_t vs = dim_ * nvec_;
    with_count<kFusedMax>(K, [&](auto kc) {
        constexpr int K_ = decltype(kc)::value;
        if (dt_ == SYK_C128)
            hipLaunchKernelGGL((k_update_dot<double, K_>), g, dim3(RB), 0, s_, (c128*)w, (const c128*)V, vs, p.p, p.G, S, part);
        else
            hipLaunchKernelGGL((k_update_dot<float, K_>), g, dim3(RB), 0, s_, (c64*)w, (const c64*)V, vs, p.p, p.G, S, part);
    });
    SYK_HIP(hipGetLastError());
    return finished(part, (int)g.x, 2 * K, (slot + "_f").c_str());
}

// Up to kDirect results the finishing kernel writes them to pinned host memory
// itself, which saves the copy; each is a store of its own over the host link, so
// that many go through device memory (16 rows, 60,000 columns: 425 us written
// directly by one workgroup each, 263 copied).
constexpr size_t kDirect = 4096;

std::vector<zd> VecOps::multidot(const void* V, int K, const void* w)
{
    const size_t n = (size_t)K * nvec_;
    double* host = 2 * n <= kDirect ? (double*)h_.pinned.get_if_used(2 * n * sizeof(double)) : nullptr;
    const bool direct = host != nullptr;
    double* out = direct ? host : (double*)h_.ws.get("md_out", 2 * n * sizeof(double));
    for (int k0 = 0; k0 < K; k0 += kFusedMax) {
        const int kk = std::min(kFusedMax, K - k0);
        const Sums p = partial_dots(V, k0, kk, w, "md_part", std::min(K, kFusedMax));
        launch_finish(p.p, p.G, 2 * kk, nvec_, out + 2 * (size_t)k0 * nvec_, s_);
    }
    // host memory for the results while the kernels run; one vector's are in order already
    std::vector<zd> res(n);
    std::vector<double> copied(direct || K == 1 ? 0 : 2 * n);
    if (!direct) {
        host = K == 1 ? reinterpret_cast<double*>(res.data()) : copied.data();
        SYK_HIP(hipMemcpyAsync(host, out, 2 * n * sizeof(double), hipMemcpyDeviceToHost, s_));
    }
    SYK_HIP(hipStreamSynchronize(s_));
    if (!direct && K == 1) return res;
    for (int k0 = 0; k0 < K; k0 += kFusedMax) {   // host: [chunk][column][k]
        const int kk = std::min(kFusedMax, K - k0);
        const double* h = host + 2 * (size_t)k0 * nvec_;
        for (int c = 0; c < nvec_; ++c)
            for (int k = 0; k < kk; ++k) {
                const double* x = h + 2 * ((size_t)c * kk + k);
                res[(size_t)(k0 + k) * nvec_ + c] = zd(x[0], x[1]);
            }
    }
    return res;
}

std::vector<double> VecOps::norm2(const void* a)
{
    std::vector<zd> d = multidot(a, 1, a);
    std::vector<double> out(d.size());
    for (size_t i = 0; i < d.size(); ++i) out[i] = d[i].real();
    return out;
}

bool VecOps::small_lanczos(int m) const { return dim_ <= kSmallRows && m <= kSmallMaxM; }

bool VecOps::one_launch_lanczos(int m, int n_masks) const
{
    return dim_ <= kOneRows && (int64_t)m * dim_ <= kOneBasis && m <= kOneMaxM && n_masks <= kOneMasks &&
           nvec_ <= kOneColumns;
}

LanczosScalars VecOps::lanczos_build(const void* psi, void* V, int m, const void* table, const MaskRec* masks, int n_masks,
                                     const int32_t* real_of_col)
{
    if (!one_launch_lanczos(m, n_masks)) throw Error(SYK_EINVAL, "lanczos_build: unsupported size");
    const LanczosScalars z = lanczos_arrays(m);
    OneColumns C{};
    for (int c = 0; c < nvec_; ++c) C.real[c] = real_of_col ? real_of_col[c] : 0;
    Shape S{dim_, nvec_};
    const dim3 g(nvec_), b(kSmallThreads);
    const int64_t vs = dim_ * nvec_;
    if (dt_ == SYK_C128)
        hipLaunchKernelGGL(k_lanczos_build<double>, g, b, 0, s_, (const c128*)psi, (c128*)V, vs, m, S, (const c128*)table,
                           masks, n_masks, C, z);
    else
        hipLaunchKernelGGL(k_lanczos_build<float>, g, b, 0, s_, (const c64*)psi, (c64*)V, vs, m, S, (const c64*)table,
                           masks, n_masks, C, z);
    SYK_HIP(hipGetLastError());
    return z;
}

LanczosScalars VecOps::lanczos_arrays(int m)
{
    const size_t B = (size_t)nvec_, mB = (size_t)m * B;
    double* d = (double*)h_.ws.get("lz_dbl", (3 * mB + 2 * B) * sizeof(double));
    int* i = (int*)h_.ws.get("lz_int", (mB + 2 * B) * sizeof(int));
    double* h = (double*)h_.pinned.get((2 * mB + B) * sizeof(double) + 2 * B * sizeof(int));
    LanczosScalars z{};
    z.alpha = d;
    z.beta = d + mB;
    z.scale = d + 2 * mB;          // [m + 1][B]
    z.nrm = d + 3 * mB + B;
    z.kdim = i;                    // [m + 1][B]
    z.flag = i + mB + B;
    z.h_alpha = h;
    z.h_beta = h + mB;
    z.h_nrm = h + 2 * mB;
    z.h_kdim = (int*)(h + 2 * mB + B);
    z.h_flag = z.h_kdim + B;
    return z;
}

LanczosScalars VecOps::lanczos_begin(const void* psi, void* V, int m)
{
    const LanczosScalars z = lanczos_arrays(m);
    Shape S{dim_, nvec_};
    const Sums n = dots(psi, 0, 1, psi, "gs_n", 1);
    const dim3 g = grid_of(S, false);
    if (dt_ == SYK_C128)
        hipLaunchKernelGGL(k_lanczos_start<double>, g, dim3(RB), 0, s_, (const c128*)psi, (c128*)V, n.p, n.G, m, S, z);
    else
        hipLaunchKernelGGL(k_lanczos_start<float>, g, dim3(RB), 0, s_, (const c64*)psi, (c64*)V, n.p, n.G, m, S, z);
    SYK_HIP(hipGetLastError());
    return z;
}

void VecOps::lanczos_step(void* w, void* V, int j, int m, const LanczosScalars& z)
{
    Shape S{dim_, nvec_};
    const int K = j + 1;
    const int64_t vs = dim_ * nvec_;
    if (small_lanczos(m)) {
        const dim3 g(1, nvec_);
        if (dt_ == SYK_C128)
            hipLaunchKernelGGL(k_lanczos_small<double>, g, dim3(kSmallThreads), 0, s_, (const c128*)w, (c128*)V, vs, j, m, S, z);
        else
            hipLaunchKernelGGL(k_lanczos_small<float>, g, dim3(kSmallThreads), 0, s_, (const c64*)w, (c64*)V, vs, j, m, S, z);
        SYK_HIP(hipGetLastError());
        return;
    }
    // two passes of classical Gram-Schmidt in chunks of kFusedMax basis vectors;
    // k0: the chunk that holds the newest vector
    const int nch = (K + kFusedMax - 1) / kFusedMax, k0 = (nch - 1) * kFusedMax, kl = K - k0;
    auto count = [&](int i) { return std::min(kFusedMax, K - i * kFusedMax); };
    auto most = [&](int i) { return std::min(kFusedMax, m - i * kFusedMax); };   // ... in the last iteration
    auto slot = [](const char* s, int i) { return s + std::to_string(i); };
    std::vector<Sums> p1(nch), p2(nch);
    for (int i = 0; i < nch; ++i) p1[i] = dots(V, i * kFusedMax, count(i), w, slot("gs_p", i), most(i));
    if (nch == 1) {
        p2[0] = subtract_dots(w, V, K, p1[0], "gs_q0", most(0));
    } else {
        for (int i = 0; i < nch; ++i) subtract(w, V, i * kFusedMax, count(i), p1[i], nullptr);
        for (int i = 0; i < nch; ++i) p2[i] = dots(V, i * kFusedMax, count(i), w, slot("gs_q", i), most(i));
    }
    Sums n{};
    for (int i = 0; i < nch; ++i) n = subtract(w, V, i * kFusedMax, count(i), p2[i], i == nch - 1 ? "gs_n" : nullptr);
    const dim3 g = j == m - 1 ? dim3(1, nvec_) : grid_of(S, false);
    void* out = (char*)V + (size_t)K * vec_bytes();   // not written by the last iteration
    const int at = 2 * (kl - 1);
    if (dt_ == SYK_C128)
        hipLaunchKernelGGL(k_lanczos_next<double>, g, dim3(RB), 0, s_, (const c128*)w, (c128*)out, p1[nch - 1].p,
                           p1[nch - 1].G, p2[nch - 1].p, p2[nch - 1].G, 2 * kl, at, n.p, n.G, j, m, S, z);
    else
        hipLaunchKernelGGL(k_lanczos_next<float>, g, dim3(RB), 0, s_, (const c64*)w, (c64*)out, p1[nch - 1].p,
                           p1[nch - 1].G, p2[nch - 1].p, p2[nch - 1].G, 2 * kl, at, n.p, n.G, j, m, S, z);
    SYK_HIP(hipGetLastError());
}

void VecOps::synchronize() { SYK_HIP(hipStreamSynchronize(s_)); }

void VecOps::combine(void* y, const void* V, int K, const std::vector<zd>& coef)
{
    Shape S{dim_, nvec_};
    dim3 g = grid_of(S, false);
    CombineArg arg{};
    const double* dc = nullptr;
    const int64_t vs = dim_ * nvec_;
    if (nvec_ == 1 && K <= CombineArg::kMax) {
        std::memcpy(arg.c, coef.data(), (size_t)K * sizeof(zd));
        if (dt_ == SYK_C128)
            hipLaunchKernelGGL((k_combine<double, true>), g, dim3(RB), 0, s_, (c128*)y, (const c128*)V, vs, K, arg, dc, S);
        else
            hipLaunchKernelGGL((k_combine<float, true>), g, dim3(RB), 0, s_, (c64*)y, (const c64*)V, vs, K, arg, dc, S);
    } else {
        // A copy from pageable memory the call owns: it has left the host buffer
        // when the call returns.
        double* d = (double*)h_.ws.get("combine_coef", coef.size() * sizeof(zd));
        SYK_HIP(hipMemcpyAsync(d, coef.data(), coef.size() * sizeof(zd), hipMemcpyHostToDevice, s_));
        SYK_HIP(hipStreamSynchronize(s_));
        dc = d;
        if (dt_ == SYK_C128)
            hipLaunchKernelGGL((k_combine<double, false>), g, dim3(RB), 0, s_, (c128*)y, (const c128*)V, vs, K, arg, dc, S);
        else
            hipLaunchKernelGGL((k_combine<float, false>), g, dim3(RB), 0, s_, (c64*)y, (const c64*)V, vs, K, arg, dc, S);
    }
    SYK_HIP(hipGetLastError());
}

void VecOps::copy(void* dst, const void* src)
{
    if (dst != src) SYK_HIP(hipMemcpyAsync(dst, src, vec_bytes(), hipMemcpyDeviceToDevice, s_));
}

}  // namespace syk

// Matrix-free H psi for the Jordan-Wigner SYK Hamiltonian on gfx950.
//
// (H psi)[r] = sum_x D_x(r) psi[r ^ x] over the flip masks x of terms.hpp.
// A workgroup owns one tile of 2^tile_bits consecutive rows of one column of a
// block (columns are whole state vectors, one after another).  For a mask, every row of the tile reads
// the tile (tile ^ (x >> tile_bits)) of psi, permuted by x's low bits, so the
// masks are processed chunk by chunk in x order: the shared source tile is
// staged once into LDS with coalesced loads, every mask of the chunk gathers
// from LDS, and each thread keeps its rows' sums in registers and writes them
// once.
//
// Grid: (tiles, column groups, parts); with fewer tiles and columns than the
// chip holds workgroups, the chunks are split over `parts` workgroups per tile
// and a second kernel adds their FP64 sums in order.  Every workgroup serves NC consecutive columns
// of one realisation (NC = 1, or 2 for the two typical states a realisation
// carries in a block), so mask records, PAIR weights and DIAG terms are
// wave-uniform (scalar loads) and the chunk's QUAD tables are staged into LDS
// next to the NC source tiles.  Everything a mask decodes (record, table
// entries, lane index and sign, PAIR coefficients) is formed once and applied
// to every column.  Up to 64 columns per launch.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <utility>

#include "apply_h.hpp"
#include "mask_classes.hpp"
#include "timing.hpp"

namespace syk {

namespace {

template <typename R>
struct KTerms {
    const cplx<R>* __restrict__ tab4;
    const uint32_t* __restrict__ qinfo;
    const cplx<R>* __restrict__ phi2;
    const R* __restrict__ w2;
    const double* __restrict__ diag;   // [n_real][dim]: the diagonal of H
    int n_real, M;
};

struct KLayout {
    const FarRec* __restrict__ far;   // QUAD masks flipping only tile bits
    int n_far;
    int n_chunks;
    int tile_bits;     // rows per tile = 2^tile_bits
    int lane_bits;     // threads per workgroup = 2^lane_bits
    uint64_t dim;      // rows per column
    int col0;          // first column of this launch (column = col0 + NC blockIdx.y + c)
    uint32_t n_tiles;  // dim >> tile_bits
    int xcd_remap;     // spread consecutive tiles over XCDs in contiguous ranges
    int n_parts;       // > 1: workgroup z sums only chunks part_chunk[z] .. part_chunk[z + 1] - 1 and its share of
                       // the far masks, into its own slice of the FP64 partial sums
    const uint32_t* __restrict__ part_chunk;
    int n_tables;           // 16-row kernel: staged QUAD tables per realisation
    uint64_t part_stride;   // elements per slice: columns of the launch * dim
    int32_t real[kColsPerLaunch];  // realisation of each column of the launch
};

static_assert(kColsPerLaunch == 64, "column slice");

// Workgroups are dispatched round-robin over the 8 XCDs; give XCD j the
// contiguous tile range [j n/8, (j+1) n/8) so that its L2 sees neighbouring
// tiles, whose source tiles overlap for low flip masks.
__device__ __forceinline__ uint32_t tile_of_block(uint32_t b, const KLayout& L)
{
    if (!L.xcd_remap || (L.n_tiles & 7u)) return b;
    return (b & 7u) * (L.n_tiles >> 3) + (b >> 3);
}

__device__ __forceinline__ uint32_t parity(uint32_t v) { return __popc(v) & 1u; }

// Flip the sign of x when s is 1 (s in {0, 1}).
__device__ __forceinline__ double flip(double x, uint32_t s)
{
    return __hiloint2double(__double2hiint(x) ^ (int)(s << 31), __double2loint(x));
}
__device__ __forceinline__ float flip(float x, uint32_t s) { return __int_as_float(__float_as_int(x) ^ (int)(s << 31)); }

__device__ __forceinline__ uint32_t bit(uint32_t r, uint32_t q) { return (r >> q) & 1u; }

// Sign flip when the count c is odd: adding c << 31 to the word holding the
// sign bit changes that bit exactly when c is odd.  Written as one
// v_lshl_add_u32 per word (plain C lets the compiler share the shift between
// words, one instruction more per table entry pair).
__device__ __forceinline__ uint32_t add_lsb31(uint32_t w, uint32_t c)
{
    uint32_t r;
    asm("v_lshl_add_u32 %0, %1, 31, %2" : "=v"(r) : "v"(c), "v"(w));
    return r;
}
__device__ __forceinline__ double flip_odd(double x, uint32_t c)
{
    return __hiloint2double((int)add_lsb31((uint32_t)__double2hiint(x), c), __double2loint(x));
}
__device__ __forceinline__ float flip_odd(float x, uint32_t c) { return __uint_as_float(add_lsb31(__float_as_uint(x), c)); }

// 4-bit QUAD table index: bit m = bit q_m of r.
__device__ __forceinline__ uint32_t quad_index(uint32_t r, uint32_t qpack)
{
    return bit(r, mask_q(qpack, 0)) | (bit(r, mask_q(qpack, 1)) << 1) | (bit(r, mask_q(qpack, 2)) << 2) |
           (bit(r, mask_q(qpack, 3)) << 3);
}

}  // namespace

namespace {

// Thread layout: row rl = tid + (k << lb) of the tile (nt = 2^lb threads,
// lb = 8 whenever a thread owns several rows, k < RPT).  A row index splits into
// lane bits (tid), k bits (the same for every lane) and tile bits (the same for
// the workgroup).
//
// QUAD masks: the tile bits of every table index and sign are folded into the
// tables while they are staged.  Inside a chunk the host sorts the QUAD masks
// by class: for each k bit, whether the mask flips it, has it in its Z string,
// or neither.  Within a class the source offset of every row and the sign each
// row adds are compile-time constants, and the rows use one table entry per
// subset of the flipped k bits.  The lane part of the table index is a byte
// gather of tid's bits (v_perm) and a dot product with the powers of two
// (v_dot4), the lane part of the sign one popcount.
constexpr int kLaneBits = 8;

// Masks per chunk of the apply kernel: complex128 keeps the LDS of a
// 2048-row tile at 40 KiB so that four workgroups share a CU.
constexpr int apply_chunk_masks(uint32_t esz) { return esz == 16 ? 32 : 64; }

template <typename R, int RPT, int NC>
struct ApplyLds {
    cplx<R> src[NC * (RPT << kLaneBits)];   // column c's tile at c * (RPT << kLaneBits)
    cplx<R> tabs[apply_chunk_masks(sizeof(cplx<R>)) * 16];
};

// Waves per SIMD the kernel is compiled for: four with one column and 8 rows
// per thread; two columns double the sums (three waves for complex64, two for
// complex128, whose two 32 KiB tiles allow two workgroups per CU anyway).
constexpr int apply_waves(int rpt, int nc, int rbytes)
{
    return rpt != 8 ? 1 : nc == 1 ? 4 : rbytes == 8 ? 2 : 3;
}

template <typename R>
__device__ __forceinline__ void cmac(R& pr, R& pi, R a, R b, const cplx<R>& v)
{
    pr = fma(a, v.re, pr);
    pr = fma(-b, v.im, pr);
    pi = fma(a, v.im, pi);
    pi = fma(b, v.re, pi);
}

// SPLIT (the masks of a tile over several workgroups) is a template argument:
// as run-time branches it cost the unsplit kernel 1% (N=52 complex128).
template <typename R, int RPT, int NC, bool SPLIT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(apply_waves(RPT, NC, sizeof(R)))))
k_apply(KTerms<R> T, const QApplyChunk* __restrict__ chunks,
                                               const QRec* __restrict__ rec, KLayout L,
                                               const cplx<R>* __restrict__ psi, cplx<R>* __restrict__ out,
                                               c128* __restrict__ parts)
{
    constexpr int KB = ilog2c(RPT);
    constexpr uint32_t esz = sizeof(cplx<R>);
    // byte weights of the four gathered index bits: esz * 2^m
    constexpr uint32_t kDotW = (esz) | (2 * esz) << 8 | (4 * esz) << 16 | (8 * esz) << 24;
    // kept in a VGPR, so that v_dot4 can take the per-mask table offset from an
    // SGPR (one scalar operand per instruction); not for two complex64 columns,
    // whose kernel is short of VGPRs at three waves (1.2% slower with it)
    uint32_t dotw = kDotW;
    if constexpr (NC == 1 || sizeof(R) == 8) asm("" : "+v"(dotw));
    __shared__ ApplyLds<R, RPT, NC> S;
    constexpr uint32_t TS = RPT << kLaneBits;   // rows of a column's tile
    const char* src_b = reinterpret_cast<const char*>(S.src);
    const char* tab_b = reinterpret_cast<const char*>(S.tabs);
    auto src_at = [&](uint32_t off) { return *reinterpret_cast<const cplx<R>*>(src_b + off); };
    auto tab_at = [&](uint32_t off) { return *reinterpret_cast<const cplx<R>*>(tab_b + off); };

    const uint32_t lb = (RPT > 1) ? (uint32_t)kLaneBits : (uint32_t)L.lane_bits;
    const uint32_t nt = 1u << lb;
    const uint32_t tile = tile_of_block(blockIdx.x, L);
    const uint32_t tid = threadIdx.x;
    const int rc = L.real[blockIdx.y * NC];   // the same for all NC columns
    const int M = T.M;
    const uint32_t base = tile << L.tile_bits;
    psi += (uint64_t)(L.col0 + blockIdx.y * NC) * L.dim;   // this workgroup's first column
    out += (uint64_t)(L.col0 + blockIdx.y * NC) * L.dim;

    // bits 0..3 and 4..7 of tid, one per byte
    uint32_t B0 = 0, B1 = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        B0 |= ((tid >> i) & 1u) << (8 * i);
        B1 |= ((tid >> (4 + i)) & 1u) << (8 * i);
    }
    const uint32_t tid_b = tid * esz;

    // complex128 sums directly in pr/pi; complex64 sums each chunk in FP32 and
    // carries the running total in FP64.
    constexpr bool kSplit = sizeof(R) < sizeof(double);
    double acc_re[NC][RPT], acc_im[NC][RPT];
    R pr[NC][RPT], pi[NC][RPT];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            acc_re[c][k] = acc_im[c][k] = 0.0;
            pr[c][k] = pi[c][k] = R(0);
        }
    auto carry = [&]() {   // complex64: chunk sums into the FP64 running totals
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < RPT; ++k) {
                acc_re[c][k] += (double)pr[c][k];
                acc_im[c][k] += (double)pi[c][k];
                pr[c][k] = pi[c][k] = R(0);
            }
    };
    // column c's source row at byte offset off of its tile
    auto src_row = [&](int c, uint32_t off) { return src_at(off + (uint32_t)c * TS * esz); };

    int g0 = 0, g1 = L.n_chunks, f0 = 0, f1 = L.n_far;
    if constexpr (SPLIT) {
        g0 = (int)L.part_chunk[blockIdx.z];
        g1 = (int)L.part_chunk[blockIdx.z + 1];
        f0 = (int)((uint32_t)L.n_far * blockIdx.z / (uint32_t)L.n_parts);
        f1 = (int)((uint32_t)L.n_far * (blockIdx.z + 1) / (uint32_t)L.n_parts);
    }
    for (int g = g0; g < g1; ++g) {
        const QApplyChunk C = chunks[g];
        uint32_t n_flat = 0;   // flat PAIR masks (no flipped k bit), first among the PAIR records
#pragma unroll
        for (int b = 0; b < 8; ++b) n_flat += (C.pcnt[b >> 2] >> (8 * (b & 3))) & 0xffu;
        __syncthreads();   // previous chunk is done with src / tabs
        if (C.new_tile || (SPLIT && g == g0)) {
            const uint64_t sbase = (uint64_t)(tile ^ C.x_high) << L.tile_bits;
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int k = 0; k < RPT; ++k)
                    S.src[c * TS + tid + k * nt] = (psi + c * L.dim)[sbase + tid + k * nt];
        }
        // Staged QUAD table entry i of slot j: sign_tile * T[i ^ index_tile].
        for (uint32_t e = tid; e < C.n_quad * 16; e += nt) {
            const QRec& qr = rec[C.first + (e >> 4)];
            const uint32_t qt = qr.tab, qp = qr.qpack, zb = qr.zbase;   // in this layout's coordinates
            const cplx<R> c = T.tab4[((size_t)qt * T.n_real + rc) * 16 + ((e & 15u) ^ quad_index(base, qp))];
            const uint32_t sg = parity(base & zb);
            cplx<R> o;
            o.re = flip(c.re, sg);
            o.im = flip(c.im, sg);
            S.tabs[e] = o;
        }
        // PAIR slots (after the QUAD tables): for each row k and term e, the part
        // of L_e(r) that does not depend on the lane, t_{k,e} = W_e + sum over
        // tile and k bits c of w_{e,c} r_c.  One slot holds RPT * 4 values (flat
        // masks, below, only row 0).
        for (uint32_t v = tid; v < C.n_pair * (RPT * 4); v += nt) {
            const uint32_t p = v / (RPT * 4), k = (v >> 2) % RPT, e = v & 3u;
            if (p < n_flat && k != 0) continue;   // flat masks use row 0 only
            const QRec& pq = rec[C.first + C.n_quad + p];
            const R* w = T.w2 + (((size_t)pq.tab * T.n_real + rc) * 4 + e) * (M + 1);
            const uint32_t rb = base | (k << lb);
            R acc = w[M];
            for (int c = (int)lb; c < M; ++c)
                if ((rb >> c) & 1u) acc += w[c];
            reinterpret_cast<R*>(reinterpret_cast<char*>(S.tabs) + pq.sel)[k * 4 + e] = acc;
        }
        __syncthreads();

        uint32_t mi = C.first;
        // The next QUAD record is loaded one mask ahead (records run one past
        // the end): complex128 at the start of a mask, complex64 after its FMAs
        // (an outstanding scalar load makes every LDS wait a full wait).
        constexpr bool kEarlyRecord = sizeof(R) == 8;
        QRec qn = rec[mi];
        // Groups of three QUAD masks (same lane flips, J = 1 or 2 flipped k
        // bits in all three ways): the lane index, the lane sign and the source
        // rows are read once for the three.  Member j's table is the (m + j)-th
        // of the chunk; the index bits of its flipped k bits sit at kof and
        // 2 kof (kof: the first record's koffs).  The next member's table
        // entries are read while the previous member's FMAs run.
        if constexpr (KB == kMaxKBits) {
            auto group_loop = [&](auto gcls) {
                constexpr int GC = decltype(gcls)::value;
                constexpr int J = 1 + (GC >> 1), P = GC & 1;
                constexpr int NE = 1 << J;   // table entries per member
                const uint32_t n = (C.cnt[(kQuadClasses + GC) >> 2] >> (8 * ((kQuadClasses + GC) & 3))) & 0xffu;
                for (uint32_t i = 0; i < n; ++i, mi += 3) {
                    const QRec q = qn;
                    if constexpr (kEarlyRecord) qn = rec[mi + 3];
                    const uint32_t ia = __builtin_amdgcn_udot4(__builtin_amdgcn_perm(B1, B0, q.sel), dotw,
                                                               (mi - C.first) * 16u * esz, false);
                    const uint32_t sl = (uint32_t)__popc(tid & q.zl);   // lane sign: its parity
                    const uint32_t kof = q.koffs;
                    auto load_member = [&](auto jc, cplx<R> (&t)[NE]) {
                        constexpr uint32_t j = decltype(jc)::value;
#pragma unroll
                        for (int e = 0; e < NE; ++e)
                            t[e] = tab_at(ia + (uint32_t)e * kof + j * 16u * esz);
                    };
                    auto member_fma = [&](auto jc, cplx<R> (&t)[NE], const cplx<R> (&v)[NC][RPT]) {
                        constexpr int j = decltype(jc)::value;
                        constexpr int XK = group_xk(J, j), ZK = group_zk(XK, P);
#pragma unroll
                        for (int e = 0; e < NE; ++e) {
                            t[e].re = flip_odd(t[e].re, sl);
                            t[e].im = flip_odd(t[e].im, sl);
                        }
#pragma unroll
                        for (int c = 0; c < NC; ++c)
#pragma unroll
                            for (int k = 0; k < RPT; ++k) {
                                const cplx<R> te = t[pack_bits3(k & XK, XK)];
                                const bool neg = (popc3(k & ZK) & 1) != 0;
                                const R a = neg ? -te.re : te.re, b = neg ? -te.im : te.im;
                                cmac(pr[c][k], pi[c][k], a, b, v[c][k ^ XK]);
                            }
                    };
                    using I0 = std::integral_constant<int, 0>;
                    using I1 = std::integral_constant<int, 1>;
                    using I2 = std::integral_constant<int, 2>;
                    cplx<R> ta[NE], tb[NE];
                    load_member(I0{}, ta);
                    __builtin_amdgcn_sched_barrier(0);
                    const uint32_t sb = tid_b ^ q.xoff;
                    cplx<R> v[NC][RPT];
#pragma unroll
                    for (int c = 0; c < NC; ++c)
#pragma unroll
                        for (int k = 0; k < RPT; ++k) v[c][k] = src_row(c, sb + ((uint32_t)k << kLaneBits) * esz);
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (J == 1) {
                        load_member(I1{}, tb);
                        member_fma(I0{}, ta, v);
                        __builtin_amdgcn_sched_barrier(0);
                        load_member(I2{}, ta);
                        member_fma(I1{}, tb, v);
                        __builtin_amdgcn_sched_barrier(0);
                        member_fma(I2{}, ta, v);
                    } else {
                        // four entries per member: no read-ahead (register pressure)
                        member_fma(I0{}, ta, v);
                        __builtin_amdgcn_sched_barrier(0);
                        load_member(I1{}, tb);
                        member_fma(I1{}, tb, v);
                        __builtin_amdgcn_sched_barrier(0);
                        load_member(I2{}, ta);
                        member_fma(I2{}, ta, v);
                    }
                    if constexpr (!kEarlyRecord) {
                        __builtin_amdgcn_sched_barrier(0);
                        qn = rec[mi + 3];
                    }
                }
            };
            for_each_class(group_loop, std::make_integer_sequence<int, kQuadGroupClasses>{});
        }
        auto class_loop = [&](auto cls) {
            constexpr int CL = decltype(cls)::value;
            constexpr uint32_t XK = (uint32_t)class_bits(CL, KB, 1);   // k bits the masks flip
            constexpr uint32_t ZK = (uint32_t)class_bits(CL, KB, 2);   // k bits in their Z string
            const uint32_t n = (C.cnt[CL >> 2] >> (8 * (CL & 3))) & 0xffu;
            for (uint32_t i = 0; i < n; ++i, ++mi) {
                const QRec q = qn;
                if constexpr (kEarlyRecord) qn = rec[mi + 1];
                const uint32_t ia = __builtin_amdgcn_udot4(__builtin_amdgcn_perm(B1, B0, q.sel), dotw,
                                                           (mi - C.first) * 16u * esz, false);
                const uint32_t sl = (uint32_t)__popc(tid & q.zl);   // lane sign: its parity
                cplx<R> te[RPT];   // entry for the k bits in p = k & XK
#pragma unroll
                for (int p = 0; p < RPT; ++p) {
                    if ((p & ~(int)XK) != 0) continue;
                    uint32_t off = 0;
#pragma unroll
                    for (int b = 0; b < KB; ++b)
                        if ((p >> b) & 1) off += (q.koffs >> (8 * b)) & 0xffu;
                    te[p] = tab_at(ia + off);
                }
                // table entries first, then the source rows in row order, so
                // that each row's FMAs wait only for its own load
                __builtin_amdgcn_sched_barrier(0);
                const uint32_t sb = tid_b ^ q.xoff;
                cplx<R> v[NC][RPT];
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int k = 0; k < RPT; ++k) v[c][k] = src_row(c, sb + (((uint32_t)k ^ XK) << kLaneBits) * esz);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int p = 0; p < RPT; ++p) {
                    if ((p & ~(int)XK) != 0) continue;
                    te[p].re = flip_odd(te[p].re, sl);
                    te[p].im = flip_odd(te[p].im, sl);
                }
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int k = 0; k < RPT; ++k) {
                        const cplx<R> t = te[k & (int)XK];
                        const bool neg = (__builtin_popcount((uint32_t)k & ZK) & 1) != 0;
                        const R a = neg ? -t.re : t.re, b = neg ? -t.im : t.im;
                        cmac(pr[c][k], pi[c][k], a, b, v[c][k]);
                    }
                if constexpr (!kEarlyRecord) {
                    __builtin_amdgcn_sched_barrier(0);
                    qn = rec[mi + 1];
                }
            }
        };
        for_each_class(class_loop, std::make_integer_sequence<int, ipow3(KB)>{});

        // PAIR: D = (-1)^{|r & zbase|} sum_e phi_e (-1)^{s_q0 e_0 + s_q1 e_1} L_e(r),
        // phi_e = Phi[idx = 3][e] (the entry with s_q0 = s_q1 = 0), L_e(r) =
        // W_e + sum_c w_{e,c} r_c: the lane bits here, the rest staged per row k.
        // The lane part of a thread's rows: l_e = sum over lane bits c of w_{e,c} tid_c.
        auto lane_forms = [&](const QRec& q, R (&l)[4]) {
            const R* w = T.w2 + ((size_t)q.tab * T.n_real + rc) * 4 * (M + 1);
#pragma unroll
            for (int e = 0; e < 4; ++e) l[e] = R(0);
#pragma unroll
            for (int c = 0; c < kLaneBits; ++c) {
                if (c >= (int)lb) break;
                const R b = (R)((tid >> c) & 1u);
#pragma unroll
                for (int e = 0; e < 4; ++e) l[e] = fma(w[e * (M + 1) + c], b, l[e]);
            }
        };
        // Flat PAIR masks (no flipped k bit), by the k bits ZK of their Z string
        // (compile-time row signs).  The qubit signs s_q0, s_q1 and the lane and
        // tile parts of the Z-string sign are the same on all of a thread's rows,
        // and L_e is linear in the k bits:
        //   D_k = (-1)^{|k & ZK|} (A + sum over set bits b of k of Om_b),
        //   A = (-1)^{s} sum_e phi_e sigma_e (l_e + t_{0,e}),
        //   Om_b = (-1)^{s} sum_e phi_e sigma_e w_{e,lb+b},
        // sigma_e = (-1)^{s_q0 e_0 + s_q1 e_1}: one complex add per row.
        auto flat_loop = [&](auto cls) {
            constexpr int ZK = decltype(cls)::value;
            const uint32_t n = (C.pcnt[ZK >> 2] >> (8 * (ZK & 3))) & 0xffu;
            for (uint32_t i = 0; i < n; ++i, ++mi) {
                const QRec q = rec[mi];
                const R* w = T.w2 + ((size_t)q.tab * T.n_real + rc) * 4 * (M + 1);
                const cplx<R>* ph = T.phi2 + (size_t)q.tab * 16 + 12;
                R l[4];
                lane_forms(q, l);
                const R* t0 = reinterpret_cast<const R*>(tab_b + q.sel);   // t_{0,e}
                const uint32_t rl = tid | base;
                const uint32_t sa = bit(rl, mask_q(q.qpack, 0)) ^ 1u, sbb = bit(rl, mask_q(q.qpack, 1)) ^ 1u;
                const uint32_t s = parity(rl & q.zbase);
                // sum_e phi_e sigma_e y_e, signed by s
                auto combine = [&](R y0, R y1, R y2, R y3) {
                    const R b1 = flip(y1, sa), b2 = flip(y2, sbb), b3 = flip(y3, sa ^ sbb);
                    cplx<R> o;
                    o.re = flip(ph[0].re * y0 + ph[1].re * b1 + ph[2].re * b2 + ph[3].re * b3, s);
                    o.im = flip(ph[0].im * y0 + ph[1].im * b1 + ph[2].im * b2 + ph[3].im * b3, s);
                    return o;
                };
                cplx<R> X[RPT];
                X[0] = combine(l[0] + t0[0], l[1] + t0[1], l[2] + t0[2], l[3] + t0[3]);
#pragma unroll
                for (int b = 0; b < KB; ++b) {
                    const int c = (int)lb + b;
                    const cplx<R> om = combine(w[c], w[(M + 1) + c], w[2 * (M + 1) + c], w[3 * (M + 1) + c]);
#pragma unroll
                    for (int k = 1 << b; k < (2 << b); ++k) {
                        X[k].re = X[k - (1 << b)].re + om.re;
                        X[k].im = X[k - (1 << b)].im + om.im;
                    }
                }
                const uint32_t sb = tid_b ^ q.xoff;
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int k = 0; k < RPT; ++k) {
                        const bool neg = (__builtin_popcount((uint32_t)k & (uint32_t)ZK) & 1) != 0;
                        const cplx<R> v = src_row(c, sb + ((uint32_t)k << kLaneBits) * esz);
                        cmac(pr[c][k], pi[c][k], neg ? -X[k].re : X[k].re, neg ? -X[k].im : X[k].im, v);
                    }
            }
        };
        if (RPT > 1) {
            for_each_class(flat_loop, std::make_integer_sequence<int, RPT>{});
        } else {
            flat_loop(std::integral_constant<int, 0>{});
        }
        for (uint32_t i = n_flat; i < C.n_pair; ++i, ++mi) {
            const QRec q = rec[mi];
            const cplx<R>* ph = T.phi2 + (size_t)q.tab * 16 + 12;
            R l[4];
            lane_forms(q, l);
            const uint32_t q0 = mask_q(q.qpack, 0), q1 = mask_q(q.qpack, 1);
            const uint32_t rl = tid | base;
            const uint32_t sa_l = bit(rl, q0) ^ 1u, sb_l = bit(rl, q1) ^ 1u, s_l = parity(rl & q.zbase);
            const uint32_t sb = tid_b ^ q.xoff;
            const R* tk = reinterpret_cast<const R*>(tab_b + q.sel);
#pragma unroll
            for (int k = 0; k < RPT; ++k) {
                const uint32_t kr = (uint32_t)k << lb;
                const uint32_t sa = sa_l ^ bit(kr, q0), sbb = sb_l ^ bit(kr, q1);
                const uint32_t s = s_l ^ parity(kr & q.zbase);
                const R a0 = l[0] + tk[k * 4 + 0];
                const R a1 = flip(l[1] + tk[k * 4 + 1], sa);
                const R a2 = flip(l[2] + tk[k * 4 + 2], sbb);
                const R a3 = flip(l[3] + tk[k * 4 + 3], sa ^ sbb);
                const R dre = flip(ph[0].re * a0 + ph[1].re * a1 + ph[2].re * a2 + ph[3].re * a3, s);
                const R dim = flip(ph[0].im * a0 + ph[1].im * a1 + ph[2].im * a2 + ph[3].im * a3, s);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const cplx<R> v = src_row(c, sb + (((uint32_t)k ^ q.koffs) << lb) * esz);
                    cmac(pr[c][k], pi[c][k], dre, dim, v);
                }
            }
        }
        // DIAG (source = own row): the precomputed diagonal of H
        for (uint32_t i = 0; i < C.n_diag; ++i, ++mi) {
            const double* dg = T.diag + (uint64_t)rc * L.dim + base + tid;
#pragma unroll
            for (int k = 0; k < RPT; ++k) {
                const R d = (R)dg[(uint32_t)k << lb];
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const cplx<R> v = src_row(c, tid_b + ((uint32_t)k << lb) * esz);
                    pr[c][k] = fma(d, v.re, pr[c][k]);
                    pi[c][k] = fma(d, v.im, pi[c][k]);
                }
            }
        }
        if (kSplit) carry();
    }

    // QUAD masks that flip only tile bits: D_x is one number per tile, the
    // source rows are the same rows of tile ^ x_high.  Streamed straight from
    // global memory with the next mask's rows loaded one mask ahead.
    if (f1 > f0) {
        cplx<R> vn[NC][RPT];
        FarRec fn = L.far[f0];
        const cplx<R>* sp = psi + ((uint64_t)(tile ^ fn.x_high) << L.tile_bits);
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < RPT; ++k) vn[c][k] = (sp + c * L.dim)[tid + k * nt];
        for (int f = f0; f < f1; ++f) {
            const FarRec fc = fn;
            cplx<R> v[NC][RPT];
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int k = 0; k < RPT; ++k) v[c][k] = vn[c][k];
            if (f + 1 < f1) {
                fn = L.far[f + 1];
                sp = psi + ((uint64_t)(tile ^ fn.x_high) << L.tile_bits);
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int k = 0; k < RPT; ++k) vn[c][k] = (sp + c * L.dim)[tid + k * nt];
            }
            const cplx<R> t = T.tab4[((size_t)fc.tab * T.n_real + rc) * 16 + quad_index(base, fc.qpack)];
            const uint32_t s = parity(base & fc.zbase);
            const R tr = flip(t.re, s), ti = flip(t.im, s);
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int k = 0; k < RPT; ++k) cmac(pr[c][k], pi[c][k], tr, ti, v[c][k]);
            if (kSplit && (f & 63) == 63) carry();
        }
        if (kSplit) carry();
    }
    if constexpr (SPLIT) {
        parts += blockIdx.z * L.part_stride + (uint64_t)(blockIdx.y * NC) * L.dim + base + tid;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < RPT; ++k)
                parts[c * L.dim + k * nt] = kSplit ? c128{acc_re[c][k], acc_im[c][k]}
                                                   : c128{(double)pr[c][k], (double)pi[c][k]};
        return;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            cplx<R> o;
            o.re = kSplit ? (R)acc_re[c][k] : pr[c][k];
            o.im = kSplit ? (R)acc_im[c][k] : pi[c][k];
            (out + c * L.dim)[(uint64_t)base + tid + k * nt] = o;
        }
}

// out[e] = sum over p of parts[p * n + e], e < n: the slices of a launch with
// its masks split over n_parts workgroups per tile.  A workgroup owns 32
// elements and eight threads share one (slices p = s, s + 8, ...; the eight sums
// are added in order through LDS), so that few rows with many slices still
// keep enough loads in flight.  n is a multiple of 32 or the tail is masked.
template <typename R>
__global__ void __launch_bounds__(256) k_sum_parts(const c128* __restrict__ parts, int n_parts, uint64_t n,
                                                   cplx<R>* __restrict__ out)
{
    __shared__ c128 red[8][32];
    const uint32_t l = threadIdx.x & 31u, s = threadIdx.x >> 5;
    const uint64_t e = (uint64_t)blockIdx.x * 32 + l;
    c128 a{0.0, 0.0};
    if (e < n) {
#pragma unroll 4
        for (int p = (int)s; p < n_parts; p += 8) {
            const c128 v = parts[(uint64_t)p * n + e];
            a.re += v.re;
            a.im += v.im;
        }
    }
    red[s][l] = a;
    __syncthreads();
    if (s == 0 && e < n) {
#pragma unroll
        for (int k = 1; k < 8; ++k) {
            a.re += red[k][l].re;
            a.im += red[k][l].im;
        }
        cplx<R> o;
        o.re = (R)a.re;
        o.im = (R)a.im;
        out[e] = o;
    }
}

// dst = transpose of src viewed as a [2^log_h] x [2^log_w] matrix (row-major),
// column by column of a block: dst[c][lo << log_h | hi] (+)= src[c][hi << log_w | lo].
// 32 x 32 tiles through LDS so that both sides are read and written along
// contiguous rows.  With ADD, complex64 sums are formed in FP64 and rounded once.
template <typename R, bool ADD>
__global__ void __launch_bounds__(256) k_transpose(const cplx<R>* __restrict__ src, cplx<R>* __restrict__ dst,
                                                   int log_h, int log_w, uint64_t dim)
{
    __shared__ cplx<R> t[32][33];
    const uint32_t lw = (uint32_t)log_w - 5u;
    const uint64_t bx = blockIdx.x & ((1u << lw) - 1u);   // tile column (lo / 32)
    const uint64_t by = blockIdx.x >> lw;                 // tile row (hi / 32)
    src += (uint64_t)blockIdx.y * dim;
    dst += (uint64_t)blockIdx.y * dim;
    const uint32_t tx = threadIdx.x & 31u, ty = threadIdx.x >> 5;
#pragma unroll
    for (uint32_t j = ty; j < 32; j += 8) t[j][tx] = src[((by * 32 + j) << log_w) | (bx * 32 + tx)];
    __syncthreads();
#pragma unroll
    for (uint32_t j = ty; j < 32; j += 8) {
        const uint64_t o = ((bx * 32 + j) << log_h) | (by * 32 + tx);
        cplx<R> v = t[tx][j];
        if (ADD) {
            const cplx<R> d = dst[o];
            v.re = (R)((double)v.re + (double)d.re);
            v.im = (R)((double)v.im + (double)d.im);
        }
        dst[o] = v;
    }
}

// diag[c][r] = sum_n dw[c][n] (-1)^{|r & dz_n|} for realisation c = blockIdx.y:
// the diagonal of H (the masks with x = 0), FP64.
__global__ void __launch_bounds__(256) k_diag_fill(const uint32_t* __restrict__ dz, const double* __restrict__ dw,
                                                   int n_diag, uint64_t dim, double* __restrict__ diag)
{
    const uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= dim) return;
    const double* d = dw + (size_t)blockIdx.y * n_diag;
    double s = 0.0;
    for (int n = 0; n < n_diag; ++n) s += (__popc((uint32_t)r & dz[n]) & 1u) ? -d[n] : d[n];
    diag[(uint64_t)blockIdx.y * dim + r] = s;
}

// Coefficient table of small states: D_x(r) itself, for every mask and row, in
// the order k_apply_table reads it: [realisation][row block][mask][kTableRows].
constexpr int kTableRows = 16, kTableThreads = 1024, kTableSlots = kTableThreads / kTableRows;
constexpr int kTableMaxBits = 12;
constexpr size_t kTableBytes = (size_t)40 << 20, kTableTraffic = (size_t)64 << 20;

template <typename R>
__global__ void __launch_bounds__(256) k_table_fill(KTerms<double> T, const MaskRec* __restrict__ masks, int n_masks,
                                                    const uint32_t* __restrict__ dz, const double* __restrict__ dw,
                                                    int n_diag, uint32_t dim, uint32_t n_blocks,
                                                    cplx<R>* __restrict__ table)
{
    const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (uint64_t)n_blocks * n_masks * kTableRows) return;
    const uint32_t m = (uint32_t)(e / kTableRows) % (uint32_t)n_masks;
    const uint32_t r = (uint32_t)(e / ((uint64_t)kTableRows * n_masks)) * kTableRows + (uint32_t)(e % kTableRows);
    const int rc = blockIdx.y;
    const MaskRec mk = masks[m];
    const uint32_t type = mk.type_tab >> 28, tab = mk.type_tab & 0x0fffffffu;
    double re = 0.0, im = 0.0;
    if (r < dim) {
        if (type == MASK_QUAD) {
            const c128 t = T.tab4[((size_t)tab * T.n_real + rc) * 16 + quad_index(r, mk.qpack)];
            re = t.re;
            im = t.im;
        } else if (type == MASK_PAIR) {
            // placeholder qubits (31) read as 0
            const uint32_t idx = bit(r, mask_q(mk.qpack, 0)) | (bit(r, mask_q(mk.qpack, 1)) << 1);
            for (int k = 0; k < 4; ++k) {
                const double* w = T.w2 + (((size_t)tab * T.n_real + rc) * 4 + k) * (T.M + 1);
                double l = w[T.M];
                for (int c = 0; c < T.M; ++c)
                    if ((r >> c) & 1u) l += w[c];
                const c128 ph = T.phi2[(size_t)tab * 16 + idx * 4 + k];
                re += ph.re * l;
                im += ph.im * l;
            }
        } else {
            const double* d = dw + (size_t)rc * n_diag;
            for (int n = 0; n < n_diag; ++n) re += parity(r & dz[n]) ? -d[n] : d[n];
        }
        const uint32_t sg = type == MASK_DIAG ? 0u : parity(r & mk.zbase);
        re = flip(re, sg);
        im = flip(im, sg);
    }
    cplx<R> o;
    o.re = (R)re;
    o.im = (R)im;
    table[(uint64_t)rc * n_blocks * n_masks * kTableRows + e] = o;
}

struct KColumns {
    int32_t real[kColsPerLaunch];
};

// H psi of a small state from its coefficient table: one multiply-add per
// (row, mask), FP64 sums.  A workgroup owns 16 rows of one column, and 64 groups
// of 16 threads take every 64th mask, so that 2^8 .. 2^12 rows keep 16 .. 256
// workgroups of 16 waves in flight with a few masks each; the groups' sums are
// added in a fixed order.  Bound by its loads' latency (table entry, mask, then
// the amplitude), up to 2^12 rows by the table's bytes from L2 and the
// Infinity Cache (37 MB at N=24 in complex128).  REC: the product goes straight
// into a Chebyshev recurrence step (RecArgs) instead of out, one launch for two
// (the reverse sweep at N=24 is mostly such pairs of short launches).
template <typename R, bool REC>
__device__ __forceinline__ void apply_table(const cplx<R>* __restrict__ table, const MaskRec* __restrict__ masks,
                                            int n_masks, int rc, uint32_t dim, const cplx<R>* __restrict__ psi,
                                            cplx<R>* out, const RecArgs& q)
{
    __shared__ c128 red[kTableThreads / 64][kTableRows];
    const uint32_t tid = threadIdx.x, rl = tid % kTableRows, slot = tid / kTableRows;
    const uint32_t r = blockIdx.x * kTableRows + rl;
    const cplx<R>* t = table + ((uint64_t)rc * gridDim.x + blockIdx.x) * n_masks * kTableRows + tid;
    psi += (uint64_t)blockIdx.y * dim;
    double ar = 0.0, ai = 0.0;
    if (r < dim) {
#pragma unroll 4
        for (int m = (int)slot; m < n_masks; m += kTableSlots) {
            const cplx<R> d = *t;
            t += kTableThreads;
            const cplx<R> v = psi[r ^ masks[m].x];
            const double dr = d.re, di = d.im, vr = v.re, vi = v.im;
            ar = fma(dr, vr, ar);
            ar = fma(-di, vi, ar);
            ai = fma(dr, vi, ai);
            ai = fma(di, vr, ai);
        }
    }
    // the four groups of a wave, then the waves in order
#pragma unroll
    for (int off = kTableRows; off < 64; off <<= 1) {
        ar += __shfl_xor(ar, off, 64);
        ai += __shfl_xor(ai, off, 64);
    }
    if ((tid & 63u) < kTableRows) red[tid >> 6][rl] = c128{ar, ai};
    __syncthreads();
    if (tid < kTableRows && r < dim) {
        double sr = 0.0, si = 0.0;
#pragma unroll
        for (int w = 0; w < kTableThreads / 64; ++w) {
            sr += red[w][rl].re;
            si += red[w][rl].im;
        }
        cplx<R> o;
        o.re = (R)sr;
        o.im = (R)si;
        if constexpr (REC) {   // one complex128 column; the formula of k_cheb_rec
            const cplx<R> yv = psi[r];
            double re = q.b * ((double)o.re - q.gamma * (double)yv.re);
            double im = q.b * ((double)o.im - q.gamma * (double)yv.im);
            if (q.z) {
                const c128 zv = q.z[r];
                re += q.s * zv.re;
                im += q.s * zv.im;
            }
            if (q.x) {
                const c128 xv = q.x[r];
                re += q.c_re * xv.re - q.c_im * xv.im;
                im += q.c_re * xv.im + q.c_im * xv.re;
            }
            o.re = (R)re;
            o.im = (R)im;
            if (q.acc) {
                const c128 a = q.acc[r];
                q.acc[r] = c128{a.re + q.ca_re * re - q.ca_im * im, a.im + q.ca_re * im + q.ca_im * re};
            }
        }
        out[(uint64_t)blockIdx.y * dim + r] = o;
    }
}

template <typename R>
__global__ void __launch_bounds__(kTableThreads) k_apply_table(const cplx<R>* __restrict__ table,
                                                               const MaskRec* __restrict__ masks, int n_masks,
                                                               KColumns C, uint32_t dim,
                                                               const cplx<R>* __restrict__ psi, cplx<R>* out)
{
    apply_table<R, false>(table, masks, n_masks, C.real[blockIdx.y], dim, psi, out, RecArgs{});
}

__global__ void __launch_bounds__(kTableThreads) k_apply_table_rec(const c128* __restrict__ table,
                                                                   const MaskRec* __restrict__ masks, int n_masks,
                                                                   uint32_t dim, const c128* __restrict__ psi, c128* out,
                                                                   RecArgs q)
{
    apply_table<double, true>(table, masks, n_masks, 0, dim, psi, out, q);
}

uint32_t table_blocks(const HamiltonianDev& H)
{
    return ((1u << H.M) + kTableRows - 1) / kTableRows;
}

size_t table_entries(const HamiltonianDev& H)
{
    return (size_t)table_blocks(H) * kTableRows * H.host_masks->size();
}

// Whether a product runs from the coefficient table: states of at most 2^12
// rows whose table over all realisations fits kTableBytes, and few enough
// columns that reading it once per column (kTableTraffic) stays cheaper than
// forming the coefficients; never when the caller has chosen a tile.
bool use_table(const HamiltonianDev& H, const ApplyPlan& P, int nvec, size_t esz)
{
    if (P.fixed_tile || H.M > kTableMaxBits) return false;
    const size_t one = table_entries(H) * esz;
    return one * H.n_real <= kTableBytes && one * std::min(nvec, kColsPerLaunch) <= kTableTraffic;
}

// Builds the table of an element type the first time it is needed.
template <typename R>
void ensure_table(const HamiltonianDev& H, TableBuf& buf, hipStream_t s)
{
    if (buf.ready) return;
    const size_t n = table_entries(H);
    buf.ensure(n * H.n_real * sizeof(cplx<R>));
    KTerms<double> T{H.tab4_d, H.qinfo, H.phi2_d, H.w2_d, nullptr, H.n_real, H.M};
    hipLaunchKernelGGL(k_table_fill<R>, dim3((uint32_t)((n + 255) / 256), (uint32_t)H.n_real), dim3(256), 0, s, T, H.masks,
                       (int)H.host_masks->size(), H.dz, H.dw_d, H.n_diag, 1u << H.M, table_blocks(H), buf.as<cplx<R>>());
    SYK_HIP(hipGetLastError());
    SYK_HIP(hipStreamSynchronize(s));   // once per handle: later calls may come on other streams
    buf.ready = true;
}

template <typename R>
void launch_table(const HamiltonianDev& H, const DevBuf& table, int nvec, const int32_t* real_of_col, const void* psi,
                  void* out, hipStream_t s)
{
    const uint32_t dim = 1u << H.M;
    for (int c0 = 0; c0 < nvec; c0 += kColsPerLaunch) {
        KColumns C{};
        const int n = std::min(kColsPerLaunch, nvec - c0);
        for (int c = 0; c < n; ++c) C.real[c] = real_of_col ? real_of_col[c0 + c] : 0;
        hipLaunchKernelGGL(k_apply_table<R>, dim3(table_blocks(H), (uint32_t)n), dim3(kTableThreads), 0, s,
                           table.as<cplx<R>>(), H.masks, (int)H.host_masks->size(), C, dim,
                           static_cast<const cplx<R>*>(psi) + (uint64_t)c0 * dim,
                           static_cast<cplx<R>*>(out) + (uint64_t)c0 * dim);
        SYK_HIP(hipGetLastError());
    }
}

void launch_table_any(const HamiltonianDev& H, syk_dtype dtype, int nvec, const int32_t* real_of_col, const void* psi,
                      void* out, hipStream_t s)
{
    if (dtype == SYK_C128) launch_table<double>(H, H.table_d, nvec, real_of_col, psi, out, s);
    else launch_table<float>(H, H.table_f, nvec, real_of_col, psi, out, s);
}

// Fills H.diag the first time it is needed (on the stream, then waits for it).
void ensure_diag(const HamiltonianDev& H, hipStream_t s)
{
    if (H.diag_ready) return;
    const uint64_t dim = (uint64_t)1 << H.M;
    H.diag.ensure((size_t)H.n_real * dim * sizeof(double));
    const dim3 grid((uint32_t)((dim + 255) / 256), (uint32_t)H.n_real);
    hipLaunchKernelGGL(k_diag_fill, grid, dim3(256), 0, s, H.dz, H.dw_d, H.n_diag, dim, H.diag.as<double>());
    SYK_HIP(hipGetLastError());
    SYK_HIP(hipStreamSynchronize(s));   // once per handle: later calls may come on other streams
    H.diag_ready = true;
}

}  // namespace

void launch_transpose(syk_dtype dtype, const void* src, void* dst, int log_h, int log_w, int ncols, uint64_t dim,
                      bool add, hipStream_t s)
{
    if (log_h < 5 || log_w < 5 || log_h + log_w > 40) throw Error(SYK_EINVAL, "transpose: unsupported shape");
    dim3 grid((uint32_t)((dim >> 10)), ncols), block(256);
    if (dtype == SYK_C128) {
        auto* i = static_cast<const c128*>(src);
        auto* o = static_cast<c128*>(dst);
        if (add) hipLaunchKernelGGL((k_transpose<double, true>), grid, block, 0, s, i, o, log_h, log_w, dim);
        else hipLaunchKernelGGL((k_transpose<double, false>), grid, block, 0, s, i, o, log_h, log_w, dim);
    } else {
        auto* i = static_cast<const c64*>(src);
        auto* o = static_cast<c64*>(dst);
        if (add) hipLaunchKernelGGL((k_transpose<float, true>), grid, block, 0, s, i, o, log_h, log_w, dim);
        else hipLaunchKernelGGL((k_transpose<float, false>), grid, block, 0, s, i, o, log_h, log_w, dim);
    }
    SYK_HIP(hipGetLastError());
}

namespace {

template <typename R, bool SPLIT>
void launch_k_apply(const ApplyPlan& P, const KTerms<R>& T, const QApplyChunk* chunks, const QRec* rec,
                    const KLayout& L, int ncols, int nc, const cplx<R>* in, cplx<R>* o, c128* parts, hipStream_t s)
{
    if (nc == 2) {
        // the caller has checked that the columns pair up by realisation
        if (ncols % 2 != 0) throw Error(SYK_EINVAL, "apply_H: odd column count for two columns per workgroup");
        dim3 grid(L.n_tiles, ncols / 2, L.n_parts), block(P.nt);
        switch (P.rpt) {
        case 4: hipLaunchKernelGGL((k_apply<R, 4, 2, SPLIT>), grid, block, 0, s, T, chunks, rec, L, in, o, parts); break;
        case 8: hipLaunchKernelGGL((k_apply<R, 8, 2, SPLIT>), grid, block, 0, s, T, chunks, rec, L, in, o, parts); break;
        default: throw Error(SYK_EINVAL, "apply_H: two columns per workgroup need 4 or 8 rows per thread");
        }
    } else {
        dim3 grid(L.n_tiles, ncols, L.n_parts), block(P.nt);
        switch (P.rpt) {
        case 1: hipLaunchKernelGGL((k_apply<R, 1, 1, SPLIT>), grid, block, 0, s, T, chunks, rec, L, in, o, parts); break;
        case 2: hipLaunchKernelGGL((k_apply<R, 2, 1, SPLIT>), grid, block, 0, s, T, chunks, rec, L, in, o, parts); break;
        case 4: hipLaunchKernelGGL((k_apply<R, 4, 1, SPLIT>), grid, block, 0, s, T, chunks, rec, L, in, o, parts); break;
        case 8: hipLaunchKernelGGL((k_apply<R, 8, 1, SPLIT>), grid, block, 0, s, T, chunks, rec, L, in, o, parts); break;
        default: throw Error(SYK_EINVAL, "apply_H: unsupported rows per thread");
        }
    }
    SYK_HIP(hipGetLastError());
}

// out = the sum of a split launch's slices (nothing otherwise)
template <typename R>
void sum_parts(const KLayout& L, const c128* parts, cplx<R>* out, hipStream_t s)
{
    if (L.n_parts <= 1) return;
    const uint64_t n = L.part_stride;
    hipLaunchKernelGGL(k_sum_parts<R>, dim3((uint32_t)((n + 31) / 32)), dim3(256), 0, s, parts, L.n_parts, n, out);
    SYK_HIP(hipGetLastError());
}

template <typename R>
void launch_t(const ApplyPlan& P, const KTerms<R>& T, const QApplyChunk* chunks, const QRec* rec, const KLayout& L,
              int ncols, int nc, const void* psi, void* out, c128* parts, hipStream_t s)
{
    auto* in = static_cast<const cplx<R>*>(psi);
    auto* o = static_cast<cplx<R>*>(out);
    if (L.n_parts > 1) launch_k_apply<R, true>(P, T, chunks, rec, L, ncols, nc, in, o, parts, s);
    else launch_k_apply<R, false>(P, T, chunks, rec, L, ncols, nc, in, o, parts, s);
    sum_parts<R>(L, parts, o, s);
}

constexpr int kSplitGroups = 1024, kMaxParts = 64, kGroupSlots = 512;

// About what a mask costs a workgroup, in single QUAD masks (a PAIR mask has
// twice the arithmetic and reads its weights with scalar loads; one that flips
// a k bit forms its coefficient row by row), and what a chunk's barriers and a
// staged source tile cost.  Only used to cut the masks into parts of similar
// cost.
constexpr double kCostFlatPair = 5.0, kCostPair = 9.0, kCostDiag = 2.0, kCostChunk = 4.0, kCostTile = 8.0;

#include "apply_groups.hpp"

template <typename R>
void launch_groups(const HamiltonianDev& H, const KTerms<R>& T, const HamiltonianDev::GroupTables& A, const KLayout& L, int ncols, const void* psi,
                   void* out, c128* parts, hipStream_t s)
{
    auto* in = static_cast<const cplx<R>*>(psi);
    auto* o = static_cast<cplx<R>*>(out);
    const auto* ch = static_cast<const GroupChunk*>(A.chunks);
    const auto* gr = static_cast<const GroupRec*>(A.groups);
    const auto* tb = static_cast<const cplx<R>*>(A.tables);
    const auto* pt = (sizeof(R) == 8 ? H.pair_tab_d : H.pair_tab_f).as<cplx<R>>();
    const auto* pr = static_cast<const PairRec*>(A.pairs);
    const dim3 grid(L.n_tiles, ncols, L.n_parts), block(256);
    if (L.n_parts > 1) hipLaunchKernelGGL((k_apply_groups<R, true>), grid, block, 0, s, T, ch, gr, tb, pt, pr, L, in, o, parts);
    else hipLaunchKernelGGL((k_apply_groups<R, false>), grid, block, 0, s, T, ch, gr, tb, pt, pr, L, in, o, parts);
    SYK_HIP(hipGetLastError());
    sum_parts<R>(L, parts, o, s);
}

// Chunks and class-sorted records of the apply kernel for tiles of 2^tile_bits
// rows, 2^lane_bits threads and elements of esz bytes.  masks must be sorted by
// x; QUAD masks that neither flip nor sign-depend on a row bit inside a tile go
// to the far list.  max_cost > 0 ends a chunk before the cost of its masks
// would pass it.
void build_apply_tables(const std::vector<MaskRec>& masks_in, int tile_bits, int lane_bits, uint32_t esz,
                        std::vector<QApplyChunk>& chunks, std::vector<QRec>& recs, std::vector<FarRec>& far,
                        double max_cost = 0.0)
{
    const uint32_t row_mask = (1u << tile_bits) - 1u;
    const uint32_t lane_mask = (1u << lane_bits) - 1u;
    const int kb = tile_bits - lane_bits;
    if (kb < 0 || kb > kMaxKBits) throw Error(SYK_EINVAL, "apply_H: unsupported rows per thread");
    const uint32_t kbits_mask = (1u << kb) - 1u;
    auto quad_class_of = [&](const MaskRec& m) { return quad_class(m.x, m.zbase, lane_bits, kb); };
    auto type_of = [](const MaskRec& m) { return m.type_tab >> 28; };
    auto xk_of = [&](const MaskRec& m) { return (m.x >> lane_bits) & kbits_mask; };
    // PAIR masks flipping no k bit, and the k-bit pattern of their Z string
    auto is_k_bit = [&](uint32_t q) { return q >= (uint32_t)lane_bits && q < (uint32_t)tile_bits; };
    auto flat_pair = [&](const MaskRec& m) {
        return type_of(m) == MASK_PAIR && !is_k_bit(mask_q(m.qpack, 0)) && !is_k_bit(mask_q(m.qpack, 1));
    };
    auto zk_of = [&](const MaskRec& m) { return (int)((m.zbase >> lane_bits) & kbits_mask); };
    // table slots (16 entries each) a mask stages
    auto slots_of = [&](const MaskRec& m) { return type_of(m) == MASK_DIAG ? 0u : 1u; };
    auto cost_of = [&](const MaskRec& m) {
        return type_of(m) == MASK_QUAD ? 1.0 : type_of(m) == MASK_DIAG ? kCostDiag : flat_pair(m) ? kCostFlatPair : kCostPair;
    };
    // Inside a run of one x_high: by lane flips, then by k flips, so that the
    // masks of a group are adjacent (a chunk boundary rarely splits one).
    std::vector<MaskRec> masks = masks_in;
    std::stable_sort(masks.begin(), masks.end(), [&](const MaskRec& a, const MaskRec& b) {
        const uint32_t ha = a.x >> tile_bits, hb = b.x >> tile_bits;
        if (ha != hb) return ha < hb;
        const uint32_t la = a.x & lane_mask, lb2 = b.x & lane_mask;
        if (la != lb2) return la < lb2;
        return xk_of(a) < xk_of(b);
    });
    size_t i = 0;
    uint32_t prev_high = 0xffffffffu;
    while (i < masks.size()) {
        // masks of one chunk: same x_high, at most apply_chunk_masks(esz)
        std::vector<uint32_t> mem;
        const uint32_t xh = masks[i].x >> tile_bits;
        const uint32_t cap = (uint32_t)apply_chunk_masks(esz);   // masks and table slots per chunk
        uint32_t used = 0;
        double cost = 0.0;
        while (i < masks.size() && (masks[i].x >> tile_bits) == xh && mem.size() < cap) {
            const MaskRec& m = masks[i];
            // far: coefficient constant over a tile (no flipped qubit and no Z-string bit inside it)
            if (type_of(m) == MASK_QUAD && (m.x & row_mask) == 0u && (m.zbase & row_mask) == 0u) {
                far.push_back({m.x >> tile_bits, m.qpack, m.zbase, m.type_tab & 0x0fffffffu});
            } else {
                if (used + slots_of(m) > cap) break;
                if (max_cost > 0.0 && !mem.empty() && cost + cost_of(m) > max_cost) break;
                used += slots_of(m);
                cost += cost_of(m);
                mem.push_back((uint32_t)i);
            }
            ++i;
        }
        if (mem.empty()) continue;
        const size_t nm = mem.size();
        // records (the PAIR / DIAG table offsets follow the final order)
        std::vector<QRec> rr(nm);
        std::vector<int> key(nm);
        for (size_t u = 0; u < nm; ++u) {
            const MaskRec& m = masks[mem[u]];
            const uint32_t t = type_of(m);
            QRec r{};
            r.zl = m.zbase & lane_mask;
            r.xoff = (m.x & lane_mask) * esz;
            r.tab = m.type_tab & 0x0fffffffu;
            r.xl = m.x & row_mask;
            r.qpack = m.qpack;
            r.zbase = m.zbase;
            if (t == MASK_QUAD) {
                for (int q = 0; q < 4; ++q) {
                    const uint32_t qb = mask_q(m.qpack, q);
                    r.sel |= (qb < (uint32_t)lane_bits ? qb : 0x0cu) << (8 * q);
                    const int b = (int)qb - lane_bits;
                    if (b >= 0 && b < kb) r.koffs |= ((1u << q) * esz) << (8 * b);
                }
                key[u] = 1000 + quad_class_of(m);
            } else {
                r.koffs = (m.x >> lane_bits) & kbits_mask;
                key[u] = t == MASK_PAIR ? (flat_pair(m) ? 2000 + zk_of(m) : 2500) : 3000;
            }
            rr[u] = r;
        }
        // Groups: three QUAD masks with the same lane flips that flip J = 1 or
        // 2 k bits in all three ways, whose classes are those of a group class
        // and whose records agree on what the kernel reads once per group.
        std::vector<int> gcls(nm, -1), gid(nm, 0), gpos(nm, 0);
        uint32_t group_kof[256] = {};
        int ng = 0;
        if (kb == kMaxKBits) {
            std::map<std::pair<uint32_t, int>, std::vector<size_t>> cand;
            for (size_t u = 0; u < nm; ++u) {
                const MaskRec& m = masks[mem[u]];
                const int J = __builtin_popcount(xk_of(m));
                if (type_of(m) == MASK_QUAD && (J == 1 || J == 2)) cand[{m.x & lane_mask, J}].push_back(u);
            }
            for (const auto& kv : cand) {
                const int J = kv.first.second;
                const std::vector<size_t>& v = kv.second;
                if (v.size() != 3) continue;
                size_t mj[3];
                bool ok = true;
                for (int j = 0; j < 3 && ok; ++j) {
                    ok = false;
                    for (size_t u : v)
                        if ((int)xk_of(masks[mem[u]]) == group_xk(J, j)) {
                            mj[j] = u;
                            ok = true;
                        }
                }
                if (!ok) continue;
                int gc = -1;
                for (int P = 0; P < 2 && gc < 0; ++P) {
                    const int g = 2 * (J - 1) + P;
                    bool all = true;
                    for (int j = 0; j < 3; ++j) all = all && quad_class_of(masks[mem[mj[j]]]) == group_member_class(g, j);
                    if (all) gc = g;
                }
                if (gc < 0) continue;
                const QRec& r0 = rr[mj[0]];
                const uint32_t kof = r0.koffs & 0xffu;   // index-bit offset of member 0's lowest flipped k bit
                ok = kof != 0u;
                for (int j = 0; j < 3 && ok; ++j) {
                    const QRec& r = rr[mj[j]];
                    ok = r.sel == r0.sel && r.zl == r0.zl && r.xoff == r0.xoff;
                    uint32_t want = 0, t = 0;
                    for (int b = 0; b < kMaxKBits; ++b)
                        if ((group_xk(J, j) >> b) & 1) want |= (kof << t++) << (8 * b);
                    ok = ok && r.koffs == want;
                }
                if (!ok) continue;
                for (int j = 0; j < 3; ++j) {
                    gcls[mj[j]] = gc;
                    gid[mj[j]] = ng;
                    gpos[mj[j]] = j;
                }
                group_kof[ng++] = kof;
            }
        }
        std::vector<size_t> ord(nm);
        for (size_t u = 0; u < nm; ++u) ord[u] = u;
        auto okey = [&](size_t u) {
            return gcls[u] >= 0 ? std::make_tuple(gcls[u], gid[u], gpos[u]) : std::make_tuple(key[u], 0, 0);
        };
        std::stable_sort(ord.begin(), ord.end(), [&](size_t a, size_t b) { return okey(a) < okey(b); });
        QApplyChunk c{};
        c.x_high = xh;
        c.first = (uint32_t)recs.size();
        c.new_tile = (xh != prev_high) ? 1u : 0u;
        prev_high = xh;
        uint32_t slot = 0;
        for (size_t u : ord) {
            const MaskRec& m = masks[mem[u]];
            const uint32_t t = type_of(m);
            QRec r = rr[u];
            if (t == MASK_QUAD) {
                ++c.n_quad;
                if (gcls[u] >= 0) {
                    if (gpos[u] == 0) {
                        const int g = kQuadClasses + gcls[u];
                        c.cnt[g >> 2] += 1u << (8 * (g & 3));
                        r.koffs = group_kof[gid[u]];
                    }
                } else {
                    const int cls = quad_class_of(m);
                    c.cnt[cls >> 2] += 1u << (8 * (cls & 3));
                }
            } else {
                r.sel = slot * 16u * esz;
                if (t == MASK_PAIR) {
                    ++c.n_pair;
                    if (flat_pair(m)) {
                        const int zk = zk_of(m);
                        c.pcnt[zk >> 2] += 1u << (8 * (zk & 3));
                    }
                } else {
                    ++c.n_diag;
                }
            }
            slot += slots_of(m);
            recs.push_back(r);
        }
        chunks.push_back(c);
    }
    recs.push_back(QRec{});   // one record past the end: loads may run one ahead
}

// Cost of every chunk (see above).
std::vector<double> chunk_costs(const std::vector<QApplyChunk>& chunks)
{
    std::vector<double> cost;
    for (const QApplyChunk& c : chunks) {
        uint32_t n_flat = 0;
        for (int b = 0; b < 8; ++b) n_flat += (c.pcnt[b >> 2] >> (8 * (b & 3))) & 0xffu;
        cost.push_back(c.n_quad + kCostFlatPair * n_flat + kCostPair * (c.n_pair - n_flat) + kCostDiag * c.n_diag +
                       kCostChunk + (c.new_tile ? kCostTile : 0.0));
    }
    return cost;
}

// Chunk boundaries of n_parts contiguous parts of similar cost
// (bounds p .. p + 1 - 1; parts may be empty).
std::vector<uint32_t> part_bounds(const std::vector<double>& cost, int n_parts)
{
    std::vector<double> sum(cost.size() + 1, 0.0);
    for (size_t g = 0; g < cost.size(); ++g) sum[g + 1] = sum[g] + cost[g];
    std::vector<uint32_t> b(n_parts + 1, (uint32_t)cost.size());
    uint32_t g = 0;
    for (int p = 0; p < n_parts; ++p) {
        // the first chunk whose middle lies at or after the part's start
        while (g < cost.size() && 0.5 * (sum[g] + sum[g + 1]) < sum.back() * p / n_parts) ++g;
        b[p] = g;
    }
    return b;
}

// Bit rotation of the second layout: bits s..M-1 of a row become bits
// 0..M-s-1 and bits 0..s-1 become the top bits.
inline uint32_t rotate_bits(uint32_t v, int M, int s)
{
    return (v >> s) | ((v & ((1u << s) - 1u)) << (M - s));
}

}  // namespace

bool quad_in_rotated(const MaskRec& m, int M, int tb)
{
    if ((m.type_tab >> 28) != MASK_QUAD) return false;
    const uint32_t row_mask = (1u << tb) - 1u;
    const int out_a = __builtin_popcount(m.x & ~row_mask);
    const int out_b = __builtin_popcount(rotate_bits(m.x, M, tb) & ~row_mask);
    return out_b < out_a;
}

MaskRec rotate_mask(const MaskRec& m, int M, int tb)
{
    MaskRec r = m;
    r.x = rotate_bits(m.x, M, tb);
    r.zbase = rotate_bits(m.zbase, M, tb);
    r.qpack = 0;   // table index bit q stays bit q; only its qubit moves
    for (int q = 0; q < 4; ++q) {
        const int b = (int)mask_q(m.qpack, q);   // 31: placeholder of an unused index bit
        r.qpack |= (uint32_t)(b == 31 ? 31 : b >= tb ? b - tb : b + (M - tb)) << (8 * q);
    }
    return r;
}

namespace {

// Masks of one layout, in that layout's row coordinates and sorted by x.  With
// two layouts, a QUAD mask goes to the rotated layout (1) when fewer of its
// flipped qubits lie outside a tile there; everything else stays in layout 0.
// A relabelling of qubits keeps every coefficient: only x, zbase and the
// qubit of each table index bit move.
std::vector<MaskRec> layout_masks(const std::vector<MaskRec>& masks, int M, int tb, bool two, int layout)
{
    std::vector<MaskRec> out;
    for (const MaskRec& m : masks) {
        const int in_b = two && quad_in_rotated(m, M, tb);
        if (in_b != layout) continue;
        out.push_back(layout == 0 ? m : rotate_mask(m, M, tb));
    }
    std::stable_sort(out.begin(), out.end(), [](const MaskRec& a, const MaskRec& b) { return a.x < b.x; });
    return out;
}

}  // namespace

std::vector<KRec> build_krecs(const std::vector<MaskRec>& masks, const std::vector<uint64_t>& bin_off, int tile_bits)
{
    const uint32_t row_mask = (1u << tile_bits) - 1u;
    std::vector<KRec> out(masks.size());
    for (size_t i = 0; i < masks.size(); ++i) {
        const MaskRec& m = masks[i];
        const uint32_t type = m.type_tab >> 28, tab = m.type_tab & 0x0fffffffu;
        KRec k{};
        k.xl = m.x & row_mask;
        k.qpack = m.qpack;
        k.zbase = m.zbase;
        k.meta = type << 28 | tab;
        k.bin0 = (uint32_t)bin_off[i];
        k.x_high = m.x >> tile_bits;
        out[i] = k;
    }
    return out;
}

namespace {

// The row layout of the 16-row kernel's second pass: the top kGroupTileBits
// qubits become the low bits of a tile (a rotation by M - kGroupTileBits, so that
// a tile's bits are neighbouring qubits at every M).  A QUAD mask runs there when
// it flips more qubits above the natural tile than below the rotated one; where
// the two tiles share qubits (M < 24) those count as the natural tile's, so that
// all masks of a group, in either layout, go the same way.  M >= 16: the rotated
// tile's k bits lie above the natural tile.
std::vector<MaskRec> group_layout_masks(const std::vector<MaskRec>& masks, int M, bool two, int layout)
{
    const int rot = M - kGroupTileBits;
    if (two && rot < kGroupKBits) throw Error(SYK_EINVAL, "apply_H groups: too few qubits for two layouts");
    const uint32_t below = (1u << std::max(kGroupTileBits, rot)) - 1u;
    std::vector<MaskRec> out;
    for (const MaskRec& m : masks) {
        const int out_a = __builtin_popcount(m.x >> kGroupTileBits);
        const int out_b = __builtin_popcount(m.x & below);
        const int in_b = two && (m.type_tab >> 28) == MASK_QUAD && out_b < out_a;
        if (in_b != layout) continue;
        out.push_back(layout == 0 ? m : rotate_mask(m, M, rot));
    }
    return out;
}

// Tables of a launch in one allocation and one upload: a handle's first product is
// mostly these (N=26, five complex64 columns, beside other handles: 290 us, 360 with
// an allocation and a copy for each).
struct TablePack {
    std::vector<char> host;
    size_t room(size_t n)   // of n bytes (at least 64), its offset
    {
        const size_t o = (host.size() + 255) & ~(size_t)255;
        host.resize(o + std::max<size_t>(n, 64));
        return o;
    }
    template <typename V>
    size_t put(const V& v)
    {
        const size_t n = v.size() * sizeof(v[0]), o = room(n);
        if (n) std::memcpy(host.data() + o, v.data(), n);
        return o;
    }
    // allocates b with `more` bytes behind the tables; returns their offset
    size_t upload(DevBuf& b, size_t more = 0)
    {
        const size_t o = (host.size() + 255) & ~(size_t)255;
        b.ensure(o + more);
        SYK_HIP(hipMemcpy(b.p, host.data(), host.size(), hipMemcpyHostToDevice));
        return o;
    }
};

int group_tables_key(const ApplyPlan& P, uint32_t esz, int layout)
{
    return (((int)esz * 2 + P.two_layouts) * 2 + layout) * 256 + P.cut;
}

const HamiltonianDev::GroupTables& group_tables_for(const HamiltonianDev& H, const ApplyPlan& P, uint32_t esz, int layout)
{
    const int key = group_tables_key(P, esz, layout);
    auto it = H.group_tables.find(key);
    if (it == H.group_tables.end()) {
        const std::vector<MaskRec> masks = group_layout_masks(*H.host_masks, H.M, P.two_layouts != 0, layout);
        // parts of a split launch: chunks of at most half a part's share, so that the parts come out even
        const double cost = (double)masks.size() + 4.0 * H.M * H.M / 2;
        const GroupTables G = build_group_tables(masks, esz, P.cut > 1 ? std::max(6.0, 0.5 * cost / P.cut) : 0.0);
        std::unique_ptr<HamiltonianDev::GroupTables> t(new HamiltonianDev::GroupTables());
        t->n_chunks = (int)G.chunks.size();
        t->n_far = (int)G.far.size();
        t->n_tables = (int)G.tabs.size();
        // the records, the table indices and (filled on the device) the QUAD tables in staging order
        const uint32_t n16 = (uint32_t)G.tabs.size() * 16u;
        TablePack pk;
        const size_t o_ch = pk.put(G.chunks), o_gr = pk.put(G.groups), o_pr = pk.put(G.pairs), o_far = pk.put(G.far);
        const size_t o_idx = pk.put(G.tabs);
        const size_t o_pc = pk.put(P.cut > 1 ? part_bounds(G.cost, P.cut) : std::vector<uint32_t>());
        const size_t o_tab = pk.upload(t->buf, std::max<size_t>((size_t)n16 * H.n_real * esz, 64));
        char* d = static_cast<char*>(t->buf.p);
        t->chunks = d + o_ch;
        t->groups = d + o_gr;
        t->pairs = d + o_pr;
        t->far = d + o_far;
        t->part_chunk = d + o_pc;
        t->tables = d + o_tab;
        // the PAIR masks' tables once per handle and element type; all finished before
        // this returns, as later calls may come on other streams
        const dim3 og((n16 + 255) / 256, (uint32_t)H.n_real), pg((uint32_t)H.host_masks->size(), (uint32_t)H.n_real);
        size_t n_pairs = 0;
        for (const MaskRec& m : *H.host_masks) n_pairs += (m.type_tab >> 28) == MASK_PAIR;
        TableBuf& pt = esz == 16 ? H.pair_tab_d : H.pair_tab_f;
        const bool need = !pt.ready;
        if (need) pt.ensure(std::max<size_t>(n_pairs * H.n_real * pair_table_size(H.M) * esz, 64));
        auto build = [&](auto zero, const auto* tab4) {
            typedef decltype(zero) R;
            if (n16)
                hipLaunchKernelGGL(k_order_tables<R>, og, dim3(256), 0, 0, tab4, reinterpret_cast<const uint32_t*>(d + o_idx),
                                   t->n_tables, H.n_real, static_cast<cplx<R>*>(t->tables));
            if (need)
                hipLaunchKernelGGL(k_pair_tables<R>, pg, dim3(256), 0, 0, H.masks, H.phi2_d, H.w2_d, H.n_real, H.M,
                                   pt.as<cplx<R>>());
        };
        if (esz == 16) build(0.0, H.tab4_d);
        else build(0.0f, H.tab4_f);
        SYK_HIP(hipGetLastError());
        SYK_HIP(hipStreamSynchronize(0));
        pt.ready = true;
        it = H.group_tables.emplace(key, std::move(t)).first;
    }
    return *it->second;
}

int apply_tables_key(const ApplyPlan& P, uint32_t esz, int layout)
{
    return ((((P.tile_bits * 16 + P.lb) * 32 + (int)esz) * 2 + P.two_layouts) * 2 + layout) * 256 + P.cut;
}

const HamiltonianDev::ApplyTables& apply_tables_for(const HamiltonianDev& H, const ApplyPlan& P, uint32_t esz,
                                                    int layout)
{
    const int key = apply_tables_key(P, esz, layout);
    auto it = H.apply_tables.find(key);
    if (it == H.apply_tables.end()) {
        std::vector<QApplyChunk> ch;
        std::vector<QRec> rc;
        std::vector<FarRec> far;
        const std::vector<MaskRec> masks = layout_masks(*H.host_masks, H.M, P.tile_bits, P.two_layouts != 0, layout);
        // parts of a split launch: chunks of at most half a part's share, so that the parts come out even
        const double cost = (double)masks.size() + 4.0 * H.M * H.M / 2;
        build_apply_tables(masks, P.tile_bits, P.lb, esz, ch, rc, far,
                           P.cut > 1 ? std::max(6.0, 0.5 * cost / P.cut) : 0.0);
        std::unique_ptr<HamiltonianDev::ApplyTables> t(new HamiltonianDev::ApplyTables());
        t->n_chunks = (int)ch.size();
        t->n_far = (int)far.size();
        TablePack pk;
        const size_t o_ch = pk.put(ch), o_rc = pk.put(rc), o_far = pk.put(far);
        const size_t o_pc = pk.put(P.cut > 1 ? part_bounds(chunk_costs(ch), P.cut) : std::vector<uint32_t>());
        (void)pk.upload(t->buf);
        const char* d = static_cast<const char*>(t->buf.p);
        t->chunks = d + o_ch;
        t->recs = d + o_rc;
        t->far = d + o_far;
        t->part_chunk = d + o_pc;
        it = H.apply_tables.emplace(key, std::move(t)).first;
    }
    return *it->second;
}

}  // namespace

ApplyPlan plan_apply(int M, int nvec, syk_dtype dtype, const ApplyTuning* tune, bool allow_groups)
{
    ApplyPlan P{};
    P.slices = (nvec + kColsPerLaunch - 1) / kColsPerLaunch;
    // 2048-row source tiles (256 threads, 8 rows each).  Where the tiles and
    // columns of a launch are fewer than kSplitGroups (four workgroups on each
    // of the 256 CUs), the masks are split over several workgroups per tile, at most
    // kMaxParts of them: up to there the full tile's arithmetic per mask is worth
    // more than the partial sums cost (16 B written and read per row and part).
    // Automatic plans come here with at most 2^12 rows (more run the 16-row kernel)
    // and too many columns or realisations for the coefficient table, or with two
    // columns per workgroup; us per call in complex128, smaller tiles unsplit ->
    // split: N=20 64 columns 67 -> 25, N=22 16 columns 89 -> 31, 64 columns 107 -> 38,
    // N=24 8 columns 129 -> 34, 64 columns 166 -> 63.  A shape given by the caller is
    // run as it is given, unsplit.
    int tb = std::min(M, 11);
    P.parts = 1;
    P.fixed_tile = tune && tune->tile_bits > 0;
    P.cols = tune ? tune->cols : 0;
    if (P.fixed_tile) {
        tb = std::min(tune->tile_bits, M);
    } else {
        const int64_t wg = ((int64_t)1 << (M - tb)) * std::min(nvec, kColsPerLaunch);
        if (wg < kSplitGroups) P.parts = (int)std::min<int64_t>(kMaxParts, (kSplitGroups + wg - 1) / wg);
    }
    // 8 lane bits; a thread owns 2^(tile_bits - 8) rows, at most 8
    if (tb > kLaneBits + kMaxKBits) throw Error(SYK_EINVAL, "apply_H: tile_bits above 11");
    // From 2^13 rows on the 16-row kernel with tiles of 2^12 rows (one column, us, 8
    // rows -> 16: complex128 N=26 19.7 -> 17.4, N=32 55 -> 42, N=36 237 -> 192, N=44
    // 7250 -> 5790; complex64 N=32 44 -> 39, N=44 4665 -> 4127; an exception in
    // plan_of_call).  Its split fills the 512 workgroups the chip holds (two per CU):
    // the parts that cost the fewest rounds of them, each part weighed with the
    // 128 KiB its sums write and read per workgroup (N=32 complex128: 42 us with 31
    // parts, 51 with 24, 53 with 64; seven columns: 195 with nine, 244 with five,
    // whose last round is part-full).
    P.groups = allow_groups && !P.fixed_tile && M > kGroupTileBits;
    if (P.groups) {
        tb = kGroupTileBits;
        const int64_t wg = ((int64_t)1 << (M - tb)) * std::min(nvec, kColsPerLaunch);
        const double n_masks = M * (M - 1) * (double)(M - 2) * (M - 3) / 24.0 + M * (M - 1) / 2.0;
        double best = 1e300;
        P.parts = 1;
        for (int p = 1; p <= kMaxParts && (p == 1 || p * wg <= kSplitGroups); ++p) {
            const double score = (double)((wg * p + kGroupSlots - 1) / kGroupSlots) / p + 0.13 * wg * (p - 1) / n_masks;
            if (score < best) {
                best = score;
                P.parts = p;
            }
        }
    }
    P.tile_bits = tb;
    P.lb = std::min(tb, kLaneBits);
    P.nt = 1 << P.lb;
    P.rpt = 1 << (tb - P.lb);
    P.xcd_remap = tune ? tune->xcd_remap : 1;
    // Two columns of one realisation per workgroup (where a launch's columns
    // pair up) need a whole 256-thread workgroup with at least 4 rows per
    // thread.  By default complex64 takes them: its 8-row kernel holds both
    // columns' sums at three waves per SIMD and decodes each mask once for
    // both; complex128 would drop to two waves per SIMD and gains nothing.
    const bool explicit_cols = P.cols > 0;
    P.nc = explicit_cols ? P.cols : (dtype == SYK_C64 ? 2 : 1);
    if (P.groups) P.nc = 1;
    if (P.nc == 2 && P.rpt < 4) {
        if (explicit_cols && tune->tile_bits > 0)
            throw Error(SYK_EINVAL, "apply_H: two columns per workgroup need tile_bits >= 10");
        P.nc = 1;
    }
    // QUAD masks whose four qubits all lie above the tile would each stream a
    // whole tile from global memory; with at least C(7,4) of them, run the
    // masks that sit better in the rotated layout there.  A split launch is
    // short enough that the second layout's launches (two transposes, another
    // product and sum) weigh more: from C(8,4) on (16-row kernel, one column, us,
    // one layout / two: N=36 complex128 190 / 199, complex64 147 / 165; N=38 430 /
    // 438, 324 / 330; N=40 1095 / 1052, 785 / 744).  The 16-row kernel unsplit: from
    // C(6,4) on (64 complex64 columns at N=36: 7.29 ms with two layouts, 7.45 with one).
    P.two_layouts = (M - tb >= (P.parts > 1 ? 8 : P.groups ? 6 : 7) && tb >= 8) ? 1 : 0;
    P.rot = P.groups ? M - tb : tb;
    P.cut = P.parts;
    return P;
}

namespace {
void launch_apply_impl(const HamiltonianDev& H, syk_dtype dtype, int nvec, const int32_t* real_of_col,
                       const void* psi, void* out, const ApplyPlan& P, hipStream_t s, void* rot_in, void* rot_out,
                       void* parts, bool timed);
}  // namespace

// The plan of one call whose columns all pair up by realisation: two columns per
// workgroup at 8 rows, if the caller asked for two, or for complex64 blocks of 2^18
// and 2^19 rows with at least kPairGroups workgroups unless the caller asked for one
// (ms, 16-row kernel -> two columns: N=36 32 columns 3.76 -> 3.65, 64 columns 7.43 ->
// 7.30; N=38 16 columns 4.64 -> 4.57, 64 columns 18.1 -> 17.9).  With half the
// workgroups it is slower (N=36 16 columns 1.89 -> 2.23, N=38 8 columns 2.33 -> 2.76),
// and so it is on smaller and larger states at every width (N=32 64 columns 1.17 ->
// 1.44, N=34 2.96 -> 3.06, N=40 43.5 -> 44.6).
constexpr int64_t kPairGroups = 2048;

static ApplyPlan plan_of_call(const HamiltonianDev& H, const ApplyPlan& P, syk_dtype dtype, int nvec, const int32_t* real)
{
    if (!P.groups || nvec % 2 != 0 || P.cols == 1) return P;
    if (P.cols != 2 && (dtype != SYK_C64 || H.M < 18 || H.M > 19 ||
                        ((int64_t)1 << (H.M - 11)) * (std::min(nvec, kColsPerLaunch) / 2) < kPairGroups))
        return P;
    for (int c = 0; real && c < nvec; c += 2)
        if (real[c] != real[c + 1]) return P;
    const ApplyTuning t{0, P.xcd_remap, P.cols};
    const ApplyPlan Q = plan_apply(H.M, nvec, dtype, &t, false);
    return Q.nc == 2 ? Q : P;
}

// Bytes of the partial sums of a split launch (FP64 for both state types): at
// most kMaxPartsBytes, 2 * kSplitGroups workgroups' 2^11 rows or half as many of 2^12.
constexpr size_t kMaxPartsBytes = (size_t)64 << 20;
static size_t parts_bytes(const ApplyPlan& P, int nvec, uint64_t dim)
{
    return P.parts > 1 ? (size_t)P.parts * std::min(nvec, kColsPerLaunch) * dim * sizeof(c128) : 0;
}

// Scratch of the allocation-free apply (syk_apply_H_noalloc): the rotated
// copy of psi and the rotated layout's output of one call, side by side.  Each
// device holds its own copy for the life of the process; host code reaches it
// only through the address hipGetSymbolAddress returns on that device.
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

void* noalloc_scratch_ptr(int device)
{
    static std::mutex mu;
    static std::map<int, void*> ptr;   // per device, set once with that device current
    std::lock_guard<std::mutex> l(mu);
    auto it = ptr.find(device);
    if (it != ptr.end()) return it->second;
    int cur = -1;
    SYK_HIP(hipGetDevice(&cur));
    if (cur != device) throw Error(SYK_EINVAL, "apply_H_noalloc: the handle's device is not the current device");
    void* p = nullptr;
    SYK_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) throw Error(SYK_EHIP, "apply_H_noalloc: no device address for the scratch array");
    ptr.emplace(device, p);
    return p;
}

namespace {

// Scratch of a launch: the rotated layout's two buffers, then the partial sums.
size_t rot_bytes(const ApplyPlan& P, int nvec, uint64_t dim, size_t esz)
{
    return P.two_layouts ? 2 * (size_t)std::min(nvec, kColsPerLaunch) * dim * esz : 0;
}

// Whether the stream is recording into a graph.
bool capturing(hipStream_t s)
{
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &c) != hipSuccess) {
        (void)hipGetLastError();   // asked of the null stream while another one records
        return false;
    }
    return c != hipStreamCaptureStatusNone;
}

// Whether the handle holds every table a launch of this plan reads.
bool has_tables(const HamiltonianDev& H, const ApplyPlan& P, uint32_t esz)
{
    auto have = [&](int layout) {
        return P.groups ? H.group_tables.count(group_tables_key(P, esz, layout)) != 0
                        : H.apply_tables.count(apply_tables_key(P, esz, layout)) != 0;
    };
    return H.diag_ready && have(0) && (!P.two_layouts || have(1));
}

// How a product runs that may build and allocate nothing.
struct Route {
    bool table = false;   // from the coefficient table, else by the plan
    ApplyPlan plan{};
};

// The call's own route if its tables exist and `fits` grants its scratch.  If they
// do not (the split of the masks, and with it the tables, goes with the number of
// columns and for complex64 with how they pair up), the same product from tables
// that another call on the handle built: the coefficient table, or any plan's,
// the split nearest to the call's own first; tables cut for a split whose partial
// sums do not fit run unsplit, which needs none.  A tile given by the caller runs
// as it is given or not at all.
template <typename Fits>
bool existing_route(const HamiltonianDev& H, const ApplyPlan& P, syk_dtype dtype, int nvec, const Fits& fits, Route& r)
{
    const uint32_t esz = (uint32_t)elem_bytes(dtype);
    const bool table = (dtype == SYK_C128 ? H.table_d : H.table_f).ready;
    r.plan = P;
    r.table = table && use_table(H, P, nvec, esz);
    if (r.table || (!use_table(H, P, nvec, esz) && has_tables(H, P, esz) && fits(P))) return true;
    if (P.fixed_tile) return false;
    r.table = table && H.M <= kTableMaxBits;
    if (r.table) return true;
    int best = -1;
    auto consider = [&](ApplyPlan Q) {
        if (!has_tables(H, Q, esz)) return;
        Q.parts = Q.cut;
        if (Q.parts > 1 && !fits(Q)) Q.parts = 1;
        if (!fits(Q)) return;
        const int away = std::abs(Q.cut - P.parts) + (Q.groups == P.groups ? 0 : 256);
        if (best >= 0 && away >= best) return;
        best = away;
        r.plan = Q;
    };
    // the keys of group_tables_key and apply_tables_key, layout 0
    for (const auto& kv : H.group_tables) {
        ApplyPlan Q = P;
        Q.cut = kv.first & 255;
        Q.two_layouts = (kv.first >> 9) & 1;
        Q.groups = 1;
        Q.tile_bits = kGroupTileBits;
        Q.rot = H.M - kGroupTileBits;
        Q.lb = kLaneBits;
        Q.nt = 1 << Q.lb;
        Q.rpt = kGroupRows;
        Q.nc = 1;
        if (((kv.first >> 8) & 1) == 0 && (uint32_t)(kv.first >> 10) == esz) consider(Q);
    }
    for (const auto& kv : H.apply_tables) {
        ApplyPlan Q = P;
        Q.cut = kv.first & 255;
        Q.two_layouts = (kv.first >> 9) & 1;
        Q.groups = 0;
        Q.tile_bits = kv.first >> 19;
        Q.rot = Q.tile_bits;
        Q.lb = (kv.first >> 15) & 15;
        Q.nt = 1 << Q.lb;
        Q.rpt = 1 << (Q.tile_bits - Q.lb);
        Q.nc = 1;
        if (((kv.first >> 8) & 1) == 0 && (uint32_t)((kv.first >> 10) & 31) == esz) consider(Q);
    }
    return best >= 0;
}

}  // namespace

void launch_apply_h_noalloc(const HamiltonianDev& H, int device, syk_dtype dtype, int nvec,
                            const int32_t* real_of_col, const void* psi, void* out, const ApplyPlan& plan,
                            hipStream_t s)
{
    const ApplyPlan own = plan_of_call(H, plan, dtype, nvec, real_of_col);
    const size_t esz = elem_bytes(dtype);
    const uint64_t dim = (uint64_t)1 << H.M;
    auto need = [&](const ApplyPlan& P) { return rot_bytes(P, nvec, dim, esz) + parts_bytes(P, nvec, dim); };
    if (!use_table(H, own, nvec, esz) && need(own) > kNoAllocScratchBytes)
        throw Error(SYK_EINVAL, "apply_H_noalloc: the call needs " + std::to_string(need(own)) +
                                    " bytes of scratch, above the maximum of " +
                                    std::to_string(kNoAllocScratchBytes));
    Route r;
    if (!existing_route(H, own, dtype, nvec, [&](const ApplyPlan& P) { return need(P) <= kNoAllocScratchBytes; }, r))
        throw Error(SYK_EINVAL, "apply_H_noalloc: the handle has no tables for this dtype and block width yet "
                                "(call syk_apply_H once with them first)");
    if (r.table) {
        launch_table_any(H, dtype, nvec, real_of_col, psi, out, s);
        return;
    }
    const size_t rot = rot_bytes(r.plan, nvec, dim, esz), part = parts_bytes(r.plan, nvec, dim);
    char* sp = rot + part > 0 ? static_cast<char*>(noalloc_scratch_ptr(device)) : nullptr;
    launch_apply_impl(H, dtype, nvec, real_of_col, psi, out, r.plan, s, rot ? sp : nullptr, rot ? sp + rot / 2 : nullptr,
                      part ? sp + rot : nullptr, false);
}

const void* coefficient_table(const HamiltonianDev& H, const ApplyPlan& P, syk_dtype dtype, int nvec, hipStream_t s)
{
    if (!use_table(H, P, nvec, elem_bytes(dtype))) return nullptr;
    if (dtype == SYK_C128) ensure_table<double>(H, H.table_d, s);
    else ensure_table<float>(H, H.table_f, s);
    return (dtype == SYK_C128 ? H.table_d : H.table_f).p;
}

bool launch_apply_rec(const HamiltonianDev& H, const ApplyPlan& P, const void* psi, void* out, const RecArgs& q, hipStream_t s)
{
    const void* table = coefficient_table(H, P, SYK_C128, 1, s);
    if (!table) return false;
    hipLaunchKernelGGL(k_apply_table_rec, dim3(table_blocks(H), 1), dim3(kTableThreads), 0, s,
                       static_cast<const c128*>(table), H.masks, (int)H.host_masks->size(), 1u << H.M,
                       static_cast<const c128*>(psi), static_cast<c128*>(out), q);
    SYK_HIP(hipGetLastError());
    return true;
}

void launch_apply_h(const HamiltonianDev& H, syk_dtype dtype, int nvec, const int32_t* real_of_col,
                    const void* psi, void* out, const ApplyPlan& plan, hipStream_t s)
{
    ApplyPlan P = plan_of_call(H, plan, dtype, nvec, real_of_col);
    const uint32_t esz = (uint32_t)elem_bytes(dtype);
    const uint64_t dim = (uint64_t)1 << H.M;
    bool table = use_table(H, P, nvec, esz);
    auto held = [&](const ApplyPlan& Q) {
        return rot_bytes(Q, nvec, dim, esz) / 2 <= std::min(H.rot_in.bytes, H.rot_out.bytes) &&
               parts_bytes(Q, nvec, dim) <= H.parts.bytes();
    };
    if (table ? !(dtype == SYK_C128 ? H.table_d : H.table_f).ready : !has_tables(H, P, esz) || !held(P)) {
        // A first call of its kind builds and allocates, unless its stream is under
        // graph capture, where that is refused: then what the handle holds serves it.
        Route r;
        if (capturing(s) && existing_route(H, P, dtype, nvec, held, r)) {
            table = r.table;
            P = r.plan;
        }
    }
    if (table) {
        if (dtype == SYK_C128) ensure_table<double>(H, H.table_d, s);
        else ensure_table<float>(H, H.table_f, s);
        timing_begin(s);
        launch_table_any(H, dtype, nvec, real_of_col, psi, out, s);
        timing_end(s);
        return;
    }
    const size_t rot = rot_bytes(P, nvec, dim, esz) / 2, part = parts_bytes(P, nvec, dim);
    if (rot) {
        H.rot_in.ensure(rot);
        H.rot_out.ensure(rot);
    }
    void* parts = part ? H.parts.get(part, kMaxPartsBytes) : nullptr;
    ensure_diag(H, s);
    launch_apply_impl(H, dtype, nvec, real_of_col, psi, out, P, s, rot ? H.rot_in.p : nullptr,
                      rot ? H.rot_out.p : nullptr, parts, true);
}

namespace {

// The launches of one apply_H call; rot_in / rot_out: state-sized buffers of
// min(nvec, 64) columns for two-layout plans.  Allocates nothing.
void launch_apply_impl(const HamiltonianDev& H, syk_dtype dtype, int nvec, const int32_t* real_of_col,
                       const void* psi, void* out, const ApplyPlan& P, hipStream_t s, void* rot_in, void* rot_out,
                       void* parts, bool timed)
{
    const int M = H.M;
    if (P.groups ? P.tile_bits != kGroupTileBits || P.nt != 256 || P.rpt != kGroupRows || P.tile_bits > M :
        P.lb > kLaneBits || (P.rpt > 1 && P.lb != kLaneBits) || P.nt != (1 << P.lb) ||
        (P.nc != 1 && (P.nc != 2 || P.rpt < 4)) ||
        (P.rpt << P.lb) != (1 << P.tile_bits) || P.tile_bits > M ||
        (P.two_layouts && (P.tile_bits < 5 || M - P.tile_bits < 5)))
        throw Error(SYK_EINVAL, "apply_H: inconsistent launch shape");
    if (P.two_layouts && (P.rot < 5 || M - P.rot < 5)) throw Error(SYK_EINVAL, "apply_H: inconsistent launch shape");
    const size_t esz = elem_bytes(dtype);
    const uint64_t dim = (uint64_t)1 << M;
    const bool two = P.two_layouts != 0;
    // the tables of both layouts exist before the first launch
    for (int l = 0; l <= P.two_layouts; ++l) {
        if (P.groups) (void)group_tables_for(H, P, (uint32_t)esz, l);
        else (void)apply_tables_for(H, P, (uint32_t)esz, l);
    }
    if (two && (!rot_in || !rot_out)) throw Error(SYK_EINVAL, "apply_H: no buffers for the rotated layout");
    if (P.parts > 1 && !parts) throw Error(SYK_EINVAL, "apply_H: no buffer for the partial sums");
    if (timed) timing_begin(s);
    for (int sl = 0; sl < P.slices; ++sl) {
        KLayout L{};
        L.tile_bits = P.tile_bits;
        L.lane_bits = P.lb;
        L.dim = dim;
        L.col0 = 0;
        L.n_tiles = (uint32_t)(dim >> P.tile_bits);
        L.xcd_remap = P.xcd_remap;
        const int col0 = sl * kColsPerLaunch;
        const int ncols = std::min(kColsPerLaunch, nvec - col0);
        for (int c = 0; c < ncols; ++c) L.real[c] = real_of_col ? real_of_col[col0 + c] : 0;
        // two columns per workgroup only where every pair of the slice shares its realisation
        int nc = P.nc;
        if (nc == 2 && ncols % 2 != 0) nc = 1;
        for (int c = 0; nc == 2 && c < ncols; c += 2)
            if (L.real[c] != L.real[c + 1]) nc = 1;
        const char* in_c = static_cast<const char*>(psi) + (size_t)col0 * dim * esz;
        char* out_c = static_cast<char*>(out) + (size_t)col0 * dim * esz;
        auto run = [&](int layout, const void* src, void* dst) {
            L.n_parts = P.parts;
            L.part_stride = (uint64_t)ncols * dim;
            c128* pt = static_cast<c128*>(parts);
            auto launch = [&](auto zero, const auto* tab4, const auto* phi2, const auto* w2) {
                typedef decltype(zero) R;
                const KTerms<R> T{tab4, H.qinfo, phi2, w2, H.diag.as<double>(), H.n_real, M};
                if (P.groups) {
                    const HamiltonianDev::GroupTables& Tb = group_tables_for(H, P, (uint32_t)esz, layout);
                    L.far = static_cast<const FarRec*>(Tb.far);
                    L.n_far = Tb.n_far;
                    L.n_chunks = Tb.n_chunks;
                    L.n_tables = Tb.n_tables;
                    L.part_chunk = static_cast<const uint32_t*>(Tb.part_chunk);
                    launch_groups<R>(H, T, Tb, L, ncols, src, dst, pt, s);
                } else {
                    const HamiltonianDev::ApplyTables& Tb = apply_tables_for(H, P, (uint32_t)esz, layout);
                    L.far = static_cast<const FarRec*>(Tb.far);
                    L.n_far = Tb.n_far;
                    L.n_chunks = Tb.n_chunks;
                    L.part_chunk = static_cast<const uint32_t*>(Tb.part_chunk);
                    launch_t<R>(P, T, static_cast<const QApplyChunk*>(Tb.chunks), static_cast<const QRec*>(Tb.recs), L, ncols, nc, src, dst, pt, s);
                }
            };
            if (dtype == SYK_C128) launch(0.0, H.tab4_d, H.phi2_d, H.w2_d);
            else launch(0.0f, H.tab4_f, H.phi2_f, H.w2_f);
        };
        if (two) {
            // rows r -> rotate_bits(r): a [2^(M-s)] x [2^s] transpose
            launch_transpose(dtype, in_c, rot_in, M - P.rot, P.rot, ncols, dim, false, s);
            run(1, rot_in, rot_out);
            run(0, in_c, out_c);
            launch_transpose(dtype, rot_out, out_c, P.rot, M - P.rot, ncols, dim, true, s);
        } else {
            run(0, in_c, out_c);
        }
    }
    if (timed) timing_end(s);
}

}  // namespace

}  // namespace syk

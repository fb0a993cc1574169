// The apply kernel with 16 rows per thread, in which every QUAD mask runs in a
// group, and its tables.  Included by apply_h.hip (helpers, KTerms, KLayout).
//
// A thread owns the rows tid + (k << 8), k < 16, of a tile of 2^12 rows.  The
// masks that agree outside the four k bits and flip J of them read the same 16
// source rows, in an order that is known at compile time; there are C(4, J) of
// them (the QUAD masks hold every choice of four qubits), and they share one
// source read, one lane index and one lane sign.  Which k bits a member has in
// its Z string follows from J, the member and one bit P per group, since the k
// bits are neighbouring qubits in both row layouts: ten group classes (J, P).
//
// Why 16 rows: per QUAD mask and thread 64 FMAs stand against ~11 (J = 0), 6
// (J = 1) or 7 (J = 2) other vector instructions and 17, 6 or 6.7 LDS reads; at 8
// rows with groups of three it is 32 FMAs against 6-7 and ~8 reads.  The price is
// two waves per SIMD (64 registers of sums and 64 of source rows in complex128)
// and 64 KiB of source tile; the tile also halves the source bytes staged per row.
// Two waves are enough because a group's rows are read from LDS while the group
// before it runs, into the registers its last member has just used, and each row
// waits only for its own read.
//
// Measured (ms per call, k_apply -> this kernel): complex128 N=40 1.37 -> 1.07,
// N=44 7.2 -> 5.7, N=48 39.0 -> 32.4 (45 TFLOP/s; the FP64 FMA rate the card holds
// under its power limit is 64); complex64 N=40 0.88 -> 0.75, N=44 4.61 -> 4.12, N=48
// 25.3 -> 22.7.  Timing copies at N=48 complex128 that step over a part: source
// tiles 4 of the 32 ms, PAIR masks ~2, table staging ~1.5.  The tiles are not hidden
// further: reading the next tile into registers during a run, or storing it later
// than it arrives, measured 4-15% slower (64 more live registers).  complex64 at
// three waves per SIMD spills (N=44 4.35 ms against 3.97 at two waves, both carrying
// once per chunk).
#pragma once

constexpr int kGroupKBits = 4, kGroupRows = 1 << kGroupKBits;
constexpr int kGroupTileBits = kLaneBits + kGroupKBits;
constexpr int kGroupClasses = 10;   // 2 J + P

// Bytes of a chunk's staged tables: with the tile, two workgroups per CU in
// complex128 (2 x 80 KiB).  The kernel's read-ahead stays inside the area if the
// tables end kGroupSlack entries before it does.
constexpr uint32_t kGroupSlack = 64;
constexpr uint32_t group_table_bytes(uint32_t esz) { return 1024u * esz; }
constexpr int kGroupsPerChunk = 64;   // a chunk's records are held one per lane

// What a group's loop reads.
struct alignas(8) GroupRec {
    uint32_t sel;    // byte selector gathering the lane bits of tid at the table's index bits (0x0c: none)
    uint32_t pack;   // lane bits of the Z string, lane bits of x << 8, index bit of the lowest flipped k bit << 16
                     // (the others follow it)
};

// Masks sharing a source tile, and QUAD masks also sharing their tables' index
// bits and sign above the tile: groups by class, then PAIR masks, then DIAG.  A
// staged table holds only the entries of the index bits that vary inside a
// tile, 2^es of them; all of the chunk's tables take the same entries, entry i
// being sign * T[(i << shift) ^ index] with the index and the sign of the tile.
struct alignas(16) GroupChunk {
    uint32_t x_high, first_group, first_table, first_pair;
    uint32_t n_tabs, es, shift, new_tile;
    uint32_t n_pair, n_diag;
    uint32_t qpack, zbase;               // of one QUAD mask: the bits above the tile are all masks'
    uint32_t pad;
    uint32_t cnt[kGroupClasses / 2];     // per J: groups with P = 0, and << 16 with P = 1
    uint32_t pad2[2];
};
static_assert(sizeof(GroupChunk) == 80, "GroupChunk layout");

// PAIR masks.  With idx the bits of r at the two flipped qubits, D_x(r) =
// (-1)^{|r & z|} A_idx(r), z the Z string without the flipped qubits and A_idx a
// linear form in the other bits of r with complex coefficients, tabulated once per
// handle (k_pair_tables) for the bits inside a tile: the sums over the low and the
// high four lane bits, 16 entries each, and the four k-bit coefficients.  A lane
// reads two sums, the tile's part and the k-bit steps from LDS, and walks its rows
// in Gray-code order, one step per row: 64 FMAs and ~50 other vector instructions
// per flat mask (no flipped k bit), where forming the linear forms from scalar
// weights took ~150 and waited for each.
constexpr int kPairEntries = 36;                  // per idx: 16 + 16 lane sums, 4 k-bit steps
constexpr int kPairStride = kPairEntries + 1;     // staged, with the tile's part
__host__ __device__ constexpr int pair_table_size(int M) { return 4 * (kPairEntries + 1 + M - kGroupTileBits); }

struct alignas(16) PairRec {
    uint32_t off;     // byte offset of the staged entries in the chunk's table area
    uint32_t xoff;    // (x & lane mask) * element size
    uint32_t z;       // Z string without the flipped qubits
    uint32_t tab;     // index into the PAIR tables
    uint32_t qpack;   // flipped qubits, one per byte (31: a placeholder, never set)
    uint32_t n_in;    // flipped qubits inside the tile: index bits that vary in it
    uint32_t sel;     // byte selector gathering the lane bits of tid at those index bits (0x0c: none)
    uint32_t cls;     // 2 (place of the flipped k bits in pair_xk) + P
};
static_assert(sizeof(PairRec) == 32, "PairRec layout");

constexpr int popc4(int v) { return (v & 1) + ((v >> 1) & 1) + ((v >> 2) & 1) + ((v >> 3) & 1); }
constexpr int choose4(int J) { return J == 0 || J == 4 ? 1 : J == 2 ? 6 : 4; }
// k bits member j of a group flips: the j-th pattern of J bits, ascending
constexpr int member_xk(int J, int j)
{
    for (int v = 0; v < 16; ++v)
        if (popc4(v) == J && j-- == 0) return v;
    return -1;
}
// ... and has in its Z string: those it does not flip with an odd number of
// flipped qubits above them
constexpr int member_zk(int xk, int P)
{
    int z = 0;
    for (int b = 0; b < kGroupKBits; ++b)
        if (!((xk >> b) & 1) && ((popc4(xk >> (b + 1)) + P) & 1)) z |= 1 << b;
    return z;
}
// k bits a PAIR mask flips, by class
constexpr int kPairPatterns = 11;
constexpr int pair_xk(int c) { return c == 0 ? 0 : c <= 4 ? member_xk(1, c - 1) : member_xk(2, c - 5); }

// the bits of p at the set bits of m, packed from bit 0
constexpr int pack_bits4(int p, int m)
{
    int r = 0, o = 0;
    for (int b = 0; b < kGroupKBits; ++b)
        if ((m >> b) & 1) r |= ((p >> b) & 1) << o++;
    return r;
}

// The i-th subset of the bits of m in Gray-code order (neighbours differ in one bit).
constexpr int gray_subset(int i, int m)
{
    const int g = i ^ (i >> 1);
    int r = 0, o = 0;
    for (int b = 0; b < kGroupKBits; ++b)
        if ((m >> b) & 1) r |= ((g >> o++) & 1) << b;
    return r;
}
constexpr int bit_place(int v) { return v == 1 ? 0 : v == 2 ? 1 : v == 4 ? 2 : 3; }

// Tables of every PAIR mask and realisation (workgroup (mask, realisation)):
// [idx][36] entries inside a tile, then [idx] the constant and the coefficients
// of the tile's bits.
template <typename R>
__global__ void __launch_bounds__(256) k_pair_tables(const MaskRec* __restrict__ masks, const c128* __restrict__ phi2,
                                                     const double* __restrict__ w2, int n_real, int M,
                                                     cplx<R>* __restrict__ out)
{
    const MaskRec m = masks[blockIdx.x];
    if ((m.type_tab >> 28) != MASK_PAIR) return;
    const uint32_t tab = m.type_tab & 0x0fffffffu;
    const int rc = blockIdx.y, nt = 1 + M - kGroupTileBits;
    const double* w = w2 + ((size_t)tab * n_real + rc) * 4 * (M + 1);
    cplx<R>* o = out + ((size_t)tab * n_real + rc) * pair_table_size(M);
    for (int t = threadIdx.x; t < 4 * (kPairEntries + nt); t += 256) {
        const bool tile = t >= 4 * kPairEntries;
        const int u = tile ? t - 4 * kPairEntries : t, idx = tile ? u / nt : u / kPairEntries;
        const int j = tile ? u % nt : u % kPairEntries;
        double re = 0.0, im = 0.0;
        for (int e = 0; e < 4; ++e) {
            const double* we = w + e * (M + 1);
            double l = 0.0;
            if (tile) {
                l = we[j == 0 ? M : kGroupTileBits + j - 1];
            } else if (j < 32) {
                for (int b = 0; b < 4; ++b)
                    if ((j >> b) & 1) l += we[(j >> 4) * 4 + b];
            } else {
                l = we[kLaneBits + j - 32];
            }
            const c128 ph = phi2[(size_t)tab * 16 + idx * 4 + e];
            re += ph.re * l;
            im += ph.im * l;
        }
        // the Z string on the flipped qubits (parity sectors) goes with idx
        uint32_t s = 0;
        for (int i = 0; i < 2; ++i) s ^= ((uint32_t)idx >> i) & (m.zbase >> (mask_q(m.qpack, i) & 31u)) & 1u;
        cplx<R> v;
        v.re = (R)flip(re, s);
        v.im = (R)flip(im, s);
        o[t] = v;
    }
}

// dst[rc][s][16] = the QUAD table of mask tab[s] in realisation rc: the tables in
// the order the chunks stage them.
template <typename R>
__global__ void __launch_bounds__(256) k_order_tables(const cplx<R>* __restrict__ tab4, const uint32_t* __restrict__ tab,
                                                      int n_tabs, int n_real, cplx<R>* __restrict__ dst)
{
    const uint32_t t = blockIdx.x * 256u + threadIdx.x;
    if (t >= (uint32_t)n_tabs * 16u) return;
    const int rc = blockIdx.y;
    dst[(size_t)rc * n_tabs * 16 + t] = tab4[((size_t)tab[t >> 4] * n_real + rc) * 16 + (t & 15u)];
}

template <typename R>
struct GroupLds {
    cplx<R> src[kGroupRows << kLaneBits];
    char tabs[group_table_bytes(sizeof(cplx<R>))];
};

// f(std::integral_constant<int, c>{}) for the c of the sequence that equals cls.
template <typename F, int... I>
__device__ __forceinline__ void dispatch_class(F& f, uint32_t cls, std::integer_sequence<int, I...>)
{
    (void)((cls == (uint32_t)I ? (f(std::integral_constant<int, I>{}), true) : false) || ...);
}


template <typename R, bool SPLIT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_apply_groups(KTerms<R> T, const GroupChunk* __restrict__ chunks, const GroupRec* __restrict__ grp,
               const cplx<R>* __restrict__ tables, const cplx<R>* __restrict__ pair_tables,
               const PairRec* __restrict__ prec, KLayout L, const cplx<R>* __restrict__ psi, cplx<R>* __restrict__ out, c128* __restrict__ parts)
{
    constexpr int RPT = kGroupRows, KB = kGroupKBits;
    constexpr uint32_t lb = kLaneBits, nt = 1u << lb;
    constexpr uint32_t esz = sizeof(cplx<R>);
    constexpr uint32_t kDotW = (esz) | (2 * esz) << 8 | (4 * esz) << 16 | (8 * esz) << 24;   // weights of the index bits
    uint32_t dotw = kDotW;
    asm("" : "+v"(dotw));   // in a VGPR: v_dot4 then takes the table offset from an SGPR
    __shared__ GroupLds<R> S;
    const char* src_b = reinterpret_cast<const char*>(S.src);
    auto src_at = [&](uint32_t off) { return *reinterpret_cast<const cplx<R>*>(src_b + off); };
    // table offsets count from the start of the tile, so that no read adds the area's base
    constexpr uint32_t kTabs = (RPT << lb) * esz;
    auto tab_at = [&](uint32_t off) { return *reinterpret_cast<const cplx<R>*>(src_b + off); };

    const uint32_t tile = tile_of_block(blockIdx.x, L);
    const uint32_t tid = threadIdx.x;
    const int rc = L.real[blockIdx.y];
    const int M = T.M;
    const uint32_t base = tile << kGroupTileBits;
    tables += (size_t)rc * L.n_tables * 16;
    psi += (uint64_t)(L.col0 + blockIdx.y) * L.dim;
    out += (uint64_t)(L.col0 + blockIdx.y) * L.dim;

    // bits 0..3 and 4..7 of tid, one per byte
    uint32_t B0 = 0, B1 = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        B0 |= ((tid >> i) & 1u) << (8 * i);
        B1 |= ((tid >> (4 + i)) & 1u) << (8 * i);
    }
    const uint32_t tid_b = tid * esz, lane = tid & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));

    // complex128 sums directly in pr/pi; complex64 sums in FP32 and carries the
    // running total in FP64 every kCarryEvery masks: the error of H psi grows with
    // the root of that number (1.7e-7 at N=44; 2.2e-7 carried once per chunk of
    // about 66 masks, which is 4% faster).
    constexpr bool kSplit = sizeof(R) < sizeof(double);
    constexpr uint32_t kCarryEvery = 36;
    uint32_t since = 0;
    double acc_re[RPT], acc_im[RPT];
    R pr[RPT], pi[RPT];
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        acc_re[k] = acc_im[k] = 0.0;
        pr[k] = pi[k] = R(0);
    }
    auto carry = [&]() {
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            acc_re[k] += (double)pr[k];
            acc_im[k] += (double)pi[k];
            pr[k] = pi[k] = R(0);
        }
    };

    int g0 = 0, g1 = L.n_chunks, f0 = 0, f1 = L.n_far;
    if constexpr (SPLIT) {
        g0 = (int)L.part_chunk[blockIdx.z];
        g1 = (int)L.part_chunk[blockIdx.z + 1];
        f0 = (int)((uint32_t)L.n_far * blockIdx.z / (uint32_t)L.n_parts);
        f1 = (int)((uint32_t)L.n_far * (blockIdx.z + 1) / (uint32_t)L.n_parts);
    }
    for (int g = g0; g < g1; ++g) {
        const GroupChunk C = chunks[g];
        const uint32_t es = C.es, n_pair = C.n_pair, n_entries = C.n_tabs << C.es;
        __syncthreads();   // previous chunk is done with src / tabs
        // The table entries are requested before the tile and stored after it: one
        // round trip to memory for both.
        const uint32_t index = quad_index(base, C.qpack), sg = parity(base & C.zbase);
        const cplx<R>* tq = tables + (size_t)C.first_table * 16;
        constexpr int NT = (int)(1024 / nt);   // entries per thread at most
        cplx<R> te[NT];
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            const uint32_t e = tid + u * nt;
            if (e < n_entries) te[u] = tq[(e >> es) * 16 + ((((e & ((1u << es) - 1u)) << C.shift) ^ index) & 15u)];
        }
        if (C.new_tile || (SPLIT && g == g0)) {
            const cplx<R>* s = psi + (((uint64_t)(tile ^ C.x_high)) << kGroupTileBits) + tid;
#pragma unroll
            for (int k = 0; k < RPT; ++k) S.src[tid + k * nt] = s[k * nt];
        }
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            const uint32_t e = tid + u * nt;
            cplx<R> o;
            o.re = flip(te[u].re, sg);
            o.im = flip(te[u].im, sg);
            if (e < n_entries) reinterpret_cast<cplx<R>*>(S.tabs)[e] = o;
        }
        // PAIR masks: every fourth to each wave; entry j of staged index i at (i * kPairStride + j)
        for (uint32_t p = wave; p < n_pair; p += 4) {
            const PairRec q = prec[C.first_pair + p];
            const cplx<R>* t = pair_tables + ((size_t)q.tab * T.n_real + rc) * pair_table_size(M);
            cplx<R>* o = reinterpret_cast<cplx<R>*>(S.tabs + q.off);
            // index bits of the flipped qubits above the tile
            const uint32_t fixed = bit(base, mask_q(q.qpack, 0)) | (bit(base, mask_q(q.qpack, 1)) << 1);
            for (uint32_t e = lane; e < ((uint32_t)kPairEntries << q.n_in); e += 64) {
                const uint32_t i = e / kPairEntries, j = e % kPairEntries;
                o[i * kPairStride + j] = t[(i ^ fixed) * kPairEntries + j];
            }
            // the tile's part: sixteen lanes per index add the constant and the tile bits' coefficients
            const uint32_t i = lane >> 4, n = 1u + (uint32_t)(M - kGroupTileBits);
            const cplx<R>* tt = t + 4 * kPairEntries + (((i ^ fixed) & 3u) * n);
            cplx<R> a{R(0), R(0)};
            for (uint32_t j = lane & 15u; j < n; j += 16) {
                const cplx<R> v = tt[j];
                const R on = j == 0 ? R(1) : (R)((tile >> (j - 1)) & 1u);
                a.re = fma(on, v.re, a.re);
                a.im = fma(on, v.im, a.im);
            }
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) {
                a.re += __shfl_xor(a.re, off, 64);
                a.im += __shfl_xor(a.im, off, 64);
            }
            if ((lane & 15u) == 0u && i < (1u << q.n_in)) o[i * kPairStride + kPairEntries] = a;
        }
        __syncthreads();

        // The chunk's group records, one per lane (no scalar loads in the loops: one
        // in flight would turn every wait for an LDS read into a full one).
        const GroupRec mine = grp[C.first_group + (tid & 63u)];
        uint32_t gi = 0;                        // group of the chunk
        uint32_t tb = kTabs;                    // byte offset of its first table
        const uint32_t stride = esz << es;      // bytes per table
        uint32_t sel = (uint32_t)__builtin_amdgcn_readlane((int)mine.sel, 0);
        uint32_t pack = (uint32_t)__builtin_amdgcn_readlane((int)mine.pack, 0);
        auto row_base = [&](uint32_t pk) { return tid_b ^ (((pk >> 8) & 0xffu) * esz); };
        // The source rows of a group are read while the last member of the group
        // before it runs, each into the registers that member has just used.
        cplx<R> v[RPT];
        {
            const uint32_t sb = row_base(pack);
#pragma unroll
            for (int k = 0; k < RPT; ++k) v[k] = src_at(sb + ((uint32_t)k << lb) * esz);
        }
        auto group_loop = [&](auto cls) {
            constexpr int J = decltype(cls)::value >> 1, P = decltype(cls)::value & 1;
            constexpr int NM = choose4(J), NE = 1 << J;
            // One or two entries per member: the lane sign goes on the entries (two
            // instructions each); more: on the source rows, once per group.
            constexpr bool kSignRows = J >= 2;
            // Up to four entries: a member's are read while the member before it runs.
            constexpr bool kAhead = J <= 2;
            constexpr bool kDirect = J == 4;   // sixteen entries (one mask per tile): read where they are used
            const uint32_t n = P ? C.cnt[J] >> 16 : C.cnt[J] & 0xffffu;
            if (n == 0) return;
            cplx<R> ta[kDirect ? 1 : NE], tn[kAhead ? NE : 1];
            uint32_t ia, sl, kof;
            auto decode = [&](uint32_t s, uint32_t pk, uint32_t t) {
                ia = __builtin_amdgcn_udot4(__builtin_amdgcn_perm(B1, B0, s), dotw, t, false);
                sl = (uint32_t)__popc(tid & pk & 0xffu);   // lane sign: its parity
                kof = esz << ((pk >> 16) & 3u);
            };
            auto load_entries = [&](auto& t) {
#pragma unroll
                for (int e = 0; e < NE; ++e) t[e] = tab_at(ia + (uint32_t)e * kof);
            };
            decode(sel, pack, tb);
            if constexpr (kAhead) {
                load_entries(ta);
                // wait here, not in the loop: there the reads in flight are then known to
                // be in row order and each row waits only for its own
#pragma unroll
                for (int e = 0; e < NE; ++e) asm volatile("" : "+v"(ta[e].re), "+v"(ta[e].im));
            }
            for (uint32_t i = 0; i < n; ++i) {
                auto member = [&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    constexpr bool kLast = j + 1 == NM;
                    constexpr int XK = member_xk(J, j), ZK = member_zk(XK, P);
                    if constexpr (!kAhead && !kDirect) load_entries(ta);
                    const uint32_t sl_now = sl, ia_now = ia, kof_now = kof;
                    uint32_t sb = 0;
                    if constexpr (kLast) {
                        // the next group; after the last of the class its entries are not used
                        ++gi;
                        sel = (uint32_t)__builtin_amdgcn_readlane((int)mine.sel, (int)gi);
                        pack = (uint32_t)__builtin_amdgcn_readlane((int)mine.pack, (int)gi);
                        sb = row_base(pack);
                        tb += NM * stride;
                        decode(sel, pack, i + 1 < n ? tb : tb - NM * stride);
                    } else {
                        ia += stride;
                    }
                    if constexpr (kAhead) load_entries(tn);
                    if constexpr (!kSignRows) {
#pragma unroll
                        for (int e = 0; e < NE; ++e) {
                            ta[e].re = flip_odd(ta[e].re, sl_now);
                            ta[e].im = flip_odd(ta[e].im, sl_now);
                        }
                    }
                    // two source rows at a time, in the order they arrive; a row's two
                    // FMAs per sum stand four instructions apart
#pragma unroll
                    for (int s = 0; s < RPT; s += 2) {
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (kSignRows && j == 0) {
#pragma unroll
                            for (int u = s; u < s + 2; ++u) {
                                v[u].re = flip_odd(v[u].re, sl_now);
                                v[u].im = flip_odd(v[u].im, sl_now);
                            }
                        }
                        const int k0 = s ^ XK, k1 = (s + 1) ^ XK;
                        const int e0 = pack_bits4(k0 & XK, XK), e1 = pack_bits4(k1 & XK, XK);
                        const cplx<R> t0 = kDirect ? tab_at(ia_now + (uint32_t)e0 * kof_now) : ta[kDirect ? 0 : e0];
                        const cplx<R> t1 = kDirect ? tab_at(ia_now + (uint32_t)e1 * kof_now) : ta[kDirect ? 0 : e1];
                        const bool n0 = (popc4(k0 & ZK) & 1) != 0, n1 = (popc4(k1 & ZK) & 1) != 0;
                        const R a0 = n0 ? -t0.re : t0.re, b0 = n0 ? -t0.im : t0.im;
                        const R a1 = n1 ? -t1.re : t1.re, b1 = n1 ? -t1.im : t1.im;
                        pr[k0] = fma(a0, v[s].re, pr[k0]);
                        pi[k0] = fma(a0, v[s].im, pi[k0]);
                        pr[k1] = fma(a1, v[s + 1].re, pr[k1]);
                        pi[k1] = fma(a1, v[s + 1].im, pi[k1]);
                        pr[k0] = fma(-b0, v[s].im, pr[k0]);
                        pi[k0] = fma(b0, v[s].re, pi[k0]);
                        pr[k1] = fma(-b1, v[s + 1].im, pr[k1]);
                        pi[k1] = fma(b1, v[s + 1].re, pi[k1]);
                        if constexpr (kLast) {
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int u = s; u < s + 2; ++u) v[u] = src_at(sb + ((uint32_t)u << lb) * esz);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (kAhead) {
#pragma unroll
                        for (int e = 0; e < NE; ++e) ta[e] = tn[e];
                    }
                };
                for_each_class(member, std::make_integer_sequence<int, NM>{});
                if constexpr (kSplit) {
                    since += NM;
                    if (since >= kCarryEvery) {
                        carry();
                        since = 0;
                    }
                }
            }
        };
        for_each_class(group_loop, std::make_integer_sequence<int, kGroupClasses>{});

        for (uint32_t p = 0; p < n_pair; ++p) {
            const PairRec q = prec[C.first_pair + p];
            // staged index of the lane's bits; the k bits' part is added per row set
            const uint32_t li = __builtin_amdgcn_udot4(__builtin_amdgcn_perm(B1, B0, q.sel), 0x00000201u, 0u, false);
            const uint32_t sl = (uint32_t)__popc((tid | base) & q.z);   // row sign but for the k bits: its parity
            const uint32_t pb = kTabs + q.off + li * (kPairStride * esz);
            const uint32_t sb = tid_b ^ q.xoff;
            auto pair_mask = [&](auto cls) {
                constexpr int XK = pair_xk(decltype(cls)::value >> 1), P = decltype(cls)::value & 1;
                constexpr int ZK = member_zk(XK, P), J = popc4(XK), FREE = (RPT - 1) ^ XK;
                // index bit of the lowest flipped k bit: above a lane qubit, if one is flipped
                const uint32_t kof = (J == 1 && q.n_in == 2 ? 2u : 1u) * (kPairStride * esz);
#pragma unroll
                for (int f = 0; f < (1 << J); ++f) {
                    const uint32_t b = pb + (uint32_t)f * kof;
                    const cplx<R> x0 = tab_at(b + (tid & 15u) * esz), x1 = tab_at(b + (16u + (tid >> 4)) * esz);
                    const cplx<R> xt = tab_at(b + kPairEntries * esz);
                    cplx<R> om[KB];
#pragma unroll
                    for (int c = 0; c < KB; ++c)
                        if ((FREE >> c) & 1) {
                            om[c] = tab_at(b + (32u + c) * esz);
                            om[c].re = flip_odd(om[c].re, sl);
                            om[c].im = flip_odd(om[c].im, sl);
                        }
                    cplx<R> X;
                    X.re = flip_odd((x0.re + x1.re) + xt.re, sl);
                    X.im = flip_odd((x0.im + x1.im) + xt.im, sl);
                    // the rows with the flipped k bits f, the others in Gray-code order
                    const int kf = XK == 0 ? 0 : [&] { int r = 0, o = 0; for (int c = 0; c < KB; ++c) if ((XK >> c) & 1) r |= ((f >> o++) & 1) << c; return r; }();
#pragma unroll
                    for (int i = 0; i < (1 << (KB - J)); ++i) {
                        const int sub = gray_subset(i, FREE), k = sub | kf;
                        if (i > 0) {
                            const int c = bit_place(sub ^ gray_subset(i - 1, FREE));
                            X.re += ((sub >> c) & 1) ? om[c].re : -om[c].re;
                            X.im += ((sub >> c) & 1) ? om[c].im : -om[c].im;
                        }
                        const bool neg = (popc4(k & ZK) & 1) != 0;
                        const cplx<R> x = src_at(sb + ((uint32_t)(k ^ XK) << lb) * esz);
                        cmac(pr[k], pi[k], neg ? -X.re : X.re, neg ? -X.im : X.im, x);
                    }
                }
            };
            dispatch_class(pair_mask, q.cls, std::make_integer_sequence<int, 2 * kPairPatterns>{});
        }
        // DIAG (source = own row): the precomputed diagonal of H
        for (uint32_t i = 0; i < C.n_diag; ++i) {
            const double* dg = T.diag + (uint64_t)rc * L.dim + base + tid;
#pragma unroll
            for (int k = 0; k < RPT; ++k) {
                const R d = (R)dg[(uint32_t)k << lb];
                const cplx<R> v = src_at(tid_b + ((uint32_t)k << lb) * esz);
                pr[k] = fma(d, v.re, pr[k]);
                pi[k] = fma(d, v.im, pi[k]);
            }
        }
        since += n_pair;
    }
    if (kSplit) carry();

    // QUAD masks that flip only tile bits: one coefficient per tile, streamed from global memory
    for (int f = f0; f < f1; ++f) {
        const FarRec fc = L.far[f];
        const cplx<R>* sp = psi + (((uint64_t)(tile ^ fc.x_high)) << kGroupTileBits) + tid;
        cplx<R> v[RPT];
#pragma unroll
        for (int k = 0; k < RPT; ++k) v[k] = sp[k * nt];
        const cplx<R> t = T.tab4[((size_t)fc.tab * T.n_real + rc) * 16 + quad_index(base, fc.qpack)];
        const uint32_t s = parity(base & fc.zbase);
        const R tr = flip(t.re, s), ti = flip(t.im, s);
#pragma unroll
        for (int k = 0; k < RPT; ++k) cmac(pr[k], pi[k], tr, ti, v[k]);
        if (kSplit && ((f - f0) & 63) == 63) carry();
    }
    if (kSplit) carry();
    if constexpr (SPLIT) {
        parts += blockIdx.z * L.part_stride + (uint64_t)blockIdx.y * L.dim + base + tid;
#pragma unroll
        for (int k = 0; k < RPT; ++k)
            parts[k * nt] = kSplit ? c128{acc_re[k], acc_im[k]} : c128{(double)pr[k], (double)pi[k]};
        return;
    }
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        cplx<R> o;
        o.re = kSplit ? (R)acc_re[k] : pr[k];
        o.im = kSplit ? (R)acc_im[k] : pi[k];
        out[(uint64_t)base + tid + k * nt] = o;
    }
}

constexpr double kGroupCostPair = 2.5;   // a PAIR mask's cost in QUAD masks, for cutting chunks and parts

struct GroupTables {
    std::vector<GroupChunk> chunks;
    std::vector<GroupRec> groups;
    std::vector<uint32_t> tabs;    // QUAD table index of every staged slot
    std::vector<PairRec> pairs;
    size_t n_diag = 0;
    std::vector<FarRec> far;
    std::vector<double> cost;  // per chunk, for cutting into parts
};

// Tables of k_apply_groups for one layout's masks (in that layout's row
// coordinates) and elements of esz bytes; max_cost > 0 ends a chunk before the
// cost of its masks would pass it.  Throws if a group is not complete or its
// members disagree on what the kernel reads once per group.
GroupTables build_group_tables(const std::vector<MaskRec>& masks, uint32_t esz, double max_cost)
{
    GroupTables G;
    const uint32_t row_mask = (1u << kGroupTileBits) - 1u, lane_mask = (1u << kLaneBits) - 1u;
    const uint32_t kmask = row_mask & ~lane_mask;
    auto type_of = [](const MaskRec& m) { return m.type_tab >> 28; };
    auto bad = [](const char* w) { throw Error(SYK_EUNSUPPORTED, std::string("apply_H groups: ") + w); };
    struct Group {
        int cls;
        std::vector<const MaskRec*> mem;
    };
    struct Run {   // masks of one source tile that share what their chunk holds once
        std::map<std::tuple<uint32_t, uint32_t, int>, Group> groups;   // lane flips, zbase outside the k bits, class
        std::vector<const MaskRec*> pairs, diag;
        int in_tile = 0;   // most flipped qubits of a QUAD mask inside the tile
        uint32_t qpack = 0, zbase = 0, shift = 0;
    };
    // index bits of a QUAD mask's qubits inside the tile (31: a placeholder) and below them
    auto bits_in = [](const MaskRec& m, int n) {
        uint32_t r = 0;
        for (int i = 0; i < n; ++i)
            if (mask_q(m.qpack, i) < (uint32_t)kGroupTileBits) r |= 1u << i;
        return r;
    };
    auto index_above = [](const MaskRec& m) {   // (index bit, tile bit) of the qubits above the tile
        uint64_t r = 0;
        for (int i = 0; i < 4; ++i) {
            const uint32_t q = mask_q(m.qpack, i);
            r = r << 8 | (q >= (uint32_t)kGroupTileBits && q != 31u ? q : 0u);
        }
        return r;
    };
    std::map<std::tuple<uint32_t, uint64_t, uint32_t, uint32_t>, Run> runs;   // x_high, index above, zbase above, index bits inside
    for (const MaskRec& m : masks) {
        const uint32_t xh = m.x >> kGroupTileBits;
        const int xk = (int)((m.x & kmask) >> kLaneBits), zk = (int)((m.zbase & kmask) >> kLaneBits);
        if (type_of(m) == MASK_DIAG) {
            runs[std::make_tuple(xh, (uint64_t)0, 0u, 0u)].diag.push_back(&m);
        } else if (type_of(m) == MASK_PAIR) {
            runs[std::make_tuple(xh, (uint64_t)0, 0u, 0u)].pairs.push_back(&m);
        } else if ((m.x & row_mask) == 0u && (m.zbase & row_mask) == 0u) {
            G.far.push_back({xh, m.qpack, m.zbase, m.type_tab & 0x0fffffffu});
        } else {
            const int J = popc4(xk);
            const int P = zk == member_zk(xk, 0) ? 0 : 1;
            if (zk != member_zk(xk, P)) bad("Z string");
            const uint32_t in = bits_in(m, 4), shift = in ? (uint32_t)__builtin_ctz(in) : 0u;
            if (((in >> shift) & ((in >> shift) + 1u)) != 0u) bad("index bits");
            Run& r = runs[std::make_tuple(xh, index_above(m), m.zbase >> kGroupTileBits, in)];
            Group& g = r.groups[std::make_tuple(m.x & lane_mask, m.zbase & ~kmask, 2 * J + P)];
            g.cls = 2 * J + P;
            g.mem.push_back(&m);
            r.in_tile = __builtin_popcount(in);
            r.qpack = m.qpack;
            r.zbase = m.zbase;
            r.shift = shift;
        }
    }
    // PAIR and DIAG masks join the QUAD masks of their source tile
    for (auto it = runs.begin(); it != runs.end();) {
        const auto nx = std::next(it);
        if (it->second.groups.empty() && nx != runs.end() && std::get<0>(nx->first) == std::get<0>(it->first)) {
            nx->second.pairs.swap(it->second.pairs);
            nx->second.diag.swap(it->second.diag);
            runs.erase(it);
        }
        it = nx;
    }
    uint32_t prev_high = 0xffffffffu;
    for (auto& kv : runs) {
        Run& r = kv.second;
        const uint32_t x_high = std::get<0>(kv.first);
        const uint32_t es = (uint32_t)r.in_tile, tab_bytes = esz << es;
        // groups in class order; within a class by lane flips
        std::vector<Group*> gs;
        for (auto& g : r.groups) gs.push_back(&g.second);
        std::stable_sort(gs.begin(), gs.end(), [](const Group* a, const Group* b) { return a->cls < b->cls; });
        // items of the run with their table bytes and cost, dealt to chunks of similar size
        struct Item {
            uint32_t bytes;
            double cost;
            Group* g;
            const MaskRec* pair;
            int kind;   // 1: PAIR, 2: DIAG
        };
        std::vector<Item> items;
        for (Group* g : gs) items.push_back({(uint32_t)g->mem.size() * tab_bytes, (double)g->mem.size(), g, nullptr, 0});
        for (const MaskRec* m : r.pairs)
            items.push_back({(uint32_t)kPairStride * esz << __builtin_popcount(bits_in(*m, 2)), kGroupCostPair, nullptr, m, 1});
        for (const MaskRec* m : r.diag) items.push_back({0u, kCostDiag, nullptr, m, 2});
        uint32_t total = 0;
        double total_cost = 0.0;
        for (const Item& it : items) {
            total += it.bytes;
            total_cost += it.cost;
        }
        const uint32_t cap = group_table_bytes(esz) - kGroupSlack * esz;
        uint32_t n = std::max(1u, (total + cap - 1) / cap);
        if (max_cost > 0.0) n = std::max(n, (uint32_t)std::ceil(total_cost / max_cost));
        n = std::min(n, (uint32_t)std::max<size_t>(1, items.size()));
        std::vector<std::vector<Item>> bins(n);
        std::vector<uint32_t> used(n, 0);
        std::vector<int> n_groups(n, 0);
        std::vector<double> cost(n, 0.0);
        // largest first onto the cheapest chunk with room, so that the classes spread evenly
        std::stable_sort(items.begin(), items.end(), [](const Item& a, const Item& b) { return a.cost > b.cost; });
        for (const Item& it : items) {
            size_t best = bins.size();
            for (size_t b = 0; b < bins.size(); ++b)
                if (used[b] + it.bytes <= cap && n_groups[b] + (it.g ? 1 : 0) <= kGroupsPerChunk && (best == bins.size() || cost[b] < cost[best])) best = b;
            if (best == bins.size()) {
                bins.push_back({});
                n_groups.push_back(0);
                used.push_back(0);
                cost.push_back(0.0);
            }
            bins[best].push_back(it);
            used[best] += it.bytes;
            n_groups[best] += it.g ? 1 : 0;
            cost[best] += it.cost;
        }
        for (size_t b = 0; b < bins.size(); ++b) {
            if (bins[b].empty()) continue;
            std::stable_sort(bins[b].begin(), bins[b].end(), [](const Item& a, const Item& c) {
                const int ka = a.g ? a.g->cls : 100 + a.kind, kc = c.g ? c.g->cls : 100 + c.kind;
                return ka < kc;
            });
            GroupChunk C{};
            C.x_high = x_high;
            C.new_tile = x_high != prev_high ? 1 : 0;
            prev_high = x_high;
            C.es = es;
            C.shift = r.shift;
            C.qpack = r.qpack;
            C.zbase = r.zbase;
            C.first_group = (uint32_t)G.groups.size();
            C.first_table = (uint32_t)G.tabs.size();
            C.first_pair = (uint32_t)G.pairs.size();
            uint32_t off = 0;
            for (const Item& it : bins[b]) {
                if (it.kind == 2) {
                    ++C.n_diag;
                    ++G.n_diag;
                    continue;
                }
                if (!it.g) {
                    const MaskRec& m = *it.pair;
                    PairRec q{};
                    q.off = off;
                    q.xoff = (m.x & lane_mask) * esz;
                    q.z = m.zbase & ~m.x;
                    q.tab = m.type_tab & 0x0fffffffu;
                    q.qpack = m.qpack;
                    const uint32_t in = bits_in(m, 2);
                    if (in == 2u) bad("PAIR index bits");
                    q.n_in = (uint32_t)__builtin_popcount(in);
                    q.sel = 0x0c0c0c0cu;
                    for (int i = 0; i < 2; ++i) {
                        const uint32_t qb = mask_q(m.qpack, i);
                        if (qb < (uint32_t)kLaneBits) q.sel = (q.sel & ~(0xffu << (8 * i))) | qb << (8 * i);
                    }
                    const int xk = (int)((m.x & kmask) >> kLaneBits), zk = (int)((q.z & kmask) >> kLaneBits);
                    q.cls = 0xffffffffu;
                    for (int c = 0; c < 2 * kPairPatterns; ++c)
                        if (q.cls == 0xffffffffu && pair_xk(c >> 1) == xk && member_zk(xk, c & 1) == zk) q.cls = (uint32_t)c;
                    if (q.cls == 0xffffffffu) bad("PAIR class");
                    off += it.bytes;
                    ++C.n_pair;
                    G.pairs.push_back(q);
                    continue;
                }
                const int J = it.g->cls >> 1;
                std::vector<const MaskRec*>& mem = it.g->mem;
                std::sort(mem.begin(), mem.end(), [&](const MaskRec* x, const MaskRec* y) { return (x->x & kmask) < (y->x & kmask); });
                if ((int)mem.size() != choose4(J)) bad("incomplete group");
                GroupRec rec{};
                for (size_t j = 0; j < mem.size(); ++j) {
                    const MaskRec& m = *mem[j];
                    if ((int)((m.x & kmask) >> kLaneBits) != member_xk(J, (int)j)) bad("member");
                    GroupRec q{0u, (m.zbase & lane_mask) | (m.x & lane_mask) << 8};
                    uint32_t first_k = 0, pos = 0, nk = 0;
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t qb = mask_q(m.qpack, i);
                        if (qb >= (uint32_t)kGroupTileBits) continue;
                        q.sel |= (qb < (uint32_t)kLaneBits ? qb : 0x0cu) << (8 * pos);
                        if (qb >= (uint32_t)kLaneBits) {
                            if (nk == 0) first_k = pos;
                            else if (first_k + nk != pos) bad("k index bits");
                            ++nk;
                        }
                        ++pos;
                    }
                    for (uint32_t i = pos; i < 4; ++i) q.sel |= 0x0cu << (8 * i);
                    if ((int)nk != J || pos != es) bad("index bits");
                    q.pack |= first_k << 16;
                    if (j == 0) rec = q;
                    if (q.sel != rec.sel || q.pack != rec.pack) bad("members differ");
                    G.tabs.push_back(m.type_tab & 0x0fffffffu);
                    ++C.n_tabs;
                    off += tab_bytes;
                }
                G.groups.push_back(rec);
                C.cnt[J] += 1u << (16 * (it.g->cls & 1));
            }
            G.chunks.push_back(C);
            G.cost.push_back(cost[b] + kCostChunk + (C.new_tile ? kCostTile : 0.0));
        }
    }
    // a chunk's lanes read up to kGroupsPerChunk records from its first, and one group ahead
    for (int i = 0; i <= kGroupsPerChunk; ++i) G.groups.push_back(GroupRec{0x0c0c0c0cu, 0u});
    return G;
}

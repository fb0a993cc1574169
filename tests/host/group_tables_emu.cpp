// Host-side check of the 16-row apply kernel's tables (no GPU).
//
// Builds them with the library's host code (build_group_tables, both row
// layouts, both element sizes) for the full space and both parity sectors and
// evaluates rows of H psi from them the way k_apply_groups reads them: for the
// row's tile, thread and k bits the groups by class from the staged tables
// (bounds-checked), the PAIR masks, the diagonal and the masks
// that flip only tile bits.  Compared with the direct sum over the term tables.
// At sizes from N = 24 to 60 the builder alone runs too (it throws where a group is not
// complete or its members disagree) and every mask must be served once.
#include "apply_h.hip"

#include <complex>
#include <cstdio>
#include <random>

using namespace syk;
typedef std::complex<double> C;

namespace {

// 4-bit QUAD table index: bit m = bit q_m of r
uint32_t table_index(uint32_t r, uint32_t qpack)
{
    uint32_t i = 0;
    for (int m = 0; m < 4; ++m) i |= ((r >> mask_q(qpack, m)) & 1u) << m;
    return i;
}

int run_case(int N, bool two, uint32_t esz, int sector, double max_cost, int n_rows)
{
    std::mt19937_64 g((uint64_t)N * 77 + esz + (two ? 5 : 0) + 100 * (uint64_t)(sector + 1));
    std::normal_distribution<double> nd;
    std::vector<double> J((size_t)N * (N - 1) * (N - 2) * (N - 3) / 24);
    for (double& v : J) v = nd(g) * 0.1;
    TermTables TF, TS;
    build_tables(N, 1, J.data(), TF);
    if (sector >= 0) build_sector_tables(TF, sector, TS);
    const TermTables& T = sector >= 0 ? TS : TF;
    const int M = sector >= 0 ? N / 2 - 1 : N / 2;
    const uint64_t D = 1ull << M;
    const int tb = kGroupTileBits, rot = M - tb;
    int bad = 0;
    size_t served = 0, groups = 0, chunks = 0;
    std::vector<C> psi(n_rows ? D : 0);
    for (C& v : psi) v = C(nd(g), nd(g));
    std::vector<uint64_t> rows;
    for (int i = 0; i < n_rows; ++i) rows.push_back(g() & (D - 1));
    std::vector<C> out(rows.size(), 0.0), ref(rows.size(), 0.0);
    auto sgn = [](uint64_t v) { return (__builtin_popcountll(v) & 1) ? -1.0 : 1.0; };
    auto lin = [&](uint32_t tab, int e, uint64_t r) {
        const double* w = &T.w2[((size_t)tab * 4 + e) * (M + 1)];
        double a = w[M];
        for (int c = 0; c < M; ++c) a += w[c] * (double)((r >> c) & 1u);
        return a;
    };
    auto diag = [&](uint64_t r) {
        double d = 0.0;
        for (int n = 0; n < T.n_diag; ++n) d += T.dw[n] * sgn(r & T.dz[n]);
        return d;
    };
    for (size_t i = 0; i < rows.size(); ++i)
        for (const MaskRec& m : T.masks) {
            const uint64_t r = rows[i];
            const uint32_t type = m.type_tab >> 28, tab = m.type_tab & 0x0fffffffu;
            C d = 0.0;
            if (type == MASK_QUAD) {
                const c128 t = T.tab4[(size_t)tab * 16 + table_index((uint32_t)r, m.qpack)];
                d = C(t.re, t.im);
            } else if (type == MASK_PAIR) {
                const int idx = (int)((r >> mask_q(m.qpack, 0)) & 1u) | (int)((r >> mask_q(m.qpack, 1)) & 1u) << 1;
                for (int e = 0; e < 4; ++e) {
                    const c128 ph = T.phi2[(size_t)tab * 16 + idx * 4 + e];
                    d += C(ph.re, ph.im) * lin(tab, e, r);
                }
            } else {
                d = diag(r);
            }
            ref[i] += (type == MASK_DIAG ? 1.0 : sgn(r & m.zbase)) * d * psi[r ^ m.x];
        }
    for (int layout = 0; layout < (two ? 2 : 1); ++layout) {
        const GroupTables G = build_group_tables(group_layout_masks(T.masks, M, two, layout), esz, max_cost);
        chunks += G.chunks.size();
        served += G.tabs.size() + G.pairs.size() + G.n_diag + G.far.size();
        auto to = [&](uint64_t r) { return layout ? (uint64_t)rotate_bits((uint32_t)r, M, rot) : r; };
        std::vector<C> ps(psi.size());
        for (uint64_t r = 0; r < psi.size(); ++r) ps[to(r)] = psi[r];
        uint32_t prev = 0xffffffffu;
        for (const GroupChunk& c : G.chunks) {
            uint32_t ng = 0, nt = 0;
            for (int J = 0; J <= 4; ++J) {
                const uint32_t n = (c.cnt[J] & 0xffffu) + (c.cnt[J] >> 16);
                ng += n;
                nt += n * choose4(J);
            }
            groups += ng;
            const uint32_t tab_end = (nt << c.es) * esz;
            if (nt != c.n_tabs || c.first_group + ng >= G.groups.size() || c.first_table + nt > G.tabs.size() ||
                c.first_pair + c.n_pair > G.pairs.size() || c.es > 4 || ng > (uint32_t)kGroupsPerChunk ||
                tab_end + kGroupSlack * esz > group_table_bytes(esz) ||
                c.first_group + kGroupsPerChunk >= G.groups.size() ||
                c.x_high >= (D >> tb) || (c.new_tile != 0) != (c.x_high != prev))
                ++bad;
            prev = c.x_high;
            // PAIR entries: after the tables, inside the area, apart
            uint32_t end = tab_end;
            for (uint32_t p = 0; p < c.n_pair; ++p) {
                const PairRec& q = G.pairs.at(c.first_pair + p);
                if (q.off < end || q.n_in > 2) ++bad;
                end = q.off + ((uint32_t)kPairStride * esz << q.n_in);
            }
            if (end > group_table_bytes(esz)) ++bad;
        }
        for (size_t ri = 0; ri < rows.size(); ++ri) {
            const uint32_t r = (uint32_t)to(rows[ri]), tile = r >> tb, base = tile << tb;
            const uint32_t tid = r & 255u;
            const int k = (int)((r >> kLaneBits) & 15u);
            C sum = 0.0;
            for (const GroupChunk& c : G.chunks) {
                const uint64_t sbase = (uint64_t)(tile ^ c.x_high) << tb;
                auto src = [&](uint32_t xoff, int ks) { return ps.at(sbase + ((tid ^ (xoff / esz)) | ((uint32_t)ks << kLaneBits))); };
                auto staged = [&](uint32_t e) {
                    const uint32_t i = (((e & ((1u << c.es) - 1u)) << c.shift) ^ table_index(base, c.qpack)) & 15u;
                    const c128 t = T.tab4.at((size_t)G.tabs.at(c.first_table + (e >> c.es)) * 16 + i);
                    return sgn(base & c.zbase) * C(t.re, t.im);
                };
                uint32_t gi = c.first_group, tab = 0;
                for (int cls = 0; cls < kGroupClasses; ++cls) {
                    const int Jf = cls >> 1, P = cls & 1;
                    const uint32_t n = P ? c.cnt[Jf] >> 16 : c.cnt[Jf] & 0xffffu;
                    for (uint32_t i = 0; i < n; ++i, ++gi) {
                        const GroupRec& q = G.groups.at(gi);
                        uint32_t ia = 0;   // v_perm / v_dot4: lane part of the table index
                        for (int m = 0; m < 4; ++m) {
                            const uint32_t b = (q.sel >> (8 * m)) & 0xffu;
                            if (b < 8) ia += ((tid >> b) & 1u) << m;
                        }
                        for (int j = 0; j < choose4(Jf); ++j, ++tab) {
                            const int XK = member_xk(Jf, j), ZK = member_zk(XK, P);
                            const uint32_t e = ia + (uint32_t)pack_bits4(k & XK, XK) * (1u << ((q.pack >> 16) & 3u));
                            if (e >> c.es) ++bad;   // inside the member's own table
                            sum += sgn(tid & q.pack & 0xffu) * sgn((uint64_t)(k & ZK)) * staged((tab << c.es) + e) *
                                   src(((q.pack >> 8) & 0xffu) * esz, k ^ XK);
                        }
                    }
                }
                for (uint32_t p = 0; p < c.n_pair; ++p) {
                    const PairRec& q = G.pairs.at(c.first_pair + p);
                    const int XK = pair_xk((int)(q.cls >> 1)), ZK = member_zk(XK, (int)(q.cls & 1));
                    // staged index: the lane's bits, then the k bits', then those above the tile
                    uint32_t i = 0;
                    for (int m = 0; m < 2; ++m) {
                        const uint32_t b = (q.sel >> (8 * m)) & 0xffu;
                        if (b < 8) i += ((tid >> b) & 1u) << m;
                    }
                    const int kp = pack_bits4(k & XK, XK);
                    i += (uint32_t)kp * (popc4(XK) == 1 && q.n_in == 2 ? 2u : 1u);
                    if (i >> q.n_in) ++bad;
                    i ^= ((base >> mask_q(q.qpack, 0)) & 1u) | ((base >> mask_q(q.qpack, 1)) & 1u) << 1;
                    const MaskRec* m = nullptr;
                    for (const MaskRec& x : T.masks)
                        if ((x.type_tab >> 28) == MASK_PAIR && (x.type_tab & 0x0fffffffu) == q.tab) m = &x;
                    C d = 0.0;
                    for (int e = 0; e < 4; ++e) {
                        const c128 ph = T.phi2[(size_t)q.tab * 16 + i * 4 + e];
                        d += C(ph.re, ph.im) * lin(q.tab, e, r);
                    }
                    const double fold = sgn((i & 1u) & (m->zbase >> mask_q(q.qpack, 0))) * sgn((i >> 1) & (m->zbase >> mask_q(q.qpack, 1)) & 1u);
                    sum += sgn((base | tid) & q.z) * sgn((uint64_t)(k & ZK)) * fold * d * src(q.xoff, k ^ XK);
                }
                if (c.n_diag) sum += diag(r) * src(0, k);   // layout 0, own tile
            }
            for (const FarRec& f : G.far) {
                const c128 t = T.tab4[(size_t)f.tab * 16 + table_index(base, f.qpack)];
                sum += sgn(base & f.zbase) * C(t.re, t.im) * ps[((uint64_t)(tile ^ f.x_high) << tb) + (r & 4095u)];
            }
            out[ri] += sum;
        }
    }
    if (served != T.masks.size()) ++bad;
    double err = 0.0, mx = 1e-300;
    for (size_t i = 0; i < rows.size(); ++i) {
        err = std::max(err, std::abs(out[i] - ref[i]));
        mx = std::max(mx, std::abs(ref[i]));
    }
    std::printf("N=%d sector=%d layouts=%d esz=%u chunks=%zu groups=%zu rel_err=%.2e table_errors=%d\n", N, sector,
                two ? 2 : 1, esz, chunks, groups, err / mx, bad);
    std::fflush(stdout);
    return (err / mx < 1e-12 && bad == 0) ? 0 : 1;
}

}  // namespace

int main()
{
    int bad = 0;
    // one and two layouts with overlapping (M = 16, 18) and disjoint (M = 25) tiles
    for (int sector : {-1, 0, 1}) {
        bad += run_case(28, false, 16u, sector, 0.0, 60);
        for (uint32_t esz : {8u, 16u}) bad += run_case(sector < 0 ? 36 : 34, true, esz, sector, esz == 8u ? 20.0 : 0.0, 60);
    }
    bad += run_case(44, true, 16u, -1, 0.0, 8);
    for (int N : {24, 26, 34, 40, 44, 46, 60})
        for (int sector : {-1, 0, 1})
            for (uint32_t esz : {N % 4 ? 8u : 16u})
                for (bool two : {false, true}) {
                    const int M = N / 2 - (sector >= 0 ? 1 : 0);
                    if (M < kGroupTileBits + (two ? kGroupKBits : 0)) continue;
                    bad += run_case(N, two, esz, sector, N < 44 ? 30.0 : 0.0, 0);
                }
    return bad;
}

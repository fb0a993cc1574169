// Host-side check of how apply_H picks its launch (no GPU).
//
// A handle that has run one product of some width, pairing of its columns and
// element type must be able to run any other one of that type without building
// tables, wherever a plan that ties the tables to the tile alone could: for each
// pair of calls the tables the first one builds are entered in the handle's maps
// (empty: only their keys are read) and existing_route must find a route for the
// second whose tables exist and whose scratch fits.  The settings of a handle with
// automatic tiles must reach the plan of every call.
#include "apply_h.hip"

#include <cstdio>

using namespace syk;

namespace {

int bad = 0;

#define CHECK(ok, ...)                     \
    do {                                   \
        if (!(ok)) {                       \
            if (bad++ < 20) {              \
                std::printf("BAD ");       \
                std::printf(__VA_ARGS__);  \
                std::printf("\n");         \
            }                              \
        }                                  \
    } while (0)

std::vector<int32_t> columns(int nvec, bool paired)
{
    std::vector<int32_t> r(nvec);
    for (int c = 0; c < nvec; ++c) r[c] = paired ? c / 2 % 2 : c % 2;
    return r;
}

// The tables a product of this plan leaves on the handle.
void built(HamiltonianDev& H, const ApplyPlan& P, syk_dtype dt, int nvec)
{
    const uint32_t esz = (uint32_t)elem_bytes(dt);
    if (use_table(H, P, nvec, esz)) {
        (dt == SYK_C128 ? H.table_d : H.table_f).ready = true;
        return;
    }
    H.diag_ready = true;
    for (int l = 0; l <= P.two_layouts; ++l) {
        if (P.groups) H.group_tables[group_tables_key(P, esz, l)];
        else H.apply_tables[apply_tables_key(P, esz, l)];
    }
}

// Tile bits of the rule that depends on the width only through the tile: the
// largest tile of at most 2^11 rows that leaves 2048 workgroups, at least 2^8.
int tile_of_width(int M, int nvec)
{
    int tb = std::min(M, 11);
    while (tb > 8 && ((int64_t)1 << (M - tb)) * nvec < 2048) --tb;
    return tb;
}

void check_routes()
{
    const int widths[] = {1, 2, 3, 4, 5, 8, 9, 16, 31, 33, 64, 65, 128, 1000};
    long pairs = 0, own = 0;
    for (int M = 2; M <= 23; ++M) {
        std::vector<MaskRec> masks(M * (M - 1) * (M - 2) * (M - 3) / 24 + M * (M - 1) / 2 + 1);
        for (int dti = 0; dti < 2; ++dti) {
            const syk_dtype dt = dti ? SYK_C64 : SYK_C128;
            const size_t esz = elem_bytes(dt);
            const uint64_t dim = (uint64_t)1 << M;
            for (int a : widths)
                for (int b : widths)
                    for (int pa = 0; pa < 2; ++pa)
                        for (int pb = 0; pb < 2; ++pb) {
                            HamiltonianDev H;
                            H.M = M;
                            H.n_real = 2;
                            H.host_masks = &masks;
                            const auto ra = columns(a, pa), rb = columns(b, pb);
                            built(H, plan_of_call(H, plan_apply(M, a, dt, nullptr), dt, a, ra.data()), dt, a);
                            const ApplyPlan P = plan_of_call(H, plan_apply(M, b, dt, nullptr), dt, b, rb.data());
                            auto need = [&](const ApplyPlan& Q) { return rot_bytes(Q, b, dim, esz) + parts_bytes(Q, b, dim); };
                            auto fits = [&](const ApplyPlan& Q) { return need(Q) <= kNoAllocScratchBytes; };
                            // what the width-only rule would accept
                            const int tb = tile_of_width(M, b);
                            const bool two = M - tb >= 7 && tb >= 8;
                            const size_t rot = two ? 2 * std::min<size_t>(b, 64) * dim * esz : 0;
                            if (tb != tile_of_width(M, a) || rot > kNoAllocScratchBytes) continue;
                            ++pairs;
                            CHECK(use_table(H, P, b, esz) || fits(P), "M=%d esz=%zu width %d: scratch of %zu bytes", M, esz, b, need(P));
                            Route r;
                            const bool ok = existing_route(H, P, dt, b, fits, r);
                            CHECK(ok, "M=%d esz=%zu: width %d (paired %d) after width %d (paired %d) has no route", M, esz, b, pb, a, pa);
                            if (!ok || r.table) continue;
                            const ApplyPlan& Q = r.plan;
                            own += Q.cut == P.cut && Q.groups == P.groups;
                            CHECK(has_tables(H, Q, (uint32_t)esz) && fits(Q), "M=%d: route without tables or scratch", M);
                            CHECK(Q.parts == Q.cut || Q.parts == 1, "M=%d: %d parts from tables cut for %d", M, Q.parts, Q.cut);
                            CHECK(Q.tile_bits <= M && (Q.rpt << Q.lb) == (1 << Q.tile_bits) && Q.nt == (1 << Q.lb) && Q.nc <= 2 &&
                                      Q.slices == P.slices && (!Q.two_layouts || (Q.rot >= 5 && M - Q.rot >= 5)),
                                  "M=%d: inconsistent plan", M);
                            if (a == b && pa == pb) CHECK(Q.cut == P.cut && Q.parts == P.parts && Q.groups == P.groups && Q.nc == P.nc,
                                                          "M=%d width %d: not its own plan", M, b);
                        }
        }
    }
    std::printf("routes: %ld pairs of calls, %ld on the call's own tables\n", pairs, own);
    CHECK(pairs > 4000, "too few pairs");
    // no product of the element type: no route
    HamiltonianDev H;
    std::vector<MaskRec> masks(1);
    H.M = 16;
    H.n_real = 1;
    H.host_masks = &masks;
    built(H, plan_apply(16, 1, SYK_C128, nullptr), SYK_C128, 1);
    Route r;
    CHECK(!existing_route(H, plan_apply(16, 1, SYK_C64, nullptr), SYK_C64, 1, [](const ApplyPlan&) { return true; }, r), "route without tables");
    // a tile given by the caller is run as given or refused
    const ApplyTuning t{9, 1, 1};
    CHECK(!existing_route(H, plan_apply(16, 1, SYK_C128, &t), SYK_C128, 1, [](const ApplyPlan&) { return true; }, r), "other tile");
}

// The settings of syk_set_apply_tuning with automatic tiles reach the plan of every
// call: one or two columns per workgroup as asked for, and the tile order.
void check_tuning()
{
    for (int M = 13; M <= 23; ++M)
        for (int dti = 0; dti < 2; ++dti)
            for (int nvec : {1, 2, 7, 8, 14, 16, 30, 32, 64, 66})
                for (int xcd = 0; xcd < 2; ++xcd)
                    for (int cols = 0; cols <= 2; ++cols)
                        for (int paired = 0; paired < 2; ++paired) {
                            const syk_dtype dt = dti ? SYK_C64 : SYK_C128;
                            HamiltonianDev H;
                            H.M = M;
                            const ApplyTuning t{0, xcd, cols};
                            const auto real = columns(nvec, paired);
                            const ApplyPlan P = plan_of_call(H, plan_apply(M, nvec, dt, &t), dt, nvec, real.data());
                            CHECK(P.xcd_remap == xcd, "M=%d nvec=%d cols=%d: tile order %d became %d", M, nvec, cols, xcd, P.xcd_remap);
                            if (cols == 1) CHECK(P.nc == 1, "M=%d nvec=%d: one column per workgroup became %d", M, nvec, P.nc);
                            if (cols == 2 && paired && nvec % 2 == 0)
                                CHECK(P.nc == 2, "M=%d esz=%zu nvec=%d: two columns per workgroup became %d", M, elem_bytes(dt), nvec, P.nc);
                            // unasked, two columns only where they are faster: complex64, 2^18 and 2^19
                            // rows, at least 2048 workgroups
                            const bool two = dt == SYK_C64 && (M == 18 || M == 19) && nvec % 2 == 0 && paired &&
                                             (1 << (M - 11)) * (std::min(nvec, 64) / 2) >= 2048;
                            if (cols == 0) CHECK(P.nc == (two ? 2 : 1), "M=%d nvec=%d paired=%d: %d columns per workgroup", M, nvec, paired, P.nc);
                        }
}

}  // namespace

int main()
{
    check_tuning();
    check_routes();
    std::printf(bad ? "%d BAD\n" : "plan checks ok\n", bad);
    return bad != 0;
}

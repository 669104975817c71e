// The piece kernels' planner and index arithmetic, walked on the CPU under AddressSanitizer + UndefinedBehaviorSanitizer (built and
// run by tests/test_host_sanitizers.py: the host side of the dispatcher and of sconv_piece.hip, included here, with everything else of the
// library, no device code, no GPU).
// Prints "ok" and exits 0 when every expectation holds.
#include "sconv_api.hip"
#include "sconv_piece.hip"

#include <random>
#include <vector>

using namespace sconv;

static int failures = 0;
#define EXPECT(cond, ...)                                                                       \
    do {                                                                                        \
        if (!(cond) && ++failures <= 20) {                                                      \
            fprintf(stderr, "line %d: %s does not hold: ", __LINE__, #cond);                    \
            fprintf(stderr, __VA_ARGS__);                                                       \
            fprintf(stderr, "\n");                                                              \
        }                                                                                       \
    } while (0)

static std::mt19937 rng(1909);
static int pick(int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); }
static int pick_log(double lo, double hi)
{
    return (int)(exp(log(lo) + (log(hi) - log(lo)) * (rng() % 10001) / 10000.0) + 0.5);
}

// A random problem with a square kernel of T taps; false where the descriptor is not valid.
static bool random_problem(int T, bool pooled, Problem* p)
{
    const int R = T == 1 ? 1 : T == 9 ? 3 : T == 25 ? 5 : 7, groups = pick(0, 3) ? 1 : pick(2, 4);
    const int H = pick_log(R, 64), W = pick(0, 2) ? H : pick_log(R, 64);
    sconv_desc_t d = {pick_log(1, 32), groups * pick_log(1, 200), H, W, groups * pick_log(1, 300), R, R, pick(0, 2) ? 1 : pick(2, 3),
                      pick(0, R - 1), groups, 0, 0, 0, SCONV_RELU};
    if (pooled) {
        d.pool_h = d.pool_w = 2;
        d.pool_stride = pick(0, 2) ? 2 : pick(1, 4);
    }
    return fill_problem(&d, pooled, p) == SCONV_OK;
}

// Filters read as stored: every read of every lane lies inside the filter tensor, or starts past its end, where the buffer's
// bounds check gives zero without a read; none straddles the end.
template <class G>
static void raw_reads(const char* name)
{
    for (int n = 0; n < 200; ++n) {
        Problem p;
        if (!random_problem(G::T, G::POOL, &p)) continue;
        const int chunks16 = (p.Cg + 16 * G::CS - 1) / (16 * G::CS) * G::CS, kblocks = (p.Kg + G::BM - 1) / G::BM;
        for (int kb : {0, kblocks - 1}) {
            const long long first = ((long long)(p.G - 1) * p.Kg + (long long)kb * G::BM) * p.L, left = ((long long)p.K * p.L - first) * 4;
            for (int row = 0; row < G::BM; ++row)
                for (int half = 0; half < 2; ++half)
                    for (int ch16 = 0; ch16 < chunks16; ++ch16)
                        for (int j = 0; j < 8; ++j) {
                            const int base = raw_base(row < p.Kg - 1 - kb * G::BM ? row : p.Kg - 1 - kb * G::BM, p.L, G::T, half);
                            for (int t = 0; t < G::T; t += G::VW) {
                                int at = base + raw_step(ch16, G::T, G::T == 1 ? 0 : j, t), bytes = 12;
                                if (G::T == 1 && raw_wide(p.Cg, ch16)) {
                                    at += j / 4 * 16;
                                    bytes = 16;
                                } else if (G::T == 1) {
                                    const int last = raw_last(base, p.L, half);
                                    at = at + 4 * j < last ? at + 4 * j : last;
                                    bytes = 4;
                                    EXPECT(at >= 0 && at < left, "%s at %d of %lld", name, at, left);
                                }
                                EXPECT(at >= 0 && (at + bytes <= left || at >= left), "%s C %d K %d G %d T %d: %d bytes at %d of %lld", name, p.C,
                                       p.K, p.G, G::T, bytes, at, left);
                                if (ch16 * 16 + half * 8 + j < p.Cg)   // a channel that counts: its own element
                                    EXPECT(at + (G::T == 1 && raw_wide(p.Cg, ch16) ? j % 4 * 4 : 0) ==
                                               ((row < p.Kg - 1 - kb * G::BM ? row : p.Kg - 1 - kb * G::BM) * p.L + (ch16 * 16 + half * 8 + j) * G::T + t) * 4,
                                           "%s", name);
                            }
                        }
        }
    }
}

template <class G>
static void taps_have_no_raw_reads(const char*)
{
}

// The strips are the best of every number of strips of four or more columns.
static void strips_are_the_best_of_all(int n)
{
    for (int i = 0; i < n; ++i) {
        Problem p;
        const int T = std::vector<int>{1, 9, 25, 49}[pick(0, 3)], BN = 64 * pick(1, 2), PXMAX = 64 * pick(1, 6);
        const bool pooled = pick(0, 2) == 0;
        if (!random_problem(T, pooled, &p)) continue;
        PieceCfg c = {}, d = {};
        c.flat = d.flat = T == 1 && p.stride == 1 && !pooled;
        const bool found = choose_strips(p, pooled, BN, PXMAX, c);
        const int cols = pooled ? p.PW : d.flat ? p.OH * p.OW : p.OW, rows = pooled ? p.PH : d.flat ? 1 : p.OH;
        double best = 0.0;
        for (int m = 1; m <= cols; ++m) {
            const int TW = (cols + m - 1) / m, strips = (cols + TW - 1) / TW;
            if (TW < 4 && m > 1) break;
            const long long px = stage_positions(p, pooled, d.flat, BN, TW), run = (long long)p.N * rows * TW * (pooled ? 4 : 1);
            if (TW > BN || px > PXMAX) continue;
            const long long nt = (run + BN - 1) / BN;
            const double cost = (double)nt * strips * (BN * (1.0 + 0.5 / TW) + px * 0.02);
            if (best != 0.0 && cost >= best) continue;
            best = cost;
            d.TW = TW;
            d.strips = strips;
            d.nrun = (int)run;
            d.ntiles = (int)nt;
            d.px = (int)px;
        }
        EXPECT(found == (best != 0.0), "T %d %dx%d", T, p.OH, p.OW);
        if (found) EXPECT(c.TW == d.TW && c.strips == d.strips && c.nrun == d.nrun && c.ntiles == d.ntiles && c.px == d.px, "T %d %dx%d", T, p.OH, p.OW);
    }
}

// A network's plans are all kept: by shape, with a workspace and without, and with the geometry that tuning found.
static void plans_are_kept()
{
    std::vector<Problem> net;
    for (int i = 0; i < 100; ++i) {
        sconv_desc_t d = {8, 64 + 32 * i, 56 >> i % 3, 56 >> i % 3, 128, i % 4 ? 1 : 3, i % 4 ? 1 : 3, 1, i % 4 ? 0 : 1, 1, 0, 0, 0, SCONV_RELU};
        Problem p;
        EXPECT(fill_problem(&d, false, &p) == SCONV_OK, "layer %d", i);
        net.push_back(p);
    }
    PlanPin pins[2];
    memset(pins, 0, sizeof(pins));
    snprintf(pins[0].geom, sizeof(pins[0].geom), "c128x64");
    snprintf(pins[1].geom, sizeof(pins[1].geom), "a128x64");
    pins[0].nwv = pins[1].nwv = 4;
    pins[0].ncs = pins[1].ncs = 1;
    for (int pass = 0; pass < 2; ++pass)
        for (size_t i = 0; i < net.size(); ++i)
            for (const PlanPin* pin : {(const PlanPin*)nullptr, (const PlanPin*)&pins[0], (const PlanPin*)&pins[1]}) {
                g_pin = pin;
                split_scratch_given(i % 2 ? nullptr : reinterpret_cast<void*>(uintptr_t(256)), i % 2 ? 0 : size_t(64) << 20, true);
                split_scratch_select(nullptr);
                double& cost = const_cast<Choice&>(choose_plan(net[i], false)).plan.cost;
                const double mark = 1e6 + i * 3.0 + (pin ? pin - pins + 1 : 0);   // (a plan that is walked again loses it)
                if (pass) EXPECT(cost == mark, "layer %zu, geometry %s", i, pin ? pin->geom : "any");
                cost = mark;
            }
    g_pin = nullptr;
    split_scratch_given(nullptr, 0, false);
}

int main()
{
    strips_are_the_best_of_all(4000);
    plans_are_kept();
#define WALK_PIECE(NAME, ...) raw_reads<PGeom<__VA_ARGS__>>(NAME);
#define WALK_TAPS(NAME, ...) taps_have_no_raw_reads<TGeom<__VA_ARGS__>>(NAME);
    PIECE_GEOMETRIES(WALK_PIECE, WALK_TAPS)
    if (failures) {
        fprintf(stderr, "%d expectation(s) failed\n", failures);
        return 1;
    }
    printf("ok\n");
    return 0;
}

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
                                unsigned at = G::T == 1 ? raw_fragment(base, p.Cg, ch16) : base + raw_step(ch16, G::T, j, t);
                                int bytes = 12;
                                if (G::T == 1 && raw_wide(p.Cg, ch16)) {
                                    at += j / 4 * 16;
                                    bytes = 16;
                                } else if (G::T == 1) {
                                    const unsigned last = raw_last(base, p.L, half);
                                    at = at + 4 * j < last ? at + 4 * j : last;
                                    bytes = 4;
                                    EXPECT(at < left, "%s at %u of %lld", name, at, left);
                                }
                                EXPECT(at + (long long)bytes <= left || at >= left, "%s C %d K %d G %d T %d: %d bytes at %u of %lld", name, p.C,
                                       p.K, p.G, G::T, bytes, at, left);
                                if (ch16 * 16 + half * 8 + j < p.Cg)   // a channel that counts: its own element
                                    EXPECT(at + (G::T == 1 && raw_wide(p.Cg, ch16) ? j % 4 * 4 : 0) ==
                                               (unsigned)((row < p.Kg - 1 - kb * G::BM ? row : p.Kg - 1 - kb * G::BM) * p.L + (ch16 * 16 + half * 8 + j) * G::T + t) * 4,
                                           "%s", name);
                            }
                        }
        }
    }
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

// The plans of one geometry: what a workgroup stages and reads in LDS, what it reads of the map and writes to the workspace, and which
// results it computes, followed as the kernels compute it.
template <class G>
static void plans(const char* name, Plan (*plan)(const Problem&, bool, bool), int CS, int PXMAX, int lds_other, int chunk_buffers, int pair_buffer = 0)
{
    const bool pairs = pair_buffer != 0;
    int walked = 0, split = 0, in_pieces = 0, rests[3] = {0, 0, 0};
    for (int tries = 0; tries < (pairs ? 40000 : 4000) && walked < 60; ++tries) {
        Problem p;
        if (!random_problem(G::T, G::POOL, &p)) continue;
        static const float some = 0.0f;
        const bool prepares = tap_supported(p, G::POOL) && p.stride == 1;
        if (pairs && walked % 4 == 3 && !prepares) continue;
        p.wprep = (pairs ? walked % 4 == 3 : pick(0, 3) == 0) && prepares ? &some : nullptr;
        // a third with the model's choice, the others with split tiles or with pieces of the filters where there is room
        const int form = walked % 3;
        char slices[16];
        snprintf(slices, sizeof(slices), "%d,1,%d", pick(0, 2), pick(2, 5));
        form == 1 ? setenv("SCONV_PIECE_SPLIT", slices, 1) : unsetenv("SCONV_PIECE_SPLIT");
        form == 2 && G::BM != 32 && !pairs ? setenv("SCONV_PIECE_SRC", "0", 1) : unsetenv("SCONV_PIECE_SRC");
        EXPECT(sconv_env_refresh() == SCONV_OK, "%s", name);
        const size_t room = form || pick(0, 1) ? plan_workspace_bytes(p, G::POOL) / (form ? 1 : (size_t)pick(1, 20)) : 0;
        split_scratch_given(room ? reinterpret_cast<void*>(uintptr_t(256)) : nullptr, room, true);
        split_scratch_select(nullptr);
        const Plan pl = plan(p, G::POOL, pick(0, 1) != 0);
        const size_t ws = usable_workspace(p, G::POOL);
        split_scratch_given(nullptr, 0, false);
        if (pl.cost < 0.0) continue;
        ++walked;
        const PieceCfg& c = pl.cfg;
        const int T = G::T, S = p.S, iH = c.flat ? 1 : p.H, iW = c.flat ? p.H * p.W : p.W, HP = iH + p.pad;
        const int prows = G::POOL ? p.PH : c.flat ? 1 : p.OH, pcols = G::POOL ? p.PW : c.flat ? p.OH * p.OW : p.OW;
        const int pitch = (G::POOL ? (c.TW - 1) * p.ps + 1 : c.TW - 1) * p.stride + S;
#define HOLDS(cond) EXPECT(cond, "%s N %d C %d %dx%d K %d G %d stride %d pad %d ps %d, %zu bytes", name, p.N, p.C, p.H, p.W, p.K, p.G, p.stride, p.pad, p.ps, ws)
        // LDS, workspace, slices
        HOLDS(c.px <= PXMAX && c.px * 48 <= c.cgb && pl.lds_bytes <= 160 * 1024);
        HOLDS((size_t)lds_other + (size_t)chunk_buffers * 2 * CS * c.cgb <= pl.lds_bytes);
        HOLDS(pl.piece_bytes + (size_t)pl.ntail * (pl.ntail ? c.nss : 0) * G::BM * G::BN * 4 <= ws);
        HOLDS(c.whole + pl.ntail == c.ntiles * c.strips * c.kblocks * p.G && (!pl.ntail || (c.nss > 1 && c.nss <= c.nch)));
        HOLDS(c.nch * 16 * CS >= p.Cg && c.kblocks * G::BM >= p.Kg && (c.nch - 1) * 16 * CS < p.Cg);
        HOLDS((pl.src == SRC_FP32) <= (p.wprep != nullptr) && (pl.src >= SRC_PAIRS) == pairs);
        if (pairs) {
            // fragments of 2048 bytes, a word for every filter behind them, and from the next 256 bytes on the pieces that the other chunks may read
            const size_t fragments = (size_t)p.G * c.kb32 * c.nch * 9, exponents = (size_t)p.G * c.kb32 * 32, both = pair_bytes(p.G, c.kb32, c.nch);
            HOLDS(both % 256 == 0 && fragments * 2048 + exponents * 4 <= both && c.kb32 * 32 >= c.kblocks * G::BM);
            HOLDS(pl.lds_bytes >= 2 * (size_t)pair_buffer);
            HOLDS(pl.piece_bytes == both + (pl.rest == SRC_PIECES ? fragments * 3072 : 0));
            HOLDS(pl.rest == (p.wprep ? SRC_FP32 : pl.rest == SRC_PIECES ? SRC_PIECES : SRC_RAW));
            if (p.wprep) HOLDS(c.kb32 == (p.Kg + 127) / 128 * 4 && p.Cg % 16 == 0);
            HOLDS(fragments / p.G / c.kb32 * 4 * 3072 < (size_t)1 << 31 && (size_t)p.L * 4 <= 128 * 1024);   // a block's offsets, a filter in LDS
            ++rests[pl.rest];
        }
        if (pl.src == SRC_PIECES) HOLDS(pl.piece_bytes == (size_t)p.G * c.kb32 * c.nch * CS * T * 3072 && c.kb32 * 32 >= c.kblocks * G::BM);
        if (pl.src == SRC_FP32) HOLDS(c.kb32 * 32 >= c.kblocks * G::BM && p.Cg % (16 * CS) == 0);
        split += pl.ntail > 0;
        in_pieces += pl.src == SRC_PIECES;
        std::vector<unsigned char> seen((size_t)p.N * prows * pcols, 0);
        const bool all = (size_t)c.ntiles * c.strips * G::BN <= 40000;
        for (int tile = 0; tile < c.ntiles; ++tile) {
            const bool look = tile < 3 || tile >= c.ntiles - 2 || pick(0, c.ntiles / 4) == 0;
            if (!look && !all) continue;
            for (int strip = 0; strip < c.strips; ++strip) {
                auto window = [&](int P, int& n, int& oh, int& ow) {
                    const int pp = G::POOL ? P >> 2 : P, q = pp / c.TW;
                    ow = pp - q * c.TW;
                    n = q / prows;
                    oh = q - n * prows;
                    if (G::POOL) {
                        oh = p.ps * oh + ((P & 3) >> 1);
                        ow = p.ps * ow + (P & 1);
                    }
                };
                int n0, oh0, ow0;
                window(tile * G::BN, n0, oh0, ow0);
                const int r0 = n0 * HP + oh0 * p.stride, first_col = strip * c.TW * (G::POOL ? p.ps : 1), w0 = first_col * p.stride - p.pad;
                for (int i = 0; i < G::BN; ++i) {
                    const int P = tile * G::BN + i;
                    int n, oh, ow;
                    window(P < c.nrun ? P : c.nrun - 1, n, oh, ow);
                    const int at = (n * HP + oh * p.stride - r0) * pitch + ow * p.stride;
                    const int col = ow + first_col, wcol = G::POOL ? (col - (P & 1)) / p.ps : col, wrow = G::POOL ? (oh - ((P & 3) >> 1)) / p.ps : oh;
                    const bool counts = P < c.nrun && wcol < pcols;
                    if (counts) {
                        HOLDS(n < p.N && wrow < prows);
                        if (n < p.N && wrow < prows) ++seen[((size_t)n * prows + wrow) * pcols + wcol];
                    }
                    for (int t = 0; look && t < T; ++t) {
                        const int q = at + t / S * pitch + t % S;
                        HOLDS(q >= 0 && q < c.px);
                        // what is staged there
                        const int sr = r0 + q / pitch, sn = sr / HP, h = sr - sn * HP - p.pad, cw = q % pitch + w0;
                        const bool staged = sn < p.N && h >= 0 && h < iH && cw >= 0 && cw < iW;
                        if (staged) {
                            const long long o = (long long)(sn - n0) * p.C * p.H * p.W + h * iW + cw + (long long)(p.Cg - 1) * p.H * p.W;
                            HOLDS(sn >= n0 && o * 4 < 0x7ffffffc && (n0 * p.C + (p.G - 1) * p.Cg) * (long long)(p.H * p.W) + o < (long long)p.N * p.C * p.H * p.W);
                        }
                        if (!counts) continue;
                        const int ih = oh * p.stride - p.pad + t / S, iw = col * p.stride - p.pad + t % S;
                        const bool inside = ih >= 0 && ih < iH && iw >= 0 && iw < iW;
                        HOLDS(staged == inside && (!inside || (sn == n && h == ih && cw == iw)));
                    }
                }
            }
        }
        for (size_t i = 0; all && i < seen.size(); ++i)
            if (seen[i] != (G::POOL ? 4 : 1)) {
                HOLDS(false);
                break;
            }
    }
    unsetenv("SCONV_PIECE_SPLIT");
    unsetenv("SCONV_PIECE_SRC");
    EXPECT(sconv_env_refresh() == SCONV_OK && walked >= 40 && split >= 10, "%s: %d plans, %d with split tiles", name, walked, split);
    if (G::BM != 32 && !pairs) EXPECT(in_pieces >= 10, "%s: %d plans with pieces of the filters", name, in_pieces);
    if (pairs) EXPECT(rests[SRC_PIECES] >= 5 && rests[SRC_RAW] >= 3 && rests[SRC_FP32] >= 5, "%s: pieces %d, prepared %d, as stored %d", name, rests[0], rests[1], rests[2]);
}

// The forms with pairs: as above, and what a wavefront writes of a chunk in LDS stays in its buffer.
template <class G>
static void pair_plans(const char* name)
{
    if constexpr (G::PAIRS) {
        constexpr int plane = G::PXMAX * 16;
        for (int unit = 0; unit < G::XU * G::NW; ++unit)
            EXPECT(unit % 2 * 2 * plane + (unit / 2 * 64 + 63) * 16 + plane + 16 <= 2 * 2 * plane, "%s: unit %d", name, unit);
        EXPECT(2 * 2 * plane + 64 + G::NW * 8 <= G::PAIR_BUF && G::NW * 4 <= 64 && G::NW == 4, "%s: words and ranges of the wavefronts", name);
        plans<G>(name, [](const Problem& p, bool pooled, bool) { return plan_pairs<G>(p, pooled); }, G::CS, G::PXMAX, 2 * G::SPARE, 2, G::PAIR_BUF);
    }
}

// The blocks: whole tiles only; every result computed once, from what is staged, in the LDS and the workspace there are.
template <class G>
static void block_plans(const char* name)
{
    constexpr int plane = G::PXMAX * 16;
    EXPECT(G::BLOCK && G::PAIRS && G::NW == 8 && G::XU == 1 && G::PXMAX == 256, "%s: one staging unit a wavefront", name);
    for (int unit = 0; unit < G::NW; ++unit)
        EXPECT(unit % 2 * 2 * plane + (unit / 2 * 64 + 63) * 16 + plane + 16 <= 2 * 2 * plane, "%s: unit %d", name, unit);
    // three buffers; flags, ranges from 64 on, and in the last 512 bytes the exponents of 128 filters
    EXPECT(3 * 2 * 2 * plane + 64 + G::NW * 8 <= 3 * G::PAIR_BUF - 512 && G::BM * 4 <= 512, "%s: what the wavefronts tell each other", name);
    int walked = 0, rests[3] = {0, 0, 0};
    for (int tries = 0; tries < 40000 && walked < 80; ++tries) {
        Problem p;
        if (!random_problem(9, G::POOL, &p)) continue;
        static const float some = 0.0f;
        const bool prepares = tap_supported(p, G::POOL) && p.stride == 1;
        if (walked % 4 == 3 && !prepares) continue;
        p.wprep = walked % 4 == 3 ? &some : nullptr;
        const size_t room = plan_workspace_bytes(p, G::POOL) / (walked % 2 ? 1 : (size_t)pick(1, 4));
        split_scratch_given(room ? reinterpret_cast<void*>(uintptr_t(256)) : nullptr, room, true);
        split_scratch_select(nullptr);
        const Plan pl = plan_pairs<G>(p, G::POOL);
        const size_t ws = usable_workspace(p, G::POOL);
        split_scratch_given(nullptr, 0, false);
        EXPECT(plan_geom<G>(p, G::POOL, false).cost < 0.0, "%s: pairs only", name);
        if (pl.cost < 0.0) continue;
        ++walked;
        const PieceCfg& c = pl.cfg;
        const int prows = G::POOL ? p.PH : p.OH, pcols = G::POOL ? p.PW : p.OW, HP = p.H + p.pad;
        const int pitch = (G::POOL ? (c.TW - 1) * p.ps + 1 : c.TW - 1) * p.stride + 3;
        HOLDS(pl.src == SRC_PAIRS && pl.ntail == 0 && c.tail == 0 && c.whole == c.ntiles * c.strips * c.kblocks * p.G);
        HOLDS(c.px <= G::PXMAX && pl.lds_bytes >= 3 * (size_t)G::PAIR_BUF && pl.lds_bytes <= 160 * 1024 && pl.piece_bytes <= ws);
        HOLDS((size_t)2 * (2 * c.cgb + G::SPARE) <= pl.lds_bytes && c.px * 48 <= c.cgb);   // what goes on from pieces
        const size_t fragments = (size_t)p.G * c.kb32 * c.nch * 9;
        HOLDS(pl.piece_bytes == pair_bytes(p.G, c.kb32, c.nch) + (pl.rest == SRC_PIECES ? fragments * 3072 : 0));
        HOLDS(c.kb32 * 32 >= c.kblocks * 128 && (!p.wprep || c.kb32 == (p.Kg + 127) / 128 * 4) && c.nch * 16 >= p.Cg && (c.nch - 1) * 16 < p.Cg);
        ++rests[pl.rest];
        std::vector<unsigned char> seen((size_t)p.N * prows * pcols, 0);
        for (int tile = 0; tile < c.ntiles; ++tile)
            for (int strip = 0; strip < c.strips; ++strip) {
                int r0 = 0;
                for (int i = 0; i < 128 && tile * 128 + i < c.nrun; ++i) {
                    const int P = tile * 128 + i, pp = G::POOL ? P >> 2 : P, q = pp / c.TW, n = q / prows, row = q - n * prows, wcol = pp - q * c.TW;
                    const int oh = G::POOL ? row * p.ps + ((P & 3) >> 1) : row, ow = G::POOL ? wcol * p.ps + (P & 1) : wcol;
                    if (i == 0) r0 = n * HP + oh * p.stride;
                    const int first = (n * HP + oh * p.stride - r0) * pitch + ow * p.stride, last = first + 2 * pitch + 2;
                    HOLDS(first >= 0 && last < c.px);
                    if (n < p.N && wcol + strip * c.TW < pcols) ++seen[((size_t)n * prows + row) * pcols + wcol + strip * c.TW];
                }
            }
        for (size_t i = 0; i < seen.size(); ++i)
            if (seen[i] != (G::POOL ? 4 : 1)) {
                HOLDS(false);
                break;
            }
    }
    EXPECT(walked >= 60 && rests[SRC_PIECES] >= 5 && rests[SRC_RAW] >= 3 && rests[SRC_FP32] >= 5, "%s: %d plans, pieces %d, stored %d, prepared %d", name, walked,
           rests[SRC_PIECES], rests[SRC_RAW], rests[SRC_FP32]);
}

// Division by multiplication: every divisor's multiples and their neighbours below 2^31, and some numbers between.
static void divisions()
{
    const int most = 0x7fffffff;
    for (int i = 0; i < 4000; ++i) {
        const int d = i < 1000 ? i + 1 : pick_log(1, most - 1.0);
        FastDiv by;
        by.by(d);
        for (int j = 0; j < 50; ++j) {
            const int n = j < 20 ? pick_log(1, most - 1.0) - 1 : (int)((long long)d * pick(0, most / d - 1)) + d - j % 2;
            EXPECT(by.of(n) == n / d, "%d / %d", n, d);
        }
        const int top = most / d * d;
        EXPECT(by.of(most) == most / d && by.of(top) == most / d && by.of(top - 1) == (top - 1) / d && by.of(0) == 0, "%d", d);
    }
    FastDiv by;
    by.by(63);
    EXPECT(by.of(1108378718) == 1108378718 / 63, "17593312 and 62 / 63");
}

// Padded rows of the whole batch are numbered in 32 bits: layers with more are not the piece kernels'.
static void rows_are_numbered()
{
    for (int N : {(1 << 29), 715827000, 715828000, (1 << 30) - 1}) {
        const sconv_desc_t d = {N, 1, 1, 1, 1, 3, 3, 3, 2, 1, 0, 0, 0, 0};   // one result of three padded rows an image
        Problem p;
        EXPECT(fill_problem(&d, false, &p) == SCONV_OK && p.OH == 1 && p.OW == 1, "%d images", N);
        const bool numbered = (long long)N * (p.H + p.pad) + 4096 < (1LL << 31);   // (a tile starts at one and stages fewer than 4096 more)
        EXPECT(shape_ok(p, false) == numbered, "%d images", N);
    }
}

int main()
{
    divisions();
    rows_are_numbered();
    strips_are_the_best_of_all(4000);
    plans_are_kept();
#define WALK_PIECE(NAME, ...)                          \
    raw_reads<PGeom<__VA_ARGS__>>(NAME);               \
    plans<PGeom<__VA_ARGS__>>(NAME, plan_geom<PGeom<__VA_ARGS__>>, PGeom<__VA_ARGS__>::CS, PGeom<__VA_ARGS__>::PXMAX, \
                              2 * PGeom<__VA_ARGS__>::SPARE, 2);                        \
    pair_plans<PGeom<__VA_ARGS__>>(NAME "/pairs");
#define WALK_TAPS(NAME, ...) \
    plans<TGeom<__VA_ARGS__>>(NAME, plan_taps<TGeom<__VA_ARGS__>>, TGeom<__VA_ARGS__>::CS, TGeom<__VA_ARGS__>::PXMAX, TGeom<__VA_ARGS__>::FB, 1);
    PIECE_GEOMETRIES(WALK_PIECE, WALK_TAPS)
#define WALK_BLOCK(NAME, ...) block_plans<PGeom<__VA_ARGS__>>(NAME);
    PIECE_BLOCKS(WALK_BLOCK)
    if (failures) {
        fprintf(stderr, "%d expectation(s) failed\n", failures);
        return 1;
    }
    printf("ok\n");
    return 0;
}

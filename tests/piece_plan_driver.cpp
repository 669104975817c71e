// The piece kernels' planner and index arithmetic, walked on the CPU under AddressSanitizer + UndefinedBehaviorSanitizer (built and
// run by tests/test_host_sanitizers.py: the host side of sconv_piece.hip with everything else of the library, no device code, no GPU).
// Prints "ok" and exits 0 when every expectation holds.
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

int main()
{
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

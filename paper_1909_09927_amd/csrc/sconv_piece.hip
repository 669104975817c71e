// Matrix kernels on exact bf16 pieces: 1x1, 3x3, 5x5 and 7x7 kernels, any grouping, optional pooling over 2x2 windows, of any stride and
// padding as far as the input positions of a tile fit its staging (stage_positions): strided 3x3 on ordinary maps, strided 1x1, 5x5 and
// 7x7, and strided or pooled 1x1 of widths that do not fill whole rows, only on small ones.
//
// What bounds the other matrix kernels on the large layers is the fp32 matrix rate (157 TFLOP/s on paper, 138 measured on a
// large product).  The bf16 matrix pipe is sixteen times as fast, and an fp32 value is the exact sum of three bf16 values
// (24 bits = 3 x 8): x = x0 + x1 + x2, every remainder of the rounding being exact.  Of the nine products of two such sums
// the six largest are issued - x0w0, x0w1, x1w0, x1w1, x0w2, x2w0 -, the other three are below 2^-24 of the product,
// i.e. below one fp32 rounding of it.  Products of pieces are exact and every instruction adds 16 of them to an fp32
// accumulator, which rounds six times per sixteen terms where an fp32 chain rounds sixteen times.  The sums of one staged
// chunk start from zero and are added to the running sums at its end (16 additions per accumulator and 54 matrix
// instructions), so that the roundings of a chunk happen at the size of its own partial sum.  Where registers allow (PGeom::apart)
// only x0w0 goes there, and the five small products have running sums of their own, whose roundings are 2^-8 of those: one rounding per sixteen
// terms is left.  Measured against 64-bit sums, relative, 512 channels of 3x3 at 50 / 70 / 85 % zeros: 0.87e-7 / 0.80e-7 / 0.72e-7 with sums
// apart, 1.86e-7 / 1.79e-7 / 1.60e-7 without; tap3x3 1.62e-7 / 1.33e-7 / 1.05e-7, quad3x3 2.24e-7 / 1.81e-7 / 1.40e-7, wide3x3 4.25e-7 /
// 3.30e-7 / 2.35e-7.  The third set of accumulators takes a third workgroup off a compute unit: no loss where LDS or filters cut on the way
// leave two anyway (128 -> 128 3x3 stride 2 @56x56 at batch 32 62.4 -> 55.8 us, 512 @28x28 at batch 8 with prepared filters 161 -> 159,
// 1x1 512 -> 256 @28x28 at batch 16 32.9 -> 32.0), nothing either with loads in their places (SPREAD), which leave two: 256 @56x56 150 (a128x64)
// and 151 (b64x128) at batch 8.
// The splitting is the one of G. Henry, P. T. P. Tang, A. Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For
// Higher-Precision Computations" (ARITH 2019).
// Both operands are multiplied by 2^24 before they are cut: the last bit of the smallest fp32 subnormal, 2^-149, becomes 2^-125,
// so every piece of every value is a normal bf16 number or zero, and the products that fall below fp32's range are those below
// 2^-174 - far under an fp32 sum's own smallest step.  The sums are multiplied by 2^-48 at the end.  What is left out of range is
// too large - elements of 2^104 and more, sums of 2^80 and more, Inf, NaN - and shows in the result as Inf or NaN (an element
// that becomes Inf leaves remainders of -Inf or NaN, which no other operand turns back into a finite sum): a lane that finds
// such a sum has its block of 32 x 32 results summed again in plain fp32, skipping zero elements.
//
// Where it is no further from 64-bit sums than what runs otherwise, a 3x3 launch with a workspace takes fp16 pairs and three products
// instead (pair_sums, pairs_for).
//
// Zeros are not skipped inside a tile (a 32-window block of 16 channels is never empty when zeros are independent): the
// rules that choose between this kernel and the element-skipping vector kernel are in sconv_api.hip (piece_first).
//
// A workgroup computes BM filters x BN windows.  The windows of a column strip (TW output columns) are numbered in format
// order - (n, oh, ow), or (n, ph, pw, py, px) for the fused call, so that a pooling window is four neighbouring lanes -
// and a tile is BN consecutive ones; the input rows they touch are staged once per chunk of 16 channels as pieces,
// [channel group of 8][position][piece][8 channels], double buffered, and all taps read the same staged tile: a tap is an
// offset.  Every lane reads its own window's address, so tiles fit any map, stride and padding; the padding is staged as
// zeros.  Filters: a lane's fragment is 8 channels of one filter and tap, straight from memory into registers, one to three
// taps ahead (no LDS, no barrier): from pieces that a kernel writes into the workspace first, from prepared filters, or
// from the filters as stored.  MT = 1, NT = 4 gives an instruction stream of 216 matrix instructions to 108 LDS reads and
// 27 loads per chunk; two workgroups a compute unit keep the matrix pipe busy 67 % of the time at 1.9 GHz, 220 - 240 TFLOP/s
// dense-equivalent on 512 channels @28x28 at batch 62 (quad3x3: 120).  Two are what all geometries have a compute unit but those that cut stored
// filters.
//
// Tiles that do not fill a last round of workgroups are split along the channels (split tiles: partial sums into the
// workspace, piece_sum_kernel adds them): the 784 tiles of 256 @56x56 at batch 8 run as 768 whole ones, three to a compute unit, and 16 in 16
// slices each (six products: 153 us against 189 with all of them whole).
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "sconv_internal.h"
#include "sconv_piece_split.h"

namespace sconv {

namespace {


typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));

// Division by a number that is known before the launch, of numbers below 2^31: with 2^l >= d > 2^(l-1) (l >= 1) and m = ceil(2^(31+l) / d), m is below 2^32
// and m d exceeds 2^(31+l) by less than 2^l, so n m / 2^(31+l) exceeds n / d by less than 1 / d.  A wavefront issues an instruction every eight clocks, and a division by a
// register's value is some 35 of them: with the dozen that place a workgroup's tile and the dozen that place its results, and results stored one by one
// behind their conditions and biases (18 000 clocks, now 5 000), a launch of one chunk took 17 us, now 10.
struct FastDiv {
    unsigned m, s;       // (m == 0: by one)
    void by(int d)
    {
        unsigned l = 1;
        while ((1u << l) < (unsigned)d) ++l;
        s = l - 1;
        m = d == 1 ? 0 : (unsigned)(((1ull << (31 + l)) + d - 1) / d);
    }
    __host__ __device__ __forceinline__ int of(int n) const
    {
        const unsigned q = (unsigned)(((unsigned long long)(unsigned)n * m) >> 32) >> s;
        return m ? (int)q : n;
    }
};

struct PieceCfg {
    int nrun;        // window rows of one column strip: N*OH*TW, or N*PH*TW*4 in PECR order
    int ntiles;      // tiles of BN window rows per strip
    int TW, strips;  // (pooled) output columns of a strip, strips
    int kblocks;     // filter blocks of BM filters per group
    int kb32;        // 32-filter blocks per group in the prepared layout
    int nch;         // staged chunks of 16*CS channels
    int whole;       // tiles run by one workgroup; the others, `tail` of them, are split along the channels over nss workgroups each
    int nss;
    int tail;
    int T, S;        // taps, kernel width
    int px, cgb;     // staged positions, bytes of one 8-channel group
    int flat;        // 1x1 / stride 1: a map is one row of H*W positions
    FastDiv by_kblocks, by_strips, by_ntiles, by_TW, by_rows, by_pitch, by_HP, by_quads;   // rows of (pooled) results of an image; quads of a tile's row
    void prepare(const Problem& p, bool pooled, int BN)
    {
        by_quads.by(BN / 4);
        by_kblocks.by(kblocks);
        by_strips.by(strips);
        by_ntiles.by(ntiles);
        by_TW.by(TW);
        by_rows.by(pooled ? p.PH : flat ? 1 : p.OH);
        by_pitch.by((pooled ? (TW - 1) * p.ps + 1 : TW - 1) * p.stride + p.S);
        by_HP.by((flat ? 1 : p.H) + p.pad);
    }
};

// Filters: cut into three pieces in the workspace; as prepared by the caller; as stored; cut into pairs in the workspace (pair_sums)
enum { SRC_PIECES = 0, SRC_FP32 = 1, SRC_RAW = 2, SRC_PAIRS = 3 };

template <int V>
struct Const {
    static constexpr int value = V;
};

constexpr int kUnpaired = -0x40000000;   // in the place of a filter's exponent: no pairs of it

// Whether a scaled sum is Inf or NaN.
__device__ __forceinline__ bool not_finite(float r) { return (__builtin_bit_cast(unsigned, r) & 0x7fffffffu) >= 0x7f800000u; }

// Filters read as stored: a lane's reads are at raw_base (its filter's row, its half of a fragment's 16 channels) plus raw_step,
// bytes from the block's first filter, all of it in the vector offset, which the buffer's bounds check covers (a scalar offset it
// may not).  Past the row's last channel lies the next filter, or the tensor's end, from where on reads give zero: either is
// multiplied by zeros of the map.  No read straddles the end: a 3x3 channel's taps are read by whole rows of three, a 1x1 filter by four
// channels where that ends inside its row or their number is a multiple of four (raw_wide), else one by one and never past the
// row's last.  (All of a filter of odd length one by one: 250 -> 1024 @14x14 at batch 16 39.9 us, by four up to the last fragment 25.7.)
__host__ __device__ constexpr int raw_base(int row, int L, int T, int half) { return (row * L + half * 8 * T) * 4; }
__host__ __device__ constexpr int raw_step(int ch16, int T, int j, int t) { return (ch16 * 16 * T + t) * 4 + j * T * 4; }
__host__ __device__ constexpr int raw_last(int base, int L, int half) { return base + (L - 1 - half * 8) * 4; }   // 1x1: the row's last channel
// 1x1, a fragment of 16 channels: its first, out of every buffer's range where all of them lie past the row (they read as zeros
// without a trip to memory); whether it is read by four channels
__host__ __device__ constexpr int raw_fragment(int base, int Cg, int ch16) { return ch16 * 16 < Cg ? base + raw_step(ch16, 1, 0, 0) : (int)0x80000000u; }
__host__ __device__ constexpr bool raw_wide(int Cg, int ch16) { return (Cg & 3) == 0 || ch16 * 16 + 16 <= Cg || ch16 * 16 >= Cg; }

template <int MT_, int NT_, int WM_, int WN_, int T_, int CS_, bool POOL_, int XU_, int OCC_, bool APART_>
struct PGeom {
    static constexpr int MT = MT_, NT = NT_, WM = WM_, WN = WN_, T = T_, CS = CS_, XU = XU_, OCC = OCC_;   // XU: staging units per wavefront
    static constexpr bool POOL = POOL_;
    // microseconds a compute unit spends on one staged chunk of one workgroup when two or three workgroups share it (fitted to the
    // launches of the benchmark layers; s128x64 on filters as stored: 512 @28x28 at batch 8 218 us)
    static constexpr double tc(int src, int taps)
    {
        if (src == SRC_PAIRS) return 1.57;
        const double wide = XU > 3 ? 0.12 : 0.0;   // (four staging units: 512 @28x28 at batch 8 158 us against 151 with three or two)
        return (MT * NT * NW == 16 ? (src == SRC_PIECES ? 4.7 : src == SRC_FP32 ? 4.9 : 5.3)
                                   : (src == SRC_PIECES ? 2.48 + wide : src == SRC_FP32 ? 2.7 + wide : APART_ && T_ == 9 ? 3.45 : 3.7) * (MT * NT * NW) / 8.0) *
               (T_ == 1 ? 0.5 : taps / 9.0);
    }
    static constexpr int NW = WM * WN, BM = 32 * MT * WM, BN = 32 * NT * WN;
    static constexpr int CG = 2 * CS;    // 8-channel groups per staged chunk
    static_assert(XU * NW % CG == 0, "every 8-channel group has the same number of staging units");
    static constexpr int PXMAX = XU * NW / CG * 64;   // staged positions
    static constexpr int AR = T == 9 ? 3 : 4;   // filter fragments in flight (ring)
    static constexpr int SPARE = 1280;          // bytes of a chunk's LDS that lanes without a position write to (64 * 16 + 32)
    static constexpr int VW = T == 9 ? 3 : 1;    // taps fetched at once from filters as stored
    // sums of their own for the five small products (see the top)
    static constexpr bool apart(int src) { return APART_ || (NT == 2 && (src == SRC_FP32 || src == SRC_PAIRS)); }
    // two tiles of 128 filters x 64 windows side by side, eight wavefronts, one workgroup a compute unit: see pair_sums
    static constexpr bool BLOCK = T == 9 && NW == 8;
    static constexpr const char* tiles = !BLOCK ? nullptr : POOL ? "u128x64" : "a128x64";
    static constexpr bool PAIRS = T == 9 && MT == 1 && NT == 2 && WM == 4 && XU * WN == 2 && APART_ == POOL;   // has the form with pairs (a128x64, u128x64, the blocks)
    // one chain on filters as stored: 168 registers, three wavefronts a SIMD (896 channels in 7 groups @14x14 at batch 32 92.0 -> 89.8 us)
    static constexpr bool three(int src, int form) { return T == 9 && src == SRC_RAW && form == 0 && XU == 2 && MT * NT * NW == 8 && !apart(src); }
    static constexpr int PAIR_BUF = 2 * 2 * PXMAX * 16 + 256;   // LDS of one chunk as pairs, and a third of flags, ranges (from 64) and exponents (the last 512 bytes)
};

// Two fp32 values times up as pairs of fp16 values: v up = p0 + 2^-12 p1, p0 of 11 bits, p1 of 11 and a sign - all but the last bit of every
// fourth value, 2^-23 of it at most, for |v up| from 2^-14 (p1 down to 2^-24) to 2^15 (p1 up to 2^15).  (Multiplication or subtraction and
// rounding to fp16 in one instruction each; up2 = 2^12 up.)
__device__ __forceinline__ void pair2(float a, float b, float up_a, float up2_a, float up_b, float up2_b, int i, u4 (&out)[2])
{
    unsigned h, r;
    const float a2 = a * up2_a, b2 = b * up2_b;
    asm("v_fma_mixlo_f16 %0, %1, %2, 0 op_sel_hi:[0,0,0]" : "=v"(h) : "v"(a), "s"(up_a));
    asm("v_fma_mixhi_f16 %0, %1, %2, 0 op_sel_hi:[0,0,0]" : "+v"(h) : "v"(b), "s"(up_b));
    asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(h), "s"(-4096.0f), "v"(a2));
    asm("v_fma_mixhi_f16 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(r) : "v"(h), "s"(-4096.0f), "v"(b2));
    out[0][i] = h;
    out[1][i] = r;
}

__device__ __forceinline__ unsigned wave_max(unsigned v)
{
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));   // row_shr 1, 2, 4, 8
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));   // row_bcast 15, 31
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// The magnitudes of some values: the largest, and the smallest but zero as 2 * bits - 1 (2^32 - 1: all are zeros).
struct Range {
    float hi = 0.0f;
    unsigned lo = 0xffffffffu;
    __device__ __forceinline__ void add(float a, float b)
    {
        asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(hi) : "v"(a), "v"(b));   // (fmaxf quiets its operands first)
        lo = min(lo, min((__builtin_bit_cast(unsigned, a) << 1) - 1, (__builtin_bit_cast(unsigned, b) << 1) - 1));
    }
    __device__ __forceinline__ uint2 of_wave() const { return make_uint2(wave_max(__builtin_bit_cast(unsigned, hi)), ~wave_max(~lo)); }
};

// The exponent sigma of the power of two that takes the largest of a set of magnitudes to 2^13 .. 2^14 (115 at most, so that 2^12 times it
// is finite).
__host__ __device__ inline int pair_exponent(unsigned hi_bits)
{
    const int e = hi_bits ? (int)(hi_bits >> 23) : 127;   // (all zeros: as good as any)
    const int sg = 140 - (e > 254 ? 254 : e);
    return sg < 115 ? sg : 115;
}
// What pairs at that scale hold: magnitudes below `hi` (bits; 2^15 after scaling), and but for zeros none below `lo` (as in Range): 2^-14 after
// scaling, under which p0 has fewer than 11 bits and the product left out weighs more than 2^-22.
struct PairLimits {
    unsigned hi, lo;
    __host__ __device__ explicit PairLimits(int sigma)
    {
        const int el = 113 - sigma;     // biased exponent of the smallest
        hi = (unsigned)(142 - sigma) << 23;
        if (hi > 0x7f800000u) hi = 0x7f800000u;
        lo = ((unsigned)(el > 0 ? el : 1) << 24) - 1;   // (nor fp32's subnormals)
    }
    __host__ __device__ bool hold(unsigned hi_bits, unsigned lo_key) const { return hi_bits < hi && lo_key >= lo; }
};
__host__ __device__ inline float power_of_two(int e) { return __builtin_bit_cast(float, (unsigned)(e + 127) << 23); }

// The sums of one tile from fp16 pairs: v = p0 + 2^-12 p1, three products p0q0, p0q1, p1q0 (the fourth is 2^-22 of the product at most) instead of
// six, two thirds of the LDS and filter traffic.  Bound by the chip's power where every unit has work (1.6 - 1.9 GHz), otherwise by what a wavefront
// issues between two matrix instructions: one instruction every eight clocks, so two wavefronts a SIMD have about seven each for the 32 clocks of one.
// Hence six a product instead of nine: the compensation carried in the sums (below), an element cut in three instructions with no wait between them,
// a flag that is written only when a scale has to move, one wait for the loads of a unit, two chunks a turn of the loop (no moves at its end).  And what
// a product needs is asked for two taps ahead (p0) and one (p1), across the chunk's end too: a chunk has one barrier, six taps before the next one's
// first staging, and three buffers, so that nobody waits in it for what was just asked for.  512 @28x28 at batch 62: 688 -> 618 us.
// Blocks (PGeom::BLOCK, 128 filters x 128 windows, eight wavefronts) read the filters once for two wavefronts - on different SIMDs, side by side: the
// second finds them in the L1 (L2 reads 9.3 -> 5.1 million at batch 8; on the same SIMD they drift apart and it does not) - and stage a quarter less of the map:
// 568 us, 1.21 PFLOP/s of fp16 products at 1.7 GHz, a matrix instruction of 32 clocks every 48 (profiles/piece_counters.txt).
// Measured and dropped: 64 x 64 a wavefront, one to a SIMD (667 us: half of what fits a matrix instruction's time can be issued there), wavefront priorities by progress (level).
// The map's pairs are scaled by a power of two, 2^sigma, that stays while the chunks' elements fit it (Range of what the workgroup
// stages, one chunk ahead), the filters' by one per filter.  Where a chunk holds a nonzero element 2^27 below its largest, or a filter such a
// weight - about one of 4 x 10^7 normally distributed values -, the tile is summed from three pieces from there on: returned is the first chunk that
// is not in the sums, `sigma` is their scale.  So every single product is within 2^-21 of its value, whatever the others in its window.  No map
// and no filters take much longer than on pieces alone.
// The sums of nine taps (p0q0) are added to the running ones once a chunk, those of the second block of windows four taps after the first's; the rounding error of
// that addition stays where the next nine taps start (error at 512 channels 1.5e-7 without, 1.07e-7 with it).  The small products' sums run through, 2^12 times their size.
// Filters: a ring of nine fragments, eight taps ahead (six with two staging units, for their registers).
template <class G, class Fetch, class Exponents, class Paired>
__device__ __forceinline__ int pair_sums(const Problem& p, const int (&pos)[G::NT], int pitch, int chb, int che, int wave, int lane,
                                         unsigned char* lds, Fetch fetch_x, __amdgpu_buffer_rsrc_t wres, Exponents fetch_exponents, Paired paired,
                                         v16f (&acc)[1][G::NT], int& sigma)
{
    constexpr int NT = G::NT, XU = G::XU, NW = G::NW, D = XU == 2 ? 6 : 8;   // (taps of filters ahead: the second staging unit's registers)
    constexpr int PLANE = G::PXMAX * 16, CGB = 2 * PLANE, BUF = 2 * CGB;
    static_assert(G::T == 9 && G::MT == 1 && NT == 2 && XU * NW == 8 && G::CS == 1, "3x3, one block of filters by two of windows");
    const int half = lane >> 5;
    int lb[NT], xst[XU];
#pragma unroll
    for (int nb = 0; nb < NT; ++nb) lb[nb] = pos[nb] * 16 + half * CGB;
#pragma unroll
    for (int u = 0; u < XU; ++u) xst[u] = wave % 2 * CGB + ((u * NW + wave) / 2 * 64 + lane) * 16;   // (all units of a wavefront are of one channel group)

    float xr[XU][8];
    u4 ap[9][2];
    auto fetch_a = [&](int ch, int t, int q) {
        ap[t][q] = __builtin_bit_cast(u4, __builtin_amdgcn_raw_buffer_load_b128(wres, lane * 16 + q * 1024, (ch * 9 + t) * 2048, 0));
    };
    // The scale.  In the rule every wavefront finds its share of the next chunk within the limits of the scale there is.  Where one does not, it
    // says so (a word for every other chunk), and all exchange their ranges: a scale that holds the chunk, or none (false).
    PairLimits lim(0);
    Range rg;
    auto flag = [&](int parity) -> unsigned& { return *reinterpret_cast<unsigned*>(lds + 3 * BUF + parity * 4); };
    auto say = [&](int parity) {
        if (__ballot(__builtin_bit_cast(unsigned, rg.hi) >= lim.hi) | __ballot(rg.lo < lim.lo)) flag(parity) = 1;
        rg = Range();
    };
    auto new_scale = [&](int& to, bool begin = false) {
        Range all;
#pragma unroll
        for (int u = 0; u < XU; ++u)
#pragma unroll
            for (int j = 0; j < 8; j += 2) all.add(xr[u][j], xr[u][j + 1]);
        const uint2 of = all.of_wave();
        if (lane == 0) *reinterpret_cast<uint2*>(lds + 3 * BUF + 64 + wave * 8) = of;
        if (begin && wave == 0) flag(0) = flag(1) = 0;
        __syncthreads();
        const u4* s = reinterpret_cast<const u4*>(lds + 3 * BUF + 64);
        unsigned h = 0, l = 0xffffffffu;
#pragma unroll
        for (int i = 0; i < NW / 2; ++i) {
            h = max(h, max(s[i][0], s[i][2]));
            l = min(l, min(s[i][1], s[i][3]));
        }
        const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)h), lo = (unsigned)__builtin_amdgcn_readfirstlane((int)l);
        to = pair_exponent(hi);
        lim = PairLimits(to);
        return lim.hold(hi, lo);
    };
    // Staging of one unit in nine parts: its channels cut two by two (p0 of a pair beside p1 of the one before, which waits for its p0), written,
    // and those of the chunk after the next fetched two by two.  up: 2^sigma
    u4 xf[2];
    float a2, b2;
    auto second = [&](int i) {
        asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(xf[1][i]) : "v"(xf[0][i]), "s"(-4096.0f), "v"(a2));
        asm("v_fma_mixhi_f16 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(xf[1][i]) : "v"(xf[0][i]), "s"(-4096.0f), "v"(b2));
    };
    auto stage = [&](int u, int part, unsigned char* buf, int after, float up, float up2) {
        if (part < 4) {
            const float a = xr[u][2 * part], b = xr[u][2 * part + 1];
            unsigned h;
            asm("v_fma_mixlo_f16 %0, %1, %2, 0 op_sel_hi:[0,0,0]" : "=v"(h) : "v"(a), "s"(up));
            if (part) second(part - 1);
            asm("v_fma_mixhi_f16 %0, %1, %2, 0 op_sel_hi:[0,0,0]" : "+v"(h) : "v"(b), "s"(up));
            xf[0][part] = h;
            a2 = a * up2;
            b2 = b * up2;
        } else if (part == 4) {
            second(3);
            *reinterpret_cast<u4*>(buf + xst[u]) = xf[0];
            *reinterpret_cast<u4*>(buf + xst[u] + PLANE) = xf[1];
        } else {
            fetch_x(xr[u], u, after, (8 - part) * 2, 2);   // (the first pair comes last: one wait for all)
        }
    };
    // channels past the group's last one count as zeros
    auto clear = [&](int ch) {
        const int left = p.Cg - (ch * 16 + wave % 2 * 8);
#pragma unroll
        for (int u = 0; u < XU; ++u)
#pragma unroll
            for (int j = 0; j < 8; ++j) xr[u][j] = left > j ? xr[u][j] : 0.0f;
    };

    const v16f zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    v16f tmp[NT], accl[NT];
    float run[NT][16];
#pragma unroll
    for (int nb = 0; nb < NT; ++nb) {
        tmp[nb] = accl[nb] = zero;
#pragma unroll
        for (int v = 0; v < 16; ++v) run[nb][v] = 0.0f;
    }
    u4 b0[3][NT], b1[2][NT];             // windows: p0 two taps ahead, p1 one
    auto load_b = [&](const unsigned char* buf, int e, int n, int q) {
        (q ? b1[e & 1][n] : b0[e % 3][n]) = *reinterpret_cast<const u4*>(buf + e / 3 * pitch * 16 + lb[n] + e % 3 * 16 + q * PLANE);
    };
    // p0q0 first and last in turn: between the last product of a block before its sums are folded and the first one after lie eight others
    constexpr int NM = 3 * NT;               // matrix instructions of a tap
    auto product = [&](int e, int m) {
        const int c = (m / NT + e % 2) % 3, n = m % NT;      // p0q0, p1q0, p0q1
        v16f& d = c ? accl[n] : tmp[n];
        d = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, ap[e][c == 1 ? 1 : 0]), __builtin_bit_cast(h8, c == 2 ? b1[e & 1][n] : b0[e % 3][n]),
                                                   d, 0, 0, 0);
    };

    // (both chunks of the map that are needed before the first product, and the filters, are asked for before any is waited for)
    float xs[XU][8];
    const int nx1 = min(chb + 1, che - 1);
#pragma unroll
    for (int u = 0; u < XU; ++u) fetch_x(xr[u], u, chb, 0, 8);
    fetch_exponents();
#pragma unroll
    for (int u = 0; u < XU; ++u) fetch_x(xs[u], u, nx1, 0, 8);
#pragma unroll
    for (int t = 0; t < D; ++t) {
        fetch_a(chb, t, 1);
        fetch_a(chb, t, 0);
    }
    if (!paired() || !new_scale(sigma, true)) return chb;
    const int first = sigma;             // (the running sums follow the scale: from 2^60 off the first one on their bits would not fit fp32's range)
    if ((chb + 1) * 16 > p.Cg) clear(chb);
#pragma unroll
    for (int u = 0; u < XU; ++u)
#pragma unroll
        for (int part = 0; part < 5; ++part) stage(u, part, lds, nx1, power_of_two(sigma), power_of_two(sigma + 12));
#pragma unroll
    for (int u = 0; u < XU; ++u)
#pragma unroll
        for (int j = 0; j < 8; j += 2) {
            xr[u][j] = xs[u][j];
            xr[u][j + 1] = xs[u][j + 1];
            rg.add(xr[u][j], xr[u][j + 1]);
        }
    say(1);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int n = 0; n < NT; ++n) load_b(lds, e, n, 0);
    unsigned said = flag(1);             // (asked for behind a barrier, needed two taps later)

    float by = 1.0f;                     // the step from the running sums' scale to that of the others
    // Some of a block's sums to the running ones; what the addition lost is where the next sums start
    auto fold = [&](int n, int from, int to) {
#pragma unroll
        for (int v = from; v < to; ++v) {
            const float t = tmp[n][v], a = run[n][v], sum = __builtin_fmaf(a, by, t);
            run[n][v] = sum;
            tmp[n][v] = t - __builtin_fmaf(a, -by, sum);
        }
    };
    int end = che, at = 0;
    auto chunk = [&](int ch, auto parity) {
        constexpr int par = decltype(parity)::value;
        const int nx = min(ch + 1, che - 1), nx2 = min(ch + 2, che - 1), to = at == 2 * BUF ? 0 : at + BUF;
        const unsigned char* buf = lds + at;
        unsigned char* nbuf = lds + to;
        at = to;
        int next = sigma;
        if (__builtin_amdgcn_readfirstlane((int)said)) {
            if (!new_scale(next) || next > first + 60 || next < first - 60) {
                next = sigma;
                end = ch + 1;            // (what is staged of the next chunk is not read)
            }
            if (wave == 0) flag(par ^ 1) = 0;   // (all have read it: there is a barrier in new_scale)
        }
        if ((nx + 1) * 16 > p.Cg) clear(nx);
        const float up = power_of_two(next), up2 = power_of_two(next + 12);
#pragma unroll
        for (int e = 0; e < 9; ++e) {
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                product(e, m);
                __builtin_amdgcn_sched_barrier(0);
                // windows; those of the next chunk behind the barrier
                if (e == 0 && m < 2) load_b(buf, 0, m, 1);
                if (e == 0 && m >= 4) load_b(buf, 1, m - 4, 1);
                if (e > 0 && e < 8 && m < 2) load_b(buf, e + 1, m, 1);
                if (m >= 2 && m < 4) load_b(e < 7 ? buf : nbuf, (e + 2) % 9, m - 2, 0);
                if (m >= 4) fetch_a(e + D < 9 ? ch : nx, (e + D) % 9, (e + D) % 9 % 2 ? m - 4 : 5 - m);
                // the next chunk
                const int item = e * NM + m - 2;
                if (item >= 0 && item < 9 * XU) stage(item / 9, item % 9, nbuf, nx2, up, up2);
                if (e == 5 && m >= 6 - 4 * XU) {
                    const int k = XU == 1 ? m - 2 : m;
                    rg.add(xr[k / 4][k % 4 * 2], xr[k / 4][k % 4 * 2 + 1]);
                }
                if (XU == 2 && e == 6 && m < 2) rg.add(xr[XU - 1][m * 2 + 4], xr[XU - 1][m * 2 + 5]);
                if (e == 6 && m == 2) say(par);
                // block 0 between taps 2 and 3, block 1 between 6 and 7
                const int k = (e - 2) % 4 * NM + m - 3;
                if (e >= 2 && k >= 0 && k < 7) fold((e - 2) / 4, k * 16 / 7, (k + 1) * 16 / 7);
                __builtin_amdgcn_sched_barrier(0);
                if (e == 6 && m == NM - 1) {
                    __syncthreads();
                    said = flag(par);
                }
            }
        }
        by = power_of_two(next - sigma);
        if (next != sigma) {
#pragma unroll
            for (int nb = 0; nb < NT; ++nb) {
                accl[nb] *= by;
                tmp[nb] *= by;
            }
            sigma = next;
        }
    };
    // (two chunks a turn: the buffers are known, and the running sums are back in their registers)
    for (int ch = chb;;) {
        chunk(ch, Const<0>());
        if (++ch >= end) break;
        chunk(ch, Const<1>());
        if (++ch >= end) break;
    }
    __syncthreads();
#pragma unroll
    for (int nb = 0; nb < NT; ++nb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[0][nb][v] = run[nb][v] * by + (tmp[nb][v] + accl[nb][v] * 0x1p-12f);
    return end;
}

// Bytes of the pairs of all filters and their exponents; behind them the pieces.
__host__ __device__ inline size_t pair_bytes(int G, int kb32, int nch16) { return ((size_t)G * kb32 * ((size_t)nch16 * 9 * 2048 + 128) + 255) / 256 * 256; }

// FORM: SRC_PAIRS (SRC: the filters' form where pairs do not do), or 0
template <class G, int SRC, int FORM>
__global__ __launch_bounds__(G::NW * 64, G::three(SRC, FORM) ? 3 : G::OCC) void piece_kernel(Problem p, PieceCfg cfg, const float* __restrict__ x,
                                                              const float* __restrict__ w, const void* __restrict__ wp,
                                                              float* __restrict__ parts, float* __restrict__ y)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int MT = G::MT, NT = G::NT, CS = G::CS, CG = G::CG, NW = G::NW, XU = G::XU, AR = G::AR;
    const int PX = cfg.px, CGB = cfg.cgb;
    constexpr int T = G::T, S = T == 9 ? 3 : 1;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // (eight wavefronts: those that read the same filters are on different SIMDs and run side by side, so that the second finds them in the L1)
    const int wm = G::NW == 8 ? wave / G::WN : wave % G::WM, wn = G::NW == 8 ? wave % G::WN : wave / G::WM;

    // workgroup -> tiles and chunks of them; ids are dealt to the eight XCDs in turn, every XCD gets a contiguous range
    const int whole = cfg.whole, nb_all = gridDim.x;
    const bool split = (int)blockIdx.x >= whole;
    int first = split ? blockIdx.x - whole : blockIdx.x;
    {
        const int cnt = split ? nb_all - whole : whole;
        const int n8 = cnt >> 3, rem = cnt & 7, xcd = first & 7, i = first >> 3;
        first = xcd * n8 + min(xcd, rem) + i;
    }

    const int ss = split ? first / cfg.tail : 0, b = split ? whole + first - ss * cfg.tail : first;
    float* const part = split ? parts + (size_t)first * (G::BM * G::BN) : nullptr;   // where a split tile's sums go
    const int chb = split ? cfg.nch * ss / cfg.nss : 0, che = split ? cfg.nch * (ss + 1) / cfg.nss : cfg.nch;
    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
    int kb, strip, tile, g;
    if (G::BLOCK) {                      // (an XCD's workgroups share the filters of few blocks)
        const int b1 = cfg.by_strips.of(b), b2 = cfg.by_ntiles.of(b1);
        strip = b - b1 * cfg.strips;
        tile = b1 - b2 * cfg.ntiles;
        g = cfg.by_kblocks.of(b2);
        kb = b2 - g * cfg.kblocks;
    } else {
        const int b1 = cfg.by_kblocks.of(b), b2 = cfg.by_strips.of(b1);
        kb = b - b1 * cfg.kblocks;
        strip = b1 - b2 * cfg.strips;
        g = cfg.by_ntiles.of(b2);
        tile = b2 - g * cfg.ntiles;
    }

    const int iH = cfg.flat ? 1 : p.H, iW = cfg.flat ? p.H * p.W : p.W;
    const int oH = cfg.flat ? 1 : p.OH, oW = cfg.flat ? p.OH * p.OW : p.OW;
    const int TW = cfg.TW;
    const int HW = p.H * p.W, HP = iH + p.pad;      // images stacked along the rows, padding rows shared
    const int pitch = (G::POOL ? (TW - 1) * p.ps + 1 : TW - 1) * p.stride + S;
    const int pcols = G::POOL ? p.PW : oW, prows = G::POOL ? p.PH : oH;
    const int plane = prows * pcols;                // stored results per image and filter
    // window row P of the strip -> image, row and column of its (pooled) result, the column counted from the strip's first; of its convolution
    auto place = [&](int P, int& n, int& row, int& c) {
        const int pp = G::POOL ? P >> 2 : P, q = cfg.by_TW.of(pp);
        c = pp - q * TW;
        n = cfg.by_rows.of(q);
        row = q - n * prows;
    };
    auto window = [&](int P, int& n, int& oh, int& ow) {
        place(P, n, oh, ow);
        if (G::POOL) {
            oh = p.ps * oh + ((P & 3) >> 1);
            ow = p.ps * ow + (P & 1);
        }
    };
    int n0, oh0, ow0;
    window(tile * G::BN, n0, oh0, ow0);
    const int r0 = n0 * HP + oh0 * p.stride;   // first staged row
    const int w0 = strip * TW * (G::POOL ? p.ps : 1) * p.stride - p.pad;   // input column of the first staged one

    // this lane's windows (one per block of 32) as positions of the staged tile
    int pos[NT];
#pragma unroll
    for (int nb = 0; nb < NT; ++nb) {
        const int P = min(tile * G::BN + (wn * NT + nb) * 32 + col, cfg.nrun - 1);
        int n, oh, ow;
        window(P, n, oh, ow);
        pos[nb] = (n * HP + oh * p.stride - r0) * pitch + ow * p.stride;
    }

    // staging: unit u of this wavefront = 64 positions of one 8-channel group
    unsigned xvo[XU];
    int xst[XU];
#pragma unroll
    for (int u = 0; u < XU; ++u) {
        const int id = u * NW + wave, cgi = id % CG, q = id / CG * 64 + lane;
        const int row = cfg.by_pitch.of(q), cw = q - row * pitch + w0;
        const int sr = r0 + row, n = cfg.by_HP.of(sr), h = sr - n * HP - p.pad;
        const bool ok = q < PX && n < p.N && h >= 0 && h < iH && cw >= 0 && cw < iW;
        xvo[u] = ok ? 4u * (unsigned)((n - n0) * p.C * HW + h * iW + cw) : 0x80000000u;
        xst[u] = q < PX ? cgi * CGB + q * 48 : CG * CGB + lane * 16;   // (lanes past the tile's positions write where nobody reads)
    }
    const float* xb = x + ((size_t)n0 * p.C + (size_t)g * p.Cg) * HW;
    const size_t xleft = ((size_t)p.N * p.C * HW - ((size_t)n0 * p.C + (size_t)g * p.Cg) * HW) * 4;
    const __amdgpu_buffer_rsrc_t xres =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(xb), 0, (int)min(xleft, (size_t)0x7ffffffc), 0x00020000);
    auto fetch_x = [&](float (&to)[8], int u, int ch, int j0 = 0, int n = 8) {
        const int c0 = ch * CS * 16 + (u * NW + wave) % CG * 8;
#pragma unroll
        for (int j = j0; j < j0 + n; ++j)
            to[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xres, (int)xvo[u], min(c0 + j, p.Cg - 1) * HW * 4, 0));
    };
    const int kblk0 = kb * (G::BM / 32) + wm * MT;
    v16f acc[MT][NT];

    int from = chb;                      // the chunks from here on are summed from pieces
    if constexpr (FORM == SRC_PAIRS) {
        const size_t blk = (size_t)cfg.nch * T * 2048;
        // the filters' exponents (kUnpaired: a filter that pairs cannot hold)
        const int* sg = reinterpret_cast<const int*>((const char*)wp + (size_t)p.G * cfg.kb32 * blk) + ((size_t)g * cfg.kb32 + kb * (G::BM / 32)) * 32;
        // (every wavefront looks at all of them, and they wait in LDS for the end)
        int* const sgl = reinterpret_cast<int*>(lds + 3 * G::PAIR_BUF - 512);
        int sgr[G::BM / 64];
        auto fetch_exponents = [&] {
#pragma unroll
            for (int i = 0; i < G::BM / 64; ++i) sgr[i] = sg[i * 64 + lane];
        };
        auto paired = [&] {
            bool all = true;
#pragma unroll
            for (int i = 0; i < G::BM / 64; ++i) {
                all &= !__any(sgr[i] == kUnpaired);
                sgl[i * 64 + lane] = sgr[i];
            }
            return all;
        };
        const __amdgpu_buffer_rsrc_t pres =
            __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)wp + ((size_t)g * cfg.kb32 + kblk0) * blk), 0, 0x7ffffffc, 0x00020000);
        int sigma = 0;
        from = pair_sums<G>(p, pos, pitch, chb, che, wave, lane, lds, fetch_x, pres, fetch_exponents, paired, acc, sigma);
        // To the scale of sums of pieces, by the exponents' sum: map and filters both small (or large) make two factors whose product fp32
        // does not hold, where the sum times both is an ordinary number.
        if (from > chb) {
            const int* e = sgl + wm * 32 + 4 * half;
#pragma unroll
            for (int v = 0; v < 16; ++v)
#pragma unroll
                for (int nb = 0; nb < NT; ++nb) acc[0][nb][v] = __builtin_amdgcn_ldexpf(acc[0][nb][v], 48 - sigma - e[8 * (v >> 2) + (v & 3)]);
            if (from < che) __syncthreads();   // (pieces are staged where the exponents are)
        } else {
            acc[0][0] = acc[0][1] = 0.0f;
            __syncthreads();             // (what pair_sums exchanged in LDS is overwritten)
        }
    }
    const void* const wrest = FORM == 0 ? wp : SRC == SRC_FP32 ? (const void*)p.wprep : (const char*)wp + pair_bytes(p.G, cfg.kb32, cfg.nch);   // (unused as stored)
    if (FORM == 0 || from < che) {
        // staging of one unit in six parts: its channels cut two by two, written, and those of the chunk after the next fetched;
        // channels past the group's last one count as zeros
        float xr[XU][8];
        u4 xf[3];
        int lb[NT];   // windows as byte offsets into the staged tile
#pragma unroll
        for (int nb = 0; nb < NT; ++nb) lb[nb] = pos[nb] * 48 + half * CGB;
        auto stage = [&](int u, int part, unsigned char* buf, int ch, int after) {
            if (part < 4) {
                const int left = p.Cg - (ch * CS * 16 + (u * NW + wave) % CG * 8) - 2 * part;
                split2<G::three(SRC, FORM)>(xr[u][2 * part], xr[u][2 * part + 1], left > 0 ? kUp : 0.0f, left > 1 ? kUp : 0.0f, part, xf);
            } else if (part == 4) {
                u4* d = reinterpret_cast<u4*>(buf + xst[u]);
                d[0] = xf[0];
                d[1] = xf[1];
                d[2] = xf[2];
            } else {
                fetch_x(xr[u], u, after);
            }
        };

        // filters: fragments of 32 filters x 16 channels of one tap
        __amdgpu_buffer_rsrc_t wres;
        int wvo[SRC == SRC_RAW ? MT : 1];
        if (SRC == SRC_PIECES) {
            const size_t blk = (size_t)cfg.nch * CS * T * 3072;
            wres = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)wrest + ((size_t)g * cfg.kb32 + kblk0) * blk), 0, 0x7ffffffc, 0x00020000);
            wvo[0] = lane * 16;
        } else if (SRC == SRC_FP32) {
            const size_t blk = (size_t)p.Cg * T * 256;
            wres = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)wrest + ((size_t)g * (cfg.kb32 >> 1) + (kblk0 >> 1)) * blk), 0, 0x7ffffffc, 0x00020000);
            wvo[0] = half * 8 * T * 256 + (kblk0 & 1) * 128 + col * 4;
        } else {
            // filters as stored; a filter past the group's last one re-reads the last
            const size_t first = ((size_t)g * p.Kg + (size_t)kb * G::BM) * p.L;
            const size_t left = ((size_t)p.K * p.L - first) * 4;
            wres = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(w + first), 0, (int)min(left, (size_t)0x7ffffffc), 0x00020000);
#pragma unroll
            for (int i = 0; i < MT; ++i)
                wvo[i] = raw_base(min((wm * MT + i) * 32 + col, p.Kg - 1 - kb * G::BM), p.L, T, half);
        }
        const int wblk = cfg.nch * CS * T * 3072;       // bytes between 32-filter blocks (pieces)
        const int wblk64 = p.Cg * T * 256;              // bytes between 64-filter blocks (fp32)
        constexpr int VW = G::VW;
        u4 ap[SRC == SRC_PIECES ? AR : 1][SRC == SRC_PIECES ? MT : 1][3];
        float af[SRC == SRC_FP32 ? AR : 1][SRC == SRC_FP32 ? MT : 1][8];
        float ar[SRC == SRC_RAW ? AR : 1][SRC == SRC_RAW ? MT : 1][8][VW];
        auto fetch_a = [&](int slot, int ch16, int t) {
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                if (SRC == SRC_PIECES) {
                    const int so = (ch16 * T + t) * 3072 + i * wblk;
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        ap[slot][i][q] = __builtin_bit_cast(u4, __builtin_amdgcn_raw_buffer_load_b128(wres, wvo[0] + q * 1024, so, 0));
                } else if (SRC == SRC_FP32) {
                    const int so = (ch16 * 16 * T + t) * 256 + (i >> 1) * wblk64;
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        af[slot][i][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wres, wvo[0] + (i & 1) * 128, so + j * T * 256, 0));
                } else if (G::T == 1) {   // eight channels are consecutive
                    const int at = raw_fragment(wvo[i], p.Cg, ch16);
                    if (raw_wide(p.Cg, ch16)) {
                        const f4 lo = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(wres, at, 0, 0));
                        const f4 hi = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(wres, at + 16, 0, 0));
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            ar[slot][i][j][0] = lo[j];
                            ar[slot][i][j + 4][0] = hi[j];
                        }
                    } else {
                        const int last = raw_last(wvo[i], p.L, half);
#pragma unroll
                        for (int j = 0; j < 8; ++j)
                            ar[slot][i][j][0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wres, min(at + 4 * j, last), 0, 0));
                    }
                } else {
                    typedef float f3 __attribute__((ext_vector_type(3)));
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const f3 q = __builtin_bit_cast(f3, __builtin_amdgcn_raw_buffer_load_b96(wres, wvo[i] + raw_step(ch16, T, j, t), 0, 0));
#pragma unroll
                        for (int e = 0; e < 3; ++e) ar[slot][i][j][e % VW] = q[e];
                    }
                }
            }
        };

        constexpr bool APART = G::apart(FORM ? FORM : SRC);
        v16f tmp[MT][NT], accl[APART ? MT : 1][APART ? NT : 1];
        const int bufb = CG * CGB + G::SPARE;
        const v16f zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int nb = 0; nb < NT; ++nb) {
                if (FORM == 0) acc[i][nb] = zero;
                if (APART) accl[APART ? i : 0][APART ? nb : 0] = zero;
            }

        static_assert(NT >= 2, "two independent accumulators at least");
        constexpr int NH = 2;                         // position blocks per half step
        constexpr int HS = NT / NH;                   // half steps per tap
        u4 bq[2][NH][3];
        u4 a[MT][3];
        auto load_b = [&](u4 (&dst)[NH][3], const unsigned char* tapbase, int imm, int h) {
#pragma unroll
            for (int n = 0; n < NH; ++n) {
#pragma unroll
                for (int q = 0; q < 3; ++q) dst[n][q] = *reinterpret_cast<const u4*>(tapbase + lb[h * NH + n] + imm + q * 16);
            }
        };
        auto take_a = [&](int slot, int e) {
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                if (SRC == SRC_PIECES) {
#pragma unroll
                    for (int q = 0; q < 3; ++q) a[i][q] = ap[slot][i][q];
                } else if (SRC == SRC_FP32) {
                    split8(af[slot][i], a[i]);
                } else {
                    float v[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) v[j] = ar[slot][i][j][e];
                    split8<G::three(SRC, FORM)>(v, a[i]);
                }
            }
        };
        // SPREAD: every load, cut and LDS write has its place between two matrix instructions; without the fences the compiler moves the
        // loads down to their uses and waits there (b64x128 197 -> 153 us and s128x64 163 -> 158 on 512 @28x28 at batch 8, 256 @56x56 with a128x64
        // 154 -> 150, 1x1 512 -> 256 @28x28 at batch 16 33.0 -> 31.2).  Not for 3x3 filters as stored, which are cut on the way: fenced, their
        // registers spill (s128x64 107 -> 138 us on 896 channels in 7 groups @14x14).
        constexpr bool SPREAD = SRC != SRC_RAW || G::T == 1;
        // Matrix instruction m of a half step.  One chain: smallest products first (x2 w0, x0 w2, x1 w1, x1 w0, x0 w1, x0 w0); sums apart:
        // x0 w0 first, so that its sums are ready when the others are still issued.
        constexpr int NM = NH * MT * 6;
        auto product = [&](const u4 (&bb)[NH][3], int h, int m, bool first) {
            constexpr int qa[6] = {0, 2, 1, 0, 1, 0}, qb[6] = {2, 0, 1, 1, 0, 0};
            const int c = APART && SPREAD ? (m / (NH * MT) + 5) % 6 : m / (NH * MT), n = m / MT % NH, i = m % MT;
            v16f& d = APART && c < 5 ? accl[APART ? i : 0][APART ? h * NH + n : 0] : tmp[i][h * NH + n];
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, a[i][qa[c]]), __builtin_bit_cast(bf8, bb[n][qb[c]]),
                                                        first && c == (APART ? 5 : 0) ? zero : d, 0, 0, 0);
        };

#pragma unroll
        for (int u = 0; u < XU; ++u) fetch_x(xr[u], u, from);
        fetch_a(0, from * CS, 0);
        if (G::T == 9 && SRC != SRC_RAW) fetch_a(1, from * CS, 1);
        if (G::T == 1) {
            fetch_a(1, from * CS + 1, 0);
            fetch_a(2, from * CS + 2, 0);
        }
#pragma unroll
        for (int u = 0; u < XU; ++u)
#pragma unroll
            for (int part = 0; part < (SPREAD ? 6 : 5); ++part) stage(u, part, lds, from, min(from + 1, che - 1));
        __syncthreads();

        constexpr int E = G::T * CS, D = AR - 1;
        constexpr int ITEMS = XU * 6, GAP = (E * HS - 1) * NM / ITEMS < 4 ? (E * HS - 1) * NM / ITEMS : 4;   // staging: a part every GAP instructions
        static_assert(GAP >= 1, "the staging of a chunk fits its products");
        for (int ch = from; ch < che; ++ch) {
            const unsigned char* buf = lds + ((ch - from) & 1) * bufb;
            unsigned char* nbuf = lds + ((ch + 1 - from) & 1) * bufb;
            const int nx = min(ch + 1, che - 1), nx2 = min(ch + 2, che - 1);
            auto off = [&](int e) { return G::T == 9 ? (e / 3) * pitch * 48 : e * 2 * CGB; };
            auto imm = [&](int e) { return G::T == 9 ? (e % 3) * 48 : 0; };
            auto next_b = [&](int e, int h, int cur) {
                if (h + 1 < HS) load_b(bq[cur ^ 1], buf + off(e), imm(e), h + 1);
                else if (e + 1 < E) load_b(bq[cur ^ 1], buf + off(e + 1), imm(e + 1), 0);
            };
            load_b(bq[0], buf + off(0), imm(0), 0);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                take_a(SRC == SRC_RAW && G::T == 9 ? 0 : e % AR, SRC == SRC_RAW && G::T == 9 ? e % 3 % VW : 0);
                if (!SPREAD) {   // three taps (one kernel row) are fetched at a time
                    if (e % 3 == 2) fetch_a(0, e < 8 ? ch : nx, e < 8 ? e + 1 : 0);
                    if (e == 0 && ch + 1 < che)
#pragma unroll
                        for (int u = 0; u < XU; ++u) fetch_x(xr[u], u, nx);
                }
#pragma unroll
                for (int h = 0; h < HS; ++h) {
                    const int cur = (e * HS + h) & 1;
                    if (!SPREAD) next_b(e, h, cur);
#pragma unroll
                    for (int m = 0; m < NM; ++m) {
                        product(bq[cur], h, m, e == 0);
                        // between the matrix instructions, where the compiler would not put them: what the next ones need
                        if (SPREAD) __builtin_amdgcn_sched_barrier(0);
                        if (SPREAD && m == 0) next_b(e, h, cur);
                        if (SPREAD && m == 1 && h == 0)
                            fetch_a((e + D) % AR, (e + D < E ? ch : nx) * CS + (G::T == 9 ? 0 : (e + D) % E), G::T == 9 ? (e + D) % E : 0);
                        const int at = (e * HS + h) * NM + m - NM;
                        if (SPREAD && at >= 0 && at % GAP == 0 && at / GAP < ITEMS) stage(at / GAP / 6, at / GAP % 6, nbuf, nx, nx2);
                        if (SPREAD) __builtin_amdgcn_sched_barrier(0);
                    }
                }
                if (!SPREAD && e == 6 && ch + 1 < che) {
                    if ((nx + 1) * CS * 16 > p.Cg)   // (once, where `stage` would pick the scale of every channel)
#pragma unroll
                        for (int u = 0; u < XU; ++u)
#pragma unroll
                            for (int j = 0; j < 8; ++j)
                                if (nx * CS * 16 + (u * NW + wave) % CG * 8 + j >= p.Cg) xr[u][j] = 0.0f;
#pragma unroll
                    for (int u = 0; u < XU; ++u) {
                        split8<G::three(SRC, FORM)>(xr[u], xf);
                        stage(u, 4, nbuf, nx, nx2);
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int nb = 0; nb < NT; ++nb) acc[i][nb] += tmp[i][nb];
            __syncthreads();
        }

        if (APART)
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int nb = 0; nb < NT; ++nb) acc[i][nb] += accl[APART ? i : 0][APART ? nb : 0];
    }

    // epilogue
    const int c_lo = chb * CS * 16, c_hi = min(che * CS * 16, p.Cg);
    auto there = [&](int nb, int& P, int& n, int& row, int& wcol) {   // a window's result, and whether there is such a one
        P = tile * G::BN + (wn * NT + nb) * 32 + col;
        place(min(P, cfg.nrun - 1), n, row, wcol);
        wcol += strip * TW;
        return P < cfg.nrun && wcol < pcols;
    };
    // sums out of the pieces' range: x times 0 is NaN where x is Inf or NaN
    float lost = 0.0f;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int nb = 0; nb < NT; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) lost = __builtin_fmaf(acc[i][nb][v], 0.0f, lost);
    const bool again = __any(lost != 0.0f);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int nb = 0; nb < NT; ++nb) {
            unsigned bad = 0;
            if (again)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float r = acc[i][nb][v];   // (a copy: the cast of a vector element reads element 0)
                    bad |= not_finite(r);
                }
            acc[i][nb] *= kDown;
            if (again && __any(bad)) {
                int P, n, oh, ow, row, wcol;
                there(nb, P, n, row, wcol);
                oh = G::POOL ? row * p.ps + ((P & 3) >> 1) : row;
                ow = G::POOL ? wcol * p.ps + (P & 1) : wcol;
                const int k0 = kb * G::BM + (wm * MT + i) * 32 + 4 * half;   // filter of element v: k0 + 8*(v/4) + v%4
                float* sc = reinterpret_cast<float*>(lds) + wave * 1024 + lane;
                for (int v = 0; v < 16; ++v) {
                    const int kk = min(k0 + 8 * (v >> 2) + (v & 3), p.Kg - 1);
                    const float* wk = w + ((size_t)g * p.Kg + kk) * p.L;
                    float s = 0.0f;
                    for (int c = c_lo; c < c_hi; ++c)
                        for (int t = 0; t < T; ++t) {
                            const int ih = oh * p.stride - p.pad + t / S, iw = ow * p.stride - p.pad + t % S;
                            if (ih < 0 || ih >= iH || iw < 0 || iw >= iW) continue;
                            const float e = x[(((size_t)n * p.G + g) * p.Cg + c) * HW + ih * iW + iw];
                            if (e != 0.0f) s = __builtin_fmaf(e, wk[c * T + t], s);
                        }
                    sc[v * 64] = s;
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][nb][v] = sc[v * 64];
            }
        }
    if (part) {
        float* const d = part + (wm * MT * 32 + 4 * half) * G::BN + wn * NT * 32 + col;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int nb = 0; nb < NT; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) d[(i * 32 + 8 * (v >> 2) + (v & 3)) * G::BN + nb * 32] = acc[i][nb][v];
        return;
    }
    // (all biases are on their way before the first is needed)
    float bias[MT][16];
    auto filter = [&](int i, int v) { return kb * G::BM + (wm * MT + i) * 32 + 4 * half + 8 * (v >> 2) + (v & 3); };
    const bool full = (kb + 1) * G::BM <= p.Kg;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) bias[i][v] = 0.0f;
    if (p.bias)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) bias[i][v] = p.bias[(size_t)g * p.Kg + min(filter(i, v), p.Kg - 1)];
#pragma unroll
    for (int nb = 0; nb < NT; ++nb) {
        int P, n, row, wcol;
        const bool ok = there(nb, P, n, row, wcol);
        float* const o = y + ((size_t)n * p.K + (size_t)g * p.Kg) * plane + row * pcols + wcol;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            if (!G::POOL) {
                float r[16];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    r[v] = acc[i][nb][v] + bias[i][v];
                    if (p.relu) r[v] = fmaxf(r[v], 0.0f);
                }
                float* const ok0 = o + (size_t)filter(i, 0) * plane;
                if (full) {
                    if (ok)
#pragma unroll
                        for (int v = 0; v < 16; ++v) ok0[(size_t)(8 * (v >> 2) + (v & 3)) * plane] = r[v];
                } else {
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        if (ok && filter(i, v) < p.Kg) ok0[(size_t)(8 * (v >> 2) + (v & 3)) * plane] = r[v];
                }
            } else {
                // the four results of a pooling window lie in four neighbouring lanes; lane e of them keeps filter v = e
                const int e = lane & 3;
#pragma unroll
                for (int vq = 0; vq < 4; ++vq) {
                    float r = 0.0f, b = 0.0f;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        float m = acc[i][nb][vq * 4 + v];
                        m = fmaxf(m, __shfl_xor(m, 1));
                        m = fmaxf(m, __shfl_xor(m, 2));
                        if (v == e) {
                            r = m;
                            b = bias[i][vq * 4 + v];
                        }
                    }
                    const int kk = filter(i, vq * 4) + e;
                    if (ok && kk < p.Kg) o[(size_t)kk * plane] = fmaxf(r + b, 0.0f);
                }
            }
        }
    }
}

// Taps dealt to the wavefronts of a workgroup: 5x5 and 7x7 kernels, and launches of 3x3 layers too small for the tiles above.
template <int T_, int CS_, int NT_, bool POOL_, int XU_>
struct TGeom {
    static constexpr int T = T_, CS = CS_, NT = NT_, XU = XU_;
    static constexpr bool POOL = POOL_;
    static constexpr int S = T == 9 ? 3 : T == 25 ? 5 : 7;
    static constexpr int NW = 8, BM = 32, BN = 32 * NT, CG = 2 * CS;
    static_assert(XU * NW % CG == 0, "as in PGeom");
    static constexpr int PXMAX = XU * NW / CG * 64;   // staged positions
    static constexpr int E = T * CS;                  // fragments of 32 filters x 16 channels per chunk
    static constexpr int FL = 16 * E, FS = FL | 1;    // floats of one filter per chunk, and their stride in LDS
    static constexpr int FR = (FL + 63) / 64;         // loads of 64 lanes per filter and chunk; a wavefront takes BM / NW filters
    static constexpr int FB = (BM * FS * 4 + 15) / 16 * 16;
};

// One workgroup computes 32 filters x 32 NT windows; its eight wavefronts share the staged chunk and take every eighth tap
// each, their sums are added through LDS at the end.  A tile is then an eighth as long as one wavefront's walk over all taps,
// and small enough that a layer of a few dozen tiles still spreads over the chip.  The filters as stored are read in runs of
// 16 channels x T taps (a fragment straight from memory would touch 64 lines per load) and kept in LDS as fp32; a lane
// cuts its eight values into pieces when it takes them.  Filters and map of the next chunk are on their way while a chunk is
// multiplied.
// Bound by the walk of one workgroup where there are few (2.0 us per chunk of 16 channels, 5x5 and 64 windows), by the matrix
// pipe and the two barriers per chunk where there are many (35 % of the busy compute
// units' matrix clocks at 5x5).  Against gen: 48 -> 128 5x5 @7x7 at
// batch 32 13 us (43), 64 -> 256 5x5 @28x28 at batch 16 90 (136), 128 -> 512 7x7 @28x28 at batch 8 293 (513); against the vector
// kernel without a workspace 256 -> 256 3x3 @14x14 at batch 1 23 (41).  More than one workgroup per compute unit needs 128
// registers: with 64 accumulators the compiler spills and the kernel takes twice as long.  Relative error against 64-bit sums
// 0.6e-7 to 1.1e-7, gen 0.8e-7 to 5.2e-7.
template <class G>
__global__ __launch_bounds__(G::NW * 64, 2) void piece_taps_kernel(Problem p, PieceCfg cfg, const float* __restrict__ x,
                                                                   const float* __restrict__ w, float* __restrict__ parts,
                                                                   float* __restrict__ y)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int T = G::T, S = G::S, CS = G::CS, CG = G::CG, NT = G::NT, NW = G::NW, XU = G::XU, E = G::E, FL = G::FL, FS = G::FS;
    const int PX = cfg.px, CGB = cfg.cgb;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;
    float* fl = reinterpret_cast<float*>(lds);
    unsigned char* buf = lds + G::FB;

    // workgroup -> (tile, slice), as in piece_kernel
    const int whole = cfg.whole, nb_all = gridDim.x;
    const bool split = (int)blockIdx.x >= whole;
    int b = split ? blockIdx.x - whole : blockIdx.x, ss = 0;
    {
        const int cnt = split ? nb_all - whole : whole;
        const int n8 = cnt >> 3, rem = cnt & 7, xcd = b & 7, i = b >> 3;
        b = xcd * n8 + min(xcd, rem) + i;
    }
    const int ns = cfg.tail, ptile0 = b;
    if (split) {
        ss = b / ns;
        b = whole + b - ss * ns;
    }
    const int b1 = cfg.by_kblocks.of(b), b2 = cfg.by_strips.of(b1), g = cfg.by_ntiles.of(b2);
    const int kb = b - b1 * cfg.kblocks, strip = b1 - b2 * cfg.strips, tile = b2 - g * cfg.ntiles;

    const int TW = cfg.TW, HW = p.H * p.W, HP = p.H + p.pad;
    const int pitch = (G::POOL ? (TW - 1) * p.ps + 1 : TW - 1) * p.stride + S;
    const int pcols = G::POOL ? p.PW : p.OW, prows = G::POOL ? p.PH : p.OH;
    const int plane = prows * pcols;
    auto place = [&](int P, int& n, int& row, int& c) {    // as in piece_kernel
        const int pp = G::POOL ? P >> 2 : P, q = cfg.by_TW.of(pp);
        c = pp - q * TW;
        n = cfg.by_rows.of(q);
        row = q - n * prows;
    };
    auto window = [&](int P, int& n, int& oh, int& ow) {
        place(P, n, oh, ow);
        if (G::POOL) {
            oh = p.ps * oh + ((P & 3) >> 1);
            ow = p.ps * ow + (P & 1);
        }
    };
    int n0, oh0, ow0;
    window(tile * G::BN, n0, oh0, ow0);
    const int r0 = n0 * HP + oh0 * p.stride;
    const int w0 = strip * TW * (G::POOL ? p.ps : 1) * p.stride - p.pad;
    int lb[NT];
#pragma unroll
    for (int nb = 0; nb < NT; ++nb) {
        int n, oh, ow;
        window(min(tile * G::BN + nb * 32 + col, cfg.nrun - 1), n, oh, ow);
        lb[nb] = ((n * HP + oh * p.stride - r0) * pitch + ow * p.stride) * 48 + half * CGB;
    }

    unsigned xvo[XU];
    int xst[XU];
#pragma unroll
    for (int u = 0; u < XU; ++u) {
        const int id = u * NW + wave, cgi = id % CG, q = id / CG * 64 + lane;
        const int row = cfg.by_pitch.of(q), cw = q - row * pitch + w0;
        const int sr = r0 + row, n = cfg.by_HP.of(sr), h = sr - n * HP - p.pad;
        const bool ok = q < PX && n < p.N && h >= 0 && h < p.H && cw >= 0 && cw < p.W;
        xvo[u] = ok ? 4u * (unsigned)((n - n0) * p.C * HW + h * p.W + cw) : 0x80000000u;
        xst[u] = q < PX ? cgi * CGB + q * 48 : -1;
    }
    const size_t xfirst = ((size_t)n0 * p.C + (size_t)g * p.Cg) * HW;
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(x + xfirst), 0, (int)min(((size_t)p.N * p.C * HW - xfirst) * 4, (size_t)0x7ffffffc), 0x00020000);
    // a filter past the group's last one re-reads the last, columns past the last re-read that one (their map elements are zeros)
    const float* wb = w + ((size_t)g * p.Kg + (size_t)kb * G::BM) * p.L;
    const int klast = p.Kg - 1 - kb * G::BM;
    constexpr int KW = G::BM / NW;

    float xr[XU][8], fr[KW][G::FR];
    auto fetch = [&](int ch) {
#pragma unroll
        for (int u = 0; u < G::FR; ++u) {
            const unsigned o = min(ch * FL + u * 64 + lane, p.L - 1);
#pragma unroll
            for (int k = 0; k < KW; ++k) fr[k][u] = wb[(size_t)min(wave * KW + k, klast) * p.L + o];
        }
#pragma unroll
        for (int u = 0; u < XU; ++u) {
            const int c0 = ch * CS * 16 + (u * NW + wave) % CG * 8;
#pragma unroll
            for (int j = 0; j < 8; ++j)
                xr[u][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xres, (int)xvo[u], min(c0 + j, p.Cg - 1) * HW * 4, 0));
        }
    };
    auto lay_out = [&](int ch) {
#pragma unroll
        for (int u = 0; u < G::FR; ++u) {
            if (u * 64 + 64 > FL && lane >= FL - u * 64) continue;
#pragma unroll
            for (int k = 0; k < KW; ++k) fl[(wave * KW + k) * FS + u * 64 + lane] = fr[k][u];
        }
#pragma unroll
        for (int u = 0; u < XU; ++u) {
            const int c0 = ch * CS * 16 + (u * NW + wave) % CG * 8;
            if (c0 + 8 > p.Cg) {   // channels past the group's last one count as zeros
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (c0 + j >= p.Cg) xr[u][j] = 0.0f;
            }
            u4 f[3];
            split8(xr[u], f);
            if (xst[u] >= 0) {
                u4* d = reinterpret_cast<u4*>(buf + xst[u]);
                d[0] = f[0];
                d[1] = f[1];
                d[2] = f[2];
            }
        }
    };

    // x0 w0 has sums of its own: one rounding per 16 terms at the size of the result, the other five at 2^-8 of it
    v16f acc[NT], accl[NT];
    const v16f zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int nb = 0; nb < NT; ++nb) acc[nb] = accl[nb] = zero;
    float av[8];
    u4 bv[NT][3];
    // fragment e of the chunk: channels 16 (e / T) and on, tap e % T
    auto take = [&](int e) {
        const int c = CS == 1 ? 0 : e / T, t = e - c * T, r = t / S;
        const float* f = fl + col * FS + (c * 16 + half * 8) * T + t;
#pragma unroll
        for (int j = 0; j < 8; ++j) av[j] = f[j * T];
        const unsigned char* tb = buf + c * 2 * CGB + (r * pitch + t - r * S) * 48;
#pragma unroll
        for (int nb = 0; nb < NT; ++nb)
#pragma unroll
            for (int q = 0; q < 3; ++q) bv[nb][q] = *reinterpret_cast<const u4*>(tb + lb[nb] + q * 16);
    };

    const int chb = split ? cfg.nch * ss / cfg.nss : 0, che = split ? cfg.nch * (ss + 1) / cfg.nss : cfg.nch;
    fetch(chb);
    for (int ch = chb; ch < che; ++ch) {
        lay_out(ch);
        __syncthreads();
        if (ch + 1 < che) fetch(ch + 1);
        take(wave);
        for (int e = wave; e < E; e += NW) {
            u4 a[3], bb[NT][3];
            split8(av, a);
#pragma unroll
            for (int nb = 0; nb < NT; ++nb)
#pragma unroll
                for (int q = 0; q < 3; ++q) bb[nb][q] = bv[nb][q];
            take(min(e + NW, E - 1));
            constexpr int qa[6] = {0, 2, 1, 0, 1, 0}, qb[6] = {2, 0, 1, 1, 0, 0};   // smallest products first
#pragma unroll
            for (int c = 0; c < 6; ++c)
#pragma unroll
                for (int nb = 0; nb < NT; ++nb) {
                    v16f& d = c == 5 ? acc[nb] : accl[nb];
                    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, a[qa[c]]), __builtin_bit_cast(bf8, bb[nb][qb[c]]), d,
                                                                0, 0, 0);
                }
        }
        __syncthreads();
    }

    // the wavefronts' sums, 32 windows at a time: element v of lane l = filter 8 (v / 4) + v % 4 + 4 (l / 32), window l % 32
    const int c_lo = chb * CS * 16, c_hi = min(che * CS * 16, p.Cg);
    float* part = split ? parts + (size_t)ptile0 * (G::BM * G::BN) : nullptr;
#pragma unroll
    for (int nb = 0; nb < NT; ++nb) {
        if (nb) __syncthreads();
#pragma unroll
        for (int v = 0; v < 16; ++v) fl[(wave * 16 + v) * 64 + lane] = acc[nb][v] + accl[nb][v];
        __syncthreads();
        const int P = tile * G::BN + nb * 32 + col;
        int n, wrow, wcol;
        place(min(P, cfg.nrun - 1), n, wrow, wcol);
        wcol += strip * TW;
        const int oh = G::POOL ? wrow * p.ps + ((P & 3) >> 1) : wrow, ow = G::POOL ? wcol * p.ps + (P & 1) : wcol;
        const bool pos_ok = P < cfg.nrun && wcol < pcols;
#pragma unroll
        for (int i = 0; i < 16 / NW; ++i) {
            const int v = i * NW + wave, kr = 8 * (v >> 2) + (v & 3) + 4 * half, k = kb * G::BM + kr;
            float s = fl[v * 64 + lane];
#pragma unroll
            for (int q = 1; q < NW; ++q) s += fl[(q * 16 + v) * 64 + lane];
            const bool ok = pos_ok && k < p.Kg;
            const bool again = ok && not_finite(s);
            s *= kDown;
            if (again) {   // out of the pieces' range: see the top
                const float* wk = w + ((size_t)g * p.Kg + k) * p.L;
                s = 0.0f;
                for (int c = c_lo; c < c_hi; ++c)
                    for (int t = 0; t < T; ++t) {
                        const int ih = oh * p.stride - p.pad + t / S, iw = ow * p.stride - p.pad + t % S;
                        if (ih < 0 || ih >= p.H || iw < 0 || iw >= p.W) continue;
                        const float e = x[(((size_t)n * p.G + g) * p.Cg + c) * HW + ih * p.W + iw];
                        if (e != 0.0f) s = __builtin_fmaf(e, wk[c * T + t], s);
                    }
            }
            if (split) {
                part[kr * G::BN + nb * 32 + col] = s;
                continue;
            }
            if (G::POOL) {   // the four results of a pooling window lie in four neighbouring lanes
                s = fmaxf(s, __shfl_xor(s, 1));
                s = fmaxf(s, __shfl_xor(s, 2));
            }
            if (!ok || (G::POOL && (lane & 3))) continue;
            s += bias_of(p, (size_t)g * p.Kg + k);
            if (G::POOL || p.relu) s = fmaxf(s, 0.0f);
            y[((size_t)n * p.K + (size_t)g * p.Kg + k) * plane + wrow * pcols + wcol] = s;
        }
    }
}

// Adds the slices of the split tiles (slice 0 first) and applies the epilogue: one thread per filter and four window rows (plain) or one
// pooling window, i.e. 16 bytes of every slice.  Bound by the slices' trip through memory; their loads are all on their way before the first
// is added, where one thread per result waited for each: 512 @14x14 at batch 8, 100 tiles x 5 slices 7.2 -> 5.7 us, 512 @7x7 at batch 1,
// 16 x 16 slices of 32 x 64 6.4 -> 4.1, 256 @56x56 16 x 16 6.2 -> 4.6.
template <bool POOL>
__global__ __launch_bounds__(256) void piece_sum_kernel(Problem p, PieceCfg cfg, int BM, int BN, const float* __restrict__ parts,
                                                        float* __restrict__ y)
{
    const int per_row = BN / 4;
    const int e = blockIdx.x * 256 + threadIdx.x, kr = cfg.by_quads.of(e), c = e - kr * per_row;
    const int b = cfg.whole + blockIdx.y, b1 = cfg.by_kblocks.of(b), b2 = cfg.by_strips.of(b1), g = cfg.by_ntiles.of(b2);
    const int kb = b - b1 * cfg.kblocks, strip = b1 - b2 * cfg.strips, tile = b2 - g * cfg.ntiles;
    const int k = kb * BM + kr;
    if (kr >= BM || k >= p.Kg || tile * BN + c * 4 >= cfg.nrun) return;
    const size_t tsz = (size_t)BM * BN, step = (size_t)cfg.tail * tsz;
    const float* src = parts + (size_t)blockIdx.y * tsz + (size_t)kr * BN + c * 4;
    f4 r = *reinterpret_cast<const f4*>(src);
    int s = 1;
    for (; s + 8 <= cfg.nss; s += 8) {
        f4 v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = *reinterpret_cast<const f4*>(src + (s + q) * step);
#pragma unroll
        for (int q = 0; q < 8; ++q) r += v[q];
    }
    if (s < cfg.nss) {
        f4 v[7];
#pragma unroll
        for (int q = 0; q < 7; ++q) v[q] = *reinterpret_cast<const f4*>(src + min(s + q, cfg.nss - 1) * step);
#pragma unroll
        for (int q = 0; q < 7; ++q)
            if (s + q < cfg.nss) r += v[q];
    }
    const int pcols = POOL ? p.PW : cfg.flat ? p.OH * p.OW : p.OW, prows = POOL ? p.PH : cfg.flat ? 1 : p.OH;
    const float bias = bias_of(p, (size_t)g * p.Kg + k);
    if (POOL) r[0] = fmaxf(fmaxf(r[0], r[1]), fmaxf(r[2], r[3]));
#pragma unroll
    for (int i = 0; i < (POOL ? 1 : 4); ++i) {
        const int P = POOL ? tile * BN / 4 + c : tile * BN + c * 4 + i;
        const int q = cfg.by_TW.of(P), n = cfg.by_rows.of(q), wrow = q - n * prows, wcol = strip * cfg.TW + P - q * cfg.TW;
        if (P >= cfg.nrun / (POOL ? 4 : 1) || wcol >= pcols) continue;
        float v = r[i] + bias;
        if (p.relu) v = fmaxf(v, 0.0f);
        y[(((size_t)n * p.K + (size_t)g * p.Kg + k) * prows + wrow) * pcols + wcol] = v;
    }
}

// w[K][Cg][T] times 2^24 -> pieces[group][32 filters][16 channels][tap][piece][64 lanes][8 channels] bf16: lane l of a fragment holds
// filter l % 32, channels 8 * (l / 32) + 0..7.  Filters past the group and channels past Cg are zero.
__global__ __launch_bounds__(64) void piece_filters_kernel(Problem p, int kb32, int nch16, int T, const float* __restrict__ w,
                                                           u4* __restrict__ out)
{
    const int t = blockIdx.x % T, ch = blockIdx.x / T, kb = blockIdx.y, g = blockIdx.z, l = threadIdx.x;
    const int k = kb * 32 + (l & 31), c0 = ch * 16 + (l >> 5) * 8;
    const float* src = w + ((size_t)g * p.Kg + min(k, p.Kg - 1)) * p.L + t;
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = src[(size_t)min(c0 + j, p.Cg - 1) * T];
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (k >= p.Kg || c0 + j >= p.Cg) v[j] = 0.0f;
    u4 f[3];
    split8(v, f);
    u4* dst = out + ((((size_t)g * kb32 + kb) * nch16 + ch) * T + t) * 192 + l;
#pragma unroll
    for (int q = 0; q < 3; ++q) dst[q * 64] = f[q];
}

// w[K][Cg][9] -> pairs[group][32 filters][16 channels][tap][pair][64 lanes][8 channels] fp16, scaled per filter, and behind them the exponent of
// every filter's scale (kUnpaired: not to be held in pairs).  Filters past the group and channels past Cg are zero.
// Where `pieces` is given, the three pieces there besides, as piece_filters_kernel writes them: what a launch reads where pairs do not do (from
// the filters as stored it took a third longer: 256 @56x56 at batch 32 with eight weights of 1e-20 729 us, now 517).
// A workgroup takes FW neighbouring filters through LDS: their ranges, then their pairs, 16 bytes a lane at a filter's place in the fragments; the
// filters' places are side by side, and those of other workgroups on the same XCD, whose L2 puts the lines together.  Bound by the stores: 512 x 512
// x 9, pairs alone / with pieces, 9.0 / 14.9 us with one filter a workgroup, 7.4 / 11.7 with two, 8.3 / 12.1 with four (half the chip), 768 x 768
// 26.0, 18.4, 15.8 with pieces, 256 x 256 7.2, 6.7, 7.2; three pieces of 512 x 512 by piece_filters_kernel 14.7.
template <int FW>
__global__ __launch_bounds__(256 * FW) void piece_pairs_kernel(Problem p, int kb32, int nch16, const float* __restrict__ w, u4* __restrict__ out,
                                                               u4* __restrict__ pieces)
{
    extern __shared__ float f[];
    __shared__ uint2 part[4 * FW];
    const int tid = threadIdx.x, g = blockIdx.y, L = p.L;
    const int k0 = ((blockIdx.x & 7) * (kb32 * 4 / FW) + (blockIdx.x >> 3)) * FW;
    Range rg;
    if (k0 + (tid >> 8) < p.Kg) {
        const float* src = w + ((size_t)g * p.Kg + k0 + (tid >> 8)) * L;
        float* dst = f + (tid >> 8) * L;
        for (int o0 = tid & 255; o0 < L; o0 += 16 * 256) {
            float v[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) v[j] = src[min(o0 + j * 256, L - 1)];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                dst[min(o0 + j * 256, L - 1)] = v[j];
                if (j & 1) rg.add(v[j - 1], v[j]);
            }
        }
    }
    const uint2 of = rg.of_wave();
    if ((tid & 63) == 63) part[tid >> 6] = of;
    __syncthreads();
    const int fw = tid % FW, k = k0 + fw;
    const uint2* r = part + 4 * fw;
    const unsigned hi = max(max(r[0].x, r[1].x), max(r[2].x, r[3].x)), lo = min(min(r[0].y, r[1].y), min(r[2].y, r[3].y));
    const int sg = pair_exponent(hi);
    const float up = power_of_two(sg);
    const bool real = k < p.Kg;
    const size_t blk = ((size_t)g * kb32 + (k >> 5)) * nch16 * 9;
    u4* dst = out + blk * 128 + (k & 31);
    u4* dst3 = pieces + blk * 192 + (k & 31);
    for (int it = tid / FW; it < nch16 * 18; it += 256) {
        const int t = it % 9, hc = it / 9;          // 8 channels of one tap
        u4 q[2], q3[3];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = hc * 8 + 2 * i;
            const float a = real && c < p.Cg ? f[fw * L + c * 9 + t] : 0.0f, b = real && c + 1 < p.Cg ? f[fw * L + c * 9 + 9 + t] : 0.0f;
            pair2(a * up, b * up, 1.0f, 4096.0f, 1.0f, 4096.0f, i, q);
            if (pieces) split2(a, b, kUp, kUp, i, q3);
        }
        const size_t at = (size_t)(hc >> 1) * 9 + t;
        u4* d = dst + at * 128 + (hc & 1) * 32;
        d[0] = q[0];
        d[64] = q[1];
        if (!pieces) continue;
        d = dst3 + at * 192 + (hc & 1) * 32;
        d[0] = q3[0];
        d[64] = q3[1];
        d[128] = q3[2];
    }
    int* exponents = reinterpret_cast<int*>(out + (size_t)p.G * kb32 * nch16 * 9 * 128) + (size_t)g * kb32 * 32;
    if (tid < FW) exponents[k] = PairLimits(sg).hold(hi, lo) ? sg : kUnpaired;
}

struct Plan {
    double cost = -1.0;   // modelled microseconds; negative = not applicable
    double stored = -1.0; // those of the cheapest split on filters as stored
    PieceCfg cfg;
    size_t lds_bytes = 0, piece_bytes = 0;
    int src = SRC_RAW, ntail = 0;
    int rest = SRC_RAW;   // with pairs: the filters' form where those do not do
};

bool shape_ok(const Problem& p, bool pooled)
{
    const int T = p.R * p.S;
    if (p.R != p.S || (T != 1 && T != 9 && T != 25 && T != 49)) return false;
    if (pooled && (p.ph != 2 || p.pw != 2)) return false;
    const long long npos = pooled ? (long long)p.N * p.PH * p.PW * 4 : (long long)p.N * p.OH * p.OW;
    if (npos >= (1LL << 30)) return false;
    // rows of the padded batch are numbered from its first one, and a tile stages fewer than 4096 (715 827 883 images of 1x1, padded by 2, at stride 3
    // have 2^31; a wrapped number reads as a row of the padding)
    return (long long)p.N * (p.H + p.pad) + 4096 < (1LL << 31);
}

// Staged positions of a tile of BN windows of a strip TW columns wide: the largest over the tiles (a tile's rows depend
// only on where it starts inside an image, so the distinct starts are walked; an upper bound where there are many).
long long stage_positions(const Problem& p, bool pooled, bool flat, int BN, int TW)
{
    const long long B = BN / (pooled ? 4 : 1), ow = TW, oh = pooled ? p.PH : flat ? 1 : p.OH, plane = oh * ow;
    const long long step = pooled ? (long long)p.ps * p.stride : p.stride, HP = (flat ? 1 : p.H) + p.pad;
    const long long ntiles = (plane * p.N + B - 1) / B, last = plane * p.N - 1;
    long long rows = 0;
    if (ntiles <= 256) {
        for (long long t = 0; t < ntiles; ++t) {
            const long long a = t * B, b = a + B - 1 < last ? a + B - 1 : last;
            const long long r = (b / plane - a / plane) * HP + (b % plane / ow - a % plane / ow) * step;
            if (r > rows) rows = r;
            if ((t + 1) * B % plane == 0) break;
        }
    } else {
        const long long rs = (ow - 1 + B - 1) / ow, ib = (plane - 1 + B - 1) / plane, jump = HP - (oh - 1) * step;
        rows = (rs - ib) * step + ib * (jump > step ? jump : step);
    }
    rows += p.R + (pooled ? p.stride : 0);
    return rows * ((long long)(pooled ? (TW - 1) * p.ps + 1 : TW - 1) * p.stride + p.S);
}

size_t usable_workspace(const Problem& p, bool pooled)
{
    if (!split_scratch_possible(nullptr)) return 0;
    const size_t have = split_scratch_bytes(), most = plan_workspace_bytes(p, pooled);
    return have < most ? have : most;
}

// Workgroups of a geometry on one compute unit.
template <class G>
int occupancy_limit(int src, size_t lds_bytes)
{
    const int by_lds = (int)(160 * 1024 / lds_bytes), by_regs = G::tc(src, 9) > 4.0 || G::apart(src) || src != SRC_RAW || G::XU > 2 ? 2 : 3;
    const int n = by_regs * 4 / G::NW;
    return by_lds < n ? by_lds : n;
}

// The most loaded of 256 compute units: na workgroups of length a dealt out first, then nb of length b wherever there is least.
double cu_load(long long na, double a, long long nb, double b)
{
    const long long q = na / 256, r = na % 256;
    double lo = q * a, hi = r ? (q + 1) * a : lo;
    if (nb == 0) return hi;
    double best = -1.0;
    for (int side = 0; side < 2; ++side)
        for (int i = 0; i <= 64; ++i) {
            const double L = (side ? hi : lo) + i * b;
            if (L + 1e-9 < hi) continue;
            const double cap = (256 - r) * floor((L - lo) / b + 1e-9) + r * floor((L - hi) / b + 1e-9);
            if (cap >= (double)nb) {
                if (best < 0.0 || L < best) best = L;
                break;
            }
        }
    return best < 0.0 ? hi + (double)(nb + 255) / 256 * b : best;
}

// Column strips of a tile of BN windows: the fewest columns past the map's edge, then the fewest staged positions.  False
// where no strip's staged positions fit.
bool choose_strips(const Problem& p, bool pooled, int BN, int PXMAX, PieceCfg& c)
{
    const int cols = pooled ? p.PW : c.flat ? p.OH * p.OW : p.OW, rows = pooled ? p.PH : c.flat ? 1 : p.OH;
    double best = 0.0;
    for (int TW = cols < BN ? cols : BN; TW >= (cols < 4 ? cols : 4); --TW) {
        const int strips = (cols + TW - 1) / TW;
        if ((cols + strips - 1) / strips != TW) continue;   // as many strips of fewer columns do
        const long long px = stage_positions(p, pooled, c.flat, BN, TW);
        if (px > PXMAX) continue;
        const long long run = (long long)p.N * rows * TW * (pooled ? 4 : 1), nt = (run + BN - 1) / BN;
        const double cost = (double)nt * strips * (BN * (1.0 + 0.5 / TW) + px * 0.02);   // (a row's end costs LDS bank conflicts)
        if (best == 0.0 || cost < best) {
            best = cost;
            c.TW = TW;
            c.strips = strips;
            c.nrun = (int)run;
            c.ntiles = (int)nt;
            c.px = (int)px;
        }
    }
    return best != 0.0;
}

// A plan remembered by sconv_tune names a geometry and leaves the split to the model; any other decomposition is not this
// kernel's.
bool pin_allows()
{
    const PlanPin* pin = current_pin();
    return !pin || !pin->nwv || (pin->nwv == 4 && pin->ncs == 1 && pin->nss <= 1);
}

// The cheapest split of a geometry's tiles, kept in pl when it beats what is there: whole tiles first, then the rest, each
// split along the channels over s workgroups (s = 1: none).  tc: microseconds of a chunk, times lone where the compute units
// hold a single workgroup; fixed: those of the launch.  in_pairs: two workgroups on a compute unit, what is left of the longer
// half runs alone.
void consider(Plan& pl, long long tiles, long long round, int NW, double tc, double lone, double fixed, int src, size_t pb, int kb32, size_t ws,
              size_t tile_bytes, bool in_pairs)
{
    PieceCfg& c = pl.cfg;
    int pin_whole = 0, pin_ncs = 0, pin_nss = 0;   // tuning aid: SCONV_PIECE_SPLIT="whole tiles,1,slices of the others"
    if (!current_pin()) pinned_split("SCONV_PIECE_SPLIT", &pin_whole, &pin_ncs, &pin_nss);
    const long long firsts[3] = {tiles, tiles / 256 * 256, tiles / round * round};
    for (int f = 0; f < (tiles < 4096 ? 4 : 1); ++f) {
        const long long whole = pin_nss ? (pin_nss > 1 ? pin_whole : tiles) : f < 3 ? firsts[f] : 0;
        const long long tail = tiles - whole;
        if (f && !pin_nss && (tail == 0 || (f == 2 && firsts[2] == firsts[1]) || (f == 3 && (firsts[1] == 0 || firsts[2] == 0)))) continue;
        if (tail < 0) continue;
        for (int s = tail ? 2 : 1; s <= (tail ? 32 : 1); s += s < 6 ? 1 : s < 16 ? 2 : 8) {
            if (pin_nss > 1 && s != pin_nss) continue;
            if (s > c.nch || pb + (size_t)tail * s * tile_bytes > ws + (tail ? 0 : pb)) break;
            const double a = (c.nch + 0.6) * tc, b = ((c.nch + s - 1) / s + 0.6) * tc;
            double load = cu_load(whole, a, tail * s, b);
            if (in_pairs) {
                const long long na = (whole + 255) / 256, nb = (tail * s + 255) / 256;
                const double rest = na % 2 ? a - (double)nb * b : nb % 2 ? b : 0.0;
                if (na + nb > 2 && rest > 0.0) load += (lone - 1.0) * rest;
            }
            const double resident = (double)(whole + tail * s) / 256.0;
            double cost = fixed + load * (resident * NW <= (lone > 1.0 ? 6.0 : 8.0) ? lone : 1.0);
            if (tail) cost += 3.0 + 2.0 * (double)(tail * s) * tile_bytes / 6e6;
            if (src == SRC_RAW && (pl.stored < 0.0 || cost < pl.stored)) pl.stored = cost;
            if (pl.cost >= 0.0 && cost >= pl.cost) continue;
            pl.cost = cost;
            pl.src = src;
            pl.piece_bytes = pb;
            pl.ntail = (int)tail;
            c.kb32 = kb32;
            c.whole = (int)whole;
            c.nss = s;
            c.tail = (int)tail;
        }
        if (pin_nss) break;
    }
}

// The same for blocks, one workgroup to a compute unit: whole tiles only, in rounds of 256.  A chunk takes 1.5 us where few units have a tile, at 2.3 GHz,
// and 2.9 where all have, at the clock that the chip's power leaves (196 tiles of 8, 16, 32 chunks 32.4, 51.7, 90.7 us with the filters' pairs, 248 of
// 32 103.9, 392 of 16 100.6, 784 of 16 192); for the same reason sharing the tiles of a last round evenly among all units won 4 % at best (392 of
// 16: 96.7) and lost where less than a round was shared (196 of 32: 98).
void consider_blocks(Plan& pl, long long tiles, double fixed, size_t pb, int kb32, size_t ws)
{
    PieceCfg& c = pl.cfg;
    if (pb > ws || (!current_pin() && env_value("SCONV_PIECE_SPLIT"))) return;   // (a decomposition of its own)
    const long long rounds = (tiles + 255) / 256;
    const double last = (double)(tiles - (rounds - 1) * 256) / 256.0;
    pl.cost = fixed + (double)(rounds - 1) * (c.nch * 2.88 + 5.0) + c.nch * (1.5 + 1.38 * last);
    pl.src = SRC_PAIRS;
    pl.piece_bytes = pb;
    pl.ntail = 0;
    c.kb32 = kb32;
    c.whole = (int)tiles;
    c.nss = 1;
    c.tail = 0;
}

// The tiles of a geometry, without a form of the filters (cost < 0); their number, 0 where it has none.
template <class G>
long long plan_tiles(const Problem& p, bool pooled, Plan& pl)
{
    if (G::POOL != pooled) return 0;
    const int T = p.R * p.S;
    if (G::T != T || p.R != p.S) return 0;
    PieceCfg& c = pl.cfg;
    c.flat = T == 1 && p.stride == 1 && !pooled;
    c.T = T;
    c.S = p.S;
    c.nch = (p.Cg + 16 * G::CS - 1) / (16 * G::CS);
    c.kblocks = (p.Kg + G::BM - 1) / G::BM;
    if (!choose_strips(p, pooled, G::BN, G::PXMAX, c)) return 0;
    c.cgb = (c.px * 48 + 255) / 256 * 256;
    pl.lds_bytes = 2 * ((size_t)G::CG * c.cgb + G::SPARE);
    if (pl.lds_bytes < (size_t)G::NW * 4096) pl.lds_bytes = (size_t)G::NW * 4096;
    if (G::PAIRS && pl.lds_bytes < 3 * (size_t)G::PAIR_BUF) pl.lds_bytes = 3 * (size_t)G::PAIR_BUF;
    if (pl.lds_bytes > 160 * 1024) return 0;
    // images a tile can touch, and the byte offsets of their elements
    const long long run_img = (long long)(pooled ? p.PH : c.flat ? 1 : p.OH) * c.TW * (pooled ? 4 : 1);
    const long long imgs = (G::BN - 1 + run_img - 1) / run_img + 1;
    if ((imgs + 1) * p.C * p.H * p.W * 4 >= (1LL << 31)) return 0;
    if ((size_t)p.Cg * T * 256 >= (1u << 31) || (size_t)p.L * 4 * (G::BM + 1) >= (1u << 31)) return 0;
    const long long tiles = (long long)c.ntiles * c.strips * c.kblocks * p.G;
    if (tiles >= (1LL << 24)) return 0;

    return pin_allows() ? tiles : 0;
}

// close: only forms with sums of their own for the small products.
template <class G>
Plan plan_geom(const Problem& p, bool pooled, bool close)
{
    Plan pl;
    if (G::BLOCK) return pl;             // (pairs only)
    const long long tiles = plan_tiles<G>(p, pooled, pl);
    if (!tiles) return pl;
    const PieceCfg& c = pl.cfg;
    const int T = G::T;
    const char* pin_src = env_value("SCONV_PIECE_SRC");
    const size_t ws = usable_workspace(p, pooled);
    const size_t tile_bytes = (size_t)G::BM * G::BN * 4;
    for (int src = SRC_PIECES; src <= SRC_RAW; ++src) {
        // filters: as prepared by the caller; else cut into pieces by a kernel of their own when the workspace has room, or as stored
        if (pin_src ? atoi(pin_src) != src : (src == SRC_FP32) != (p.wprep && G::T == 9)) continue;
        if (src == SRC_FP32 && (!p.wprep || G::T != 9)) continue;
        if (close && !G::apart(src)) continue;
        size_t pb = 0;
        const int kb32 = src == SRC_FP32 ? (p.Kg + 127) / 128 * 4 : c.kblocks * (G::BM / 32);
        if (src == SRC_PIECES) {
            const size_t blk = (size_t)c.nch * G::CS * T * 3072;
            if (blk * (G::BM / 32) >= (1u << 31) || c.nch * G::CS > 65535 || kb32 > 65535 || p.G > 65535) continue;
            pb = (size_t)p.G * kb32 * blk;
            if (pb > ws) continue;
        }
        const double tc = G::tc(src, T);
        const int occ = occupancy_limit<G>(src, pl.lds_bytes);
        const double pre = src == SRC_PIECES ? 6.0 + (double)p.K * p.L * 10.0 / 4e6 : 0.0;
        consider(pl, tiles, 256LL * occ, G::NW, tc, 1.25, 6.0 + pre, src, pb, kb32, ws, tile_bytes, G::T == 9 && src != SRC_FP32 && (src == SRC_PIECES || G::apart(src)));
    }
    return pl;
}

// The form with pairs of geometries that have it.
template <class G>
Plan plan_pairs(const Problem& p, bool pooled)
{
    Plan pl;
    if constexpr (G::PAIRS) {
        const char* pin_src = env_value("SCONV_PIECE_SRC");
        if (pin_src && atoi(pin_src) < SRC_PAIRS) return pl;
        const long long tiles = plan_tiles<G>(p, pooled, pl);
        if (!tiles) return pl;
        const int kb32 = pl.cfg.kblocks * (G::BM / 32);
        const size_t blk = (size_t)pl.cfg.nch * 9 * 3072, ws = usable_workspace(p, pooled);
        if (blk * 4 >= (1u << 31) || p.G > 65535 || (size_t)p.L * 4 > 128 * 1024) return pl;
        // What pairs do not hold is summed from the prepared filters, or from pieces written behind the pairs; from the filters as stored, which
        // takes a third longer, where the pieces leave no room for the plan (a workspace of 16 MiB and 512 channels of 512 filters).
        const size_t room[2] = {p.wprep ? 0 : (size_t)p.G * kb32 * blk, 0};
        const int rest[2] = {p.wprep ? SRC_FP32 : SRC_PIECES, SRC_RAW};
        const Plan empty = pl;
        for (int i = 0; i < (p.wprep ? 1 : 2); ++i) {
            Plan q = empty;
            const size_t pb = pair_bytes(p.G, kb32, pl.cfg.nch) + room[i];
            if (pb > ws) continue;
            const double fixed = 11.0 + 2e-6 * p.K * p.L;
            if (G::BLOCK) consider_blocks(q, tiles, fixed, pb, kb32, ws);
            else consider(q, tiles, 256LL * occupancy_limit<G>(SRC_PAIRS, q.lds_bytes), G::NW, G::tc(SRC_PAIRS, 9), 1.25, fixed, SRC_PAIRS, pb, kb32, ws,
                          (size_t)G::BM * G::BN * 4, true);
            q.rest = rest[i];
            if (q.cost >= 0.0 && (pl.cost < 0.0 || q.cost < 0.9 * pl.cost)) pl = q;
        }
    }
    return pl;
}

template <class G, int SRC, int FORM = 0>
int launch_src(const Plan& pl, const Problem& p, const float* x, const float* w, const void* wp, float* parts, float* y, hipStream_t stream)
{
    auto kern = piece_kernel<G, SRC, FORM>;
    static_assert(FORM == 0 || G::PAIRS, "the forms with pairs are those of some geometries");
    static size_t opted = 0;
    if (pl.lds_bytes > opted) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)pl.lds_bytes) != hipSuccess)
            return SCONV_ELAUNCH;
        opted = pl.lds_bytes;
    }
    PieceCfg cfg = pl.cfg;
    cfg.prepare(p, G::POOL, G::BN);
    hipLaunchKernelGGL(kern, dim3((unsigned)(pl.cfg.whole + pl.ntail * pl.cfg.nss)), dim3(G::NW * 64), pl.lds_bytes, stream, p, cfg, x,
                       w, wp, parts, y);
    return launch_status();
}

template <int FW>
int launch_pairs(const Problem& p, const PieceCfg& cfg, const float* w, u4* pairs, u4* pieces, hipStream_t stream)
{
    const size_t rows = (size_t)p.L * 4 * FW;
    static size_t opted = 0;
    if (rows > opted) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(piece_pairs_kernel<FW>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)rows) != hipSuccess)
            return SCONV_ELAUNCH;
        opted = rows;
    }
    hipLaunchKernelGGL(piece_pairs_kernel<FW>, dim3((unsigned)cfg.kb32 * 32 / FW, (unsigned)p.G), dim3(256 * FW), rows, stream, p, cfg.kb32, cfg.nch, w,
                       pairs, pieces);
    return launch_status();
}

template <class G>
int launch_sum(const Plan& pl, const Problem& p, const float* parts, float* y, hipStream_t stream)
{
    PieceCfg cfg = pl.cfg;
    cfg.prepare(p, G::POOL, G::BN);
    hipLaunchKernelGGL(piece_sum_kernel<G::POOL>, dim3((unsigned)((G::BM * G::BN / 4 + 255) / 256), (unsigned)pl.ntail), dim3(256), 0, stream, p, cfg,
                       G::BM, G::BN, parts, y);
    return launch_status();
}

template <class G>
int launch_plan(const Plan& pl, const Problem& p, bool pooled, const float* x, const float* w, float* y, hipStream_t stream)
{
    char* ws = reinterpret_cast<char*>(split_scratch(stream));
    float* parts = pl.ntail ? reinterpret_cast<float*>(ws + pl.piece_bytes) : nullptr;
    int rc = SCONV_EUNSUPPORTED;
    if (pl.src == SRC_PAIRS) {
        if constexpr (G::PAIRS) {
            u4* const pairs = reinterpret_cast<u4*>(ws);
            u4* const pieces = pl.rest == SRC_PIECES ? reinterpret_cast<u4*>(ws + pair_bytes(p.G, pl.cfg.kb32, pl.cfg.nch)) : nullptr;
            rc = p.L <= 16 * 1024 ? launch_pairs<2>(p, pl.cfg, w, pairs, pieces, stream) : launch_pairs<1>(p, pl.cfg, w, pairs, pieces, stream);   // (by LDS)
            if (rc) return rc;
            auto launch = pl.rest == SRC_FP32     ? launch_src<G, SRC_FP32, SRC_PAIRS>
                          : pl.rest == SRC_PIECES ? launch_src<G, SRC_PIECES, SRC_PAIRS>
                                                  : launch_src<G, SRC_RAW, SRC_PAIRS>;
            rc = launch(pl, p, x, w, ws, parts, y, stream);
        }
    } else if constexpr (!G::BLOCK) {
        if (pl.src == SRC_FP32) {
            if constexpr (G::T == 9) rc = launch_src<G, SRC_FP32>(pl, p, x, w, p.wprep, parts, y, stream);
        } else if (pl.src == SRC_PIECES) {
            const int nch16 = pl.cfg.nch * G::CS, T = pl.cfg.T;
            hipLaunchKernelGGL(piece_filters_kernel, dim3((unsigned)(nch16 * T), (unsigned)pl.cfg.kb32, (unsigned)p.G), dim3(64), 0, stream, p,
                               pl.cfg.kb32, nch16, T, w, reinterpret_cast<u4*>(ws));
            rc = launch_status();
            if (rc) return rc;
            rc = launch_src<G, SRC_PIECES>(pl, p, x, w, ws, parts, y, stream);
        } else {
            rc = launch_src<G, SRC_RAW>(pl, p, x, w, nullptr, parts, y, stream);
        }
    }
    return rc || !pl.ntail ? rc : launch_sum<G>(pl, p, parts, y, stream);
}

template <class G>
Plan plan_taps(const Problem& p, bool pooled, bool)
{
    Plan pl;
    if (G::POOL != pooled || p.R != p.S || p.S != G::S || p.wprep) return pl;
    PieceCfg& c = pl.cfg;
    c = PieceCfg();
    c.nch = (p.Cg + 16 * G::CS - 1) / (16 * G::CS);
    c.kblocks = (p.Kg + G::BM - 1) / G::BM;
    if (!choose_strips(p, pooled, G::BN, G::PXMAX, c)) return pl;
    c.cgb = (c.px * 48 + 255) / 256 * 256;
    pl.lds_bytes = G::FB + (size_t)G::CG * c.cgb;
    if (pl.lds_bytes < (size_t)G::NW * 4096) pl.lds_bytes = (size_t)G::NW * 4096;
    if (pl.lds_bytes > 160 * 1024) return pl;
    const long long run_img = (long long)(pooled ? p.PH : p.OH) * c.TW * (pooled ? 4 : 1);
    const long long imgs = (G::BN - 1 + run_img - 1) / run_img + 1;
    if ((imgs + 1) * p.C * p.H * p.W * 4 >= (1LL << 31)) return pl;
    if (((size_t)p.L + G::FL) * 4 * (G::BM + 1) >= (1u << 31)) return pl;
    const long long tiles = (long long)c.ntiles * c.strips * c.kblocks * p.G;
    if (tiles >= (1LL << 24) || !pin_allows()) return pl;
    if (env_value("SCONV_PIECE_SRC") && atoi(env_value("SCONV_PIECE_SRC")) != SRC_RAW) return pl;
    // a chunk: the matrix instructions of its busiest SIMD (32 clocks each), and barriers and staging that nothing hides (one
    // workgroup per compute unit).  Measured: 2.0 us with few workgroups and 2.6 with all (5x5, 64 windows), 3.9 and 5.9 (7x7)
    const double tc = (((G::E + 3) / 4) * G::NT * 6 * 32 / 2000.0 / 0.75 + 0.8) * (G::T == 49 ? 1.2 : 1.0);
    consider(pl, tiles, 256LL, G::NW, tc, 0.75, 7.0, SRC_RAW, 0, 0, usable_workspace(p, pooled), (size_t)G::BM * G::BN * 4, false);
    return pl;
}

template <class G>
int launch_taps(const Plan& pl, const Problem& p, bool, const float* x, const float* w, float* y, hipStream_t stream)
{
    auto kern = piece_taps_kernel<G>;
    static size_t opted = 0;
    if (pl.lds_bytes > opted) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)pl.lds_bytes) != hipSuccess)
            return SCONV_ELAUNCH;
        opted = pl.lds_bytes;
    }
    float* parts = pl.ntail ? split_scratch(stream) : nullptr;
    PieceCfg cfg = pl.cfg;
    cfg.prepare(p, G::POOL, G::BN);
    hipLaunchKernelGGL(kern, dim3((unsigned)(cfg.whole + cfg.tail * cfg.nss)), dim3(G::NW * 64), pl.lds_bytes, stream, p, cfg, x, w, parts, y);
    const int rc = launch_status();
    return rc || !pl.ntail ? rc : launch_sum<G>(pl, p, parts, y, stream);
}

struct Candidate {
    const char* name;
    Plan (*plan)(const Problem&, bool, bool);
    Plan (*pairs)(const Problem&, bool);
    int (*launch)(const Plan&, const Problem&, bool, const float*, const float*, float*, hipStream_t);
    bool (*apart)(int);
    const char* tiles;   // a block's tiles; null: no block
};

bool always_apart(int) { return true; }

// The geometries, for the table below and for the test that walks their plans; the blocks.
#define PIECE_GEOMETRIES(CAND, TAPS) \
    /* 32-filter and 32-window blocks of a wavefront, wavefronts along filters and windows, taps, 16-channel groups per chunk, pooled, */ \
    /* staging units, wavefronts per SIMD, small products apart */ \
    CAND("a128x128", 1, 4, 4, 1, 9, 1, false, 3, 2, false) \
    CAND("a128x64", 1, 2, 4, 1, 9, 1, false, 2, 2, false) \
    CAND("a64x128", 1, 2, 2, 2, 9, 1, false, 3, 2, false) \
    CAND("s128x64", 1, 2, 4, 1, 9, 1, false, 2, 2, true) /* as many positions as two units stage; more with four */ \
    CAND("s128x64", 1, 2, 4, 1, 9, 1, false, 4, 2, true) \
    CAND("b64x128", 1, 2, 2, 2, 9, 1, false, 3, 2, true) \
    CAND("p128x128", 1, 4, 4, 1, 9, 1, true, 3, 2, false) \
    CAND("p128x64", 1, 2, 4, 1, 9, 1, true, 2, 2, false) \
    CAND("u128x64", 1, 2, 4, 1, 9, 1, true, 2, 2, true) \
    CAND("c128x64", 1, 2, 4, 1, 1, 4, false, 2, 2, true) \
    CAND("q128x64", 1, 2, 4, 1, 1, 4, true, 2, 2, true) \
    /* taps, 16-channel groups per chunk, window blocks, pooled, staging units */ \
    TAPS("t3x64", 9, 2, 2, false, 2) \
    TAPS("t5x64", 25, 1, 2, false, 1) \
    TAPS("t5x128", 25, 1, 4, false, 2) \
    TAPS("t7x64", 49, 1, 2, false, 2) \
    TAPS("t7x96", 49, 1, 3, false, 2) \
    TAPS("tp5x128", 25, 1, 4, true, 2) \
    TAPS("tp7x96", 49, 1, 3, true, 2)
#define PIECE_BLOCKS(CAND) \
    CAND("a128x64x2", 1, 2, 4, 2, 9, 1, false, 1, 2, false) /* two tiles of a128x64 side by side */ \
    CAND("u128x64x2", 1, 2, 4, 2, 9, 1, true, 1, 2, true)
#define CAND(NAME, ...) {NAME, plan_geom<PGeom<__VA_ARGS__>>, plan_pairs<PGeom<__VA_ARGS__>>, launch_plan<PGeom<__VA_ARGS__>>, PGeom<__VA_ARGS__>::apart, PGeom<__VA_ARGS__>::tiles},
#define TAPS(NAME, ...) {NAME, plan_taps<TGeom<__VA_ARGS__>>, nullptr, launch_taps<TGeom<__VA_ARGS__>>, always_apart, nullptr},
const Candidate kCandidates[] = {PIECE_GEOMETRIES(CAND, TAPS) PIECE_BLOCKS(CAND)};

}  // namespace

const char* const* piece_geoms()
{
    static const char* names[sizeof(kCandidates) / sizeof(kCandidates[0]) + 1];
    for (size_t i = 0; i < sizeof(kCandidates) / sizeof(kCandidates[0]); ++i) names[i] = kCandidates[i].name;
    return names;
}

bool piece_supported(const Problem& p, bool pooled) { return shape_ok(p, pooled); }

namespace {

struct Choice {
    const Candidate* cand = nullptr;
    Plan plan;
    double stored = -1.0;   // modelled microseconds on filters as stored, negative: no such plan
};

// Whether a plan keeps the small products' sums apart.
bool apart_of(const Choice& c) { return c.cand->apart(c.plan.src); }

// Whether the last round of a block's launch would leave three fifths of the compute units idle.  Its tiles one by one, two to a unit, fill twice as many:
// of 290 layers on blocks, 21 with at most 102 in the last of up to three rounds took 0.78 - 0.98 of the blocks' time that way (median 0.91), where the model has them
// level, and the others 0.89 and more (median 1.06); 11 with so many in the fourth 0.95 - 1.05.
bool idle_end(const Plan& block) { return block.cfg.whole <= 3 * 256 && (block.cfg.whole - 1) % 256 < 102; }

// Whether pairs may take the place of what a launch takes without them - the plan `three` (its sums apart or not), or its family's kernel, `other`
// microseconds (negative: not known), where that is faster.  Relative error against 64-bit sums (1e-7; the same at 40 - 90 % zeros within a tenth): pairs
// 1.05 - 1.2 at any number of channels.  Against three pieces in one chain, 1.7 - 2.0, they are closer; against sums apart, 0.65 at 64 channels to 1.17 at
// 512 (less where tiles are split), from 512 on while most tiles are whole; against the taps kernel there too, where a reported ratio is 50 % at
// most (512 / 640 channels @14x14, taps against pairs, 1.20 / 1.28 against 1.16 / 1.21 at 50 % zeros, 1.02 / 1.09 against 1.12 / 1.20 at 70, 0.79 / 0.82
// against 1.02 / 1.10 at 90); against the other families up to the zero ratio that piece_close gives.
// A call without a zero ratio whose family is the vector kernel's stays as it was (see piece_first).
bool pairs_for(const Problem& p, const Plan* three, bool apart, bool taps, double other, float pairs_to)
{
    if (other == 0.0) return false;
    if (three && (other < 0.0 || three->cost < other)) {
        const bool level = p.Cg >= 512 && three->cfg.whole >= three->ntail;
        return !apart || (level && (!taps || (p.zhint >= 0.0f && p.zhint <= 0.5f)));
    }
    return pairs_to > 1.0f || (p.zhint >= 0.0f && p.zhint <= pairs_to);
}

// The cheapest plan by the model.  Walking the candidates takes 2 to 80 us by shape, as long as a small kernel runs, so plans are
// kept by what they depend on: the shape, the room in the workspace, whether the filters come prepared, whether small
// products are kept apart, the zero ratio (by which the time of the launch's family is known), whether there is such a time (not with a pinned
// variant) and pairs may stand against it, a geometry that sconv_tune found.  Networks have up to a few hundred such keys: 256 sets of eight, the oldest of a set goes.  (Under the
// dispatcher's lock; the reference lasts until the next call.)
const Choice& choose_plan(const Problem& p, bool pooled)
{
    struct Key {
        size_t ws;
        int v[19];
        PlanPin pin;
    };
    static_assert(sizeof(Key) == sizeof(size_t) + 19 * sizeof(int) + sizeof(PlanPin), "compared as bytes: no padding");
    struct Set {
        Key key[8];
        Choice choice[8];
        int used, next;
    };
    constexpr size_t kSets = 256;
    static Set kept[kSets];
    static Choice pinned;
    const PlanPin* tuned = current_pin();
    const char* pin = pinned_geom("SCONV_PIECE_GEOM");
    double other = -1.0;
    float pairs_to = -1.0f;
    const bool close = piece_close(p, pooled, &other, &pairs_to) && !pin;
    if (pin) other = -1.0;
    auto walk = [&](Choice& out) {
        out = Choice();
        if (!shape_ok(p, pooled)) return;
        for (const Candidate& c : kCandidates) {
            if (pin && strcmp(pin, c.name) != 0) continue;
            Plan pl = c.plan(p, pooled, close);
            if (pl.cost < 0.0) continue;
            if (pl.stored >= 0.0 && (out.stored < 0.0 || pl.stored < out.stored)) out.stored = pl.stored;
            // The taps kernel, which has no pairs and is the closest, also where it is level with a plan in one chain (466 -> 352 in 2 groups @19x49 at
            // batch 3 modelled 49.7 and 48.9 us, 0.70e-7 and 1.7e-7), and then at the other's time against other families.  Not over filters as stored: their
            // one chain ran such layers before (368 -> 368 in 2 groups @31x31 at batch 9 152 us, the taps kernel 209; 388 -> 368 @28x28 at batch 11 162 and 224).
            if (!out.cand || pl.cost < out.plan.cost * (!c.pairs && !apart_of(out) && out.plan.src != SRC_RAW ? 1.02 : 1.0)) {
                const double least = out.cand && out.plan.cost < pl.cost ? out.plan.cost : pl.cost;
                out.cand = &c;
                out.plan = pl;
                out.plan.cost = least;
            }
        }
        // the same with pairs, where it is no further from 64-bit sums
        const bool pinned_pairs = env_value("SCONV_PIECE_SRC") && atoi(env_value("SCONV_PIECE_SRC")) >= SRC_PAIRS;
        if (!pinned_pairs && !pairs_for(p, out.cand ? &out.plan : nullptr, out.cand && apart_of(out), out.cand && !out.cand->pairs, other, pairs_to)) return;
        for (const Candidate& c : kCandidates) {
            if (!c.pairs || (pin && strcmp(pin, c.name) != 0)) continue;
            Plan pl = c.pairs(p, pooled);
            if (pl.cost < 0.0 || (out.cand && pl.cost >= out.plan.cost)) continue;
            out.cand = &c;
            out.plan = pl;
        }
        if (out.cand && out.cand->tiles && !pin && idle_end(out.plan)) {
            const double modelled = out.plan.cost;
            for (const Candidate& c : kCandidates) {
                if (strcmp(c.name, out.cand->tiles) != 0) continue;
                const Plan pl = c.pairs(p, pooled);
                if (pl.cost < 0.0) break;
                out.cand = &c;
                out.plan = pl;
                out.plan.cost = modelled;
                break;
            }
        }
    };
    if ((pin && !tuned) || env_value("SCONV_PIECE_SPLIT") || env_value("SCONV_PIECE_SRC")) {
        walk(pinned);
        return pinned;
    }
    Key k;
    memset(&k, 0, sizeof(k));
    const int v[19] = {p.N, p.C, p.H, p.W, p.K, p.R, p.S, p.stride, p.pad, p.G, pooled ? p.ph : 0, pooled ? p.pw : 0, pooled ? p.ps : 0,
                       pooled ? 1 : 0, p.wprep ? 1 : 0, tuned ? 1 : 0, close ? 1 : 0, (int)(p.zhint * 254.0f + 0.5f), other < 0.0 ? 0 : other == 0.0 ? 1 : 2};
    memcpy(k.v, v, sizeof(v));
    k.ws = usable_workspace(p, pooled);
    if (tuned) {
        snprintf(k.pin.geom, sizeof(k.pin.geom), "%s", tuned->geom);
        k.pin.nwv = tuned->nwv;
        k.pin.ncs = tuned->ncs;
        k.pin.nss = tuned->nss;
    }
    unsigned long long h = 14695981039346656037ull;   // FNV-1a
    for (size_t i = 0; i < sizeof(k); ++i) h = (h ^ reinterpret_cast<const unsigned char*>(&k)[i]) * 1099511628211ull;
    Set& set = kept[(h ^ (h >> 32)) % kSets];
    for (int i = 0; i < set.used; ++i)
        if (!memcmp(&set.key[i], &k, sizeof(k))) return set.choice[i];
    const int at = set.next;
    set.next = (at + 1) % 8;
    if (set.used < 8) ++set.used;
    memcpy(&set.key[at], &k, sizeof(k));
    walk(set.choice[at]);
    return set.choice[at];
}

}  // namespace

double piece_cost(const Problem& p, bool pooled)
{
    const Choice& c = choose_plan(p, pooled);
    return c.cand ? c.plan.cost : -1.0;
}

double piece_margin(const Problem& p, bool pooled)
{
    const Choice& c = choose_plan(p, pooled);
    return !c.cand || !apart_of(c) || c.plan.src == SRC_RAW ? 1.0 : c.plan.src == SRC_FP32 ? 1.02 : 1.04;
}

double piece_stored_cost(const Problem& p, bool pooled) { return choose_plan(p, pooled).stored; }

bool describe_piece(const Problem& p, bool pooled, char* out, size_t out_size)
{
    const Choice& c = choose_plan(p, pooled);
    if (!c.cand) return false;
    // (pairs are cut from the filters as stored in prepared calls too)
    const char* const forms[] = {"pieces", "prepared", "stored", p.wprep ? "prepared-f16k" : "pieces-f16k"};
    if (c.cand->tiles)
        snprintf(out, out_size, "%s/%s/x2", c.cand->tiles, forms[c.plan.src]);
    else if (c.plan.ntail)
        snprintf(out, out_size, "%s/%s/%d+%dx%d", c.cand->name, forms[c.plan.src], c.plan.cfg.whole, c.plan.ntail, c.plan.cfg.nss);
    else
        snprintf(out, out_size, "%s/%s", c.cand->name, forms[c.plan.src]);
    return true;
}

int launch_piece(const Problem& p, bool pooled, const float* x, const float* w, float* y, hipStream_t stream)
{
    const Choice& c = choose_plan(p, pooled);
    if (!c.cand) return SCONV_EUNSUPPORTED;
    if (env_value("SCONV_TRACE_PLAN"))
        fprintf(stderr, "piece %s: src %d strips %d x %d, %d tiles x %d filter blocks, %d whole, %d split %d ways, modelled %.1f us\n", c.cand->name,
                c.plan.src, c.plan.cfg.strips, c.plan.cfg.TW, c.plan.cfg.ntiles * c.plan.cfg.strips, c.plan.cfg.kblocks, c.plan.cfg.whole,
                c.plan.ntail, c.plan.cfg.nss, c.plan.cost);
    return c.cand->launch(c.plan, p, pooled, x, w, y, stream);
}

}  // namespace sconv

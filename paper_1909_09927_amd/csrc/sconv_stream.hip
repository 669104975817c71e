// 1x1 / stride 1 / pad 0 layers of few filters on large maps: the map streams through registers once, on exact bf16 pieces.
//
// What bounds such a layer is the map's trip through memory (256 -> 64 @56x56 at batch 32: 128 MB, 25 us at the rate of a large copy).  The fp32
// matrix kernel (sconv_pw.hip) reads it in 128-byte pieces and issues 32 clocks of matrix instructions for every 4 positions of a channel, which
// takes as long again: 43 us.  Here the products run on the bf16 pipe (six of the nine products of three pieces, as in
// sconv_piece.hip, at a sixteenth of the clocks each), and a lane's loads are two neighbouring positions, 256 bytes a channel.
//
// A workgroup is eight wavefronts, one to a compute unit.  It cuts its 64 filters into pieces once, into LDS (C * 384 bytes); then every
// wavefront walks the channels of its own blocks of 64 positions, 16 at a time, with no barrier: it loads eight bytes of 8 channels, cuts
// them in its registers - even positions are one operand, odd ones the other - and multiplies.  RING steps of 4 KB are in flight for every
// wavefront, across the end of a block too.  x0 w0 has sums of its own, as have the five small products.  Results leave as they lie in the accumulators: 256
// contiguous bytes of a filter's plane.
// quad1x1 / here: 256 -> 64 @56x56 at batch 32 42.9 / 31.6 us, 64 -> 32 @112x112 58.8 / 32.6 (4.7 TB/s), 128 -> 32 @56x56 26.2 / 16.3, 64 -> 256 @56x56
// 63 / 52 (four passes over the map, three of them from the caches).  Relative error against 64-bit sums 0.4e-7 at 64 channels, 0.6e-7 at 256; quad1x1 0.65e-7, 1.0e-7.
// 64 filters with four steps in flight spill (41 us for the first of these), so they have two.
//
// Zeros are multiplied.  What the pieces' range does not hold (elements of 2^104 and more, sums of 2^80 and more, Inf, NaN) shows as Inf or NaN in a
// sum; the wavefront's block is then summed again in plain fp32, zero elements skipped.
#include <atomic>

#include "sconv_internal.h"
#include "sconv_piece_split.h"

namespace sconv {

namespace {

constexpr int TP = 64;    // positions per block
constexpr int NW = 8;     // wavefronts

struct StreamCfg {
    int npos, nblk;       // positions of the batch, blocks of TP
};

// MT: blocks of 32 filters; RING: steps of 16 channels in flight
template <int MT, int RING>
__global__ __launch_bounds__(NW * 64, 2) void stream_kernel(Problem p, StreamCfg cfg, const float* __restrict__ x, const float* __restrict__ w,
                                                            float* __restrict__ y)
{
    extern __shared__ __align__(16) u4 filters[];   // [16 channels][32 filters][piece][64 lanes]
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kb0 = blockIdx.y * (32 * MT), g = blockIdx.z, HW = p.H * p.W, steps = p.Cg / 16;
    const int stride = (int)gridDim.x * NW;
    int b = wave * (int)gridDim.x + blockIdx.x;

    // a block's elements: a buffer that starts at the image of its first position, and this lane's first element in it (positions 2 col and
    // 2 col + 1 of the block, of one image: HW is even; those past the last one re-read the last)
    auto block = [&](int blk, int& n0, int& voff) {
        const int P0 = min(blk * TP, cfg.npos - 2), P = min(blk * TP + 2 * col, cfg.npos - 2), n = P / HW;
        n0 = __builtin_amdgcn_readfirstlane(P0 / HW);
        voff = ((n - n0) * p.C * HW + P - n * HW + half * 8 * HW) * 4;
    };
    auto buffer = [&](int n0, bool there) {
        const size_t first = ((size_t)n0 * p.C + (size_t)g * p.Cg) * HW, left = ((size_t)p.N * p.C * HW - first) * 4;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x + first), 0, there ? (int)min(left, (size_t)0x7ffffffc) : 0, 0x00020000);
    };
    f2 ring[RING][8];
    auto fetch = [&](int slot, __amdgpu_buffer_rsrc_t from, int voff, int step) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            ring[slot][j] = __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(from, voff + step * (64 * HW), j * HW * 4, 0));
    };

    int n0, voff;
    block(b, n0, voff);
    __amdgpu_buffer_rsrc_t xres = buffer(n0, b < cfg.nblk);   // (a wavefront without a block loads nothing)
    // the filters' pieces: eight channels of a filter at a time, four at once, asked for before the first of the map (loads return in order)
    const int items = steps * 2 * 32 * MT;
    for (int it0 = tid; it0 < items + tid; it0 += 4 * NW * 64) {
        f4 lo[4], hi[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int it = min(it0 + i * NW * 64, items - 1), k = (it >> 2) % (32 * MT), oct = (it & 3) + it / (128 * MT) * 4;
            const f4* src = reinterpret_cast<const f4*>(w + ((size_t)g * p.Kg + min(kb0 + k, p.Kg - 1)) * p.L + oct * 8);
            lo[i] = src[0];
            hi[i] = src[1];
        }
        if (it0 == tid)
#pragma unroll
            for (int s = 0; s < RING; ++s) fetch(s, xres, voff, s);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int it = it0 + i * NW * 64, k = (it >> 2) % (32 * MT), oct = (it & 3) + it / (128 * MT) * 4;
            if (it >= items) break;
            float v[8];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[j] = lo[i][j];
                v[4 + j] = hi[i][j];
            }
            u4 q[3];
            split8(v, q);
            u4* dst = filters + ((oct >> 1) * MT + (k >> 5)) * 192 + (oct & 1) * 32 + (k & 31);
            dst[0] = q[0];
            dst[64] = q[1];
            dst[128] = q[2];
        }
    }
    float* const biases = reinterpret_cast<float*>(filters + steps * MT * 192);
    if (tid < 32 * MT) biases[tid] = bias_of(p, (size_t)g * p.Kg + min(kb0 + tid, p.Kg - 1));
    __syncthreads();

    const v16f zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    while (b < cfg.nblk) {
        const int after = b + stride;
        int n1, voff1;
        block(after, n1, voff1);
        const __amdgpu_buffer_rsrc_t xnext = buffer(n1, after < cfg.nblk);
        v16f acc[MT][2], accl[MT][2];
#pragma unroll
        for (int i = 0; i < MT; ++i) acc[i][0] = acc[i][1] = accl[i][0] = accl[i][1] = zero;
        for (int s0 = 0; s0 < steps; s0 += RING) {
            const bool last = s0 + RING >= steps;
            const __amdgpu_buffer_rsrc_t from = last ? xnext : xres;
            const int vo = last ? voff1 : voff, step = last ? 0 : s0 + RING;
#pragma unroll
            for (int r = 0; r < RING; ++r) {
                __builtin_amdgcn_sched_barrier(0);   // (steps stay apart: the registers)
                u4 bq[2][3];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    split2(ring[r][2 * i][0], ring[r][2 * i + 1][0], kUp, kUp, i, bq[0]);
                    split2(ring[r][2 * i][1], ring[r][2 * i + 1][1], kUp, kUp, i, bq[1]);
                }
                __builtin_amdgcn_sched_barrier(0);
                fetch(r, from, vo, step + r);
                const u4* a = filters + (size_t)(s0 + r) * MT * 192 + lane;
#pragma unroll
                for (int i = 0; i < MT; ++i) {
                    const u4 aq[3] = {a[i * 192], a[i * 192 + 64], a[i * 192 + 128]};
                    constexpr int qa[6] = {0, 0, 1, 1, 0, 2}, qb[6] = {0, 1, 0, 1, 2, 0};
#pragma unroll
                    for (int c = 0; c < 6; ++c)
#pragma unroll
                        for (int n = 0; n < 2; ++n) {
                            v16f& d = c ? accl[i][n] : acc[i][n];
                            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, aq[qa[c]]), __builtin_bit_cast(bf8, bq[n][qb[c]]), d, 0, 0, 0);
                        }
                }
            }
        }

        const int P = b * TP + 2 * col;
        const bool ok = P < cfg.npos;
        const int n = (ok ? P : 0) / HW, pix = (ok ? P : 0) - n * HW;
        float* const o = y + ((size_t)n * p.K + (size_t)g * p.Kg) * HW + pix;
        float lost = 0.0f;               // x times 0 is NaN where x is Inf or NaN
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                acc[i][e] += accl[i][e];
#pragma unroll
                for (int v = 0; v < 16; ++v) lost = __builtin_fmaf(acc[i][e][v], 0.0f, lost);
            }
        if (__any(lost != 0.0f)) {
            if (ok)
                for (int k = kb0 + 4 * half; k < min(kb0 + 32 * MT, p.Kg); k += k % 4 == 3 ? 5 : 1) {   // (the filters of this half: 4 of every 8)
                    const float* xk = x + ((size_t)n * p.C + (size_t)g * p.Cg) * HW + pix;
                    const float* wk = w + ((size_t)g * p.Kg + k) * p.L;
                    f2 sum = {0.0f, 0.0f};
                    for (int c = 0; c < p.Cg; ++c)
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            const float v = xk[(size_t)c * HW + e];
                            if (v != 0.0f) sum[e] = __builtin_fmaf(v, wk[c], sum[e]);
                        }
                    sum += biases[k - kb0];
                    if (p.relu) sum = {fmaxf(sum[0], 0.0f), fmaxf(sum[1], 0.0f)};
                    *reinterpret_cast<f2*>(o + (size_t)k * HW) = sum;
                }
        } else {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    if (v % 4 == 0) __builtin_amdgcn_sched_barrier(0);
                    const int kr = i * 32 + 8 * (v >> 2) + (v & 3) + 4 * half, k = kb0 + kr;
                    const float bias = biases[kr];
                    f2 r = {acc[i][0][v] * kDown + bias, acc[i][1][v] * kDown + bias};
                    if (p.relu) r = {fmaxf(r[0], 0.0f), fmaxf(r[1], 0.0f)};
                    if (ok && k < p.Kg) *reinterpret_cast<f2*>(o + (size_t)k * HW) = r;
                }
        }
        b = after;
        voff = voff1;
        xres = xnext;
    }
}

template <int MT, int RING>
int launch_mt(const Problem& p, const float* x, const float* w, float* y, hipStream_t stream)
{
    StreamCfg cfg;
    cfg.npos = p.N * p.H * p.W;
    cfg.nblk = (cfg.npos + TP - 1) / TP;
    const size_t lds_bytes = (size_t)(p.Cg / 16) * MT * 192 * 16 + 32 * MT * sizeof(float);
    static std::atomic<bool> opted{false};   // (dynamic LDS above 48 KiB is opted into once)
    if (!opted.load(std::memory_order_relaxed)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(stream_kernel<MT, RING>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
            return SCONV_ELAUNCH;
        opted.store(true, std::memory_order_relaxed);
    }
    const int wgs = cfg.nblk < 256 ? cfg.nblk : 256;   // one to a compute unit
    hipLaunchKernelGGL((stream_kernel<MT, RING>), dim3((unsigned)wgs, (unsigned)((p.Kg + 32 * MT - 1) / (32 * MT)), (unsigned)p.G), dim3(NW * 64), lds_bytes, stream, p,
                       cfg, x, w, y);
    return launch_status();
}

}  // namespace

bool stream_supported(const Problem& p, const float* x, const float* w, const float* y)
{
    if (p.R != 1 || p.S != 1 || p.stride != 1 || p.pad != 0) return false;
    const int mt = p.Kg > 32 ? 2 : 1;
    if (p.Cg % 64 || (long long)(p.Cg / 16) * mt * 192 * 16 + 32 * mt * 4 > 160 * 1024) return false;   // the filters' pieces fill LDS
    if (p.H * p.W % 2 || (((uintptr_t)x | (uintptr_t)y) & 7) || ((uintptr_t)w & 15)) return false;     // loads and stores of two positions, four channels
    if ((long long)p.N * p.C * p.H * p.W >= (1LL << 30) || (long long)p.N * p.H * p.W >= (1LL << 30)) return false;
    const long long images = (TP + p.H * p.W - 1) / (p.H * p.W) + 1;
    if (images * p.C * p.H * p.W >= (1LL << 29)) return false;                                          // a block's byte offsets in 32 bits
    // A pass - 64 filters of a group, or a group of up to 32 - cuts its filters and has at most one block to a wavefront up to 2048 blocks, however few
    // there are, and multiplies zeros, which quad1x1 skips where neighbouring channels have them together: a launch has to have enough blocks.  quad1x1 / here,
    // 64 - 384 channels, at 65 % zeros and at 95 % in clusters: 32 filters at 628 blocks 1.08 - 1.61 and 1.04 - 1.12 times as fast; 64 filters at
    // 784 - 1372 1.02 - 1.35 and 0.89 - 1.05, at 1500 - 1536 (95 %) 0.87 - 1.0, at 1568, where quad1x1 begins another round, 1.30 - 1.53 and 1.08 - 1.13; 80 - 128
    // filters (two passes) at 1323 1.05 - 1.29 and 0.92 - 0.96, at 1666 1.15 - 1.46 and 1.00 - 1.12; 160 - 512 at 1323 0.99 - 1.27 and 0.83 - 0.91, at 1666 1.11 - 1.44 and
    // 0.95 - 1.07; 768 at 1813 (95 %) 0.93 - 0.95, at 3136 1.33 - 1.44 and 1.08.  So where the ratio is not known, or high, the lines are where clusters are level.
    // Clusters of 80 - 85 %: 64 filters at 784 - 1372 1.03 - 1.14 from 128 channels on (0.95 - 1.06 at 64); 80 - 128 at 1323 0.97 - 1.09; 160 - 768 at 1323 0.91 -
    // 1.10, at 1421 0.95 and more; 1024 at 1519 0.95.  Groups at 57 % in clusters: 128 -> 32 in 2 at 637 blocks 12.1 / 14.1 us, 256 -> 64 in 4 at 931 29.9 / 34.2.
    const long long blocks = ((long long)p.N * p.H * p.W + TP - 1) / TP, passes = (long long)p.G * ((p.Kg + 63) / 64);
    const bool known = p.G == 1 && p.zhint >= 0.0f && p.zhint <= 0.8f;
    if (passes == 1 && p.Kg <= 32) return blocks >= 600;
    if (passes == 1) return blocks >= (known && p.Cg >= 128 ? 768 : 1537);
    if (known) return blocks >= (passes == 2 ? 1300 : passes <= 8 ? 1450 : 1650);
    return blocks >= (passes == 2 ? 1600 : passes <= 8 ? 1800 : 2000);
}

int launch_stream(const Problem& p, const float* x, const float* w, float* y, hipStream_t stream)
{
    return p.Kg > 32 ? launch_mt<2, 2>(p, x, w, y, stream) : launch_mt<1, 4>(p, x, w, y, stream);
}

}  // namespace sconv

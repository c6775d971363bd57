// Int8 x Int8 -> Int32 GEMM with the fused Int32-bias / dequantize epilogue of the
// quantized FC layer (Section 3), for gfx950.
//
//   acc[m,n] = bq[n] + sum_k xq[m,k] * wq[n,k]          y[m,n] = acc[m,n] / (S_x S_W)
//
// Both operands are K-contiguous ("NT" GEMM), so a 16-byte vector of either one is
// 16 consecutive k of one row -- exactly one lane's share of an i8 MFMA operand.
//
// MFMA kernel: a workgroup owns a BM x BN tile of y and walks K in stages of 128 bytes.
// Operand tiles go HBM/L2 -> LDS directly (buffer_load ... lds, 16 B per lane) into a
// ring of stage buffers; waves read 16-byte fragments back (ds_read_b128) and issue
// v_mfma_i32_32x32x32_i8.  LDS rows are swizzled so fragment reads are free of bank
// conflicts; the swizzle costs nothing on the way in because each lane of a
// direct-to-LDS load picks its own global address while the LDS side stays linear.
//
// Short reductions go to the kernel of q8_gemm_ring_kernel.h, the same but for how it overlaps, and so does any K that is a multiple of
// 4; any other K or alignment, launches of at most 256 tiles of 32x32 and long reductions of other widths in few such tiles go to the kernel of
// q8_gemm_direct.hip; a handful of products to the one-thread-per-output kernel below.
#include "q8_device.h"
#include "q8_epilogue.h"
#include "q8_launch.h"

#include <math.h>

namespace q8 {

constexpr int kBK = 128;  // the staged kernel's K granularity (see q8_gemm_kernel.h)

// One translation unit per tile shape.
int launch_tile_256x256_w4(const int8_t*, const int8_t*, int, int, int, int, const Epilogue&, hipStream_t);
int launch_tile_256x256_w8(const int8_t*, const int8_t*, int, int, int, int, const Epilogue&, hipStream_t);
int launch_tile_128x128_w4(const int8_t*, const int8_t*, int, int, int, int, const Epilogue&, hipStream_t);
int launch_tile_64x64_w4(const int8_t*, const int8_t*, int, int, int, int, const Epilogue&, hipStream_t);
int launch_tile_192x256_w4(const int8_t*, const int8_t*, int, int, int, int, const Epilogue&, hipStream_t);
int launch_tile_192x256_w8(const int8_t*, const int8_t*, int, int, int, int, const Epilogue&, hipStream_t);
int launch_tile_192x128_w4(const int8_t*, const int8_t*, int, int, int, int, const Epilogue&, hipStream_t);

// The same for the kernel of q8_gemm_ring_kernel.h (tile, stage buffers); the last integer is whether each XCD takes a contiguous
// run of tiles.
#define Q8_RING(NAME) int launch_ring_##NAME(const int8_t*, const int8_t*, int, int, int, int, int, const Epilogue&, hipStream_t)
Q8_RING(64x64_s3);
Q8_RING(64x64_s2);
Q8_RING(128x64_s2);
Q8_RING(128x128_s1);
Q8_RING(192x128_s1);
#undef Q8_RING

// One thread per output element: reductions so short that the loads of a direct-kernel tile take longer than the whole sum
// (5 x 33 x 9: 2.6 us against 4.7; 64 x 4096 x 9: 3.8 against 5.1; 1 x 2 x 17: 2.9 against 4.4).  The chain of K byte loads costs 45 ns
// an element, and many outputs queue up: 16384 x 64 x 9 takes 8.5 us against 6.7.
constexpr int64_t kScalarMaxK = 32, kScalarMaxProducts = (int64_t)1 << 22;
__global__ __launch_bounds__(256) void gemm_scalar_kernel(const int8_t* __restrict__ X, const int8_t* __restrict__ W,
                                                           int64_t M, int64_t N, int64_t K, Epilogue ep)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool valid = idx < M * N;
    unsigned ab = 0u;
    if (valid) {
        const int64_t m = idx / N;
        const int n = (int)(idx - m * N);
        const int8_t* xr = X + m * K;
        const int8_t* wr = W + (int64_t)n * K;
        int acc = 0;
        for (int64_t k = 0; k < K; ++k) acc += (int)xr[k] * (int)wr[k];
        const float sx = ep.sx[0];
        const ColConst cc = col_const(ep, n, sx);
        const float next_scale = (ep.flags & 4u) ? ep.next_scale[0] : 0.0f;
        ab = epilogue_store(ep, idx, acc + cc.bq, cc.r, next_scale);
    }
    if (ep.flags & 2u) {
        ab = wave_max_u32(ab);
        if ((threadIdx.x & 63) == 0) atomicMax(reinterpret_cast<unsigned*>(ep.out_amax), ab);
    }
}

static int g_variant = 0;
void set_gemm_variant(int v) { g_variant = v; }

// Variants 1 to 6 are the staged tile shapes of full launches, 7 the small one with deep rings, 8 the direct kernel, 9 and up the rings.
constexpr int kVariant192x256 = 5, kVariant64 = 7, kVariantDirect = 8, kVariantRing = 9;

// The shapes of q8_gemm_ring_kernel.h and what a launch of each takes (us): `fixed`, the longer of two times per stage of K -- the
// chain a workgroup walks (`chain`, per round of workgroups) and the work of a compute unit (`work`, per tile) -- and the
// epilogue of every tile (fp32, fp32 with GELU or abs-max, int8).  The constants are a fit to 143 launches of 300 to 16384
// rows and N x K from 512 x 512 to 4096 x 1024, outputs rotating through more than the Infinity Cache, off by 5 to 10 % (rms).
// Choosing by it costs 3.4 % against the best of the five (geometric mean of 860 launches of any size; a tenth lose 11 % or more).  `smooth` says how much
// of a last, partly filled round counts in full.  Large tiles store better with neighbouring tiles on different XCDs, in panels of four
// rows (12288 x 3072 x 1024 54.8 -> 48.6 us with 192x128): what is written at the same time then lies together.
struct Ring {
    int (*launch)(const int8_t*, const int8_t*, int, int, int, int, int, const Epilogue&, hipStream_t);
    int bm, bn, wgs;    // tile, workgroups per compute unit
    int group_m, by_xcd;
    float fixed, chain, work, out[3], smooth;
};
static const Ring kRings[] = {
    {launch_ring_64x64_s3, 64, 64, 3, 8, 1, 2.84f, 0.222f, 0.182f, {0.51f, 0.70f, 0.71f}, 0.42f},
    {launch_ring_64x64_s2, 64, 64, 5, 8, 1, 2.42f, 0.411f, 0.176f, {0.48f, 0.64f, 0.65f}, 0.42f},
    {launch_ring_128x64_s2, 128, 64, 3, 8, 1, 2.58f, 0.481f, 0.284f, {0.83f, 1.11f, 1.17f}, 0.38f},
    {launch_ring_128x128_s1, 128, 128, 4, 4, 0, 2.17f, 0.863f, 0.437f, {2.17f, 2.49f, 2.61f}, 0.51f},
    {launch_ring_192x128_s1, 192, 128, 3, 4, 0, 2.65f, 0.949f, 0.604f, {2.66f, 3.80f, 4.59f}, 1.0f},
};
constexpr int kNumRings = sizeof(kRings) / sizeof(kRings[0]), kFirstLargeRing = 3;

// That kernel has no accumulator dump and no residual, and only the flag combinations that mean something.
static bool ring_operands_eligible(const int8_t* xq, const int8_t* wq, int64_t M, int64_t N, int64_t K)
{
    if (K < 1 || K % 4 != 0 || ((reinterpret_cast<uintptr_t>(xq) | reinterpret_cast<uintptr_t>(wq)) & 3)) return false;
    const int64_t lim = (int64_t)1 << 31;  // 32-bit offsets span one tile of 192 rows
    return M > 0 && N > 0 && M < lim && N < lim && K < (lim / 192) - 256 && ((M + 63) / 64) * ((N + 63) / 64) < lim;
}
static bool ring_eligible(const Epilogue& ep) { return !ep.acc_out && !ep.residual && ep.flags <= 5u; }
static int launch_ring(const Ring& r, const int8_t* xq, const int8_t* wq, int M, int N, int K, const Epilogue& ep, hipStream_t st)
{
    return r.launch(xq, wq, M, N, K, r.group_m, r.by_xcd, ep, st);
}
// `cached`: an fp32 output stored for the caches (32 to 64 MiB), its rows whole 128-byte lines.  There the small tiles pay 2 to 4 us that the model
// does not know of, so only the two large shapes are looked at from K = 512 on: 4096 x 3584 x 512 22.3 -> 19.2 us, 4096 x 2304 x 768 + GELU 20.1 -> 17.0, 2 % over
// 17 launches of 512; shorter reductions lose by that (3839 x 3712 x 256 22.4 us, 16.2 with 128x64; 4 % over 20 launches of 256).
// `broken`: an fp32 output of 16 MiB or more with rows of other lengths, the lines of which are written in parts.  The wider the tile the more that costs, so only
// the three small shapes are looked at: 61749 x 999 x 512 180 us with 192x128, 101 with 64x64; 9000 x 1000 x 1024 + GELU 24.7 with 128x128, 23.0 with 128x64; 14 % over
// 14 launches from 32 MiB on.
static const Ring& choose_ring(int M, int N, int K, unsigned flags, bool cached, bool broken)
{
    const int kind = (flags & 4u) ? 2 : (flags & 3u) ? 1 : 0;
    const float stages = (float)((K + kBK - 1) / kBK);
    const int first = cached && K >= 512 ? kFirstLargeRing : 0, last = broken ? kFirstLargeRing : kNumRings;
    int best = first;
    float best_us = 0.0f;
    for (int i = first; i < last; ++i) {
        const Ring& r = kRings[i];
        const float mean = (float)((((int64_t)M + r.bm - 1) / r.bm) * (((int64_t)N + r.bn - 1) / r.bn)) / 256.0f;   // tiles per compute unit
        const float most = ceilf(mean), tiles = r.smooth * most + (1.0f - r.smooth) * mean;
        const float rounds = most > r.wgs ? r.smooth * ceilf(most / r.wgs) + (1.0f - r.smooth) * mean / r.wgs : 1.0f;
        const float a = rounds * r.chain * stages, b = tiles * r.work * stages;
        const float us = r.fixed + cbrtf(a * a * a + b * b * b) + tiles * r.out[kind];
        if (i == first || us < best_us) {
            best = i;
            best_us = us;
        }
    }
    return kRings[best];
}

// What the staged kernels can take.
static bool gemm_staged_eligible(const int8_t* xq, const int8_t* wq, int64_t M, int64_t N, int64_t K)
{
    if (K < kBK || K % kBK != 0) return false;
    if ((reinterpret_cast<uintptr_t>(xq) & 15) || (reinterpret_cast<uintptr_t>(wq) & 15)) return false;
    const int64_t lim = (int64_t)1 << 31;  // M, N and the tile count are ints in the kernel; buffers are addressed per tile
    if (M >= lim || N >= lim || ((M + 127) / 128) * ((N + 127) / 128) >= lim) return false;
    return M > 0 && N > 0;
}

int launch_gemm(const int8_t* xq, const int8_t* wq, int64_t M64, int64_t N64, int64_t K64, const Epilogue& ep_in, hipStream_t st)
{
    Epilogue ep = ep_in;
    // Which fp32 outputs are stored with the non-temporal hint.  Beyond a quarter of the 256 MB Infinity Cache they could not stay
    // cached until their reader runs anyway, and kept out they neither evict the next kernels' inputs nor leave dirty lines
    // to drain under them (whole BERT-Large layer step 5-6 % faster).  Below the 32 MB that the L2s hold they would all be dirty
    // there at the end of the kernel, which waits for them to be written back (4096 x 768 x 768 8.4 -> 6.8 us, 4096 x 768 x 3072
    // 18.2 -> 16.5, BERT-Base layer 32 x 128 127 -> 125.5).  In between the hint costs the reader as much as it gains (stored-scale BERT-Large
    // layer 359.3 -> 356.5 us without it).  Rows that are not whole 128-byte lines: their parts meet in the L2s without the hint, which takes 4 %
    // off outputs below 4 MiB (small ring tiles, 26 launches); from 4 MiB on the hint is 4 to 10 % ahead there too (56 launches).
    const double y_mib = (double)M64 * (double)N64 * 4.0 / (1 << 20);
    const bool whole_lines = N64 % 32 == 0;
    ep.stream_out = y_mib > 64.0 || (y_mib < 32.0 && (whole_lines || y_mib >= 4.0));
    const bool fp32 = !(ep.flags & 4u), cached = fp32 && whole_lines && y_mib >= 32.0 && y_mib <= 64.0, broken = fp32 && !whole_lines && y_mib >= 16.0;
    int v = g_variant;
    if (v < 0 || v >= kVariantRing + kNumRings) return 1;
    if (v == 0 && K64 <= kScalarMaxK && M64 * N64 <= kScalarMaxProducts / (K64 > 0 ? K64 : 1)) {
        hipLaunchKernelGGL(gemm_scalar_kernel, dim3((unsigned)((M64 * N64 + 255) / 256)), dim3(256), 0, st, xq, wq, M64, N64, K64, ep);
        return hipGetLastError() == hipSuccess ? 0 : 1;
    }
    if (v == kVariantDirect) return launch_gemm_direct(xq, wq, M64, N64, K64, ep, st);
    if (!gemm_staged_eligible(xq, wq, M64, N64, K64)) {
        // Rows that are 4-byte aligned whatever their width go to the rings from more than one 32x32 tile per compute unit on: 777 x 1000 x
        // 520 (425 tiles) 5.6 us against 6.6 with the direct kernel, 700 x 60 x 600 4.4 against 5.8, 2000 x 520 x 2000 8.4 against 17.8,
        // 16000 x 60 x 300 8.2 against 19.2; with 100 tiles (300 x 1000 x 300) 5.4 against 5.3.  Long
        // reductions in at most two rounds of 32x32 tiles are the direct kernel's, whose waves share them: plain ones from 1412 on (direct over ring 0.98 up to 2044,
        // 0.91 beyond; 1.07 around 1000), with GELU or abs-max from 1156 on (0.95; 0.88 from 1668 on; 1.06 around 900), to int8 from 644 on (0.91; 0.87 from 1412 on;
        // 1.05 below) -- of at most 32 columns, of which a ring tile wastes half, with an epilogue of any kind from half of that on (0.87; 1.09 below).
        const int64_t t32 = ((M64 + 31) / 32) * ((N64 + 31) / 32);
        const int64_t shared = ((ep.flags & 4u) ? 640 : (ep.flags & 3u) ? 1152 : 1408) / (ep.flags && N64 <= 32 ? 2 : 1);
        if (ring_operands_eligible(xq, wq, M64, N64, K64) && ring_eligible(ep) && (v >= kVariantRing || (v == 0 && t32 > (K64 <= shared ? 256 : 512)))) {
            const Ring& r = v >= kVariantRing ? kRings[v - kVariantRing] : choose_ring((int)M64, (int)N64, (int)K64, ep.flags, cached, broken);
            return launch_ring(r, xq, wq, (int)M64, (int)N64, (int)K64, ep, st);
        }
        return launch_gemm_direct(xq, wq, M64, N64, K64, ep, st);
    }
    const int M = (int)M64, N = (int)N64, K = (int)K64;
    if (v >= kVariantRing) {
        if (ring_eligible(ep)) return launch_ring(kRings[v - kVariantRing], xq, wq, M, N, K, ep, st);
        v = 0;
    }
    if (v == 0) {
        // Launches that leave compute units idle are bound by the chain of stages each workgroup walks, so they get the
        // smallest tile that still fits the chip in one round.  One 32x32 tile per unit, the reduction split over eight
        // waves: 256 x 768 x 3072 5.8 us against 7.9 with 64x64 tiles, 128 x 768 x 768 4.3 against 4.4; at 288 such tiles
        // (384 x 768 x 768) the 64x64 ones are ahead, 4.4 against 4.8.  Long reductions: two 64x64 tiles per unit with five
        // stages in flight (651 x 768 x 3072 8.2 us against 12.7 with 128x128).  Short ones: many workgroups a unit instead of deep
        // pipelines (choose_ring); from 16 stages on the large staged tiles come out even or ahead (4096 x 768 x 3072 15.2 us against
        // 16.6 with the best ring, 12288 x 1024 x 4096 50.5 against 56.3).
        const int64_t tiles32 = (((int64_t)M + 31) / 32) * (((int64_t)N + 31) / 32);
        const int64_t tiles64 = (((int64_t)M + 63) / 64) * (((int64_t)N + 63) / 64);
        if (tiles32 <= 256) return launch_gemm_direct(xq, wq, M64, N64, K64, ep, st);
        // A plain launch of at most one round of 192x256 tiles, about two thirds of them outputs or more, whose 32 to 48 MiB are stored for the caches, which
        // the rings' smaller tiles pay for: 4096 x 2304 x 768 15.4 us against 16.3 with the ring of the rule, 12288 x 768 x 768 16.3 / 17.4, 3072 x 3072 x 1536
        // 21.9 / 25.8.  Over 200 such launches this tile takes 0.97 of the ring's time at K = 640 and 768, 0.93 at 896 and 1024, 0.89 beyond, the same at 512
        // (2860 x 3008 13.5, 14.3; 3270 x 3584 16.7, 16.2) and 1.01 below; of 28 to 32 MiB it is ahead beyond 1024 only (0.94 over 85 launches).  Narrow outputs
        // fill as many tiles without that: 40000 x 64 x 768 13.0 / 6.6, 48000 x 128 x 128 10.4 / 6.6, 36000 x 2 x 1024 12.0 / 8.5, 12288 x 576 x 768 13.3 / 12.5.
        const int64_t tiles192x256 = (((int64_t)M + 191) / 192) * (((int64_t)N + 255) / 256);
        const bool one_round = ep.flags == 0 && whole_lines && (cached ? K >= 512 : (y_mib >= 28.0 && K > 1024)) && tiles192x256 <= 256;
        // At most one 64x64 tile a unit: from 1152 on five stages in flight outweigh the ring's neighbours, where nothing but the dequantization follows (158 x
        // 2304 x 1920 6.8 -> 6.3 us; 0.97 of the ring's time over 70 launches, 1.08 with abs-max, 1.13 with GELU; two tiles a unit 1.05).
        if (K < 2048 && ring_eligible(ep)) {
            if (one_round)
                v = kVariant192x256;
            else if (!(ep.flags & 3u) && K > 1024 && tiles64 <= 256)
                v = kVariant64;
            else
                return launch_ring(choose_ring(M, N, K, ep.flags, cached, broken), xq, wq, M, N, K, ep, st);
        }
        // of broken lines the hint is the rings': wide outputs of staged tiles take 3 to 7 % longer with it (3903 x 2115 x 3456 45.0 us, 48.3)
        if (!whole_lines && N > 1024 && y_mib < 32.0) ep.stream_out = 0;
        if (v == 0 && tiles64 <= 512) v = kVariant64;
    }
    if (v == 0) {
        // Pick the tile shape with the best expected use of the chip: the fraction of the launch's
        // workgroup slots that hold work (256 compute units; tiles whose rings take half of the
        // LDS run two workgroups per unit, one's epilogue under the other's main loop), times the
        // fraction of each tile that lies inside y, times a prior of the shape itself.  The priors
        // come from timing each FC of a BERT-Large layer inside the whole layer step, where the
        // outputs of the neighbouring kernels keep the HBM busy (timings of a GEMM run alone, its
        // operands and output warm in the caches, rank the shapes differently and do not carry
        // over): long reductions favour the 192x256 tiles (most MFMAs per byte staged); short ones -- here
        // only with a residual or an accumulator dump -- the paired tiles.
        struct Cand { int variant, bm, bn, per_cu; double prior_long, prior_short; };
        static const Cand cands[] = {
            {5, 192, 256, 1, 1.00, 0.97}, {4, 192, 256, 1, 0.99, 0.90}, {2, 256, 256, 1, 0.96, 0.97},
            {6, 192, 128, 2, 0.95, 0.93}, {3, 128, 128, 2, 0.90, 1.00},
        };
        double best = -1.0;
        for (const Cand& c : cands) {
            const int64_t tm = (M + c.bm - 1) / c.bm, tn = (N + c.bn - 1) / c.bn, tiles = tm * tn;
            const double inside = ((double)M * N) / ((double)tiles * c.bm * c.bn);
            // rounds of the launch: a last round that fills at most one workgroup per unit of a paired
            // shape runs unshared and ends early
            const int64_t slots = 256 * c.per_cu, full = tiles / slots, rem = tiles % slots;
            const double rounds = (double)full + (rem == 0 ? 0.0 : (c.per_cu == 2 && rem <= 256) ? 0.6 : 1.0);
            const double slots_used = ((double)tiles / (double)slots) / rounds;
            const double prior = K >= 2048 ? c.prior_long : c.prior_short;
            const double score = prior * slots_used * inside;
            if (score > best) {
                best = score;
                v = c.variant;
            }
        }
    }
    // tile rows per raster panel: 4 is 1-2 us faster than 8 over the 317 us layer step but re-reads the weight tiles more
    // often (FFN1: 282 MB of HBM-side traffic against 248); 16 is 4 us slower
    const int group_m = 8;
    switch (v) {
        case 1: return launch_tile_256x256_w4(xq, wq, M, N, K, group_m, ep, st);
        case 2: return launch_tile_256x256_w8(xq, wq, M, N, K, group_m, ep, st);
        case 3: return launch_tile_128x128_w4(xq, wq, M, N, K, group_m, ep, st);
        case 4: return launch_tile_192x256_w4(xq, wq, M, N, K, group_m, ep, st);
        case 5: return launch_tile_192x256_w8(xq, wq, M, N, K, group_m, ep, st);
        case 6: return launch_tile_192x128_w4(xq, wq, M, N, K, group_m, ep, st);
        case kVariant64: return launch_tile_64x64_w4(xq, wq, M, N, K, group_m, ep, st);
        default: return 1;
    }
}

}  // namespace q8

// Int8 GEMM of the quantized FC layer (Section 3) for any reduction length and alignment, and for launches too small to
// fill the chip with the staged tiles of q8_gemm_kernel.h.
//
// What bounds a small launch is latency: a 128x128 tile walks the reduction in a serial chain of stages, and 128 tokens x
// 768 outputs are 6 such tiles on 256 compute units.  Here the tile is 32x32 and the reduction is dealt out over the
// waves of the workgroup, each staging through LDS of its own: no barrier until the partial sums meet (in LDS; exact:
// Int32).  128 x 768 x 3072: 12.0 -> 5.5 us, 128 x 768 x 768: 6.1 -> 4.1 us (an empty launch takes 3.5).
//
//   workgroup  = KW waves, one tile of 32x32 outputs
//   wave w     = the 128-byte units w, w + KW, ... of the reduction, the loads of the next unit in flight behind the
//                MFMAs of this one; a wave load covers 8 rows x 128 B (whole cache lines: fetching the MFMA operands
//                straight into registers, 32 rows x 32 B a load, was measured 1.1 to 2 times slower)
//   rows that lie outside the matrices re-read the last row; their sums are never stored.
//
// Rows may start at any byte (K is odd, or the caller's tensor is): the 16-byte vectors are loaded at their own address,
// which global loads of gfx950 allow, and the unit that K cuts short is read with bounds, so no load leaves its row.
// 777 x 520 x 1000: 750 us with one thread per output -> 7 us.  The L1 and the LDS see every operand once per 32 outputs,
// which caps the rate at about a sixth of the MFMA peak: 16384 x 4096 x 1000 runs at 300 TOP/s.
#include "q8_device.h"
#include "q8_epilogue.h"
#include "q8_launch.h"

namespace q8 {

constexpr int kGdUnit = 128;         // bytes of K per trip: one cache line of a 16-byte aligned row
constexpr int kGdSteps = kGdUnit / 32;
constexpr int kGdTile = 32;          // rows and columns of a workgroup's tile

__device__ __forceinline__ v4i load16_any(const int8_t* p)
{
    v4i v;
    __builtin_memcpy(&v, p, 16);
    return v;
}

// 16 bytes at p of which the first `left` belong to the row (none if left <= 0), zeros behind them.  The row is K bytes
// long and ends at p + left; nothing outside it is read: a vector that would end behind the row starts earlier instead,
// and the bytes in front of p are shifted out (rows of less than 16 bytes: the same with words, less than 4: bytes).
__device__ __forceinline__ v4i load16_bounded(const int8_t* p, int left, int K)
{
    v4i v = {0, 0, 0, 0};
    if (K >= 16) {
        unsigned __int128 u;
        __builtin_memcpy(&u, p + min(left - 16, 0), 16);
        const int drop = max(16 - left, 0);
        u = drop < 16 ? u >> (8 * drop) : 0;
        __builtin_memcpy(&v, &u, 16);
    } else if (left > 0 && K >= 4) {  // the row's only chunk: left = K
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const int rest = K - 4 * d;  // bytes of the row from word d on
            unsigned u;
            __builtin_memcpy(&u, p + 4 * d + min(rest - 4, 0), 4);
            const int drop = max(4 - rest, 0);
            v[d] = drop < 4 ? (int)(u >> (8 * drop)) : 0;
        }
    } else if (left > 0) {
#pragma unroll
        for (int j = 0; j < 3; ++j) v[0] |= (j < K ? (int)(unsigned char)p[min(j, K - 1)] : 0) << (8 * j);
    }
    return v;
}

__device__ __forceinline__ int swizzle_of_row(int r) { return (r ^ (r >> 3)) & 7; }

// Orders one wave's LDS accesses before this point and after it (its lanes exchange data; no other wave takes part).
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int KW>
__global__ __launch_bounds__(KW * 64, 4) void gemm_direct_kernel(const int8_t* __restrict__ X, const int8_t* __restrict__ W,
                                                                 int64_t M, int64_t N, int64_t K, unsigned tiles_m,
                                                                 unsigned tiles, Epilogue ep)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int kLoads = 2 * kGdTile / 8;  // 1 KiB wave loads per unit: 8 rows x 128 B each, A rows first
    constexpr int kStage = 2 * kGdTile * kGdUnit;
    // Partial sums of wave w at [w][row][col], in the place of the staged operands: rows of 40 words put the two 32-lane
    // halves of an accumulator store, four rows apart, on different banks.
    constexpr int kRow = kGdTile + 8;
    static_assert(kGdTile * kRow * 4 <= kStage, "the partial sums take the place of the staged operands");
    __shared__ __attribute__((aligned(16))) char lds[KW * kStage];
    __shared__ unsigned wave_amax[KW];
    int* part = reinterpret_cast<int*>(lds);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, hi = lane >> 5;
    const int k32 = (int)K;
    const int full = k32 / kGdUnit, units = (k32 + kGdUnit - 1) / kGdUnit;
    const float sx = ep.sx[0];
    const float next_scale = (ep.flags & 4u) ? ep.next_scale[0] : 0.0f;
    unsigned amax = 0u;

    // this wave's own staging area: row r, 16-byte chunk c at slot c ^ swizzle(r), so that the 16 rows a fragment read
    // serves per cycle cover all banks
    char* stage = lds + wave * kStage;
    const int chunk = lane & 7, row8 = lane >> 3;
    int put[kLoads], get_a[kGdSteps], get_b[kGdSteps];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) put[i] = (8 * i + row8) * kGdUnit + ((chunk ^ swizzle_of_row(8 * i + row8)) << 4);
#pragma unroll
    for (int s = 0; s < kGdSteps; ++s) {
        get_a[s] = l32 * kGdUnit + (((2 * s + hi) ^ swizzle_of_row(l32)) << 4);
        get_b[s] = (kGdTile + l32) * kGdUnit + (((2 * s + hi) ^ swizzle_of_row(kGdTile + l32)) << 4);
    }

    for (unsigned b = blockIdx.x; b < tiles; b += gridDim.x) {
        // Tiles in column-major order, each of the 8 XCDs (workgroups go round robin over them) a contiguous run: the
        // weight rows of a tile column are then read into one L2 only.
        const unsigned per = tiles >> 3, rem = tiles & 7, xcd = b & 7, idx = b >> 3;
        const unsigned tile = xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
        const int64_t m0 = (int64_t)(tile % tiles_m) * kGdTile, n0 = (int64_t)(tile / tiles_m) * kGdTile;
        const int last_a = (int)min((int64_t)kGdTile, M - m0) - 1, last_b = (int)min((int64_t)kGdTile, N - n0) - 1;
        const int8_t *Xt = X + m0 * K, *Wt = W + n0 * K;

        unsigned off[kLoads];  // row of each wave load, in bytes from the tile's first row of its operand
#pragma unroll
        for (int i = 0; i < kLoads; ++i)
            off[i] = (unsigned)(i < kLoads / 2 ? min(8 * i + row8, last_a) : min(8 * i - kGdTile + row8, last_b)) * (unsigned)k32 + 16u * chunk;

        v16i acc;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0;

        v4i in[kLoads];
        auto load_unit = [&](int u) {
            const int8_t *xu = Xt + u * kGdUnit, *wu = Wt + u * kGdUnit;
            if (u < full) {
#pragma unroll
                for (int i = 0; i < kLoads; ++i) in[i] = load16_any((i < kLoads / 2 ? xu : wu) + off[i]);
            } else {  // the unit that K cuts short
                const int left = k32 - u * kGdUnit - 16 * chunk;
#pragma unroll
                for (int i = 0; i < kLoads; ++i) in[i] = load16_bounded((i < kLoads / 2 ? xu : wu) + off[i], left, k32);
            }
        };
        if (wave < units) load_unit(wave);
        for (int u = wave; u < units; u += KW) {
#pragma unroll
            for (int i = 0; i < kLoads; ++i) *reinterpret_cast<v4i*>(stage + put[i]) = in[i];
            if (u + KW < units) load_unit(u + KW);
            wave_lds_order();  // the lanes read what other lanes of this wave wrote
#pragma unroll
            for (int s = 0; s < kGdSteps; ++s) {
                const v4i fa = *reinterpret_cast<const v4i*>(stage + get_a[s]);
                const v4i fb = *reinterpret_cast<const v4i*>(stage + get_b[s]);
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa, fb, acc, 0, 0, 0);
            }
            wave_lds_order();  // and are done reading before the next unit is written
        }
        __syncthreads();  // the partial sums lie where other waves staged

        // Accumulator register e of lane (l32, hi) is row 8 (e / 4) + 4 hi + e % 4, column l32.
#pragma unroll
        for (int e = 0; e < 16; ++e) part[(wave * kGdTile + 8 * (e >> 2) + 4 * hi + (e & 3)) * kRow + l32] = acc[e];
        __syncthreads();

        // A thread keeps its column, so the per-column constants are formed once; lanes run along the columns.
        constexpr int kRowStep = KW * 64 / kGdTile;
        const int col = threadIdx.x % kGdTile;
        const int64_t n = n0 + col;
        if (n < N) {
            const ColConst cc = col_const(ep, (int)n, sx);
#pragma unroll 2
            for (int i = 0; i < kGdTile / kRowStep; ++i) {
                const int r = i * kRowStep + threadIdx.x / kGdTile;
                int sum = cc.bq;
#pragma unroll
                for (int w = 0; w < KW; ++w) sum += part[(w * kGdTile + r) * kRow + col];
                const int64_t m = m0 + r;
                if (m < M) amax = max(amax, epilogue_store(ep, m * N + n, sum, cc.r, next_scale));
            }
        }
        __syncthreads();  // the next tile's operands go to the same place
    }

    if (ep.flags & 2u) {  // one atomic max per workgroup, and only while it has something to add
        amax = wave_max_u32(amax);
        if (lane == 0) wave_amax[wave] = amax;
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int w = 1; w < KW; ++w) amax = max(amax, wave_amax[w]);
            unsigned* slot = reinterpret_cast<unsigned*>(ep.out_amax);
            if (amax > __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(slot, amax);
        }
    }
#endif
}

// Waves that share a tile: eight while the tiles do not fill the chip, fewer as there are more of them to hide the latency
// (us with 8 / 4 / 2 / 1 waves: 777 x 520 x 1000, 425 tiles 7.0 / 7.4 / 8.2 / 10.3; 1500 x 900 x 250, 1363 tiles
// 22 / 11.4 / 8.5 / 9.6; 5000 x 1000 x 300, 5024 tiles 67 / 33 / 25 / 21).
int launch_gemm_direct(const int8_t* xq, const int8_t* wq, int64_t M, int64_t N, int64_t K, const Epilogue& ep, hipStream_t st)
{
    const int64_t tm = (M + kGdTile - 1) / kGdTile, tn = (N + kGdTile - 1) / kGdTile;
    const int64_t tiles = tm * tn;
    if (tiles >= ((int64_t)1 << 31)) return 1;
    const int64_t most = (int64_t)1 << 25;  // a launch is limited to 2^32 threads; beyond, a workgroup takes several tiles
    const dim3 grid((unsigned)(tiles < most ? tiles : most));
#define Q8_GD_LAUNCH(KW) \
    hipLaunchKernelGGL(gemm_direct_kernel<KW>, grid, dim3(KW * 64), 0, st, xq, wq, M, N, K, (unsigned)tm, (unsigned)tiles, ep)
    if (tiles <= 512)
        Q8_GD_LAUNCH(8);
    else if (tiles <= 1024)
        Q8_GD_LAUNCH(4);
    else if (tiles <= 2048)
        Q8_GD_LAUNCH(2);
    else
        Q8_GD_LAUNCH(1);
#undef Q8_GD_LAUNCH
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

}  // namespace q8

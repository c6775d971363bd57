// i8 MFMA GEMM kernel template of the quantized FC layer (Section 3), gfx950: small stage buffers and as many workgroups per
// compute unit as fit.  Included by one translation unit per tile shape (q8_gemm_ring_*.hip).
//
// The kernel of q8_gemm_kernel.h keeps one or two workgroups on a unit and overlaps inside each of them: rings of two to
// five stages, every load placed by hand.  Where the reduction is short, or the launch is not many times the chip, what
// it cannot overlap is a large part of a tile's life: filling the ring, the epilogue with its stores, the last round of
// workgroups.  Here a workgroup holds kSlots stage buffers of 128 bytes of K (one: it loads a stage, waits, multiplies) and
// the overlap is between the three to five workgroups of a unit, each at another point of its tile; tiles are also small
// enough to spread a launch evenly over the units.  Operand and LDS layout are those of the other kernel.
// The best tile of the other kernel -> the one that the launcher takes here, outputs rotating through more than the Infinity Cache, each warmed up by
// itself, us:
//   4096 x  768 x  768   6.7 ->  6.5 (128x64, two slots)           8192 x 2304 x  768        26.2 -> 24.6 (128x128, one slot)
//   1536 x 1024 x 1024   6.3 ->  6.0 (64x64, three slots)         12288 x 3072 x 1024        54.9 -> 51.6 (192x128, one slot)
//   8192 x 3072 x  768 + GELU + abs-max 37.9 -> 33 (128x128)      12288 x 4096 x 1024 + GELU + abs-max 76.5 -> 70.3 (192x128)
//   4096 x 3072 x  768 + GELU + abs-max 21.7 -> 20.0 (128x128)     1536 x 3072 x  768 + GELU + abs-max 10.4 -> 10.1 (192x128)
// Long reductions stay with the other kernel (12288 x 1024 x 4096 50.5 against 56.3, 8192 x 768 x 3072 26.1 against 28.7, 4096 x 768 x 3072 15.2 against
// 16.6): there the bytes staged per MFMA count, and its tiles are the largest.
// What bounds the large launches: 12288 x 4096 x K with GELU and abs-max takes 41 us at K = 128, 42 at 256 -- the stores, at 4.8 TB/s -- and from there on
// 0.040 us a unit of K (2.5 POP/s), 72 at 1024: what does not hide behind the stores adds.  In those 72 us the matrix pipes are busy in 42 % of the cycles,
// the L1 waits for outstanding requests in 47 % and is held by the L2's request path in 9 % (12288 x 3072 x 1024: 38, 42 and 20 %).
#pragma once
#include "q8_gemm_kernel.h"

namespace q8 {

// kWgs: workgroups per compute unit the kernel is compiled for (they share the unit's 160 KiB of LDS and its registers).
// kEpi: the combination of Q8_EPI_GELU (1), Q8_EPI_ABSMAX (2) and Q8_EPI_REQUANT (4); no accumulator dump, no residual.
// kTail: K is any multiple of 4 and rows are 4-byte aligned (all that the loads need); the last stage then holds the front of the next
// rows behind the end of K -- or zeros, behind the end of the tile -- and the x operand is cleared there.  Else K is a multiple of 128.
template <int BM, int BN, int WGM, int WGN, int kSlots, int kWgs, int kEpi, bool kTail>
__global__ __launch_bounds__(WGM* WGN * 64, kWgs* WGM* WGN / 4) void gemm_ring_kernel(const int8_t* __restrict__ X, const int8_t* __restrict__ W, int M, int N,
                                                                                     int K, int tiles_n, int group_m, int by_xcd, Epilogue ep)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr bool do_gelu = (kEpi & 1) != 0, do_amax = (kEpi & 2) != 0, do_req = (kEpi & 4) != 0;
    constexpr int NW = WGM * WGN;
    constexpr int TM = BM / WGM, TN = BN / WGN;  // wave tile
    constexpr int FM = TM / 32, FN = TN / 32;    // 32x32 MFMA blocks per wave tile
    constexpr int A_BYTES = BM * kBK, B_BYTES = BN * kBK, SLOT = A_BYTES + B_BYTES;
    constexpr int A_LOADS = BM / 8 / NW, B_LOADS = BN / 8 / NW, LOADS = A_LOADS + B_LOADS;  // 1 KiB wave loads per stage
    static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "tile rows must split over the waves");
    static_assert(TM % 32 == 0 && TN % 32 == 0, "wave tile must be made of 32x32 blocks");
    static_assert(kWgs * kSlots * SLOT <= 160 * 1024, "LDS is 160 KiB per compute unit");
    static_assert(kSlots < 2 || (kSlots - 1) * LOADS <= 63, "vmcnt is a 6-bit counter");

    __shared__ __attribute__((aligned(1024))) char lds[kSlots * SLOT];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned lds_base = (unsigned)(size_t)(lds_ptr_t)lds;
    const int pid = tile_of_workgroup(by_xcd ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x, gridDim.x / tiles_n, tiles_n, group_m);
    const int m0 = (pid / tiles_n) * BM;
    const int n0 = (pid % tiles_n) * BN;

    // Descriptors start at the tile's first row; rows beyond the matrix edge re-read the last row, their products are never stored.
    const int rows_a = min(BM, M - m0), rows_b = min(BN, N - n0);
    const unsigned bytes_a = (unsigned)rows_a * (unsigned)K, bytes_b = (unsigned)rows_b * (unsigned)K;
    const int8_t* Xt = X + (int64_t)m0 * K;
    const int8_t* Wt = W + (int64_t)n0 * K;
    unsigned a_off[A_LOADS], b_off[B_LOADS];
#pragma unroll
    for (int i = 0; i < A_LOADS; ++i) {
        const int r = (wave * A_LOADS + i) * 8 + (lane >> 3);
        a_off[i] = (unsigned)min(r, rows_a - 1) * (unsigned)K + (unsigned)(((lane & 7) ^ swizzle_of_row(r)) * 16);
    }
#pragma unroll
    for (int i = 0; i < B_LOADS; ++i) {
        const int r = (wave * B_LOADS + i) * 8 + (lane >> 3);
        b_off[i] = (unsigned)min(r, rows_b - 1) * (unsigned)K + (unsigned)(((lane & 7) ^ swizzle_of_row(r)) * 16);
    }
    const int KT = kTail ? (K + kBK - 1) / kBK : K / kBK;
    auto load_stage = [&](int kt, int slot) {
        const bool live = kt < KT;  // past the end of K: empty descriptor, nothing is fetched
        const unsigned koff = live ? (unsigned)(kt * kBK) : 0u, dst = lds_base + (unsigned)(slot * SLOT);
        if constexpr (kTail) {
            // The last row's operands may end behind the matrix, so the stage is part of the descriptor: the bounds check is documented for
            // the vector offset alone.  No immediate offsets either: with rows shorter than 128 bytes the vector offset would fall below them.
            const v4i qa = make_rsrc(Xt + koff, live ? bytes_a - koff : 0u), qb = make_rsrc(Wt + koff, live ? bytes_b - koff : 0u);
            static_for<0, A_LOADS>([&](auto ic) { lds_dma16_first(qa, a_off[decltype(ic)::value], 0u, dst + (wave * A_LOADS + decltype(ic)::value) * 1024); });
            static_for<0, B_LOADS>([&](auto ic) { lds_dma16_first(qb, b_off[decltype(ic)::value], 0u, dst + A_BYTES + (wave * B_LOADS + decltype(ic)::value) * 1024); });
        } else {
            const v4i qa = make_rsrc(Xt, live ? bytes_a : 0u), qb = make_rsrc(Wt, live ? bytes_b : 0u);
            static_for<0, A_LOADS>([&](auto ic) { lds_dma16_run<decltype(ic)::value>(qa, a_off[decltype(ic)::value], koff, dst + wave * A_LOADS * 1024); });
            static_for<0, B_LOADS>([&](auto ic) { lds_dma16_run<decltype(ic)::value>(qb, b_off[decltype(ic)::value], koff, dst + A_BYTES + wave * B_LOADS * 1024); });
        }
    };

    const int wm = wave / WGN, wn = wave % WGN;
    const int l32 = lane & 31, hi = lane >> 5;
    int a_row[FM], b_row[FN], a_sw[FM], b_sw[FN];  // this lane's row of each block: byte offset in a slot, swizzle
#pragma unroll
    for (int f = 0; f < FM; ++f) {
        const int r = wm * TM + f * 32 + l32;
        a_row[f] = r * kBK;
        a_sw[f] = swizzle_of_row(r);
    }
#pragma unroll
    for (int f = 0; f < FN; ++f) {
        const int r = wn * TN + f * 32 + l32;
        b_row[f] = A_BYTES + r * kBK;
        b_sw[f] = swizzle_of_row(r);
    }

    v16i acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0;

    // The epilogue's per-column inputs, fetched ahead of the main loop.
    const float sx = ep.sx[0];
    float sw_col[FN], bias_col[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int n = min(n0 + wn * TN + j * 32 + l32, N - 1);
        sw_col[j] = ep.sw[n / ep.cols_per_group];
        bias_col[j] = ep.bias ? ep.bias[n] : 0.0f;
    }

    static_for<0, kSlots - 1>([&](auto pc) { load_stage(decltype(pc)::value, decltype(pc)::value); });
    int slot = 0;
    for (int kt = 0; kt < KT; ++kt) {
        if constexpr (kSlots == 1) {
            if (kt) {  // every wave has read the last stage
                __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(63));
                __syncthreads();
            }
            load_stage(kt, 0);
            __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
            __syncthreads();
        } else {
            // own loads of stage kt have landed, own reads of stage kt-1 are complete; the slot of stage kt-1 is free behind the barrier
            __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((kSlots - 2) * LOADS));
            __syncthreads();
            load_stage(kt + kSlots - 1, slot == 0 ? kSlots - 1 : slot - 1);
        }
        const char* stage = lds + slot * SLOT;
        slot = (slot + 1 == kSlots) ? 0 : slot + 1;
        v4i fa[2][FM], fb[2][FN];
        auto read_step = [&](int ks) {
#pragma unroll
            for (int f = 0; f < FM; ++f) fa[ks & 1][f] = *reinterpret_cast<const v4i*>(stage + a_row[f] + (((ks * 2 + hi) ^ a_sw[f]) << 4));
#pragma unroll
            for (int f = 0; f < FN; ++f) fb[ks & 1][f] = *reinterpret_cast<const v4i*>(stage + b_row[f] + (((ks * 2 + hi) ^ b_sw[f]) << 4));
            if constexpr (kTail) {
                if (kt == KT - 1) {
                    const int left = K - kt * kBK - ks * 32 - hi * 16;  // bytes of K this lane's operand still covers
#pragma unroll
                    for (int f = 0; f < FM; ++f)
#pragma unroll
                        for (int w = 0; w < 4; ++w) fa[ks & 1][f][w] = 4 * w < left ? fa[ks & 1][f][w] : 0;
                }
            }
        };
        read_step(0);
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) {
            if (ks + 1 < kKS) read_step(ks + 1);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[ks & 1][i], fb[ks & 1][j], acc[i][j], 0, 0, 0);
        }
    }
    // The (empty) loads past the end of K have landed before the stage buffers are given up or used for the abs-max.
    if constexpr (kSlots > 1) __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));

    // Epilogue: accumulator register e of lane l is row 8*(e/4) + 4*(l/32) + e%4 and column l%32 of its block.
    float next_scale = 0.0f;
    if (do_req) next_scale = ep.next_scale[0];
    unsigned amax = 0u;
    if ((m0 + BM <= M) && (n0 + BN <= N) && ((int64_t)N * BM * 4 < ((int64_t)1 << 31))) {
        constexpr int esize = do_req ? 1 : 4;
        const __amdgpu_buffer_rsrc_t ry =
            __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char*>(ep.y) + (int64_t)m0 * N * esize, 0, BM * N * esize, 0x00020000);
        const int row0 = wm * TM + 4 * hi;
        float famax = 0.0f;
        auto store_tile = [&](auto ntc) {
            constexpr int kAux = decltype(ntc)::value ? 2 : 0;  // aux bit 1 = nt
            static_for<0, FN>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                const int n = n0 + wn * TN + j * 32 + l32;
                const ColConst cc = ColConst{ep.bias ? quantize_bias(bias_col[j], sx, sw_col[j]) : 0, dequant_factor(sx, sw_col[j])};
                const int elem0 = row0 * N + n;
                static_for<0, FM>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    static_for<0, 16>([&](auto ec) {
                        constexpr int e = decltype(ec)::value;
                        constexpr int dm = i * 32 + 8 * (e >> 2) + (e & 3);
                        const int row_elems = dm * N;  // wave-uniform: lives in an SGPR
                        float yv = (float)(acc[i][j][e] + cc.bq) * cc.r;
                        if (do_gelu) yv = gelu_erf(yv);
                        if (do_amax) famax = __builtin_fmaxf(famax, __builtin_fabsf(yv));
                        if (do_req)
                            __builtin_amdgcn_raw_buffer_store_b8((unsigned char)quantize_code(yv, next_scale), ry, elem0, row_elems, 0);
                        else
                            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(yv), ry, elem0 * 4, row_elems * 4, kAux);
                        if constexpr ((e & 3) == 3) __builtin_amdgcn_sched_barrier(0);  // stores trickle out between the arithmetic
                    });
                });
            });
        };
        if (ep.stream_out && !do_req)
            store_tile(std::true_type{});
        else
            store_tile(std::false_type{});
        amax = __float_as_uint(famax);
    } else {
        static_for<0, FN>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            const int n = n0 + wn * TN + j * 32 + l32;
            if (n < N) {
                const ColConst cc = ColConst{ep.bias ? quantize_bias(bias_col[j], sx, sw_col[j]) : 0, dequant_factor(sx, sw_col[j])};
                static_for<0, FM>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    const int mb = m0 + wm * TM + i * 32 + 4 * hi;
                    static_for<0, 16>([&](auto ec) {
                        constexpr int e = decltype(ec)::value;
                        const int m = mb + 8 * (e >> 2) + (e & 3);
                        if (m < M) {
                            const int64_t idx = (int64_t)m * N + n;
                            float yv = (float)(acc[i][j][e] + cc.bq) * cc.r;
                            if (do_gelu) yv = gelu_erf(yv);
                            if (do_req)
                                reinterpret_cast<int8_t*>(ep.y)[idx] = (int8_t)quantize_code(yv, next_scale);
                            else
                                reinterpret_cast<float*>(ep.y)[idx] = yv;
                            if (do_amax) amax = max(amax, f32_abs_bits(yv));
                        }
                    });
                });
            }
        });
    }
    if constexpr (do_amax) publish_amax<NW>(amax, reinterpret_cast<unsigned*>(lds), ep.out_amax);
#endif
}

template <int BM, int BN, int WGM, int WGN, int kSlots, int kWgs>
int launch_ring(const int8_t* xq, const int8_t* wq, int M, int N, int K, int group_m, int by_xcd, const Epilogue& ep, hipStream_t st)
{
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    const dim3 grid(tiles_m * tiles_n), block(WGM * WGN * 64);
    const bool tail = K % kBK != 0;
#define Q8_LAUNCH_EPI(E)                                                                                                                       \
    case E:                                                                                                                                    \
        if (tail)                                                                                                                              \
            hipLaunchKernelGGL((gemm_ring_kernel<BM, BN, WGM, WGN, kSlots, kWgs, E, true>), grid, block, 0, st, xq, wq, M, N, K, tiles_n, group_m, \
                               by_xcd, ep);                                                                                                    \
        else                                                                                                                                   \
            hipLaunchKernelGGL((gemm_ring_kernel<BM, BN, WGM, WGN, kSlots, kWgs, E, false>), grid, block, 0, st, xq, wq, M, N, K, tiles_n, group_m, \
                               by_xcd, ep);                                                                                                    \
        break
    switch (ep.flags) {
        Q8_LAUNCH_EPI(0);
        Q8_LAUNCH_EPI(1);
        Q8_LAUNCH_EPI(2);
        Q8_LAUNCH_EPI(3);
        Q8_LAUNCH_EPI(4);
        Q8_LAUNCH_EPI(5);
        default: return 1;
    }
#undef Q8_LAUNCH_EPI
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

}  // namespace q8

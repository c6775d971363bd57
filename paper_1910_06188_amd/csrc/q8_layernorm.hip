// FP32 glue next to the quantized FC layers: Layer Normalization (Section 3 keeps it in FP32)
// fused with what surrounds it on the dynamic-quantization path -- the residual addition or the
// three-table int8 embedding lookup in front, and behind it the abs-max of its output, which is
// the first half of the next FC layer's quantizer (Section 4.1).  One pass over HBM instead of
// three or four: per element 4 B (+ 4 B residual, or 3 B of int8 codes) read and 4 B written.
//
// A wave owns a row.  The row lives in registers (up to 2048 columns); its sum and its sum of
// squared deviations are accumulated in binary64 and reduced across the wave in a fixed order,
// and the normalisation itself runs in binary64 with one final rounding, so the result is within
// an ulp of the exact one and the same bytes come out on every run.  The kernel is bound by
// memory: the binary64 arithmetic (about ten operations per element) hides under the loads where there are other rows to load; what is
// left in small launches is the chain load - two reductions - store.  8192 x 768 with residual 17.0 -> 15.4 us, 12288 x 1024
// 28.9 -> 28.4 (5.3 TB/s) and 19.8 -> 18.9 without, from rows behind descriptors, the estimate of 1 / sqrt and the skipped vectors.
#include "q8_device.h"
#include "q8_launch.h"

namespace q8 {

constexpr int kLnThreads = 256;            // four waves = four rows per workgroup per trip
constexpr int kLnMaxVec = 8;               // float4 vectors per lane: rows up to 64 * 4 * 8 = 2048 columns
constexpr int kLnRowsShort = 2;           // rows a wave carries side by side: plain LayerNorm of rows of at most 1024 columns (with a
                                          // residual or the embedding rows in front the extra registers cost more than they win)
constexpr int kLnOneTrip = 4096;          // rows that 1024 workgroups take in one trip
constexpr int kLnSlots = 2048;             // abs-max slots (= Q8_AMAX_SLOTS): one per workgroup, the rest zero

// Sum of a double over the 64 lanes, the same value in every lane, in a fixed order (so the same bytes come out on
// every run): an inclusive scan inside each row of 16 lanes with DPP row shifts (1, 2, 4, 8; lanes shifted in from
// outside the row contribute zero), then the row totals carried across rows with the two row broadcasts, and lane
// 63's total read back as a scalar.  A 64-bit value moves as two 32-bit DPP moves; the cross-lane traffic stays in
// the vector ALU (a butterfly of ds_bpermute exchanges costs ten times the latency, and a wave does two of these
// reductions per row with nothing else to do meanwhile).
template <int kCtrl, int kRowMask>
__device__ __forceinline__ double dpp_move_f64(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), kCtrl, kRowMask, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), kCtrl, kRowMask, 0xf, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum_f64(double v)
{
    v += dpp_move_f64<0x111, 0xf>(v);  // row_shr:1
    v += dpp_move_f64<0x112, 0xf>(v);  // row_shr:2
    v += dpp_move_f64<0x114, 0xf>(v);  // row_shr:4
    v += dpp_move_f64<0x118, 0xf>(v);  // row_shr:8   -> lane 15 of each row holds its row's sum
    v += dpp_move_f64<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_move_f64<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3 -> lane 63 holds the total
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63), __builtin_amdgcn_readlane(__double2loint(v), 63));
}

// 16-byte load with the non-temporal hint: the inputs of a LayerNorm are read exactly once, and streamed
// past the Infinity Cache they leave it to the tensors that are read again (layer step with the fused
// LayerNorms 5 % faster with dynamic scales, 9 % with stored ones).
// Rows are addressed through a descriptor that ends with the row (and is empty for a row that does not exist): what lies behind
// it reads as zeros and is not stored, without a branch around every access.
typedef unsigned u32x4_ln __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* base, int64_t row, int64_t rows, int row_bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(reinterpret_cast<const char*>(base)) + (row < rows ? row * row_bytes : 0), 0,
                                             row < rows ? row_bytes : 0, 0x00020000);
}
template <int kAux>
__device__ __forceinline__ float4 load_f4_ln(__amdgpu_buffer_rsrc_t r, int off)
{
    const u32x4_ln v = __builtin_bit_cast(u32x4_ln, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kAux));
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}
constexpr int kNt = 2;  // non-temporal

// 1 / sqrt(v), v >= 0: the hardware's estimate (about 2^-23) and two Newton steps, good to the last places of binary64.  The
// library's square root and division are four times as many dependent operations, and every row waits for them.
__device__ __forceinline__ double rsqrt_f64(double v)
{
    double y = __builtin_amdgcn_rsq(v);
    const double h = 0.5 * v;
#pragma unroll
    for (int i = 0; i < 2; ++i) y = __builtin_fma(y, __builtin_fma(-h * y, y, 0.5), y);
    return h == v ? __builtin_amdgcn_rsq(v) : y;   // the ends, where a step would be 0 times infinity: v = 0 and an infinite eps
}

struct EmbedSrc {
    const unsigned *word, *pos, *typ;  // int8 tables viewed as packed dwords
    int64_t Vw, Vp, Vt;
    const float* scales;
    const int32_t *wid, *pid, *tid;
    int32_t* err_flag;
};

__device__ __forceinline__ float4 dequant4_ln(unsigned packed, float r)
{
    float4 o;
    o.x = (float)(int)(int8_t)(packed & 0xff) * r;
    o.y = (float)(int)(int8_t)((packed >> 8) & 0xff) * r;
    o.z = (float)(int)(int8_t)((packed >> 16) & 0xff) * r;
    o.w = (float)(int)(int8_t)(packed >> 24) * r;
    return o;
}

// kSrc: 0 = x is a; 1 = x is a + r (one binary32 addition); 2 = x is the sum of three
// dequantized embedding rows, (word + position) + type as in the plain lookup.
// kEarly: launches of one trip, rows of up to 1024 columns.  gamma and beta are requested under the statistics instead of where they are
// used, no next trip's rows are (128 x 768 with residual 3.7 -> 3.2 us, 1024 x 768 5.3 -> 4.7, 4096 x 768 9.7 -> 9.1).  Longer launches have other rows of the
// workgroup to wait under, and no registers for it.
// H % 4 == 0, H <= 256 * kVec (kVec float4 vectors per lane: 4 for rows of up to 1024 columns -- fewer registers, more
// waves in flight -- 8 up to 2048), every pointer 16-byte aligned (tables 4-byte).
template <int kSrc, int kVec, int kRows, bool kEarly>
__global__ __launch_bounds__(kLnThreads, kEarly ? 4 : 1) void layernorm_rows_kernel(const float* a, const float* r, EmbedSrc es,
                                                                     const float* __restrict__ gamma,
                                                                     const float* __restrict__ beta, double eps, double inv_h,
                                                                     int64_t M, int H, float* y,
                                                                     unsigned* __restrict__ amax_slots,
                                                                     const float* __restrict__ q_scale,
                                                                     unsigned* __restrict__ q_out)
{
    __shared__ unsigned wave_amax[kLnThreads / 64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (amax_slots)  // slots no workgroup owns
        for (int i = gridDim.x + blockIdx.x * kLnThreads + threadIdx.x; i < kLnSlots; i += gridDim.x * kLnThreads) amax_slots[i] = 0u;
    const int nvec = H >> 2;
    const float qs = q_out ? q_scale[0] : 0.0f;
    float amax = 0.0f;
    float r0 = 0.f, r1 = 0.f, r2 = 0.f;
    if (kSrc == 2) {
        r0 = __fdiv_rn(1.0f, es.scales[0]);
        r1 = __fdiv_rn(1.0f, es.scales[1]);
        r2 = __fdiv_rn(1.0f, es.scales[2]);
    }
    // A wave takes kRows consecutive rows per trip and carries them side by side: all their loads are in flight
    // together and their reductions -- chains of dependent cross-lane exchanges -- interleave, so a wave spends its
    // time waiting for memory once per trip instead of once per row.  Each row's arithmetic is unchanged.
    constexpr int kWaves = kLnThreads / 64;
    const int64_t row_step = (int64_t)gridDim.x * kWaves * kRows;
    // kSrc 0 and 1: the rows of the NEXT trip are requested as soon as this trip's have arrived, so their flight
    // covers this trip's reductions, normalisation and stores (a wave otherwise has nothing in flight while it
    // computes, and with four or five waves per SIMD the pass ran at 5 TB/s where a copy gets 6.5).
    float4 na[kRows][kVec], nr[kRows][kVec];
    auto request_rows = [&](int64_t r0) {
#pragma unroll
        for (int q = 0; q < kRows; ++q) {
            const auto av = row_rsrc(a, r0 + q, M, 4 * H), rv = row_rsrc(kSrc == 1 ? r : a, r0 + q, M, 4 * H);
#pragma unroll
            for (int j = 0; j < kVec; ++j) {
                na[q][j] = load_f4_ln<kNt>(av, 16 * (j * 64 + lane));
                if (kSrc == 1) nr[q][j] = load_f4_ln<kNt>(rv, 16 * (j * 64 + lane));
            }
        }
    };
    const int64_t first_row0 = ((int64_t)blockIdx.x * kWaves + wave) * kRows;
    if (kSrc != 2 && first_row0 < M) request_rows(first_row0);
    const auto rg = row_rsrc(gamma, 0, 1, 4 * H), rb = row_rsrc(beta, 0, 1, 4 * H);
    for (int64_t row0 = first_row0; row0 < M; row0 += row_step) {
        float4 x[kRows][kVec];
        bool live[kRows];
#pragma unroll
        for (int q = 0; q < kRows; ++q) {
            const int64_t row = row0 + q;
            live[q] = row < M;
#pragma unroll
            for (int j = 0; j < kVec; ++j) x[q][j] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (kSrc != 2) {   // this trip's rows were requested a trip ago
#pragma unroll
                for (int j = 0; j < kVec; ++j)
                    x[q][j] = kSrc == 1 ? make_float4(__fadd_rn(na[q][j].x, nr[q][j].x), __fadd_rn(na[q][j].y, nr[q][j].y),
                                                      __fadd_rn(na[q][j].z, nr[q][j].z), __fadd_rn(na[q][j].w, nr[q][j].w))
                                        : na[q][j];
                continue;
            }
            if (!live[q]) continue;
            if (kSrc == 2) {
                const int64_t ia = es.wid[row], ib = es.pid[row], ic = es.tid[row];
                const bool ok = ia >= 0 && ia < es.Vw && ib >= 0 && ib < es.Vp && ic >= 0 && ic < es.Vt;
                if (!ok && es.err_flag && lane == 0) es.err_flag[0] = 1;
                const unsigned* wr = es.word + (ok ? ia : 0) * nvec;
                const unsigned* pr = es.pos + (ok ? ib : 0) * nvec;
                const unsigned* tr = es.typ + (ok ? ic : 0) * nvec;
#pragma unroll
                for (int j = 0; j < kVec; ++j) {
                    const int v = j * 64 + lane;
                    if (v < nvec && ok) {
                        const float4 p = dequant4_ln(wr[v], r0), t1 = dequant4_ln(pr[v], r1), t2 = dequant4_ln(tr[v], r2);
                        x[q][j] = make_float4((p.x + t1.x) + t2.x, (p.y + t1.y) + t2.y, (p.z + t1.z) + t2.z, (p.w + t1.w) + t2.w);
                    }
                }
            }
        }
        if (kSrc != 2 && !kEarly && row0 + row_step < M) request_rows(row0 + row_step);
        float4 ge[kVec], be[kVec];
        if (kEarly) {
            int lane16 = 16 * lane;
            asm volatile("" : "+v"(lane16));   // here: as loop invariants they would be converted ahead of the loop, which takes 32 registers more
#pragma unroll
            for (int j = 0; j < kVec; ++j) {
                ge[j] = load_f4_ln<0>(rg, 1024 * j + lane16);
                be[j] = load_f4_ln<0>(rb, 1024 * j + lane16);
            }
        }
        double mean[kRows], rstd[kRows];
#pragma unroll
        for (int q = 0; q < kRows; ++q) {
            double s = 0.0;
#pragma unroll
            for (int j = 0; j < kVec; ++j) {  // lanes past the row hold zeros
                if (j * 64 >= nvec) continue;
                s += ((double)x[q][j].x + (double)x[q][j].y) + ((double)x[q][j].z + (double)x[q][j].w);
            }
            mean[q] = s;
        }
#pragma unroll
        for (int q = 0; q < kRows; ++q) {  // the quotient by H, rounded once: a row of equal numbers has that number as its mean
            const double sum = wave_sum_f64(mean[q]), m0 = sum * inv_h;
            mean[q] = __builtin_fma(__builtin_fma(-m0, (double)H, sum), inv_h, m0);
        }
#pragma unroll
        for (int q = 0; q < kRows; ++q) {
            double ss = 0.0;
#pragma unroll
            for (int j = 0; j < kVec; ++j) {
                if (j * 64 >= nvec) continue;
                const double d0 = (double)x[q][j].x - mean[q], d1 = (double)x[q][j].y - mean[q];
                const double d2 = (double)x[q][j].z - mean[q], d3 = (double)x[q][j].w - mean[q];
                const double part = __builtin_fma(d0, d0, d1 * d1) + __builtin_fma(d2, d2, d3 * d3);
                ss += j * 64 + lane < nvec ? part : 0.0;
            }
            rstd[q] = ss;
        }
#pragma unroll
        for (int q = 0; q < kRows; ++q) rstd[q] = rsqrt_f64(wave_sum_f64(rstd[q]) * inv_h + eps);
#pragma unroll
        for (int q = 0; q < kRows; ++q) {
            const auto ry = row_rsrc(y, row0 + q, M, 4 * H), rq = row_rsrc(q_out, row0 + q, q_out ? M : 0, H);
#pragma unroll
            for (int j = 0; j < kVec; ++j) {
                if (j * 64 >= nvec) continue;
                const int v = j * 64 + lane;
                const float4 g = kEarly ? ge[j] : load_f4_ln<0>(rg, 16 * v), b = kEarly ? be[j] : load_f4_ln<0>(rb, 16 * v);
                float4 o;   // zero where gamma and beta end
                o.x = (float)__builtin_fma(((double)x[q][j].x - mean[q]) * rstd[q], (double)g.x, (double)b.x);
                o.y = (float)__builtin_fma(((double)x[q][j].y - mean[q]) * rstd[q], (double)g.y, (double)b.y);
                o.z = (float)__builtin_fma(((double)x[q][j].z - mean[q]) * rstd[q], (double)g.z, (double)b.z);
                o.w = (float)__builtin_fma(((double)x[q][j].w - mean[q]) * rstd[q], (double)g.w, (double)b.w);
                const u32x4_ln ob = {__float_as_uint(o.x), __float_as_uint(o.y), __float_as_uint(o.z), __float_as_uint(o.w)};
                __builtin_amdgcn_raw_buffer_store_b128(ob, ry, 16 * v, 0, 0);
                if (q_out)  // stored-scale quantizer of the next FC (Eq. 1 on the rounded fp32 value), 4 codes per lane
                    __builtin_amdgcn_raw_buffer_store_b32(((unsigned)quantize_code(o.x, qs) & 0xffu) | (((unsigned)quantize_code(o.y, qs) & 0xffu) << 8) |
                                                              (((unsigned)quantize_code(o.z, qs) & 0xffu) << 16) | ((unsigned)quantize_code(o.w, qs) << 24),
                                                          rq, 4 * v, 0, 0);
                const float most = __builtin_fmaxf(__builtin_fmaxf(__builtin_fabsf(o.x), __builtin_fabsf(o.y)), __builtin_fmaxf(__builtin_fabsf(o.z), __builtin_fabsf(o.w)));
                if (live[q]) amax = __builtin_fmaxf(amax, most);
            }
        }
    }
    if (amax_slots) {
        unsigned m = wave_max_u32(__float_as_uint(amax));  // non-negative floats order like their bit patterns
        if (lane == 0) wave_amax[wave] = m;
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int w = 1; w < kLnThreads / 64; ++w) m = max(m, wave_amax[w]);
            amax_slots[blockIdx.x] = m;
        }
    }
}

// Any H and alignment: a wave per row, three passes over the row (the second and third come
// from cache).  Same arithmetic; rows are read element by element.
template <int kSrc>
__global__ __launch_bounds__(kLnThreads) void layernorm_generic_kernel(const float* a, const float* r, EmbedSrc es,
                                                                        const int8_t* word8, const int8_t* pos8,
                                                                        const int8_t* typ8,
                                                                        const float* __restrict__ gamma,
                                                                        const float* __restrict__ beta, double eps,
                                                                        int64_t M, int64_t H, float* y,
                                                                        unsigned* __restrict__ amax_slots,
                                                                        const float* __restrict__ q_scale,
                                                                        int8_t* __restrict__ q_out)
{
    __shared__ unsigned wave_amax[kLnThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float amax = 0.0f;
    const float qs = q_out ? q_scale[0] : 0.0f;
    float r0 = 0.f, r1 = 0.f, r2 = 0.f;
    if (kSrc == 2) {
        r0 = __fdiv_rn(1.0f, es.scales[0]);
        r1 = __fdiv_rn(1.0f, es.scales[1]);
        r2 = __fdiv_rn(1.0f, es.scales[2]);
    }
    for (int64_t row = ((int64_t)blockIdx.x * (kLnThreads / 64)) + wave; row < M;
         row += (int64_t)gridDim.x * (kLnThreads / 64)) {
        int64_t ia = 0, ib = 0, ic = 0;
        bool ok = true;
        if (kSrc == 2) {
            ia = es.wid[row], ib = es.pid[row], ic = es.tid[row];
            ok = ia >= 0 && ia < es.Vw && ib >= 0 && ib < es.Vp && ic >= 0 && ic < es.Vt;
            if (!ok && es.err_flag && lane == 0) es.err_flag[0] = 1;
        }
        auto value = [&](int64_t h) -> float {
            if (kSrc == 2) {
                if (!ok) return 0.0f;
                const float p = (float)(int)word8[ia * H + h] * r0, q = (float)(int)pos8[ib * H + h] * r1;
                const float t = (float)(int)typ8[ic * H + h] * r2;
                return (p + q) + t;
            }
            const float v = a[row * H + h];
            return kSrc == 1 ? __fadd_rn(v, r[row * H + h]) : v;
        };
        double s = 0.0;
        for (int64_t h = lane; h < H; h += 64) s += (double)value(h);
        const double mean = wave_sum_f64(s) / (double)H;
        double ss = 0.0;
        for (int64_t h = lane; h < H; h += 64) {
            const double d = (double)value(h) - mean;
            ss += d * d;
        }
        const double rstd = 1.0 / sqrt(wave_sum_f64(ss) / (double)H + eps);
        for (int64_t h = lane; h < H; h += 64) {
            const float o = (float)(((double)value(h) - mean) * rstd * (double)gamma[h] + (double)beta[h]);
            y[row * H + h] = o;
            if (q_out) q_out[row * H + h] = (int8_t)quantize_code(o, qs);
            amax = __builtin_fmaxf(amax, __builtin_fabsf(o));
        }
    }
    if (amax_slots) {
        unsigned m = wave_max_u32(__float_as_uint(amax));
        if (lane == 0) wave_amax[wave] = m;
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int w = 1; w < kLnThreads / 64; ++w) m = max(m, wave_amax[w]);
            amax_slots[blockIdx.x] = m;
        }
        if (blockIdx.x == 0)
            for (int i = gridDim.x + threadIdx.x; i < kLnSlots; i += kLnThreads) amax_slots[i] = 0u;
    }
}

__global__ void amax_slots_clear_kernel(unsigned* slots)
{
    for (int i = threadIdx.x; i < kLnSlots; i += kLnThreads) slots[i] = 0u;
}

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

static int ln_grid(int64_t M, int rows_per_wave = 1)
{
    // one slot per workgroup caps the grid; within the cap, spread the rows evenly over the trips
    const int64_t per_wg = (int64_t)(kLnThreads / 64) * rows_per_wave;
    const int64_t need = (M + per_wg - 1) / per_wg;
    if (need <= 1) return 1;
    // at most 1024 workgroups (four per compute unit, all resident at once; fewer than the slots): beyond that a
    // workgroup makes several trips and fetches the next trip's rows under the arithmetic of the current one
    const int64_t cap = kLnSlots < 1024 ? kLnSlots : 1024;
    const int64_t trips = (need + cap - 1) / cap;
    return (int)((need + trips - 1) / trips);
}

int launch_layernorm(const float* a, const float* r, const float* gamma, const float* beta, float eps, int64_t M,
                     int64_t H, float* y, float* amax_slots, const float* q_scale, int8_t* q_out, hipStream_t st)
{
    unsigned* slots = reinterpret_cast<unsigned*>(amax_slots);
    if (M == 0) {
        if (slots) hipLaunchKernelGGL(amax_slots_clear_kernel, dim3(1), dim3(kLnThreads), 0, st, slots);
        return hipGetLastError() == hipSuccess ? 0 : 1;
    }
    EmbedSrc es = {};
    const bool fast = H % 4 == 0 && H <= 64 * 4 * kLnMaxVec && aligned16(a) && aligned16(y) && aligned16(gamma) &&
                      aligned16(beta) && (!r || aligned16(r)) && (reinterpret_cast<uintptr_t>(q_out) & 3) == 0;
    const dim3 grid(ln_grid(M)), block(kLnThreads);
    if (fast) {
        if (r)
            if (H <= 1024)
                hipLaunchKernelGGL((M <= kLnOneTrip ? layernorm_rows_kernel<1, 4, 1, true> : layernorm_rows_kernel<1, 4, 1, false>), dim3(ln_grid(M, 1)), block, 0, st, a, r,
                                   es, gamma, beta, (double)eps, 1.0 / (double)H, M, (int)H, y, slots, q_scale, reinterpret_cast<unsigned*>(q_out));
            else
                hipLaunchKernelGGL((layernorm_rows_kernel<1, 8, 1, false>), grid, block, 0, st, a, r, es, gamma, beta, (double)eps, 1.0 / (double)H, M,
                               (int)H, y, slots, q_scale, reinterpret_cast<unsigned*>(q_out));
        else
            if (H <= 1024)
                hipLaunchKernelGGL((layernorm_rows_kernel<0, 4, kLnRowsShort, false>), dim3(ln_grid(M, kLnRowsShort)), block, 0, st, a, r, es, gamma, beta, (double)eps, 1.0 / (double)H, M,
                               (int)H, y, slots, q_scale, reinterpret_cast<unsigned*>(q_out));
            else
                hipLaunchKernelGGL((layernorm_rows_kernel<0, 8, 1, false>), grid, block, 0, st, a, r, es, gamma, beta, (double)eps, 1.0 / (double)H, M,
                               (int)H, y, slots, q_scale, reinterpret_cast<unsigned*>(q_out));
    } else {
        if (r)
            hipLaunchKernelGGL(layernorm_generic_kernel<1>, grid, block, 0, st, a, r, es, nullptr, nullptr, nullptr,
                               gamma, beta, (double)eps, M, H, y, slots, q_scale, q_out);
        else
            hipLaunchKernelGGL(layernorm_generic_kernel<0>, grid, block, 0, st, a, r, es, nullptr, nullptr, nullptr,
                               gamma, beta, (double)eps, M, H, y, slots, q_scale, q_out);
    }
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

int launch_embedding_sum3_layernorm(const int8_t* word, int64_t Vw, const int8_t* pos, int64_t Vp, const int8_t* typ,
                                    int64_t Vt, const float* scales, int64_t H, const int32_t* wid,
                                    const int32_t* pid, const int32_t* tid, int64_t T, const float* gamma,
                                    const float* beta, float eps, float* y, float* amax_slots, const float* q_scale,
                                    int8_t* q_out, int32_t* err_flag, hipStream_t st)
{
    unsigned* slots = reinterpret_cast<unsigned*>(amax_slots);
    if (T == 0) {
        if (slots) hipLaunchKernelGGL(amax_slots_clear_kernel, dim3(1), dim3(kLnThreads), 0, st, slots);
        return hipGetLastError() == hipSuccess ? 0 : 1;
    }
    EmbedSrc es;
    es.word = reinterpret_cast<const unsigned*>(word);
    es.pos = reinterpret_cast<const unsigned*>(pos);
    es.typ = reinterpret_cast<const unsigned*>(typ);
    es.Vw = Vw, es.Vp = Vp, es.Vt = Vt;
    es.scales = scales;
    es.wid = wid, es.pid = pid, es.tid = tid;
    es.err_flag = err_flag;
    const auto a4 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3) == 0; };
    const bool fast = H % 4 == 0 && H <= 64 * 4 * kLnMaxVec && a4(word) && a4(pos) && a4(typ) && aligned16(y) &&
                      aligned16(gamma) && aligned16(beta) && a4(q_out);
    const dim3 grid(ln_grid(T)), block(kLnThreads);
    if (fast)
        if (H <= 1024)
                hipLaunchKernelGGL((T <= kLnOneTrip ? layernorm_rows_kernel<2, 4, 1, true> : layernorm_rows_kernel<2, 4, 1, false>), dim3(ln_grid(T, 1)), block, 0, st,
                                   nullptr, nullptr, es, gamma, beta, (double)eps, 1.0 / (double)H, T, (int)H, y, slots, q_scale, reinterpret_cast<unsigned*>(q_out));
            else
                hipLaunchKernelGGL((layernorm_rows_kernel<2, 8, 1, false>), grid, block, 0, st, nullptr, nullptr, es, gamma, beta,
                           (double)eps, 1.0 / (double)H, T, (int)H, y, slots, q_scale, reinterpret_cast<unsigned*>(q_out));
    else
        hipLaunchKernelGGL(layernorm_generic_kernel<2>, grid, block, 0, st, nullptr, nullptr, es, word, pos, typ, gamma,
                           beta, (double)eps, T, H, y, slots, q_scale, q_out);
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

}  // namespace q8

// FP32 multi-head softmax attention, the operation between the fused Q|K|V FC layer and the
// attention-output FC layer of an encoder layer.  Section 3 keeps Softmax in FP32 and quantizes
// only Embedding and FC layers, so both matrix products around the softmax stay FP32 as well:
//     s[i,j] = scale * <Q[i,:], K[j,:]> (+ mask[j]),   p = softmax_j(s),   ctx[i,:] = sum_j p[i,j] V[j,:]
// Behind it sits the first half of the next FC layer's quantizer (Section 4.1): the abs-max of
// ctx goes to per-workgroup slots, or, with a stored scale (Eq. 4), the int8 codes of ctx are
// written directly (Eq. 1) and ctx itself need not be stored at all.
//
// FP32 products on the bf16 matrix pipes.  A binary32 number is the exact sum of three bf16 numbers h + m + l (8 + 8 + 8
// significant bits, each part the rounded remainder of the ones before it), so a product is nine bf16 products.  Eight of
// them run on v_mfma_f32_32x32x16_bf16; l l, below 2^-34 of the product, is left out.  (m l and l m reach 2^-24 of it, half
// a last place of binary32: without them a score of one nonzero term is up to 1.7 times as far from 64 bits as one rounded
// product.)  The h h products have an accumulator of their own and the others share one, joined by one addition of the
// vector ALU: an MFMA adds up products of like size exactly, and rounds to nearest where the accumulator is the larger, but
// cuts an accumulator that is much smaller than its products off at the last place of the result (measured: errors up to one
// last place instead of half, and a bias).  The bf16 pipes are 16 times as fast as the fp32 ones, so eight products take half the time of
// one fp32 MFMA pass, and -- unlike the fp32 MFMAs, which share their lanes with the vector ALU -- they run beside the
// softmax arithmetic.  Error against 64 bits, rms of ctx over rms: normal inputs 32 x 128 tokens 1.5e-7 (fp32 pipes
// 3.4e-7, six products in one accumulator 2.6e-7), 8 x 384 2.1e-7 (4.5e-7, 3.8e-7); scores of one nonzero column 2.30e-6
// (2.30e-6, 2.58e-6).  BERT-Large attention: fp32 pipes 175 us, six products 117 us, eight 140 us
// (144 with the look at the range).  Six products against a reference that stays at zero while the scores are small (106 to 109 us, eight on the
// same box 127) are no way out: the mean error over normal inputs falls, but a score of one term loses what m l and l m are, and a
// query with one visible key, whose probability is exactly 1 against the maximum of its scores, no longer gets its V row back bit for bit.
//
// Range.  The sum is exact, and the products lose nothing, while no number is near the ends of the type: from 3.3953e38 on
// h rounds to infinity, and the lower parts of numbers below 2^-110 fall under the smallest bf16.  The kernels keep the largest
// magnitude of the rows they split (a vector instruction for every two numbers) and look at their results: rows that saw a
// number above 2^96 or an infinity, or whose results are infinite or so small that lost parts could matter in them, are formed
// again in plain binary32 (attention_rows_plain).  Slow, but values that occur in earnest never lead there.  (Not for a NaN: it
// makes the same results NaN either way.)
//
// Kernel (head widths up to 128): a workgroup of four waves owns 128 queries of one (sequence, head); each wave keeps
// its 32 query rows, split, in registers (pre-multiplied by scale * log2 e) and walks the keys in stages of 32.  The K
// and V rows of a stage are split once per workgroup on their way into LDS, V transposed.  Scores are formed
// transposed, S^T = K Q^T: a lane then holds 16 keys of ONE query, so the softmax statistics are per-lane loops plus
// a single exchange between the two half-waves, and the probabilities sit exactly where the B operand of
// O^T += V^T P^T wants them (the keys of a V row are stored in that order) -- no data movement between the two
// products.  Softmax is the running-maximum form (scores never exist in memory), evaluated with exp2.
// The key loop is skewed by one stage: the scores of stage i+1 are formed while the softmax of stage i runs, and the
// split of the stages ahead runs under P V; a wave issues in order, so the pieces are interleaved by hand.
#include "q8_device.h"
#include "q8_launch.h"

#include <type_traits>

namespace q8 {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr int kAtWaves = 4;                // waves per workgroup
constexpr int kAtThreads = kAtWaves * 64;
constexpr int kAtQW = 32;                  // queries per wave
constexpr int kAtQB = kAtQW * kAtWaves;    // queries per workgroup
constexpr int kAtKB = 32;                  // keys per stage
constexpr int kAtMaxD = 128;               // head widths of the MFMA kernel: multiples of 4 up to here
constexpr int kAtSlots = 2048;             // abs-max slots (= Q8_AMAX_SLOTS)

// LDS of one stage, for heads padded to 32 * kDB columns: three parts of the K tile (a row per key), three parts of the
// V tile (a row per column, its 32 keys in the order the P V operands take them), the stage's mask row.  Rows carry 16
// bytes of padding: strides of 16 kDB + 4 and 20 dwords put the 16 rows a 16-byte read serves per cycle on all 64 banks.
template <int kDB>
struct AttnTile {
    static constexpr int kKStride = 64 * kDB + 16, kVStride = 2 * kAtKB + 16;   // bytes
    static constexpr int kKPart = kAtKB * kKStride, kVPart = 32 * kDB * kVStride;
    static constexpr int kMask = 3 * kKPart;                                    // the mask row sits behind the K parts
    static constexpr int kKTile = 3 * kKPart + 4 * kAtKB, kVTile = 3 * kVPart;
    static constexpr int kBytes = 2 * (kKTile + kVTile);
};

struct AttnArgs {
    const float* qkv;     // [B*S, 3*heads*d]
    const float* mask;    // [B, S] additive, or null
    float* ctx;           // [B*S, heads*d] or null
    unsigned* slots;      // abs-max slots or null
    const float* q_scale; // stored scale of the next FC or null
    unsigned* q_out;      // int8 codes of ctx, packed four to a dword, or null
    int64_t S;
    int heads;
    int d;
    int n_qblocks;        // ceil(S / 128)
    int slots_atomic;     // more workgroups than slots: fold with atomics into cleared slots
    float c;              // scale * log2(e)
};

template <int I, int E, class F>
__device__ __forceinline__ void at_static_for(F&& f)
{
    if constexpr (I < E) {
        f(std::integral_constant<int, I>{});
        at_static_for<I + 1, E>(f);
    }
}

// The maximum that the three-operand instruction takes directly (the other one first quiets each operand).  A NaN stays one.
__device__ __forceinline__ float at_max(float a, float b) { return __builtin_elementwise_maximum(a, b); }

// Two binary32 numbers as three packed pairs of bf16 numbers whose sums they are, exactly: each part is the
// nearest bf16 of what the parts before it leave, and the differences are exact (inside the range named above).  In two halves, so that the pieces that
// go between two MFMAs stay small.  (v_dot2_f32_bf16 would unpack and subtract in one instruction, 7 for the pair
// instead of 11, but it waits for the MFMA in flight: measured 62 cycles per MFMA with four of them between, 33 with
// four ordinary instructions.)
__device__ __forceinline__ unsigned pack_bf16(float a, float b)
{
    v2f v;
    v.x = a;
    v.y = b;
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, v2bf));
}
struct Bf16x3 {
    unsigned h, m, l;
    float ra, rb;   // what h leaves
    __device__ __forceinline__ void first(float a, float b)
    {
        h = pack_bf16(a, b);
        ra = a - __uint_as_float(h << 16);
        rb = b - __uint_as_float(h & 0xffff0000u);
    }
    __device__ __forceinline__ void first(float a, float b, float& largest)
    {
        largest = at_max(largest, at_max(__builtin_fabsf(a), __builtin_fabsf(b)));
        asm volatile("" : "+v"(largest));   // here, and not gathered behind the trip
        first(a, b);
    }
    __device__ __forceinline__ void second()
    {
        m = pack_bf16(ra, rb);
        l = pack_bf16(ra - __uint_as_float(m << 16), rb - __uint_as_float(m & 0xffff0000u));
    }
};

__device__ __forceinline__ Bf16x3 split_bf16(float a, float b)
{
    Bf16x3 s;
    s.first(a, b);
    s.second();
    return s;
}
__device__ __forceinline__ Bf16x3 split_bf16(float a, float b, float& largest)
{
    Bf16x3 s;
    s.first(a, b, largest);
    s.second();
    return s;
}

// Three-part operand of an MFMA: eight numbers of one lane, two to a dword.
struct Frag3 {
    v4u part[3];
    __device__ __forceinline__ void set(int i, const Bf16x3& s)
    {
        part[0][i] = s.h;
        part[1][i] = s.m;
        part[2][i] = s.l;
    }
};
__device__ __forceinline__ v8bf as_bf(v4u v) { return __builtin_bit_cast(v8bf, v); }

// Partial product I of a . b: number 0 is h h.  The parts of a are used up one after the other (h, l, m).
constexpr int kAtParts = 8;
template <int I>
__device__ __forceinline__ v16f mfma_part(const Frag3& a, const Frag3& b, v16f acc)
{
    constexpr int pa[kAtParts] = {0, 0, 0, 2, 2, 1, 1, 1}, pb[kAtParts] = {0, 2, 1, 1, 0, 2, 1, 0};
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf(a.part[pa[I]]), as_bf(b.part[pb[I]]), acc, 0, 0, 0);
}
__device__ __forceinline__ v16f zero16()
{
    v16f z;
#pragma unroll
    for (int e = 0; e < 16; ++e) z[e] = 0.0f;
    return z;
}
// The sum of the leading products and the sum of the others, joined: one rounding of the vector ALU.
__device__ __forceinline__ void join_parts(v16f& lead, const v16f& rest)
{
#pragma unroll
    for (int e = 0; e < 16; ++e) lead[e] += rest[e];
}

// A mask value in log2 units.  The lowest values of the type would overflow to -inf, and a stage of nothing else has no
// maximum to take its probabilities against: they stay finite, far below any score.  (A NaN stays one.)
__device__ __forceinline__ float mask_log2(float m)
{
    const float v = m * 1.44269504088896341f;
    return v < -3.0e38f ? -3.0e38f : v;
}

// Loads through a descriptor.  The whole offset is in the vector operand: that is what the bounds check is documented to
// compare with the descriptor's size (the scalar operand is left out of it), and rows beyond the sequence rely on the check.
__device__ __forceinline__ float buf_f1(__amdgpu_buffer_rsrc_t r, unsigned off)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}
__device__ __forceinline__ float4 buf_f4(__amdgpu_buffer_rsrc_t r, unsigned off)
{
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    const u4 v = __builtin_bit_cast(u4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}

// Global -> registers -> (split) -> LDS staging of a stage.  An item is eight numbers: of the K tile eight columns of one
// key, of the V tile the eight keys one half-wave takes to a 16-key step, of one column.  Descriptors span one stage
// of one sequence, so offsets are 32 bits whatever the size of qkv, and rows beyond the sequence read as zeros.
template <int kDB>
struct AttnStager {
    using T = AttnTile<kDB>;
    static constexpr int kItems = (kAtKB * 4 * kDB + kAtThreads - 1) / kAtThreads;   // items of each tile per thread
    static constexpr int kAll = kAtKB * 4 * kDB;
    const float *kbase, *vbase;   // K and V of token 0 of this sequence and head (wave-uniform)
    const float* mrow;            // mask row of the sequence, or null
    char *k_tiles, *v_tiles;      // two (K tile + mask row); two V tiles
    int64_t ld;
    int S32, d, tid;
    unsigned k_off[kItems][2];    // byte offsets of an item's two float4 inside a stage
    unsigned v_off[kItems];
    int k_dst[kItems], v_dst[kItems];
    // Rows in flight.  Set st & 1 holds what trip st stores: K of stage st + 2 and V of stage st + 1, requested two trips
    // earlier; sets 2 and 3 are the prologue's.
    float4 k[4][kItems][2];
    float v[3][kItems][8];
    float m[4];
    float largest;                // magnitude of the numbers split so far
    bool masked;                  // the mask row of the K stage stashed last is not all zeros (wave-uniform)

    __device__ __forceinline__ void init(int t)
    {
        tid = t;
        m[0] = m[1] = m[2] = m[3] = 0.0f;
        largest = 0.0f;
        const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            const int it = min(i * kAtThreads + t, kAll - 1), key = it / (4 * kDB), c = it % (4 * kDB);
#pragma unroll
            for (int u = 0; u < 2; ++u) k_off[i][u] = 4u * ((unsigned)key * (unsigned)ld + (unsigned)min(8 * c + 4 * u, d - 4));
            k_dst[i] = key * T::kKStride + 16 * c;
            const int col = min(64 * i + lane, 32 * kDB - 1);
            v_off[i] = 4u * (unsigned)min(col, d - 1);
            v_dst[i] = col * T::kVStride + 16 * wave;   // wave = 2 * (16-key step) + half-wave
        }
    }
    // rows of a stage that exist, as a descriptor
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const float* base, int stage) const
    {
        const int rows = min(S32 - stage * kAtKB, kAtKB);
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base) + (int64_t)stage * kAtKB * ld, 0,
                                                 rows > 0 ? 4 * ((rows - 1) * (int)ld + d) : 0, 0x00020000);
    }
    template <int kSet>
    __device__ __forceinline__ void fetch_k(int stage)
    {
        const auto r = rsrc(kbase, stage);
#pragma unroll
        for (int i = 0; i < kItems; ++i)
#pragma unroll
            for (int u = 0; u < 2; ++u) k[kSet][i][u] = buf_f4(r, k_off[i][u]);
        if (mrow) m[kSet] = mrow[min(stage * kAtKB + (tid & (kAtKB - 1)), S32 - 1)];
    }
    template <int kSet>
    __device__ __forceinline__ void fetch_v(int stage)
    {
        const auto r = rsrc(vbase, stage);
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int row0 = 16 * (wave >> 1) + 4 * (wave & 1);
#pragma unroll
        for (int i = 0; i < kItems; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                v[kSet][i][e] = buf_f1(r, v_off[i] + 4u * (unsigned)(row0 + (e & 3) + 8 * (e >> 2)) * (unsigned)ld);
    }
    template <int kSet>
    __device__ __forceinline__ void stash_mask(int buf, int stage)
    {
        const int key = tid & (kAtKB - 1);   // eight threads write each value: no branch
        const float v = (stage * kAtKB + key < S32) ? mask_log2(m[kSet]) : -__builtin_inff();   // beyond the sequence: weight 0 whatever the row holds
        *reinterpret_cast<float*>(k_tiles + buf * T::kKTile + T::kMask + 4 * key) = v;
        masked = __builtin_amdgcn_ballot_w64(v != 0.0f) != 0;
    }
    // What a trip does for the stages ahead, in pieces: per item the two halves of four splits of its K numbers, then their
    // three stores; the mask row; the request of the K rows after those; the same for V.
    static constexpr int kPieces = 18 * kItems + 4;
    Frag3 f;
    Bf16x3 part;
    template <int kSet, bool kIsV, int kItem, int Q>
    __device__ __forceinline__ void stash_piece(int buf)
    {
        constexpr int u = Q / 2;
        if constexpr (u < 4) {
            if constexpr (Q % 2 == 0) {
                if constexpr (kIsV)
                    part.first(v[kSet][kItem][2 * u], v[kSet][kItem][2 * u + 1], largest);
                else if constexpr ((u & 1) == 0)
                    part.first(k[kSet][kItem][u >> 1].x, k[kSet][kItem][u >> 1].y, largest);
                else
                    part.first(k[kSet][kItem][u >> 1].z, k[kSet][kItem][u >> 1].w, largest);
            } else {
                part.second();
                f.set(u, part);
            }
        } else {
            // threads past the last item (their loads repeated one) store nothing
            constexpr bool all_live = kIsV ? 64 * (kItem + 1) <= 32 * kDB : (kItem + 1) * kAtThreads <= kAll;
            if (all_live || (kIsV ? 64 * kItem + (tid & 63) < 32 * kDB : kItem * kAtThreads + tid < kAll)) {
                char* w = kIsV ? v_tiles + buf * T::kVTile + v_dst[kItem] : k_tiles + buf * T::kKTile + k_dst[kItem];
#pragma unroll
                for (int p = 0; p < 3; ++p) *reinterpret_cast<v4u*>(w + p * (kIsV ? T::kVPart : T::kKPart)) = f.part[p];
            }
        }
    }
    // kSet: parity of the current stage; k_stage: the K stage to store (two ahead; the V stage is the one before it)
    template <int kSet, int P>
    __device__ __forceinline__ void piece(int k_stage)
    {
        constexpr int kHalf = 9 * kItems + 2;
        if constexpr (P < 9 * kItems)
            stash_piece<kSet, false, P / 9, P % 9>(kSet);
        else if constexpr (P == 9 * kItems)
            stash_mask<kSet>(kSet, k_stage);
        else if constexpr (P == kHalf - 1)
            fetch_k<kSet>(k_stage + 2);
        else if constexpr (P < kHalf + 9 * kItems)
            stash_piece<kSet, true, (P - kHalf) / 9, (P - kHalf) % 9>(kSet ^ 1);
        else if constexpr (P == kPieces - 1)
            fetch_v<kSet>(k_stage + 1);   // past the last stage: empty descriptors, nothing is read
    }
    // the same, all at once
    template <int kSet>
    __device__ __forceinline__ void stash_k(int buf, int stage)
    {
        at_static_for<0, 9 * kItems>([&](auto pc) { stash_piece<kSet, false, decltype(pc)::value / 9, decltype(pc)::value % 9>(buf); });
        stash_mask<kSet>(buf, stage);
    }
    template <int kSet>
    __device__ __forceinline__ void stash_v(int buf)
    {
        at_static_for<0, 9 * kItems>([&](auto pc) { stash_piece<kSet, true, decltype(pc)::value / 9, decltype(pc)::value % 9>(buf); });
    }
    template <int kSet>
    __device__ __forceinline__ void all_pieces(int k_stage)
    {
        at_static_for<0, kPieces>([&](auto pc) { piece<kSet, decltype(pc)::value>(k_stage); });
    }
};

// Running state of a wave's 32 queries (lane (lq, hi) and lane (lq, 1 - hi) belong to the same query).
template <int kDB>
struct AttnWave {
    Frag3 q[2 * kDB];   // the queries, times scale * log2 e, split: step j holds columns 16 j + 8 hi .. + 7
    v16f o[kDB];        // O^T: o[blk][e] = ctx[query lq][column 32 blk + 8 (e/4) + 4 hi + e%4], not yet normalised
    float m_run;        // reference maximum (log2 units)
    float l_run;        // this lane's share of the running denominator
};

// First MFMA of the small products of a stage's scores: their sums start at the stage's mask row, or at zero where that is all
// zeros (the leading products start at zero, where the matrix pipes add them up exactly).  Number e of lane (lq, hi)
// belongs to key 8 (e/4) + 4 hi + e%4.
template <int kDB>
__device__ __forceinline__ v16f attention_first_mfma(const char* mask_row, int hi, const AttnWave<kDB>& w, const Frag3& kf, bool masked)
{
    if (!masked) return mfma_part<1>(kf, w.q[0], zero16());
    v16f s;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const float4 mk = *reinterpret_cast<const float4*>(mask_row + 16 * hi + 32 * g);
        s[4 * g + 0] = mk.x;
        s[4 * g + 1] = mk.y;
        s[4 * g + 2] = mk.z;
        s[4 * g + 3] = mk.w;
    }
    return mfma_part<1>(kf, w.q[0], s);
}

// Part kP of 2 of the maximum of a lane's sixteen scores.
template <int kP>
__device__ __forceinline__ void attention_max_piece(const v16f& s, float& mx)
{
    if constexpr (kP == 0) mx = s[0];
#pragma unroll
    for (int e = 8 * kP; e < 8 * kP + 8; e += 2) mx = at_max(mx, at_max(s[e], s[e + 1]));
    asm volatile("" : "+v"(mx));   // here, and not where it is used
}

// The reference against which a stage's probabilities are taken, from the maximum of the lane's scores.  It moves only
// when some query of the wave outgrows it by more than 2^8: below that the probabilities are merely up to 256 times larger
// (harmless in binary32, and the final division takes it out again), and the operations that shrink O are saved.  The
// first stage always moves it (it starts at -inf; key 0 is inside the sequence).
template <int kDB>
__device__ __forceinline__ void attention_move_reference(AttnWave<kDB>& w, float mx)
{
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    const float row_max = at_max(__uint_as_float(sw[0]), __uint_as_float(sw[1]));   // both half-waves hold keys of the query
    if (__builtin_amdgcn_ballot_w64(row_max > w.m_run + 8.0f) != 0) {
        const float m_up = at_max(w.m_run, row_max), alpha = __builtin_amdgcn_exp2f(w.m_run - m_up);
        w.m_run = m_up;
        w.l_run *= alpha;
#pragma unroll
        for (int b = 0; b < kDB; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) w.o[b][e] *= alpha;
    }
}

// One trip of the key loop, skewed by a stage: the softmax of the current stage's scores `sc` while -- kMore -- the
// matrix pipes form the next stage's, `sn`, from the K tile; then O^T += V^T P^T of the current stage while the rows
// requested two trips ago (K of `k_stage`, two ahead, and V of the stage before it) are split and stored and the next ones
// requested.  A wave issues in order, so the vector work goes between the MFMAs in pieces of a few instructions: an
// MFMA takes 32 cycles, and up to six vector instructions behind it are free; and the operands of a group of eight MFMAs
// are read from LDS 13 MFMAs ahead, each part into the place of one that is used up (six ahead, a group waited 50 to 100
// cycles for them; whole groups two ahead take twelve registers more, which spill at width 64).  kSet: parity of the
// current stage.
template <int kDB, bool kMore, int kSet>
__device__ __forceinline__ void attention_trip(const char* Kn, const char* Vs, int lq, int hi, v16f& sc, v16f& sn, AttnWave<kDB>& w,
                                               AttnStager<kDB>& sg, int k_stage)
{
    using T = AttnTile<kDB>;
    const char* krow = Kn + lq * T::kKStride + 16 * hi;
    const char* vrow = Vs + lq * T::kVStride + 16 * hi;
    constexpr int kKG = kMore ? 2 * kDB : 0, kGroups = kKG + 2 * kDB;   // groups of eight MFMAs: K steps, then column blocks x V steps
    Frag3 frag[2];
    // part p of the operands of group g
    auto read_part = [&](auto gc, auto pc) {
        constexpr int g = decltype(gc)::value, p = decltype(pc)::value;
        if constexpr (g < kKG) {
            frag[g % 2].part[p] = *reinterpret_cast<const v4u*>(krow + p * T::kKPart + 32 * g);
        } else if constexpr (g < kGroups) {
            constexpr int n = g - kKG;   // column block n / 2, step n % 2
            frag[g % 2].part[p] = *reinterpret_cast<const v4u*>(vrow + p * T::kVPart + (n / 2) * 32 * T::kVStride + 32 * (n % 2));
        }
    };
    // in front of MFMA i of group g: what takes the place of the part that the MFMAs before it used last
    auto read_ahead = [&](auto gc, auto ic) {
        constexpr int g = decltype(gc)::value, i = decltype(ic)::value;
        if constexpr (i == 0 && g > 0) read_part(std::integral_constant<int, g + 1>{}, std::integral_constant<int, 1>{});
        if constexpr (i == 3) read_part(std::integral_constant<int, g + 2>{}, std::integral_constant<int, 0>{});
        if constexpr (i == 5) read_part(std::integral_constant<int, g + 2>{}, std::integral_constant<int, 2>{});
    };
    at_static_for<0, 2>([&](auto gc) { at_static_for<0, 3>([&](auto pc) { read_part(gc, pc); }); });

    Frag3 pf[2];        // the probabilities, split: step j holds s[8 j .. 8 j + 7]
    Bf16x3 part;
    constexpr int kSoft = 24, kSoftFirst = kMore ? 6 : kSoft;   // the first ones go under the latency of the first operands
    auto soft = [&](auto pc) {   // per pair of keys: their probabilities, then the halves of their split
        constexpr int P = decltype(pc)::value, i = P / 3, q = P % 3;
        if constexpr (q == 0) {
            sc[2 * i] = __builtin_amdgcn_exp2f(sc[2 * i] - w.m_run);
            sc[2 * i + 1] = __builtin_amdgcn_exp2f(sc[2 * i + 1] - w.m_run);
            w.l_run += sc[2 * i] + sc[2 * i + 1];
            asm volatile("" : "+v"(w.l_run));   // here, and not gathered into one chain behind the trip
        } else if constexpr (q == 1) {
            part.first(sc[2 * i], sc[2 * i + 1]);
        } else {
            part.second();
            pf[i >> 2].set(i & 3, part);
        }
    };
    at_static_for<0, kSoftFirst>(soft);
    __builtin_amdgcn_sched_barrier(0);
    v16f rest;   // sums of the small partial products
    if constexpr (kMore) {
        constexpr int kNqk = kAtParts * kKG;
        at_static_for<0, kNqk>([&](auto nc) {
            constexpr int n = decltype(nc)::value, g = n / kAtParts, i = n % kAtParts;
            read_ahead(std::integral_constant<int, g>{}, std::integral_constant<int, i>{});
            if constexpr (i == 0)
                sn = mfma_part<0>(frag[g % 2], w.q[g], n == 0 ? zero16() : sn);
            else if constexpr (n == 1)
                rest = attention_first_mfma(Kn + T::kMask, hi, w, frag[0], sg.masked);
            else
                rest = mfma_part<i>(frag[g % 2], w.q[g], rest);
            at_static_for<kSoftFirst + (kSoft - kSoftFirst) * n / kNqk, kSoftFirst + (kSoft - kSoftFirst) * (n + 1) / kNqk>(soft);
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    // P V, a column block after the other: step j joins the keys of s[8 j .. 8 j + 7] of both half-waves
    constexpr int kBlock = 2 * kAtParts, kNpv = kBlock * kDB;
    float mx = 0.0f;
    at_static_for<0, kNpv>([&](auto nc) {
        constexpr int n = decltype(nc)::value, b = n / kBlock, j = (n / kAtParts) % 2, i = n % kAtParts, g = kKG + n / kAtParts;
        read_ahead(std::integral_constant<int, g>{}, std::integral_constant<int, i>{});
        if constexpr (i == 0)
            w.o[b] = mfma_part<0>(frag[g % 2], pf[j], w.o[b]);
        else
            rest = mfma_part<i>(frag[g % 2], pf[j], j == 0 && i == 1 ? zero16() : rest);
        if constexpr (n % kBlock == 0) {   // under an MFMA of another accumulator: the sums of the block before, or the scores
            if constexpr (b > 0)
                join_parts(w.o[b - 1], rest);
            else if constexpr (kMore)
                join_parts(sn, rest);
        }
        if constexpr (kMore) {
            if constexpr (n == 3) attention_max_piece<0>(sn, mx);
            if constexpr (n == 4) attention_max_piece<1>(sn, mx);
            constexpr int kP = AttnStager<kDB>::kPieces, kFrom = 5;
            if constexpr (n >= kFrom)
                at_static_for<kP*(n - kFrom) / (kNpv - kFrom), kP*(n + 1 - kFrom) / (kNpv - kFrom)>(
                    [&](auto pc) { sg.template piece<kSet, decltype(pc)::value>(k_stage); });
        }
        __builtin_amdgcn_sched_barrier(0);
    });
    join_parts(w.o[kDB - 1], rest);
    if constexpr (kMore) attention_move_reference(w, mx);
}

// Magnitudes are compared as bit patterns, which order like the numbers (a NaN above all).
// The bits minus one, doubled, for the smallest magnitude of numbers that are not zero: zero becomes the largest of all.
__device__ __forceinline__ unsigned nonzero_bits(float x) { return (__float_as_uint(x) << 1) - 1u; }

__device__ __forceinline__ void attention_ends(float4 v, unsigned& smallest, float& amax)
{
    smallest = min(smallest, min(min(nonzero_bits(v.x), nonzero_bits(v.y)), min(nonzero_bits(v.z), nonzero_bits(v.w))));
    // a NaN is passed over, as everywhere in the abs-max of ctx
    amax = __builtin_fmaxf(amax, __builtin_fmaxf(__builtin_fmaxf(__builtin_fabsf(v.x), __builtin_fabsf(v.y)), __builtin_fmaxf(__builtin_fabsf(v.z), __builtin_fabsf(v.w))));
}

// Four neighbouring results: ctx, or its codes under the stored scale of the next FC layer (Eq. 1), or both.
__device__ __forceinline__ void attention_store(const AttnArgs& a, int64_t off, float4 v, float qs)
{
    if (a.ctx) *reinterpret_cast<float4*>(a.ctx + off) = v;
    if (a.q_out)
        a.q_out[off >> 2] = ((unsigned)quantize_code(v.x, qs) & 0xffu) | (((unsigned)quantize_code(v.y, qs) & 0xffu) << 8) |
                            (((unsigned)quantize_code(v.z, qs) & 0xffu) << 16) | ((unsigned)quantize_code(v.w, qs) << 24);
}

// Whether results come out of the split products as they would of binary32 ones.  `largest`: bits of the largest magnitude
// that went into them; `smallest` and `amax`: of the smallest (nonzero_bits) and the largest result.  What lower parts under the smallest bf16 can do to
// a result is 2^-134 by a V row of weight 1 and, by the parts of the weights, 2^-134 of `largest` for each of up to 2^20 keys;
// both stay below 2^-24 of a result above this bound.
__device__ __forceinline__ bool attention_in_range(unsigned largest, unsigned smallest, unsigned amax)
{
    const float f = __uint_as_float(largest);
    if (largest > 0x7f800000u) return true;   // a NaN among the inputs
    return f <= 0x1p96f && amax < 0x7f800000u && smallest >= nonzero_bits(__builtin_fmaxf(0x1p-100f, f * 0x1p-90f));
}

// Rows q0 .. q0 + n - 1 of the context by one wave in plain binary32: 64 keys at a time, one per lane, then the columns of V
// (lane, lane + 64).  Returns this lane's abs-max.
__device__ __forceinline__ float attention_rows_plain(const AttnArgs& a, int64_t b, int h, int64_t q0, int n)
{
    const int lane = threadIdx.x & 63;
    const int64_t HD = (int64_t)a.heads * a.d, ld = 3 * HD;
    const float* base = a.qkv + b * a.S * ld + (int64_t)h * a.d;
    const float qs = a.q_out ? a.q_scale[0] : 0.0f;
    float amax = 0.0f;
    for (int64_t q = q0; q < q0 + n && q < a.S; ++q) {
        float m = -__builtin_inff(), l = 0.0f, acc[2] = {0.0f, 0.0f};
        for (int64_t j0 = 0; j0 < a.S; j0 += 64) {
            const int64_t j = j0 + lane;
            float s = -__builtin_inff();
            if (j < a.S) {
                const float *qp = base + q * ld, *kp = base + j * ld + HD;
                s = 0.0f;
#pragma unroll 4
                for (int k = 0; k < a.d; k += 4) {   // the width is a multiple of 4 and rows are 16-byte aligned here
                    const float4 qv = *reinterpret_cast<const float4*>(qp + k), kv = *reinterpret_cast<const float4*>(kp + k);
                    s = __builtin_fmaf(qv.x * a.c, kv.x, s);
                    s = __builtin_fmaf(qv.y * a.c, kv.y, s);
                    s = __builtin_fmaf(qv.z * a.c, kv.z, s);
                    s = __builtin_fmaf(qv.w * a.c, kv.w, s);
                }
                if (a.mask) s += mask_log2(a.mask[b * a.S + j]);
            }
            float m_up = s;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) m_up = __builtin_fmaxf(m_up, __shfl_xor(m_up, off, 64));
            m_up = __builtin_fmaxf(m, m_up);
            const float alpha = __builtin_amdgcn_exp2f(m - m_up), p = j < a.S ? __builtin_amdgcn_exp2f(s - m_up) : 0.0f;
            m = m_up;
            l = l * alpha + p;
            acc[0] *= alpha;
            acc[1] *= alpha;
            const int keys = (int)min((int64_t)64, a.S - j0);
#pragma unroll 8
            for (int t = 0; t < keys; ++t) {
                const float pt = __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(p), t));
                const float* vp = base + (j0 + t) * ld + 2 * HD;
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (lane + 64 * i < a.d) acc[i] = __builtin_fmaf(pt, vp[lane + 64 * i], acc[i]);
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
        const float inv = 1.0f / l;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (lane + 64 * i < a.d) {
                const float v = acc[i] * inv;
                const int64_t off = (b * a.S + q) * HD + (int64_t)h * a.d + lane + 64 * i;
                if (a.ctx) a.ctx[off] = v;
                if (a.q_out) reinterpret_cast<int8_t*>(a.q_out)[off] = (int8_t)quantize_code(v, qs);
                amax = __builtin_fmaxf(amax, __builtin_fabsf(v));
            }
    }
    return amax;
}

template <int kDB>
__global__ __launch_bounds__(kAtThreads, kDB <= 2 ? 2 : 1) void attention_mfma_kernel(AttnArgs a)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using T = AttnTile<kDB>;
    extern __shared__ __align__(16) char lds[];   // K tiles (+ mask rows) of two stages, then V tiles of two stages
    __shared__ uint4 wave_ends[kAtWaves];   // bits of the largest input, the smallest and the largest result of each wave

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, lq = lane & 31, hi = lane >> 5;
    // Workgroups of one (sequence, head) are neighbours in the logical order; each XCD takes a contiguous
    // run of it so that they find the K and V rows in the same L2.
    int wid = blockIdx.x;
    const int total = gridDim.x;
    if ((total & 7) == 0) wid = (wid & 7) * (total >> 3) + (wid >> 3);
    const int qb = wid % a.n_qblocks;
    const int bh = wid / a.n_qblocks;
    const int h = bh % a.heads;
    const int64_t b = bh / a.heads;
    const int64_t S = a.S, HD = (int64_t)a.heads * a.d, ld = 3 * HD;
    const float* base = a.qkv + b * S * ld + (int64_t)h * a.d;   // Q of token 0 of this sequence and head
    const int64_t q0 = (int64_t)qb * kAtQB + wave * kAtQW;
    const bool wave_live = q0 < S;      // a wave whose queries all lie beyond the sequence only helps with the staging

    AttnStager<kDB> sg;
    sg.kbase = base + HD;
    sg.vbase = base + 2 * HD;
    sg.mrow = a.mask ? a.mask + b * S : nullptr;
    sg.k_tiles = lds;
    sg.v_tiles = lds + 2 * T::kKTile;
    sg.ld = ld;
    sg.S32 = (int)S;
    sg.d = a.d;
    sg.init(tid);
    const int n_stages = (sg.S32 + kAtKB - 1) / kAtKB, last = n_stages - 1;

    // Everything the first trips need is requested at once -- a 128-token sequence in full -- so that its way from memory
    // is waited for once; columns beyond d are zeros in the queries (whatever K holds there).
    sg.template fetch_k<2>(0);
    AttnWave<kDB> w;
    float4 qraw[2 * kDB][2];
    {
        const int64_t qrow = (q0 + lq < S) ? q0 + lq : S - 1;
        const float* qp = base + qrow * ld;
#pragma unroll
        for (int j = 0; j < 2 * kDB; ++j)
#pragma unroll
            for (int u = 0; u < 2; ++u) qraw[j][u] = *reinterpret_cast<const float4*>(qp + min(16 * j + 8 * hi + 4 * u, a.d - 4));
    }
    sg.template fetch_v<2>(0);
    sg.template fetch_k<3>(1);
    sg.template fetch_k<0>(2);
    sg.template fetch_v<0>(1);
    sg.template fetch_k<1>(3);
    sg.template fetch_v<1>(2);
    __builtin_amdgcn_sched_barrier(0);
    sg.template stash_k<2>(0, 0);
#pragma unroll
    for (int j = 0; j < 2 * kDB; ++j)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const float c = (16 * j + 8 * hi + 4 * u < a.d) ? a.c : 0.0f;
            Bf16x3 part;
            part.first(qraw[j][u].x * c, qraw[j][u].y * c, sg.largest);
            part.second();
            w.q[j].set(2 * u, part);
            part.first(qraw[j][u].z * c, qraw[j][u].w * c, sg.largest);
            part.second();
            w.q[j].set(2 * u + 1, part);
        }
#pragma unroll
    for (int blk = 0; blk < kDB; ++blk)
#pragma unroll
        for (int e = 0; e < 16; ++e) w.o[blk][e] = 0.0f;
    w.m_run = -__builtin_inff();
    w.l_run = 0.0f;
    __syncthreads();
    v16f s0, s1;
    {
        const char* krow = sg.k_tiles + lq * T::kKStride + 16 * hi;
        v16f rest;
        at_static_for<0, 2 * kDB>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            Frag3 f;
#pragma unroll
            for (int p = 0; p < 3; ++p) f.part[p] = *reinterpret_cast<const v4u*>(krow + p * T::kKPart + 32 * j);
            s0 = mfma_part<0>(f, w.q[j], j == 0 ? zero16() : s0);
            if constexpr (j == 0) rest = attention_first_mfma(sg.k_tiles + T::kMask, hi, w, f, sg.masked);
            at_static_for<(j == 0 ? 2 : 1), kAtParts>([&](auto ic) { rest = mfma_part<decltype(ic)::value>(f, w.q[j], rest); });
        });
        join_parts(s0, rest);
    }
    sg.template stash_v<2>(0);
    sg.template stash_k<3>(1, 1);
    {
        float mx;
        attention_max_piece<0>(s0, mx);
        attention_max_piece<1>(s0, mx);
        attention_move_reference(w, mx);
    }
    __syncthreads();

    // Two trips per turn, so that the scores of the next stage become those of the current one without a copy.  A wave
    // without queries passes the same barriers.
    char *const k0 = sg.k_tiles, *const k1 = k0 + T::kKTile, *const v0 = sg.v_tiles, *const v1 = v0 + T::kVTile;
    int st = 0;
    if (wave_live) {
        for (; st + 2 <= last; st += 2) {
            attention_trip<kDB, true, 0>(k1, v0, lq, hi, s0, s1, w, sg, st + 2);
            __syncthreads();
            attention_trip<kDB, true, 1>(k0, v1, lq, hi, s1, s0, w, sg, st + 3);
            __syncthreads();
        }
        if (st < last) {
            attention_trip<kDB, true, 0>(k1, v0, lq, hi, s0, s1, w, sg, st + 2);
            __syncthreads();
            s0 = s1;
        }
        attention_trip<kDB, false, 0>(k0, (last & 1) ? v1 : v0, lq, hi, s0, s1, w, sg, 0);
    } else {
        for (; st + 2 <= last; st += 2) {
            sg.template all_pieces<0>(st + 2);
            __syncthreads();
            sg.template all_pieces<1>(st + 3);
            __syncthreads();
        }
        if (st < last) {
            sg.template all_pieces<0>(st + 2);
            __syncthreads();
        }
    }

    const auto l2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(w.l_run), __float_as_uint(w.l_run), false, false);
    const float inv = 1.0f / (__uint_as_float(l2[0]) + __uint_as_float(l2[1]));
    const bool live = q0 + lq < S;
    const float qs = a.q_out ? a.q_scale[0] : 0.0f;
    const int64_t out_off = (b * S + q0 + lq) * HD + (int64_t)h * a.d + 4 * hi;
    // Lanes beyond the sequence or the width repeat results of the last query or column: they change neither end.
    unsigned smallest = ~0u;
    float ctx_max = 0.0f;
#pragma unroll
    for (int blk = 0; blk < kDB; ++blk)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 v = make_float4(w.o[blk][4 * g + 0] * inv, w.o[blk][4 * g + 1] * inv, w.o[blk][4 * g + 2] * inv, w.o[blk][4 * g + 3] * inv);
            if (live && 32 * blk + 8 * g + 4 * hi < a.d) attention_store(a, out_off + 32 * blk + 8 * g, v, qs);
            attention_ends(v, smallest, ctx_max);   // 0 / 0 in a wave without queries: neither
        }
    unsigned largest = wave_max_u32(__float_as_uint(sg.largest));
    smallest = ~wave_max_u32(~smallest);
    unsigned amax = wave_max_u32(__float_as_uint(ctx_max));
    if (lane == 0) wave_ends[wave] = make_uint4(largest, smallest, amax, 0u);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kAtWaves; ++i) {
        largest = max(largest, wave_ends[i].x);
        smallest = min(smallest, wave_ends[i].y);
        amax = max(amax, wave_ends[i].z);
    }
    if (__builtin_expect(!attention_in_range(largest, smallest, amax), 0)) {
        __threadfence();   // behind the stores above
        amax = wave_max_u32(__float_as_uint(attention_rows_plain(a, b, h, q0, kAtQW)));
        __syncthreads();   // wave_ends has been read
        if (lane == 0) wave_ends[wave].z = amax;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kAtWaves; ++i) amax = max(amax, wave_ends[i].z);
    }
    if (a.slots) {
        if (tid == 0) {
            if (a.slots_atomic) {
                if (amax) atomicMax(a.slots + (blockIdx.x % kAtSlots), amax);
            } else {
                a.slots[blockIdx.x] = amax;
            }
        }
        if (!a.slots_atomic && blockIdx.x == 0)  // slots no workgroup owns
            for (int i = gridDim.x + tid; i < kAtSlots; i += kAtThreads) a.slots[i] = 0u;
    }
#endif
}

// The same products for launches that leave most of the chip idle: 32 queries of one (sequence, head) a workgroup, the
// key stages dealt out over its four waves, each with running statistics of its own that meet in LDS at the end.  A short
// sequence is a chain of latencies -- rows from memory, then per stage 64 MFMAs (of 32 cycles, at width 64) that the
// kernel above walks one after the other on an eighth of the compute units.  No wave shares its keys, so K and V go straight
// from memory into operand registers and nothing is staged: for every 32 queries they are read and split again, which is
// why full launches keep the kernel above.  One sequence of 128 tokens, 12 heads of 64: 11.2 -> 7.6 us; of 512: 28.9 ->
// 15.6; 2 x 256 of width 32: 13.1 -> 7.0.  Error against 64 bits no larger (1.3e-7 against 1.5e-7 at 128 tokens).
template <int kDB>
__global__ __launch_bounds__(kAtThreads, kDB <= 2 ? 2 : 1) void attention_split_kernel(AttnArgs a)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int kRow = 32 * kDB + 4;   // floats of a query's row of partial sums; the padding spreads rows over the banks
    __shared__ __attribute__((aligned(16))) float part_o[kAtWaves * kAtQW * kRow];
    __shared__ float part_m[kAtWaves * kAtQW], part_l[kAtWaves * kAtQW];
    __shared__ uint4 wave_ends[kAtWaves];   // bits of the largest input, the smallest and the largest result of each wave

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, lq = lane & 31, hi = lane >> 5;
    int wid = blockIdx.x;
    const int total = gridDim.x;
    if ((total & 7) == 0) wid = (wid & 7) * (total >> 3) + (wid >> 3);   // as above: an XCD takes whole (sequence, head)s
    const int qb = wid % a.n_qblocks, bh = wid / a.n_qblocks, h = bh % a.heads;
    const int64_t b = bh / a.heads;
    const int S = (int)a.S, d = a.d;
    const int64_t HD = (int64_t)a.heads * d, ld = 3 * HD;
    const float* base = a.qkv + b * S * ld + (int64_t)h * d;
    const float *kbase = base + HD, *vbase = base + 2 * HD;
    const float* mrow = a.mask ? a.mask + b * S : nullptr;
    const int q0 = qb * kAtQW, n_stages = (S + kAtKB - 1) / kAtKB;

    unsigned k_off[2 * kDB][2], v_off[kDB];   // byte offsets inside a stage
#pragma unroll
    for (int j = 0; j < 2 * kDB; ++j)
#pragma unroll
        for (int u = 0; u < 2; ++u) k_off[j][u] = 4u * ((unsigned)lq * (unsigned)ld + (unsigned)min(16 * j + 8 * hi + 4 * u, d - 4));
#pragma unroll
    for (int c = 0; c < kDB; ++c) v_off[c] = 4u * ((unsigned)(4 * hi) * (unsigned)ld + (unsigned)min(32 * c + lq, d - 1));
    // rows of a stage that exist, as a descriptor: the others read as zeros
    auto rsrc = [&](const float* p, int stage) {
        const int rows = min(S - stage * kAtKB, kAtKB);
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p) + (int64_t)stage * kAtKB * ld, 0, rows > 0 ? 4 * ((rows - 1) * (int)ld + d) : 0, 0x00020000);
    };
    float4 k[2 * kDB][2];
    float v[2][kDB][8], mk = 0.0f;   // mk: the mask of key lq
    auto fetch_k = [&](int stage) {
        const auto r = rsrc(kbase, stage);
#pragma unroll
        for (int j = 0; j < 2 * kDB; ++j)
#pragma unroll
            for (int u = 0; u < 2; ++u) k[j][u] = buf_f4(r, k_off[j][u]);
        if (mrow) mk = mrow[min(stage * kAtKB + lq, S - 1)];
    };
    auto fetch_v = [&](int stage) {   // step j, column block c: the eight keys this half-wave takes to the step
        const auto r = rsrc(vbase, stage);
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int c = 0; c < kDB; ++c) {
                unsigned col = v_off[c];
                asm volatile("" : "+v"(col));   // added up here: kept across the loop, the sixteen row offsets cost registers that spill
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    v[j][c][e] = buf_f1(r, col + 4u * (unsigned)(16 * j + (e & 3) + 8 * (e >> 2)) * (unsigned)ld);
            }
    };

    AttnWave<kDB> w;
    w.m_run = -__builtin_inff();
    w.l_run = 0.0f;
#pragma unroll
    for (int c = 0; c < kDB; ++c)
#pragma unroll
        for (int e = 0; e < 16; ++e) w.o[c][e] = 0.0f;
    float largest = 0.0f;   // magnitude of the numbers split so far
    if (wave < n_stages) {
        float4 qraw[2 * kDB][2];
        const float* qp = base + (int64_t)min(q0 + lq, S - 1) * ld;
#pragma unroll
        for (int j = 0; j < 2 * kDB; ++j)
#pragma unroll
            for (int u = 0; u < 2; ++u) qraw[j][u] = *reinterpret_cast<const float4*>(qp + min(16 * j + 8 * hi + 4 * u, d - 4));
        fetch_k(wave);
        fetch_v(wave);
#pragma unroll
        for (int j = 0; j < 2 * kDB; ++j)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float c = (16 * j + 8 * hi + 4 * u < d) ? a.c : 0.0f;   // columns beyond d are zeros here, whatever K holds
                w.q[j].set(2 * u, split_bf16(qraw[j][u].x * c, qraw[j][u].y * c, largest));
                w.q[j].set(2 * u + 1, split_bf16(qraw[j][u].z * c, qraw[j][u].w * c, largest));
            }
    }
    for (int st = wave; st < n_stages; st += kAtWaves) {
        // a stage that is walked has a key inside the sequence, so its maximum is above -inf
        v16f s = zero16(), rest = zero16();
        const int keys = S - st * kAtKB;
        if (mrow || keys < kAtKB) {   // every lane makes its key's value, the lanes that score the key fetch it
            const float m0 = lq < keys ? mask_log2(mk) : -__builtin_inff();
#pragma unroll
            for (int e = 0; e < 16; ++e) rest[e] = __uint_as_float((unsigned)__builtin_amdgcn_ds_bpermute(16 * hi + 4 * (8 * (e >> 2) + (e & 3)), (int)__float_as_uint(m0)));
        }
#pragma unroll
        for (int j = 0; j < 2 * kDB; ++j) {
            Frag3 f;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                f.set(2 * u, split_bf16(k[j][u].x, k[j][u].y, largest));
                f.set(2 * u + 1, split_bf16(k[j][u].z, k[j][u].w, largest));
            }
            s = mfma_part<0>(f, w.q[j], s);
            at_static_for<1, kAtParts>([&](auto ic) { rest = mfma_part<decltype(ic)::value>(f, w.q[j], rest); });
        }
        join_parts(s, rest);
        const bool more = st + kAtWaves < n_stages;
        if (more) fetch_k(st + kAtWaves);
        float mx;
        attention_max_piece<0>(s, mx);
        attention_max_piece<1>(s, mx);
        attention_move_reference(w, mx);
        Frag3 pf[2];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float p0 = __builtin_amdgcn_exp2f(s[2 * i] - w.m_run), p1 = __builtin_amdgcn_exp2f(s[2 * i + 1] - w.m_run);
            w.l_run += p0 + p1;
            pf[i >> 2].set(i & 3, split_bf16(p0, p1));
        }
#pragma unroll
        for (int c = 0; c < kDB; ++c) {
            rest = zero16();
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                Frag3 f;
#pragma unroll
                for (int u = 0; u < 4; ++u) f.set(u, split_bf16(v[j][c][2 * u], v[j][c][2 * u + 1], largest));
                w.o[c] = mfma_part<0>(f, pf[j], w.o[c]);
                at_static_for<1, kAtParts>([&](auto ic) { rest = mfma_part<decltype(ic)::value>(f, pf[j], rest); });
            }
            join_parts(w.o[c], rest);
        }
        if (more) fetch_v(st + kAtWaves);
    }

    // The waves' shares, each against its own reference; a wave without a stage has reference -inf and weight 0.
    {
        const auto l2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(w.l_run), __float_as_uint(w.l_run), false, false);
        if (hi == 0) {
            part_m[wave * kAtQW + lq] = w.m_run;
            part_l[wave * kAtQW + lq] = __uint_as_float(l2[0]) + __uint_as_float(l2[1]);
        }
        float* row = part_o + (wave * kAtQW + lq) * kRow + 4 * hi;
#pragma unroll
        for (int c = 0; c < kDB; ++c)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<float4*>(row + 32 * c + 8 * g) = make_float4(w.o[c][4 * g], w.o[c][4 * g + 1], w.o[c][4 * g + 2], w.o[c][4 * g + 3]);
    }
    const unsigned large_bits = wave_max_u32(__float_as_uint(largest));
    if (lane == 0) wave_ends[wave].x = large_bits;
    __syncthreads();
    const int q = tid >> 3;   // eight threads a query, four columns of every 32 each
    float m_all = part_m[q];
#pragma unroll
    for (int i = 1; i < kAtWaves; ++i) m_all = at_max(m_all, part_m[i * kAtQW + q]);
    float f[kAtWaves], den = 0.0f;
    unsigned all_large = 0u;
#pragma unroll
    for (int i = 0; i < kAtWaves; ++i) {
        f[i] = __builtin_amdgcn_exp2f(part_m[i * kAtQW + q] - m_all);
        den += f[i] * part_l[i * kAtQW + q];
        all_large = max(all_large, wave_ends[i].x);
    }
    const float inv = 1.0f / den;
    const float qs = a.q_out ? a.q_scale[0] : 0.0f;
    const int64_t out_off = (b * S + q0 + q) * HD + (int64_t)h * d;
    unsigned smallest = ~0u;   // lanes beyond the sequence or the width repeat other results, as above
    float ctx_max = 0.0f;
#pragma unroll
    for (int c = 0; c < kDB; ++c) {
        const int col = 32 * c + 4 * (tid & 7);
        float4 o = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
        for (int i = 0; i < kAtWaves; ++i) {
            const float4 p = *reinterpret_cast<const float4*>(part_o + (i * kAtQW + q) * kRow + col);
            o.x += f[i] * p.x;
            o.y += f[i] * p.y;
            o.z += f[i] * p.z;
            o.w += f[i] * p.w;
        }
        o.x *= inv;
        o.y *= inv;
        o.z *= inv;
        o.w *= inv;
        if (q0 + q < S && col < d) attention_store(a, out_off + col, o, qs);
        attention_ends(o, smallest, ctx_max);
    }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!attention_in_range(all_large, smallest, __float_as_uint(ctx_max))) != 0, 0)) {
        __threadfence();   // behind the stores above
        ctx_max = attention_rows_plain(a, b, h, q0 + 8 * wave, 8);   // a wave ends up with eight queries
    }
    if (a.slots) {   // never more workgroups than slots here
        unsigned amax = wave_max_u32(__float_as_uint(ctx_max));
        if (lane == 0) wave_ends[wave].z = amax;
        __syncthreads();
        if (tid == 0) {
#pragma unroll
            for (int i = 1; i < kAtWaves; ++i) amax = max(amax, wave_ends[i].z);
            a.slots[blockIdx.x] = amax;
        }
        if (blockIdx.x == 0)
            for (int i = gridDim.x + tid; i < kAtSlots; i += kAtThreads) a.slots[i] = 0u;
    }
#endif
}

// Any head width and alignment: one wave per (sequence, head, query).  Scores go to LDS, the softmax is the
// plain three-step form, then each lane sums its columns of V.  Slow; same tolerance.
__global__ __launch_bounds__(64) void attention_generic_kernel(const float* __restrict__ qkv, const float* __restrict__ mask,
                                                               float* __restrict__ ctx, unsigned* __restrict__ slots,
                                                               const float* __restrict__ q_scale, int8_t* __restrict__ q_out,
                                                               int64_t S, int heads, int d, float c)
{
    extern __shared__ __align__(16) float p[];   // S scores / probabilities
    const int lane = threadIdx.x;
    const int64_t i = blockIdx.x % S;
    const int64_t bh = blockIdx.x / S;
    const int h = (int)(bh % heads);
    const int64_t b = bh / heads;
    const int64_t HD = (int64_t)heads * d, ld = 3 * HD;
    const float* qrow = qkv + (b * S + i) * ld + (int64_t)h * d;
    float mx = -__builtin_inff();
    for (int64_t j = lane; j < S; j += 64) {
        const float* krow = qkv + (b * S + j) * ld + HD + (int64_t)h * d;
        float dot = 0.0f;
        for (int k = 0; k < d; ++k) dot = __builtin_fmaf(qrow[k] * c, krow[k], dot);
        if (mask) dot += mask_log2(mask[b * S + j]);
        p[j] = dot;
        mx = __builtin_fmaxf(mx, dot);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = __builtin_fmaxf(mx, __shfl_xor(mx, off, 64));
    float den = 0.0f;
    for (int64_t j = lane; j < S; j += 64) {
        const float e = __builtin_amdgcn_exp2f(p[j] - mx);
        p[j] = e;
        den += e;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) den += __shfl_xor(den, off, 64);
    __syncthreads();
    const float inv = 1.0f / den;
    const float qs = q_out ? q_scale[0] : 0.0f;
    float amax = 0.0f;
    for (int k = lane; k < d; k += 64) {
        const float* vcol = qkv + b * S * ld + 2 * HD + (int64_t)h * d + k;
        float acc = 0.0f;
        for (int64_t j = 0; j < S; ++j) acc = __builtin_fmaf(p[j], vcol[j * ld], acc);
        const float v = acc * inv;
        const int64_t off = (b * S + i) * HD + (int64_t)h * d + k;
        if (ctx) ctx[off] = v;
        if (q_out) q_out[off] = (int8_t)quantize_code(v, qs);
        amax = __builtin_fmaxf(amax, __builtin_fabsf(v));
    }
    if (slots) {
        const unsigned m = wave_max_u32(__float_as_uint(amax));
        if (lane == 0 && m) atomicMax(slots + (blockIdx.x % kAtSlots), m);
    }
}

__global__ void attention_slots_clear_kernel(unsigned* slots)
{
    for (int i = threadIdx.x; i < kAtSlots; i += 256) slots[i] = 0u;
}

static bool at_aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

int attention_generic_max_s() { return 16384; }   // scores of one query in 64 KiB of LDS

bool attention_mfma_eligible(const float* qkv, int64_t B, int64_t S, int heads, int d, const float* ctx, const int8_t* q_out)
{
    const int64_t wgs = B * heads * ((S + kAtQB - 1) / kAtQB);
    // 32-bit arithmetic inside: the workgroup count, the row index, and byte offsets within 32 rows of qkv
    return d % 4 == 0 && d <= kAtMaxD && at_aligned(qkv, 16) && (!ctx || at_aligned(ctx, 16)) && at_aligned(q_out, 4) &&
           wgs < ((int64_t)1 << 31) && S < ((int64_t)1 << 30) && (int64_t)kAtKB * 3 * heads * d < ((int64_t)1 << 29);
}

template <int kDB>
static int launch_attention_width(AttnArgs a, int64_t wgs, hipStream_t st)
{
    // The split kernel while each of its workgroups has one of the 256 compute units for itself: at 256 workgroups of width 64
    // it takes 7.9 us against 11.4 on sequences of 4 stages, 10.1 against 17.0 on 8, 22.3 against 50.7 on 32, of width 128 28.3
    // against 60.4 on 16.  With two on a unit (widths up to 64): width 32 always (384 workgroups of 1 / 2 / 3 / 4 / 8 / 16
    // stages 5.1 / 6.2 / 6.5 / 6.9 / 9.3 / 13.2 us against 6.4 / 6.3 / 7.7 / 8.8 / 13.4 / 22.6), width 64 but for
    // sequences of two and three stages (1 / 2 / 3 / 4 / 5 / 6 / 7 / 8 / 16 stages 7.0 / 9.3 / 10.2 / 10.9 / 13.5 / 14.4 /
    // 15.4 / 14.8 / 21.5 against 8.8 / 8.1 / 9.9 / 11.8 / 13.9 / 14.8 / 16.6 / 17.6 / 29.0).  Beyond, its third round
    // costs more than the chain it shortens (576 of width 64: 4 / 8 / 16 stages 15.3 / 20.0 / 31.7 against 12.5 / 18.1 / 29.5).
    const int64_t bh = wgs / a.n_qblocks, n_q32 = (a.S + kAtQW - 1) / kAtQW, wgs32 = bh * n_q32;
    const bool split = wgs32 <= 256 || (wgs32 <= 512 && (kDB == 1 || (kDB == 2 && (n_q32 == 1 || n_q32 >= 4))));
    if (split) {
        a.n_qblocks = (int)n_q32;
        hipLaunchKernelGGL(attention_split_kernel<kDB>, dim3((unsigned)wgs32), dim3(kAtThreads), 0, st, a);
        return hipGetLastError() == hipSuccess ? 0 : 1;
    }
    constexpr int lds_bytes = AttnTile<kDB>::kBytes;
    if constexpr (lds_bytes > 64 * 1024) {   // more than 64 KiB of dynamic LDS has to be asked for
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(attention_mfma_kernel<kDB>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                lds_bytes) != hipSuccess)
            return 1;
    }
    hipLaunchKernelGGL(attention_mfma_kernel<kDB>, dim3((unsigned)wgs), dim3(kAtThreads), lds_bytes, st, a);
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

int launch_attention(const float* qkv, int64_t B, int64_t S, int heads, int d, const float* mask, float scale, float* ctx,
                     float* amax_slots, const float* q_scale, int8_t* q_out, hipStream_t st)
{
    unsigned* slots = reinterpret_cast<unsigned*>(amax_slots);
    if (B == 0) {
        if (slots) hipLaunchKernelGGL(attention_slots_clear_kernel, dim3(1), dim3(256), 0, st, slots);
        return hipGetLastError() == hipSuccess ? 0 : 1;
    }
    const float c = scale * 1.44269504088896341f;
    const int64_t n_qblocks = (S + kAtQB - 1) / kAtQB;
    const int64_t wgs = B * heads * n_qblocks;
    if (attention_mfma_eligible(qkv, B, S, heads, d, ctx, q_out)) {
        AttnArgs a;
        a.qkv = qkv;
        a.mask = mask;
        a.ctx = ctx;
        a.slots = slots;
        a.q_scale = q_scale;
        a.q_out = reinterpret_cast<unsigned*>(q_out);
        a.S = S;
        a.heads = heads;
        a.d = d;
        a.n_qblocks = (int)n_qblocks;
        a.slots_atomic = wgs > kAtSlots;
        a.c = c;
        if (slots && a.slots_atomic) hipLaunchKernelGGL(attention_slots_clear_kernel, dim3(1), dim3(256), 0, st, slots);
        switch ((d + 31) / 32) {
            case 1: return launch_attention_width<1>(a, wgs, st);
            case 2: return launch_attention_width<2>(a, wgs, st);
            case 3: return launch_attention_width<3>(a, wgs, st);
            default: return launch_attention_width<4>(a, wgs, st);
        }
    } else {
        const int64_t blocks = B * heads * S;
        if (blocks >= ((int64_t)1 << 31)) return 1;
        if (slots) hipLaunchKernelGGL(attention_slots_clear_kernel, dim3(1), dim3(256), 0, st, slots);
        hipLaunchKernelGGL(attention_generic_kernel, dim3((unsigned)blocks), dim3(64), (size_t)S * sizeof(float), st, qkv,
                           mask, ctx, slots, q_scale, q_out, S, heads, d, c);
    }
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

}  // namespace q8

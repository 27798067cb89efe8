// Routing kernels of the BrownoutMoE layer for gfx950:
//   prep     split fp32 gate weights into three bf16 pieces (also the one-time repack behind moe_pack_gate), clear the
//            expert counters (large batches over at most 16 experts; the logit kernel does it for more)
//   gate     affinities s = x.e_i on MFMA (bf16 x 3-piece weights, fp64 running sums, pieces and x rows staged in LDS) or,
//            for at most 16 experts and small batches, in plain fp64; TopK by wavefront shuffles, weights g, expert
//            histogram.  More than 16 experts: two launches, logits (blocks of 16, 64 or 128 tokens by 64 experts by a
//            slice of K) and TopK                                    (Architecture of BrownoutMoE)
//   rows     up to 8192 tokens, one launch: expert counts, Algorithm 1's S1/S2 split and unit map (Brownout Approach,
//            Algorithm 1), the row lists row_token, row_weight, token_rows (stable: ascending token inside a unit) and the
//            GEMM tile tables; for few tokens it takes TopK as well
//   count, scan, scatter   the same for larger batches: the rows each 64-token segment gives each unit, offsets of segments
//            inside units and unit totals, row lists and tile tables
// No floating-point atomics anywhere; integer atomics only where the result does not depend on order.
#include "internal.h"
#include "tiles.h"

#include <algorithm>
#include <type_traits>

namespace bmoe {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned short f32_to_bf16_bits(float f)
{
    unsigned int u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest, ties to even
    return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf16_bits_to_f32(unsigned short b) { return __uint_as_float(((unsigned int)b) << 16); }

// ------------------------------------------------------------------------------------------------
// prep: expert_cnt = 0; gate_w = hi + mid + lo with bf16 pieces (the three pieces carry 24 bits of
// significand, so x(bf16) * piece products are exact in fp32 and their sum equals x*w to fp32 accuracy).
// Rows m..m_pad-1 of every piece are zero.
// ------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) prep_kernel(const float* __restrict__ gate_w, int m, int m_pad, int d,
                                                   unsigned short* __restrict__ split, int32_t* __restrict__ expert_cnt)
{
    const size_t n = split != nullptr ? (size_t)m_pad * d : 0;   // split == nullptr: only clear the counters
    const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (expert_cnt != nullptr && gid < (size_t)m) expert_cnt[gid] = 0;
    for (size_t i = gid; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int e = (int)(i / d);
        const float w = e < m ? gate_w[i] : 0.0f;
        const unsigned short hi = f32_to_bf16_bits(w);
        const float r1 = w - bf16_bits_to_f32(hi);
        const unsigned short mid = f32_to_bf16_bits(r1);
        const float r2 = r1 - bf16_bits_to_f32(mid);
        const unsigned short lo = f32_to_bf16_bits(r2);
        split[i] = hi;
        split[n + i] = mid;
        split[2 * n + i] = lo;
    }
}

// ------------------------------------------------------------------------------------------------
// gate: affinities on MFMA.  Each k chunk is accumulated from zero by 16x16x32 bf16 MFMAs over the low,
// middle and high piece of the gate weights and folded into an fp64 running sum at least every 64 k, which
// keeps the logit within a few 1e-8 of the exact dot product whatever d is.
// ------------------------------------------------------------------------------------------------
struct GateArgs {
    const bf16_t* x; const unsigned short* split; const float* bias;
    int T, d, m, m_pad, K, score_fn;
    int32_t* topk_idx; float* topk_w; uint8_t* near_tie;
    int32_t* expert_cnt;   // the batch's expert counts (atomics on cleared counters); null where the row kernel counts the
                           // experts itself
    int n_slice;           // 17 experts and more: slices of K, each leaving fp64 partial logits
    void* logits;          // one slice: [T][m_pad] fp32, bias added; else [n_slice][T][m_pad] fp64
    int32_t* clear_cnt;    // expert counters the logit kernel clears for the TopK launch behind it (or null)
    unsigned long long* bits;   // [n_seg][m]: which of a segment's 64 tokens name the expert (null: not wanted).  The last
                                // segment's quarters without tokens are not written
    int t_base;            // token of the batch that token 0 of this launch is (a multiple of 16 with bits)
};

// What a block of 16 tokens leaves of its winners besides the lists: a map of its tokens per expert (p.bits: a quarter of a
// segment's word), or counts for the launches behind it.
__device__ __forceinline__ void note_winner(const GateArgs& p, int* hist, int tl, int e)
{
    if (p.bits != nullptr) atomicOr(&hist[e], 1 << tl);
    else atomicAdd(&hist[e], 1);
}
template <int THREADS>
__device__ __forceinline__ void flush_winners(const GateArgs& p, const int* hist, int tid)
{
    if (p.bits != nullptr) {
        const int t16 = p.t_base / 16 + (int)blockIdx.x;
        unsigned short* out = reinterpret_cast<unsigned short*>(p.bits) + (size_t)(t16 >> 2) * p.m * 4 + (t16 & 3);
        for (int i = tid; i < p.m; i += THREADS) out[4 * i] = (unsigned short)hist[i];
    } else if (p.expert_cnt != nullptr) {
        for (int i = tid; i < p.m; i += THREADS)
            if (hist[i] > 0) atomicAdd(&p.expert_cnt[i], hist[i]);
    }
}

// row_ror:n of a 16-lane row (DPP control 0x120 + n): lane l reads lane (l - n) mod 16 of its row
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false); }
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) { return __int_as_float(dpp_i<CTRL>(__float_as_int(v))); }

// A logit as an integer of the same order (-0 as +0, NaN as -infinity) and back.
__device__ __forceinline__ int order_key(float v)
{
    const int i = __float_as_int(v + 0.0f);
    return v != v ? (int)0x807fffff : i ^ ((i >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float key_value(int k) { return __int_as_float(k ^ ((k >> 31) & 0x7fffffff)); }
// the other operand comes through the instruction itself
template <int CTRL>
__device__ __forceinline__ int max_dpp(int v) { return max(v, __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, true)); }
template <int CTRL>
__device__ __forceinline__ int min_dpp(int v) { return min(v, __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, true)); }

// TopK(.,K) of one token by one wavefront: lane holds experts lane, lane+64, ...; K (+1 for the best loser) rounds of "largest key of
// the wavefront, then the lowest id that holds it" (experts already taken are no candidates).  Lane j keeps the j-th winner, weights are
// normalised over lanes 0..K-1.  What bounds it is the issue of the rounds: by keys some 30 instructions each, with value and id carried
// together through every exchange and compared as floats some 75 (routing of 1024 tokens x 32 of 128 experts 53 us, now 32).
// put(j, expert, weight): called by the lanes that hold a winner, besides the store to the output arrays.
template <typename Put>
__device__ __forceinline__ void topk_token(const GateArgs& p, const float (&v)[4], int t, int lane, Put put)
{
    const int K = p.K;
    const int n_pick = K < p.m ? K + 1 : K;    // one extra pick: the best loser, for the near-tie flag
    constexpr int kTaken = (int)0x80000000;
    int k[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) k[c] = lane + 64 * c < p.m ? order_key(v[c]) : kTaken;
    int my_k = 0, my_i = 0;
    for (int j = 0; j < n_pick; ++j) {
        int mx = max(max(k[0], k[1]), max(k[2], k[3]));
        mx = max_dpp<0x128>(max_dpp<0x124>(max_dpp<0x122>(max_dpp<0x121>(mx))));
        mx = max(max(__builtin_amdgcn_readlane(mx, 0), __builtin_amdgcn_readlane(mx, 16)),
                 max(__builtin_amdgcn_readlane(mx, 32), __builtin_amdgcn_readlane(mx, 48)));
        int id = 0;
#pragma unroll
        for (int c = 3; c >= 0; --c) {
            const unsigned long long b = __ballot(k[c] == mx);
            if (b != 0ull) id = 64 * c + __builtin_ctzll(b);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) k[c] = lane + 64 * c == id ? kTaken : k[c];
        if (lane == j) { my_k = mx; my_i = id; }
    }
    const float my_v = key_value(my_k);
    const float top = __shfl(my_v, 0);
    float num = 0.0f;
    if (lane < K) num = p.score_fn == 0 ? expf(my_v - top) : 1.0f / (1.0f + expf(-my_v));
    float den = num;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) den += __shfl_xor(den, off);
    const float nxt = __shfl_down(my_v, 1);
    const bool close = lane + 1 < n_pick && (my_v - nxt) < 1e-6f;
    const unsigned long long any_close = __ballot(close);
    if (lane < K) {
        const float w = num / den;
        p.topk_idx[(size_t)t * K + lane] = my_i;
        p.topk_w[(size_t)t * K + lane] = w;
        put(lane, my_i, w);
    }
    if (lane == 0 && p.near_tie != nullptr) p.near_tie[t] = any_close != 0ull ? 1 : 0;
}

// Weights and outputs of four tokens, a row of 16 lanes each: lane j of a row holds the key and the id of the j-th winner.  LIKE_TOKEN:
// the weights are added up in topk_token's order.
template <bool LIKE_TOKEN, typename Put>
__device__ __forceinline__ void weights_rows(const GateArgs& p, int my_k, int my_i, int t, bool valid, int lane, Put put)
{
    const int K = p.K, r = lane & 15, n_pick = K < p.m ? K + 1 : K;
    const float my_v = key_value(my_k);
    const float top = dpp_f<0x150>(my_v);                   // row_newbcast: lane 0 of the row
    float num = 0.0f;
    if (r < K) num = p.score_fn == 0 ? expf(my_v - top) : 1.0f / (1.0f + expf(-my_v));
    float den = num;
    if constexpr (LIKE_TOKEN) {
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) den += __shfl_xor(den, off);
    } else {
        den += dpp_f<0x121>(den);
        den += dpp_f<0x122>(den);
        den += dpp_f<0x124>(den);
        den += dpp_f<0x128>(den);
    }
    const float nxt = __shfl(my_v, (lane & ~15) | ((r + 1) & 15));
    const bool close = r + 1 < n_pick && (my_v - nxt) < 1e-6f;
    const unsigned long long any_close = __ballot(close);
    if (valid) {
        if (r < K) {
            const float w = num / den;
            p.topk_idx[(size_t)t * K + r] = my_i;
            p.topk_w[(size_t)t * K + r] = w;
            put(r, my_i, w);
        }
        if (r == 0 && p.near_tie != nullptr) p.near_tie[t] = ((any_close >> (lane & 48)) & 0xFFFFull) != 0ull ? 1 : 0;
    }
}

// The same for four tokens at a time: token `row` = lane >> 4 of the four is handled by the 16 lanes of its
// row, lane r of the row holding experts r, r+16, ... (NC of them: NC >= m_pad / 16); every reduction stays
// inside the row (rotations), so the four selections run side by side.  A lane's experts that do not exist or
// have been picked hold -infinity (a row that has nothing above that left picks expert 0 again).  A round first takes the
// maximum, over NC registers and four rotations, then the lowest id that holds it, the same way: about 6 NC / 2 + 16
// instructions (value and id carried together: 9 a rotation; a block with 16 wavefronts is bound by their issue).
// Needs K + 1 <= 16 (lane j of the row keeps the j-th winner).
// v[c]: the logit of expert r + 16 c (-infinity: no such expert), t: the row's token, valid: whether it exists.
template <int NC, typename Put>
__device__ __forceinline__ void topk_rows(const GateArgs& p, const float (&v)[NC], int t, bool valid, int lane, Put put)
{
    const int K = p.K, r = lane & 15;
    const int n_pick = K < p.m ? K + 1 : K;
    constexpr int kNone = (int)0x807fffff;                  // -infinity
    int k[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) k[c] = order_key(v[c]);
    int my_k = 0, my_i = 0;
    for (int j = 0; j < n_pick; ++j) {
        int mx = k[0];
#pragma unroll
        for (int c = 1; c < NC; ++c) mx = max(mx, k[c]);
        mx = max_dpp<0x128>(max_dpp<0x124>(max_dpp<0x122>(max_dpp<0x121>(mx))));
        int id = 0x7fffffff;
#pragma unroll
        for (int c = NC - 1; c >= 0; --c) id = k[c] == mx ? 16 * c + r : id;
        id = min_dpp<0x128>(min_dpp<0x124>(min_dpp<0x122>(min_dpp<0x121>(id))));
        const int wc = (id & 15) == r ? (id >> 4) : -1;     // the winner leaves its lane's candidates
#pragma unroll
        for (int c = 0; c < NC; ++c) k[c] = c == wc ? kNone : k[c];
        if (r == j) { my_k = mx; my_i = id; }
    }
    weights_rows<false>(p, my_k, my_i, t, valid, lane, put);
}

// The same for at most 16 experts, lane r of the row holding expert r, with topk_token's winners and weights: an expert already
// taken is no candidate (so experts of logit -infinity are picked one after the other, not repeated), and the weights are added
// up in its order.
template <typename Put>
__device__ __forceinline__ void topk_few(const GateArgs& p, float v, int t, bool valid, int lane, Put put)
{
    const int K = p.K, r = lane & 15;
    const int n_pick = K < p.m ? K + 1 : K;
    constexpr int kTaken = (int)0x80000000;
    int k = r < p.m ? order_key(v) : kTaken;
    int my_k = 0, my_i = 0;
    for (int j = 0; j < n_pick; ++j) {
        const int mx = max_dpp<0x128>(max_dpp<0x124>(max_dpp<0x122>(max_dpp<0x121>(k))));
        int id = k == mx ? r : 16;
        id = min_dpp<0x128>(min_dpp<0x124>(min_dpp<0x122>(min_dpp<0x121>(id))));
        if (id == r) k = kTaken;
        if (r == j) { my_k = mx; my_i = id; }
    }
    weights_rows<true>(p, my_k, my_i, t, valid, lane, put);
}

// gate for at most 16 experts in batches beyond kFewExpertsTokens tokens: one block = 16 tokens x the one tile of
// experts, 8 wavefronts that split K.  A stage is 256 k: the 48 rows of the three gate pieces and the 16 x rows,
// as four pieces of 64 k (rows of 128 bytes = whole lines, brought in by direct global->LDS loads, 8 rows per
// wave instruction; a wave that lets every lane fetch its own 16-byte fragment instead spends its time on tag
// look-ups: 16 rows x 64 bytes per instruction).  Wave w multiplies the 32-wide half w&1 of piece w>>1 of every
// stage, three MFMAs (low, middle, high piece) folded into fp64 sums; the eight partial sums of a logit are added
// in wave order through LDS.  Three stages: two in flight while one is multiplied.
__global__ void __launch_bounds__(512) gate_few_kernel(GateArgs p)
{
    constexpr int RB = 128, SUB = 64 * RB, STAGE = 4 * SUB, NST = 3;
    extern __shared__ __attribute__((aligned(16))) char gsm[];
    __shared__ int hist[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wave_s = __builtin_amdgcn_readfirstlane(wave);
    const int t0 = blockIdx.x * 16;
    if (tid < 16) hist[tid] = 0;
    const int n_sub = p.d >> 6, n_stage = (n_sub + 3) >> 2;
    const int sub = wave_s >> 1, sl = wave_s & 1;

    // loader: the four loads of wave w bring rows 8 (4 (w&1) + i) .. +7 of piece w>>1; 16-byte chunk c of row r
    // sits in slot c ^ ((r/2)&7) (conflict-free ds_read_b128)
    const unsigned short* srcp[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = (sl * 4 + i) * 8 + (lane >> 3);
        const int chunk = (lane & 7) ^ ((row >> 1) & 7);
        const unsigned short* src = row < 48 ? p.split + (size_t)row * p.d
                                             : reinterpret_cast<const unsigned short*>(p.x) +
                                                   (size_t)min(t0 + row - 48, p.T - 1) * p.d;
        srcp[i] = src + chunk * 8;
    }
    auto issue = [&](int st, int buf) {
        const int piece = min(st * 4 + sub, n_sub - 1);   // past the end of K: the last piece again, never multiplied
        char* dst = gsm + buf * STAGE + sub * SUB + sl * 4096;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(srcp[i] + piece * 64),
                                             (__attribute__((address_space(3))) void*)(dst + i * 1024), 16, 0, 0);
    };
    // fragment of row (base + lane&15), 32-wide half sl: chunks 4 sl + (lane>>4); bases are multiples of 16 rows
    const int coff = ((sl * 4 + (lane >> 4)) ^ (((lane & 15) >> 1) & 7)) << 4;
    const int roff = (lane & 15) * RB + coff;
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    for (int q = 0; q < NST - 1; ++q)
        if (q < n_stage) issue(q, q);
    int buf = 0;
    for (int st = 0; st < n_stage; ++st) {
        // loads complete in order: stage st has landed once only the four loads of stage st+1 are outstanding
        if (st + 1 < n_stage) __builtin_amdgcn_s_waitcnt(0x0F74);
        else __builtin_amdgcn_s_waitcnt(0x0F70);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();                     // stage st is in LDS for everyone; stage st-1 is free
        asm volatile("" ::: "memory");
        if (st + NST - 1 < n_stage) issue(st + NST - 1, buf == 0 ? NST - 1 : buf - 1);
        if (st * 4 + sub < n_sub) {
            const char* St = gsm + buf * STAGE + sub * SUB + roff;
            const bf16x8 a = *reinterpret_cast<const bf16x8*>(St + 48 * RB);
            const bf16x8 b_hi = *reinterpret_cast<const bf16x8*>(St);
            const bf16x8 b_mid = *reinterpret_cast<const bf16x8*>(St + 16 * RB);
            const bf16x8 b_lo = *reinterpret_cast<const bf16x8*>(St + 32 * RB);
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b_lo, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b_mid, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b_hi, acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) sum[v] += (double)acc[v];
        }
        buf = buf + 1 == NST ? 0 : buf + 1;
    }
    __syncthreads();                                      // every wave is done with the stages: reuse them
    double* part = reinterpret_cast<double*>(gsm);        // [wave][token][expert]
    float* logit = reinterpret_cast<float*>(gsm + 8 * 256 * 8);
    // MFMA 16x16 result layout: lane holds column (lane&15) = expert, rows 4*(lane>>4)+v = tokens
#pragma unroll
    for (int v = 0; v < 4; ++v) part[(wave * 16 + 4 * (lane >> 4) + v) * 16 + (lane & 15)] = sum[v];
    __syncthreads();
    if (tid < 256) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < 8; ++w) s += part[w * 256 + tid];
        const int e = tid & 15;
        if (p.bias != nullptr && e < p.m) s += (double)p.bias[e];
        logit[tid] = (float)s;
    }
    __syncthreads();
    if (wave < 4) {                                       // four tokens per wavefront (K + 1 <= m_pad = 16 picks)
        const int tl = wave * 4 + (lane >> 4);
        const bool valid = t0 + tl < p.T;
        float v[1] = {(lane & 15) < p.m ? logit[tl * 16 + (lane & 15)] : -__builtin_inff()};
        topk_rows<1>(p, v, t0 + tl, valid, lane, [&](int, int e, float) { note_winner(p, hist, tl, e); });
    }
    __syncthreads();
    flush_winners<512>(p, hist, tid);
}

// ------------------------------------------------------------------------------------------------
// gate for at most 16 experts and at most kFewExpertsTokens tokens: plain fp64 arithmetic, no matrix cores.
// With so few experts and tokens what the gate needs is many blocks in flight (a CU pulls its share of x and
// the whole gate matrix at the rate of the few loads it keeps in flight), not MFMA tiles padded from m to 16
// columns: 15 us instead of 24 for 256 tokens of width 4096.  (Beyond a few thousand tokens the MFMA gate, which
// reads the gate matrix once per 16 tokens, is faster again: 28 us against 44 at 4096 tokens.)  One block = TPB tokens, 256 threads; thread t multiplies the k range
// 8t .. 8t+7 (+2048, ...) of the tokens' rows with every centroid, products and sums in double (a bf16 times an
// fp32 value is exact there), the 256 partial sums of a (token, expert) pair are added in a fixed order through
// LDS, and one wavefront per token takes TopK.  The centroids are read as fp32 rows (for at most 16 experts the
// packed form of the gate is a copy of them).
// ------------------------------------------------------------------------------------------------
template <int M, int TPB>
__global__ void __launch_bounds__(256) gate_small_kernel(GateArgs p, const float* __restrict__ gate_w)
{
    constexpr int NP = TPB * M;                           // (token, expert) pairs of the block
    __shared__ double part[NP][33];
    __shared__ float logit[TPB][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t0 = blockIdx.x * TPB;
    double acc[TPB][M];
#pragma unroll
    for (int q = 0; q < TPB; ++q)
#pragma unroll
        for (int e = 0; e < M; ++e) acc[q][e] = 0.0;
    for (int k = tid * 8; k < p.d; k += 2048) {
        double xv[TPB][8];
#pragma unroll
        for (int q = 0; q < TPB; ++q) {
            const int t = min(t0 + q, p.T - 1);
            const uint4 raw = *reinterpret_cast<const uint4*>(p.x + (size_t)t * p.d + k);
            const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                xv[q][2 * c] = (double)__uint_as_float(w[c] << 16);
                xv[q][2 * c + 1] = (double)__uint_as_float(w[c] & 0xFFFF0000u);
            }
        }
        // eight rows of the gate matrix on their way at a time (past the last one: that one again, the sums are not used)
#pragma unroll
        for (int e0 = 0; e0 < M; e0 += 8) {
            float4 wv[8][2];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float* row = gate_w + (size_t)min(e0 + e, p.m - 1) * p.d + k;
                wv[e][0] = *reinterpret_cast<const float4*>(row);
                wv[e][1] = *reinterpret_cast<const float4*>(row + 4);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int q = 0; q < TPB; ++q)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        acc[q][e0 + e] = fma(xv[q][4 * h], (double)wv[e][h].x, acc[q][e0 + e]);
                        acc[q][e0 + e] = fma(xv[q][4 * h + 1], (double)wv[e][h].y, acc[q][e0 + e]);
                        acc[q][e0 + e] = fma(xv[q][4 * h + 2], (double)wv[e][h].z, acc[q][e0 + e]);
                        acc[q][e0 + e] = fma(xv[q][4 * h + 3], (double)wv[e][h].w, acc[q][e0 + e]);
                    }
        }
    }
    // the 256 partial sums of a pair: eight neighbouring lanes first (three exchange steps), then the 32 group
    // sums in order by one thread
#pragma unroll
    for (int q = 0; q < TPB; ++q)
#pragma unroll
        for (int e = 0; e < M; ++e) {
            double v = acc[q][e];
            v += __shfl_xor(v, 1);
            v += __shfl_xor(v, 2);
            v += __shfl_xor(v, 4);
            if ((lane & 7) == 0) part[q * M + e][tid >> 3] = v;
        }
    __syncthreads();
    if (tid < NP) {
        const int q = tid / M, e = tid - q * M;
        if (e < p.m) {
            double s = 0.0;
            for (int i = 0; i < 32; ++i) s += part[tid][i];
            if (p.bias != nullptr) s += (double)p.bias[e];
            if (p.logits == nullptr) logit[q][e] = (float)s;
            else if (t0 + q < p.T) static_cast<float*>(p.logits)[(size_t)(t0 + q) * p.m_pad + e] = (float)s;
        }
    }
    if (p.logits != nullptr) return;                      // TopK is the routing block's
    __syncthreads();
    if (wave < TPB && t0 + wave < p.T)                    // the row kernel counts the experts, from the lists
        topk_few(p, (lane & 15) < p.m ? logit[wave][lane & 15] : 0.0f, t0 + wave, lane < 16, lane, [](int, int, float) {});
}

// ------------------------------------------------------------------------------------------------
// gate with more than 16 experts: logits as a tiled GEMM cut over (token tiles, expert tiles of 64, slices of K).
// One block = 16 MT WM tokens x 64 experts x its slice, four wavefronts as WM x WN, a wave multiplies MT token
// tiles by NE expert tiles of 16.  A stage holds 64 k (rows of 128 bytes = whole lines) of the block's 3 x 64 piece
// rows and its x rows, brought in by direct global->LDS loads (8 rows per wave instruction); 16-byte chunk c of row
// r sits in slot c ^ ((r/2)&7) (conflict-free ds_read_b128).  After every 64 k the fp32 accumulators are folded into
// fp64 sums; with several slices those leave as fp64 partial logits, which the TopK launch adds in slice order.
// What bounds it: the bytes a CU pulls into LDS (about 55 a clock), so tokens AND experts are cut over blocks (a
// block that holds every expert pulls the whole gate matrix) and K as well while the chip is not full.  Against one
// launch with all experts in a block and TopK behind them, logits + TopK launch: 28.7 -> 4.4 + 8.0 us (1 token, 128
// experts, d 2048), 274 -> 23 + 14 (1021, 256, d 7168), 48.8 -> 13.4 + 9.9 (5003, 60, d 2048), 49.6 -> 26.7 + 15.5
// (8192, 128, d 2048), 350 -> 207 + 19 (16384, 256, d 7168: 0.87 PFLOP/s on the three pieces, bound by LDS reads and
// the fp64 folds).
// ------------------------------------------------------------------------------------------------
// How a batch is cut: 16-token blocks up to kGateSmallTokens tokens x blocks of experts (64-token blocks leave the
// chip idle there; at 1021 x 256 experts they are ahead, 31 us against 56, K cut alike), 128-token blocks from
// kGateLargeTokens on (half the gate bytes per token; the 64-token blocks already fill the chip: 252 -> 207 us at 16384
// x 256), and K in up to kGateSlices slices until two blocks per CU are there (one per CU: 36 us instead of 26 at 8192
// x 128; 16 slices: no faster, and TopK reads twice the partial sums).
constexpr int kGateExperts = 64;       // experts of a block
constexpr int kGateSmallTokens = 2048, kGateLargeTokens = 32768, kGateBlocks = 512, kGateSlices = 8;   // kGate..Tokens: x n_eb
template <int MT, int WM>
constexpr int gate_rows() { return 3 * kGateExperts + 16 * MT * WM; }

template <int MT, int NE, int WM, int WN, int NST>
__global__ void __launch_bounds__(256) gate_logits_kernel(GateArgs p)
{
    static_assert(WM * WN == 4 && NE * WN * 16 == kGateExperts, "four waves over 64 experts");
    constexpr int RB = 128, BE = kGateExperts, W_ROWS = 3 * BE, BM = 16 * MT * WM;
    constexpr int GROUPS = gate_rows<MT, WM>() / 8;
    constexpr int LD = (GROUPS + 3) / 4;                 // loads of a wave and stage (the last ones may repeat a group)
    constexpr int STAGE = GROUPS * 1024;
    extern __shared__ __attribute__((aligned(16))) char gsm[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_tb = (p.T + BM - 1) / BM, n_eb = (p.m_pad + BE - 1) / BE;
    const int tb = blockIdx.x % n_tb, rest = blockIdx.x / n_tb;
    const int e0 = (rest % n_eb) * BE, slice = rest / n_eb, t0 = tb * BM;
    if (p.clear_cnt != nullptr && blockIdx.x == 0 && tid < p.m) p.clear_cnt[tid] = 0;
    const int all = p.d >> 6, per = (all + p.n_slice - 1) / p.n_slice;
    const int k_lo = slice * per, nk = min(all, k_lo + per) - k_lo;   // no slice is empty (the launcher's choice)

    const unsigned short* srcp[LD];
    int dsto[LD];
#pragma unroll
    for (int i = 0; i < LD; ++i) {
        const int g = min(wave + 4 * i, GROUPS - 1);
        const int row = g * 8 + (lane >> 3);
        const int chunk = (lane & 7) ^ ((row >> 1) & 7);
        // experts past the padded matrix and tokens past the batch repeat the last row (never used)
        const unsigned short* src =
            row < W_ROWS ? p.split + ((size_t)(row / BE) * p.m_pad + min(e0 + row % BE, p.m_pad - 1)) * p.d
                         : reinterpret_cast<const unsigned short*>(p.x) + (size_t)min(t0 + row - W_ROWS, p.T - 1) * p.d;
        srcp[i] = src + chunk * 8 + (size_t)k_lo * 64;
        dsto[i] = g * 1024;
    }
    auto issue = [&](int kt, int buf) {
#pragma unroll
        for (int i = 0; i < LD; ++i)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(srcp[i] + kt * 64),
                                             (__attribute__((address_space(3))) void*)(gsm + buf * STAGE + dsto[i]), 16, 0, 0);
    };
    const int wm = wave / WN, wn = wave % WN;
    double sum[MT][NE][4];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NE; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) sum[i][j][v] = 0.0;
    const int swz = ((lane & 15) >> 1) & 7;
    const int aoff = (W_ROWS + wm * MT * 16 + (lane & 15)) * RB;
    const int boff = (wn * NE * 16 + (lane & 15)) * RB;
#pragma unroll
    for (int q = 0; q < NST - 1; ++q)
        if (q < nk) issue(q, q);
    int buf = 0;
    for (int kt = 0; kt < nk; ++kt) {
        // a wave's loads complete in order: stage kt has landed once only those of stages kt+1 .. kt+NST-2 are out
        if (kt + NST - 2 < nk) __builtin_amdgcn_s_waitcnt((((NST - 2) * LD) & 0xF) | ((((NST - 2) * LD) >> 4) << 14) | 0x0F70);
        else __builtin_amdgcn_s_waitcnt(0x0F70);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();                    // stage kt is in LDS for everyone; stage kt-1 is free
        asm volatile("" ::: "memory");
        if (kt + NST - 1 < nk) issue(kt + NST - 1, buf == 0 ? NST - 1 : buf - 1);
        const char* St = gsm + buf * STAGE;
        buf = buf + 1 == NST ? 0 : buf + 1;
        f32x4 acc[MT][NE];
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NE; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) {
            const int coff = ((sl * 4 + (lane >> 4)) ^ swz) << 4;
            bf16x8 a[MT], b[3][NE];
#pragma unroll
            for (int i = 0; i < MT; ++i) a[i] = *reinterpret_cast<const bf16x8*>(St + aoff + i * 16 * RB + coff);
#pragma unroll
            for (int pz = 0; pz < 3; ++pz)
#pragma unroll
                for (int j = 0; j < NE; ++j)
                    b[pz][j] = *reinterpret_cast<const bf16x8*>(St + boff + (pz * BE + j * 16) * RB + coff);
            // low piece first (the sum of a logit is taken in that order); consecutive MFMAs are independent
#pragma unroll
            for (int pz = 2; pz >= 0; --pz)
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NE; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[pz][j], acc[i][j], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NE; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) sum[i][j][v] += (double)acc[i][j][v];
    }
    // MFMA 16x16 result layout: lane holds column (lane&15) = expert, rows 4*(lane>>4)+v = tokens
#pragma unroll
    for (int j = 0; j < NE; ++j) {
        const int e = e0 + (wn * NE + j) * 16 + (lane & 15);
        if (e >= p.m_pad) continue;
        const double bias = p.bias != nullptr && e < p.m ? (double)p.bias[e] : 0.0;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int t = t0 + (wm * MT + i) * 16 + 4 * (lane >> 4) + v;
                if (t >= p.T) continue;
                if (p.n_slice == 1) static_cast<float*>(p.logits)[(size_t)t * p.m_pad + e] = (float)(sum[i][j][v] + bias);
                else static_cast<double*>(p.logits)[((size_t)slice * p.T + t) * p.m_pad + e] = sum[i][j][v];
            }
    }
}

// Logits of token t for experts e0 + STRIDE c (past the m experts: `none`), the partial sums of the slices added in order,
// loaded QB slices at a time.
template <int NC, int STRIDE, int QB>
__device__ __forceinline__ void read_logits(const GateArgs& p, int t, int e0, float none, float (&v)[NC])
{
    if (p.n_slice == 1) {
        const float* l = static_cast<const float*>(p.logits) + (size_t)t * p.m_pad;
#pragma unroll
        for (int c = 0; c < NC; ++c) v[c] = e0 + STRIDE * c < p.m ? l[e0 + STRIDE * c] : none;
        return;
    }
    const double* l = static_cast<const double*>(p.logits) + (size_t)t * p.m_pad;
    const size_t plane = (size_t)p.T * p.m_pad;
    double s[NC];
    int e[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        s[c] = 0.0;
        e[c] = min(e0 + STRIDE * c, p.m_pad - 1);            // loads without a branch: all of a batch in flight
    }
    for (int q0 = 0; q0 < p.n_slice; q0 += QB) {
        double x[QB][NC];
#pragma unroll
        for (int q = 0; q < QB; ++q)
#pragma unroll
            for (int c = 0; c < NC; ++c) x[q][c] = l[min(q0 + q, p.n_slice - 1) * plane + e[c]];
#pragma unroll
        for (int q = 0; q < QB; ++q)
#pragma unroll
            for (int c = 0; c < NC; ++c) s[c] += q0 + q < p.n_slice ? x[q][c] : 0.0;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (p.bias != nullptr) s[c] += (double)p.bias[min(e[c], p.m - 1)];
        v[c] = e0 + STRIDE * c < p.m ? (float)s[c] : none;
    }
}

// TopK behind the logit kernel: 16 lanes per token (NC > 0, K + 1 <= 16 picks), else a wavefront per token.  The experts' tokens
// leave as bitmaps (16 tokens per block: p.bits, a quarter of a segment's 64-bit word per expert) where the row kernel
// takes the whole batch in, else as counts.
template <int NC, int THREADS>
__global__ void __launch_bounds__(THREADS) gate_topk_kernel(GateArgs p)
{
    constexpr int QB = THREADS == 1024 && NC > 0 ? 1 : NC > 8 ? 4 : THREADS == 256 ? 8 : 4;
    __shared__ int hist[kMaxExperts];                      // counts, or 16-bit maps of the block's tokens
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid; i < p.m; i += THREADS) hist[i] = 0;
    __syncthreads();
    const int per = NC > 0 ? 16 : 64;                      // lanes of a token
    const int tl = tid / per, t = (int)blockIdx.x * (THREADS / per) + tl;
    auto put = [&](int, int e, float) { note_winner(p, hist, tl, e); };
    if constexpr (NC > 0) {
        float v[NC];
        read_logits<NC, 16, QB>(p, min(t, p.T - 1), lane & 15, -__builtin_inff(), v);
        topk_rows<NC>(p, v, t, t < p.T, lane, put);
    } else if (t < p.T) {
        float v[4];
        read_logits<4, 64, QB>(p, t, lane, 0.0f, v);
        topk_token(p, v, t, lane, put);
    }
    __syncthreads();
    flush_winners<THREADS>(p, hist, tid);
}

struct RowArgs {
    const int32_t* topk_idx; const float* topk_w; const int32_t* expert_cnt;
    int32_t* expert_unit; uint8_t* expert_in_s1;
    int T, K, m, way, G, Ns, U, n_seg, full;
    int lk;                                                // log2 of the lanes a token gets: K rounded up to a power of two
    double threshold;
    int32_t* seg_cnt; int32_t* seg_off;
    int32_t* unit_cnt; int32_t* unit_off; int32_t* n_rows;
    int32_t* row_token; float* row_weight; int32_t* token_rows;
    int32_t* expert_cnt_out;                               // route_rows_kernel counts the experts itself
    const unsigned long long* bits;                        // its input where it does not build them: [n_seg][m] (GateArgs::bits)
    TileJobs jobs;                                         // GEMM tile tables to build (jobs.n == 0: none)
};

// The row kernels give every TopK entry a lane of its own: a token's K entries lie in 2^lk neighbouring lanes (never
// across a wavefront, K <= 32), entry e of a block is entry e mod 2^lk of its token e >> lk.  (One lane per token walked its
// entries one after the other, each a chain of global read, LDS read and atomic.)
template <int NT>
constexpr int entry_batch() { return kSegTokens * kMaxTopK / NT; }     // entries a thread holds: a segment's fit NT threads
static_assert(kMaxTopK <= 32, "lanes of a token");

// Entries q NT + tid, q = 0.., of the tokens [t0, t1): expert (-1: no such entry) and weight.
template <int NT, bool WEIGHTS>
__device__ __forceinline__ void load_entries(const RowArgs& p, int t0, int t1, int tid, int (&ex)[entry_batch<NT>()],
                                             float (&w)[entry_batch<NT>()])
{
    const int j = tid & ((1 << p.lk) - 1);                 // 2^lk divides NT: the same in every entry of the thread
#pragma unroll
    for (int q = 0; q < entry_batch<NT>(); ++q) {
        const int t = t0 + ((q * NT + tid) >> p.lk);
        ex[q] = -1;
        w[q] = 0.0f;
        if (t < t1 && j < p.K) {
            ex[q] = p.topk_idx[(size_t)t * p.K + j];
            if (WEIGHTS) w[q] = p.topk_w[(size_t)t * p.K + j];
        }
    }
}

// The row of one entry (token t, slot j; u: its unit or -1, w: its weight), called by whole wavefronts.  A united unit
// that several entries of the token name gets one row, at the first of them, with the sum of their weights in TopK
// order.  bmw: bitmaps of the token's segment, soff: rows of every unit in earlier segments.
__device__ __forceinline__ void scatter_entry(const RowArgs& p, const unsigned long long* bmw, const int* off_s,
                                              const int* soff, int t, int j, int u, float w, bool valid, int lane)
{
    bool first = u >= 0;
    if (__ballot(u >= p.m) != 0) {
        const int base = lane & ~((1 << p.lk) - 1);
        const float own = w;
        for (int q = 0; q < p.K; ++q) {
            const int uq = __shfl(u, base + q);
            const float wq = __shfl(own, base + q);
            if (u >= p.m && uq == u) {
                if (q < j) first = false;
                if (q > j) w += wq;
            }
        }
    }
    int row = -1;
    if (first) {
        row = off_s[u] + soff[u] + __popcll(bmw[u] & ((1ull << (t & 63)) - 1ull));
        p.row_token[row] = t;
        p.row_weight[row] = w;
    }
    if (valid) p.token_rows[(size_t)t * (p.K + p.Ns) + j] = row;
}

// A token names an expert twice only where TopK ran out of logits above -infinity (or met NaN); all but the first of those
// entries then have no positive weight.  They share the expert's row, whose weight the lanes have written in no stated
// order: once those writes are done, the last entry's is written over them.  A pass of its own, off the common path (looked
// for among the shuffles of scatter_entry, with the counts' sum taken by every wavefront, it cost the one-block routing of
// 1000 x 2 entries 0.7 us of 6.7; so 0.1).
template <int NT>
__device__ __forceinline__ void rewrite_repeated(const RowArgs& p, const int* unit_s, int t0, int t1, int tid)
{
    __syncthreads();                                       // (waits for the block's stores)
    for (int e = tid; e < (t1 - t0) * p.K; e += NT) {
        const int t = t0 + e / p.K, j = e % p.K;
        const int32_t* idx = p.topk_idx + (size_t)t * p.K;
        if (unit_s[idx[j]] != idx[j]) continue;            // united (one row with the sum of its entries) or dropped
        bool before = false, behind = false;
        for (int q = 0; q < p.K; ++q)
            if (q != j && idx[q] == idx[j]) (q < j ? before : behind) = true;
        if (before && !behind) p.row_weight[p.token_rows[(size_t)t * (p.K + p.Ns) + j]] = p.topk_w[(size_t)t * p.K + j];
    }
}

// Rows of the shared experts: every token has one in each, in token order.
template <int NT>
__device__ __forceinline__ void scatter_shared(const RowArgs& p, const int* off_s, int t0, int t1, int tid)
{
    for (int s = 0; s < p.Ns; ++s) {
        const int first = off_s[p.m + p.G + s];
        for (int t = t0 + tid; t < t1; t += NT) {
            p.row_token[first + t] = t;
            p.row_weight[first + t] = 1.0f;
            p.token_rows[(size_t)t * (p.K + p.Ns) + p.K + s] = first + t;
        }
    }
}

// Workgroup barrier for what goes through LDS: the stores and loads of a wave to memory stay in flight across it (waiting for
// the outputs of every step cost the rows kernel about 1 us a barrier).
__device__ __forceinline__ void lds_sync()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Algorithm 1 on the expert counts, in 1024 threads, four neighbouring lanes per expert (m <= 256).  Sorting is implicit: expert j precedes
// expert i in the order "count descending, id ascending" iff cnt_j > cnt_i or (equal and j < i); P_i = tokens covered before i is the
// sum of the counts of those j.  Sums in 32 bits (the counts add up to T K <= 2^30); cnt_s is 16-byte aligned and zero from m up to
// kMaxExperts.  What bounds it is the issue of m^2 comparisons on one CU: a wave's 16 experts lie in step `wave` of its walk over the counts, so in all other steps the order
// "count descending, id ascending" is one comparison with c or c - 1.  grp_s: zero; *any_s is set where a unit is united.
__device__ __forceinline__ void decide_rows(const int* cnt_s, int* unit_s, int* grp_s, int* sum_s, int* any_s, const RowArgs& p,
                                            int tid, bool write)
{
    const int ex = tid >> 2, part = tid & 3;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    bool in_s1 = false, s2 = false;
    int gr = 0;
    if (p.threshold == 1.0) {
        // P < S but for experts without tokens: nobody is browned out.  The sum of the counts, for the caller
        if (ex < p.m) in_s1 = cnt_s[ex] > 0;
        if (wave == 15) {
            const int4 v = reinterpret_cast<const int4*>(cnt_s)[tid & 63];
            const int S = wave_scan((v.x + v.y) + (v.z + v.w));
            if ((tid & 63) == 63) *sum_s = S;
        }
    } else if (ex < p.m) {
        const int c = cnt_s[ex];
        int P = 0, S = 0;
        const int4* c4 = reinterpret_cast<const int4*>(cnt_s) + part;
        const int steps = (p.m + 15) >> 4;                  // (counts past m are zero)
        gr = ex / p.way;
        auto add = [&](int it, int th) {
            const int4 v = c4[4 * it];
            S += (v.x + v.y) + (v.z + v.w);
            P += (v.x > th ? v.x : 0) + (v.y > th ? v.y : 0);
            P += (v.z > th ? v.z : 0) + (v.w > th ? v.w : 0);
        };
#pragma unroll 4
        for (int it = 0; it < wave; ++it) add(it, c - 1);
        {
            const int4 v = c4[4 * wave];
            const int j = 16 * wave + 4 * part;
            S += (v.x + v.y) + (v.z + v.w);
            P += v.x > c - (j < ex) ? v.x : 0;
            P += v.y > c - (j + 1 < ex) ? v.y : 0;
            P += v.z > c - (j + 2 < ex) ? v.z : 0;
            P += v.w > c - (j + 3 < ex) ? v.w : 0;
        }
#pragma unroll 4
        for (int it = wave + 1; it < steps; ++it) add(it, c);
        S += dpp_i<0xB1>(S);                                // quad_perm: lanes l ^ 1, then l ^ 2
        P += dpp_i<0xB1>(P);
        S += dpp_i<0x4E>(S);
        P += dpp_i<0x4E>(P);
        in_s1 = (double)P < (double)S * p.threshold;
        s2 = !in_s1 && c > 0;
        if (part == 0 && s2) atomicAdd(&grp_s[gr], 1);
        if (tid == 0) *sum_s = S;
    }
    lds_sync();
    if (ex < p.m && part == 0) {
        const int unit = !s2 ? ex : p.full ? -1 : grp_s[gr] >= 2 ? p.m + gr : ex;
        unit_s[ex] = unit;
        if (unit >= p.m) *any_s = 1;
        if (write) {
            if (p.expert_unit) p.expert_unit[ex] = unit;
            if (p.expert_in_s1) p.expert_in_s1[ex] = in_s1 ? 1 : 0;
        }
    }
    lds_sync();
}

// One segment (64 tokens) per block: which tokens have a row in unit u, as one bit per token, and how many.
__global__ void __launch_bounds__(1024) route_count_kernel(RowArgs p)
{
    __shared__ __attribute__((aligned(16))) int cnt_s[kMaxExperts];
    __shared__ int unit_s[kMaxExperts], grp_s[kMaxExperts], sum_s, any_s;
    __shared__ unsigned long long bm[kMaxUnits];
    const int tid = threadIdx.x, seg = blockIdx.x;
    const int t0 = seg * kSegTokens, t1 = min(p.T, t0 + kSegTokens);
    constexpr int NE = entry_batch<1024>();
    int ex[NE];
    float w[NE];
    load_entries<1024, false>(p, t0, t1, tid, ex, w);       // on their way while Algorithm 1 runs
    if (tid < kMaxExperts) {
        cnt_s[tid] = tid < p.m ? p.expert_cnt[tid] : 0;
        grp_s[tid] = 0;
    }
    for (int i = tid; i < p.U; i += 1024) bm[i] = 0ull;
    __syncthreads();
    decide_rows(cnt_s, unit_s, grp_s, &sum_s, &any_s, p, tid, seg == 0);
#pragma unroll
    for (int q = 0; q < NE; ++q) {
        const int u = ex[q] >= 0 ? unit_s[ex[q]] : -1;
        // a repeated united unit sets the same bit again
        if (u >= 0) atomicOr(&bm[u], 1ull << (((q * 1024 + tid) >> p.lk) & 63));
    }
    __syncthreads();
    for (int u = tid; u < p.U; u += 1024)
        p.seg_cnt[(size_t)seg * p.U + u] = u < p.m + p.G ? __popcll(bm[u]) : t1 - t0;
}

// One wavefront per unit: exclusive scan of the unit's rows over the segments (lane l owns a contiguous
// chunk of segments), and the unit's total.
__global__ void __launch_bounds__(256) route_scan_kernel(RowArgs p)
{
    const int lane = threadIdx.x & 63;
    const int u = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (u >= p.U) return;
    const int per = (p.n_seg + 63) / 64;
    const int s_lo = min(p.n_seg, lane * per), s_hi = min(p.n_seg, s_lo + per);
    int local = 0;
    for (int sgm = s_lo; sgm < s_hi; ++sgm) local += p.seg_cnt[(size_t)sgm * p.U + u];
    int incl = local;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
    }
    int run = incl - local;
    for (int sgm = s_lo; sgm < s_hi; ++sgm) {
        const int c = p.seg_cnt[(size_t)sgm * p.U + u];
        p.seg_off[(size_t)sgm * p.U + u] = run;
        run += c;
    }
    if (lane == 63) p.unit_cnt[u] = incl;
}

// Unit counts into cnt_s and their exclusive scan into off_s (every block of the scatter needs all unit offsets);
// off_s[U] = total.
__device__ __forceinline__ void unit_offsets(const int32_t* unit_cnt, int U, int* cnt_s, int* off_s, int* wsum, int tid)
{
    const int lane = tid & 63, wave = tid >> 6;
    constexpr int PER = (kMaxUnits + 255) / 256;
    const int per = (U + 255) / 256;
    int c[PER];
    int local = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int u = tid * per + q;
        c[q] = q < per && u < U ? unit_cnt[u] : 0;
        local += c[q];
    }
    int incl = local;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int base = incl - local;
    for (int w = 0; w < wave; ++w) base += wsum[w];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int u = tid * per + q;
        if (q < per && u < U) {
            off_s[u] = base;
            cnt_s[u] = c[q];
            base += c[q];
            if (u == U - 1) off_s[U] = base;
        }
    }
    __syncthreads();
}

// One segment per block; the last block has none and writes the unit offsets and the GEMM tile tables instead.
__global__ void __launch_bounds__(256) route_scatter_kernel(RowArgs p)
{
    __shared__ int unit_s[kMaxExperts];
    __shared__ unsigned long long bm[kMaxUnits];
    __shared__ int off_s[kMaxUnits + 1], ucnt_s[kMaxUnits];
    __shared__ int wsum[4], repeated_s;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, seg = blockIdx.x;
    if (tid == 0) repeated_s = 0;
    const int t0 = seg * kSegTokens, t1 = min(p.T, t0 + kSegTokens);
    constexpr int NE = entry_batch<256>();
    int ex[NE];
    float w[NE];
    load_entries<256, true>(p, t0, t1, tid, ex, w);
    if (tid < p.m) unit_s[tid] = p.expert_unit[tid];
    for (int i = tid; i < p.U; i += 256) bm[i] = 0ull;
    unit_offsets(p.unit_cnt, p.U, ucnt_s, off_s, wsum, tid);
    if (seg == p.n_seg) {
        for (int u = tid; u <= p.U; u += 256) p.unit_off[u] = off_s[u];
        if (tid == 0 && p.n_rows) p.n_rows[0] = off_s[p.U];
        build_tables<true>(ucnt_s, off_s, p.jobs, wave, lane);
        return;
    }
#pragma unroll
    for (int q = 0; q < NE; ++q) {
        ex[q] = ex[q] >= 0 ? unit_s[ex[q]] : -1;
        if (ex[q] >= 0) atomicOr(&bm[ex[q]], 1ull << (((q * 256 + tid) >> p.lk) & 63));
    }
    __syncthreads();
    const int32_t* soff = p.seg_off + (size_t)seg * p.U;
    const int j = tid & ((1 << p.lk) - 1);
    bool repeated = false;                                 // an entry without a positive weight may repeat its expert
#pragma unroll
    for (int q = 0; q < NE; ++q) {
        if (q * 256 >= (kSegTokens << p.lk)) break;
        const int t = t0 + ((q * 256 + tid) >> p.lk);
        repeated |= ex[q] >= 0 && !(w[q] > 0.0f);
        scatter_entry(p, bm, off_s, soff, t, j, ex[q], w[q], t < t1 && j < p.K, lane);
    }
    scatter_shared<256>(p, off_s, t0, t1, tid);
    if (repeated) repeated_s = 1;
    __syncthreads();
    if (repeated_s) rewrite_repeated<256>(p, unit_s, t0, t1, tid);
}

// Batches whose bitmaps fit a block's LDS: everything behind the TopK lists in one launch, a block per segment and one more that
// writes what the whole batch has one of (counts, unit maps and offsets, tile tables).  Nothing passes between blocks: each
// counts the whole batch from the bitmaps of its TopK entries (token t of segment g names expert i: bit t mod 64 of word
// [g][i]), takes Algorithm 1's decision and the unit offsets from that and scatters its own segment.
//   kBits  the bitmaps come from the launch that takes TopK 16 tokens to a block (more than 16 experts; at most 16 beyond
//          kFewExpertsTokens tokens)
//   kLists every block makes them from the TopK lists (at most 16 experts: a mask per token, then a ballot per expert; more: LDS
//          atomics).  A ballot per entry and expert made few experts with long lists slow: routing of 2048 tokens x 16 of 16
//          experts 68 us, now 50; 300 x 8 of 16 19.8, 15.4; beyond, lists read by every block instead of bitmaps: 8192 x 8 of 16
//          81, now 17.4, x 16 of 16 146, 19.6
//   kTopK  one segment: the block takes TopK of the logits itself and is the only one (NC: 1 topk_few, more topk_rows, 0
//          topk_token)
// Bound by latency: some ten barriers, two trips to the L2 and what a block reads of the bitmaps (8 m bytes per segment).  TopK
// and rows in us, before (TopK launch, then one block up to 1024 tokens or three launches) and now: 1 token x 8 of 128
// experts 8.6 + 9.2, 9.4; 37 x 4 of 60 4.8 + 8.2, 10.9; 1021 x 8 of 256 14.7 + 32.2, 13.8 + 14.4; 3001 x 8 of 128 12.3 + 6.0 + 3.0 +
// 6.4, 7.9 + 9.0; 8192 x 8 of 128 16.3 + 7.2 + 5.0 + 10.6, 11.2 + 18.5.
enum { kBits, kLists, kTopK };
// A row of bitmaps in LDS: a word of padding after every eight, so that lanes that walk groups of eight experts find
// different banks.
__host__ __device__ constexpr int bit_slot(int e) { return e + (e >> 3); }
__host__ __device__ constexpr int bit_pitch(int m) { return m + (m >> 3) + 1; }

template <int SRC, int NC, bool STREAM>
__global__ void __launch_bounds__(1024) route_rows_kernel(RowArgs p, GateArgs g)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char rsm[];      // bitmaps [n_seg][bit_pitch(m)]; kTopK: logits
    __shared__ __attribute__((aligned(16))) int cnt_s[kMaxExperts], wsum[16];
    __shared__ int unit_s[kMaxExperts], tok_s[kMaxExperts], grp_s[kMaxExperts];
    __shared__ unsigned long long bm[kMaxUnits];           // this block's segment
    __shared__ int ucnt_s[kMaxUnits], pre_s[kMaxUnits];    // rows of a unit: in all, in earlier segments
    __shared__ int off_s[kMaxUnits + 1], sum_s, any_s;
    __shared__ int ex_s[SRC == kTopK ? kSegTokens * kMaxTopK : 1];
    __shared__ float w_s[SRC == kTopK ? kSegTokens * kMaxTopK : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, seg = blockIdx.x;
    const int t0 = seg * kSegTokens, t1 = min(p.T, t0 + kSegTokens);
    const bool writer = SRC == kTopK || seg == p.n_seg;
    unsigned long long* local = reinterpret_cast<unsigned long long*>(rsm);
    const int bp = bit_pitch(p.m);
    int ex[entry_batch<1024>()];
    float w[entry_batch<1024>()];
    if (SRC != kTopK) load_entries<1024, true>(p, t0, t1, tid, ex, w);
    if (tid < p.U) {
        bm[tid] = 0ull;
        ucnt_s[tid] = 0;
        pre_s[tid] = 0;
    }
    if (tid < kMaxExperts) { cnt_s[tid] = 0; tok_s[tid] = 0; grp_s[tid] = 0; }
    if (tid == 0) any_s = 0;
    if (SRC == kLists && p.m > 16)
        for (int i = tid; i < p.n_seg * bp; i += 1024) local[i] = 0ull;
    lds_sync();

    // bitmaps, and the tokens of every expert
    if constexpr (SRC == kTopK) {
        constexpr int per = NC > 0 ? 16 : 64;
        const int pitch = g.m_pad + 16;                    // floats: the four tokens of a wavefront on different banks
        float* logit_s = reinterpret_cast<float*>(rsm);
        // A few tokens leave lanes for every (token, expert) pair: four lanes count the experts ahead of theirs, and there is no
        // round per winner (one token, 8 of 128 experts: 2.4 us in rounds, 0.8 so).  LDS then holds the logits' keys.
        bool by_rank = false;
        int l_m = 5;                                       // log2 of the lanes' experts: m_pad up to a power of two
        if constexpr (NC > 1) {
            while ((1 << l_m) < g.m_pad) ++l_m;
            by_rank = p.T << (l_m + 2) <= 1024;
        }
        auto keep = [&](float v) { return by_rank ? __int_as_float(order_key(v)) : v; };
        if constexpr (NC != 1) {
            // a thread per logit: the slices' partial sums, four tokens' at a time in flight, added in order
            const float none = NC > 0 ? -__builtin_inff() : 0.0f;
            int lm = 5;
            while ((1 << lm) < g.m_pad) ++lm;
            const int e = tid & ((1 << lm) - 1), tq = tid >> lm, rows = 1024 >> lm;
            const int eb = min(e, g.m_pad - 1), plane = p.T * g.m_pad;
            const double bias = g.bias != nullptr && e < p.m ? (double)g.bias[e] : 0.0;
            if (g.n_slice == 1) {
                for (int t = tq; t < p.T; t += rows)
                    if (e < g.m_pad) logit_s[t * pitch + e] = keep(e < p.m ? static_cast<const float*>(g.logits)[t * g.m_pad + e] : none);
            } else {
                const double* l = static_cast<const double*>(g.logits);
                for (int tb = 0; tb < p.T; tb += 4 * rows) {
                    double x[4][kGateSlices];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (tb + q * rows >= p.T) break;
                        const int at = min(tb + q * rows + tq, p.T - 1) * g.m_pad + eb;
#pragma unroll
                        for (int sl = 0; sl < kGateSlices; ++sl) x[q][sl] = l[min(sl, g.n_slice - 1) * plane + at];
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int t = tb + q * rows + tq;
                        double v = 0.0;
#pragma unroll
                        for (int sl = 0; sl < kGateSlices; ++sl) v += sl < g.n_slice ? x[q][sl] : 0.0;
                        if (g.bias != nullptr) v += bias;
                        if (t < p.T && e < g.m_pad) logit_s[t * pitch + e] = keep(e < p.m ? (float)v : none);
                    }
                }
            }
            lds_sync();
        }
        bool ranked = false;
        if constexpr (NC > 1) {
            if (by_rank) {
                const int part = tid & 3, e = (tid >> 2) & ((1 << l_m) - 1), t = tid >> (l_m + 2);
                if (t < p.T && e < p.m) {
                    const int* row = reinterpret_cast<const int*>(logit_s) + t * pitch;
                    const int key = row[e];
                    int rank = 0;
#pragma unroll 4
                    for (int q = 4 * part; q < g.m_pad; q += 16) {
                        const int4 v = *reinterpret_cast<const int4*>(row + q);
                        rank += v.x > key - (q < e ? 1 : 0);
                        rank += v.y > key - (q + 1 < e ? 1 : 0);
                        rank += v.z > key - (q + 2 < e ? 1 : 0);
                        rank += v.w > key - (q + 3 < e ? 1 : 0);
                    }
                    rank += dpp_i<0xB1>(rank);
                    rank += dpp_i<0x4E>(rank);
                    if (part == 0 && rank < (g.K < p.m ? g.K + 1 : g.K)) {
                        ex_s[t * kMaxTopK + rank] = e;
                        w_s[t * kMaxTopK + rank] = __int_as_float(key);
                        if (key == (int)0x807fffff) any_s = 1;      // a winner of logit -infinity: the rounds decide
                    }
                }
                lds_sync();
                ranked = any_s == 0;
                lds_sync();
                if (tid == 0) any_s = 0;
            }
        }
        for (int t = tid / per; t < (p.T + 64 / per - 1) / (64 / per) * (64 / per); t += 1024 / per) {      // whole wavefronts
            auto put = [&](int j, int e, float wt) {
                ex_s[t * kMaxTopK + j] = e;
                w_s[t * kMaxTopK + j] = wt;
                atomicOr(&bm[e], 1ull << t);
            };
            if (ranked) {
                const int at = min(t, p.T - 1) * kMaxTopK + (lane & 15);
                weights_rows<false>(g, __float_as_int(w_s[at]), ex_s[at], t, t < p.T, lane, put);
                continue;
            }
            const int r = lane & (per - 1), tt = min(t, p.T - 1);
            if constexpr (NC == 1) {
                topk_few(g, r < p.m ? static_cast<const float*>(g.logits)[(size_t)tt * 16 + r] : 0.0f, t, t < p.T, lane, put);
            } else {
                constexpr int N = NC > 0 ? NC : 4;
                float v[N];
#pragma unroll
                for (int c = 0; c < N; ++c)
                    v[c] = r + per * c < g.m_pad ? logit_s[tt * pitch + r + per * c] : NC > 0 ? -__builtin_inff() : 0.0f;
                if (NC > 1 && by_rank) {
#pragma unroll
                    for (int c = 0; c < N; ++c)
                        if (r + per * c < g.m_pad) v[c] = key_value(__float_as_int(v[c]));
                }
                if constexpr (NC > 0) topk_rows<NC>(g, v, t, t < p.T, lane, put);
                else topk_token(g, v, t, lane, put);
            }
        }
        lds_sync();
        if (tid < p.m) cnt_s[tid] = tok_s[tid] = __popcll(bm[tid]);
    } else {
        if constexpr (SRC == kLists) {
            if (p.m <= 16) {
                for (int sgm = wave; sgm < p.n_seg; sgm += 16) {
                    const int t = sgm * kSegTokens + lane;
                    const int32_t* list = p.topk_idx + (size_t)min(t, p.T - 1) * p.K;
                    unsigned named = 0u;                   // the token's experts, eight entries on their way at a time
                    for (int j = 0; j < p.K; j += 8) {
                        int e[8];
#pragma unroll
                        for (int q = 0; q < 8; ++q)
                            if (j + q < p.K) e[q] = list[j + q];
#pragma unroll
                        for (int q = 0; q < 8; ++q)
                            if (j + q < p.K) named |= 1u << e[q];
                    }
                    if (t >= p.T) named = 0u;
                    unsigned long long mine = 0ull;
                    for (int i = 0; i < p.m; ++i) {
                        const unsigned long long b = __ballot((named >> i) & 1u);
                        if (lane == i) mine = b;
                    }
                    if (lane < p.m) local[sgm * bp + bit_slot(lane)] = mine;
                }
            } else {
                for (int e = tid; e < p.T * p.K; e += 1024) {
                    const int t = e / p.K;
                    atomicOr(&local[(t >> 6) * bp + bit_slot(p.topk_idx[e])], 1ull << (t & 63));
                }
            }
            lds_sync();
        }
        // an expert's segments are shared out to 1024 / 2^lm threads (2^lm: m up to a power of two)
        int lm = 0;
        while ((1 << lm) < p.m) ++lm;
        const int e = tid & ((1 << lm) - 1), parts = 1024 >> lm;
        const unsigned long long last = (p.T & 63) ? (1ull << (p.T & 63)) - 1ull : ~0ull;     // tokens of the last segment
        if (e < p.m) {
            int c = 0, pre = 0;
#pragma unroll 8
            for (int sgm = tid >> lm; sgm < p.n_seg; sgm += parts) {
                unsigned long long b;
                if constexpr (SRC == kLists) {
                    b = local[sgm * bp + bit_slot(e)];
                } else {
                    b = p.bits[(size_t)sgm * p.m + e];
                    if (sgm == p.n_seg - 1) b &= last;
                    local[sgm * bp + bit_slot(e)] = b;
                }
                const int n = __popcll(b);
                c += n;
                pre += sgm < seg ? n : 0;
                if (sgm == seg) bm[e] = b;
            }
            if (c > 0) atomicAdd(&cnt_s[e], c);
            if (pre > 0) atomicAdd(&pre_s[e], pre);
        }
        lds_sync();
        if (tid < p.m) tok_s[tid] = cnt_s[tid];
    }
    lds_sync();

    // Algorithm 1.  Its input counts entries: where a token names an expert twice (see rewrite_repeated) these are more than
    // the tokens.
    bool repeated = false;
    for (;;) {
        decide_rows(cnt_s, unit_s, grp_s, &sum_s, &any_s, p, tid, writer);
        if (repeated || sum_s == p.T * p.K) break;
        repeated = true;
        lds_sync();                                        // everyone has read the sum
        if (tid < kMaxExperts) { cnt_s[tid] = 0; grp_s[tid] = 0; }
        if (tid == 0) any_s = 0;
        lds_sync();
        for (int e = tid; e < p.T * p.K; e += 1024)
            atomicAdd(&cnt_s[SRC == kTopK ? ex_s[e / p.K * kMaxTopK + e % p.K] : p.topk_idx[e]], 1);
        lds_sync();
    }
    if (writer && tid < p.m) p.expert_cnt_out[tid] = cnt_s[tid];

    // united units: the union of the bitmaps of the experts they stand for
    if (any_s) {
        if constexpr (SRC == kTopK) {
            if (tid < p.G) {
                const int lo = tid * p.way, hi = min(p.m, lo + p.way);
                unsigned long long b = 0ull;
#pragma unroll 4
                for (int i = lo; i < hi; ++i) b |= unit_s[i] == p.m + tid ? bm[i] : 0ull;
                bm[p.m + tid] = b;
                ucnt_s[p.m + tid] = __popcll(b);
            }
        } else {
            int lg = 0;
            while ((1 << lg) < p.G) ++lg;
            const int gr = tid & ((1 << lg) - 1), parts = 1024 >> lg;
            if (gr < p.G) {
                const int lo = gr * p.way, hi = min(p.m, lo + p.way);
                int c = 0, pre = 0;
                for (int sgm = tid >> lg; sgm < p.n_seg; sgm += parts) {
                    unsigned long long b = 0ull;
#pragma unroll 4
                    for (int i = lo; i < hi; ++i) b |= unit_s[i] == p.m + gr ? local[sgm * bp + bit_slot(i)] : 0ull;
                    const int n = __popcll(b);
                    c += n;
                    pre += sgm < seg ? n : 0;
                    if (sgm == seg) bm[p.m + gr] = b;
                }
                if (c > 0) atomicAdd(&ucnt_s[p.m + gr], c);
                if (pre > 0) atomicAdd(&pre_s[p.m + gr], pre);
            }
        }
        lds_sync();
    }

    // rows of every unit and their exclusive scan, a thread per unit
    {
        const int u = tid;
        int c = 0;
        if (u < p.m) c = unit_s[u] == u ? tok_s[u] : 0;    // else its tokens have a row in the united unit, or none
        else if (u < p.m + p.G) c = ucnt_s[u];
        else if (u < p.U) c = p.T;                         // a shared expert: every token
        const int incl = wave_scan(c);
        if (lane == 63) wsum[wave] = incl;
        lds_sync();
        static_assert(kMaxUnits <= 12 * 64, "units lie in the first 12 wavefronts");
        int base = 0;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int4 v = reinterpret_cast<const int4*>(wsum)[q];
            base += (4 * q < wave ? v.x : 0) + (4 * q + 1 < wave ? v.y : 0) + (4 * q + 2 < wave ? v.z : 0) +
                    (4 * q + 3 < wave ? v.w : 0);
        }
        if (u < p.U) {
            ucnt_s[u] = c;
            off_s[u] = base + incl - c;
            if (writer) { p.unit_cnt[u] = c; p.unit_off[u] = base + incl - c; }
            if (u == p.U - 1) {
                off_s[p.U] = base + incl;
                if (writer) {
                    p.unit_off[p.U] = base + incl;
                    if (p.n_rows) p.n_rows[0] = base + incl;
                }
            }
        }
        lds_sync();
    }
    // the GEMM tile tables, by the last wavefronts (with kTopK the first ones hold the tokens of a short batch)
    if (writer) build_tables<STREAM>(ucnt_s, off_s, p.jobs, 15 - wave, lane);
    if (SRC != kTopK && writer) return;

    const int j = tid & ((1 << p.lk) - 1);
#pragma unroll
    for (int q = 0; q < entry_batch<1024>(); ++q) {
        if (q * 1024 + tid - lane >= (t1 - t0) << p.lk) break;                     // whole wavefronts leave
        const int tl = (q * 1024 + tid) >> p.lk;
        const bool valid = t0 + tl < t1 && j < p.K;
        if (SRC == kTopK) {
            ex[q] = valid ? ex_s[tl * kMaxTopK + j] : -1;
            w[q] = valid ? w_s[tl * kMaxTopK + j] : 0.0f;
        }
        scatter_entry(p, bm, off_s, pre_s, t0 + tl, j, ex[q] >= 0 ? unit_s[ex[q]] : -1, w[q], valid, lane);
    }
    scatter_shared<1024>(p, off_s, t0, t1, tid);
    if (repeated) rewrite_repeated<1024>(p, unit_s, t0, t1, tid);
}

// Where the rows kernel takes a batch: up to kRowSegs segments whose bitmaps fit the LDS beside what it declares.
constexpr int kRowSegs = 128, kRowLds = 145 * 1024;
static bool rows_fit(int n_seg, int m) { return n_seg <= kRowSegs && (size_t)n_seg * bit_pitch(m) * 8 <= kRowLds; }

constexpr int kGateFewLds = 3 * 4 * 64 * 128;          // three stages of four 64-row pieces (gate_few_kernel)
// The block shapes of the logit kernel: 16 tokens with three stages, 64 and 128 tokens with two (two blocks fit a CU).
constexpr int kGateLds16 = 3 * gate_rows<1, 1>() * 128;
constexpr int kGateLds64 = 2 * gate_rows<2, 2>() * 128;
constexpr int kGateLds128 = 2 * gate_rows<4, 2>() * 128;

template <bool STREAM>
static hipError_t init_rows()
{
    const void* topk[] = {reinterpret_cast<const void*>(route_rows_kernel<kTopK, 0, STREAM>),
                          reinterpret_cast<const void*>(route_rows_kernel<kTopK, 4, STREAM>),
                          reinterpret_cast<const void*>(route_rows_kernel<kTopK, 8, STREAM>),
                          reinterpret_cast<const void*>(route_rows_kernel<kTopK, 16, STREAM>)};
    hipError_t e;
    for (const void* k : topk)
        if ((e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kSegTokens * (kMaxExperts + 16) * 4)) != hipSuccess)
            return e;
    const void* rows[] = {reinterpret_cast<const void*>(route_rows_kernel<kBits, 0, STREAM>),
                          reinterpret_cast<const void*>(route_rows_kernel<kLists, 0, STREAM>)};
    for (const void* k : rows)
        if ((e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kRowLds)) != hipSuccess) return e;
    return hipSuccess;
}

hipError_t init_route_kernels()
{
    hipError_t e;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(gate_logits_kernel<1, 1, 1, 4, 3>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kGateLds16);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(gate_logits_kernel<2, 2, 2, 2, 2>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kGateLds64);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(gate_logits_kernel<4, 2, 2, 2, 2>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kGateLds128);
    if (e != hipSuccess) return e;
    if ((e = init_rows<true>()) != hipSuccess || (e = init_rows<false>()) != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(gate_few_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               kGateFewLds);
}

hipError_t launch_pack_gate(const float* gate_w, int m, int m_pad, int d, bf16_t* packed, hipStream_t s)
{
    if (m_pad == 16)     // at most 16 experts: the fp64 gate reads fp32 rows, the packed form is a copy of them
        return hipMemcpyAsync(packed, gate_w, (size_t)m * d * 4, hipMemcpyDeviceToDevice, s);
    const size_t n = (size_t)m_pad * d;
    const int blocks = (int)std::min<size_t>((n + 255) / 256, 2048);
    prep_kernel<<<blocks, 256, 0, s>>>(gate_w, m, m_pad, d, reinterpret_cast<unsigned short*>(packed), nullptr);
    return hipGetLastError();
}

template <int THREADS>
static void launch_topk(const GateArgs& p, hipStream_t s)
{
    const int blocks = ceil_div(p.T, THREADS / 16);
    if (p.K + 1 > 16) gate_topk_kernel<0, 1024><<<ceil_div(p.T, 16), 1024, 0, s>>>(p);
    else if (p.m_pad <= 64) gate_topk_kernel<4, THREADS><<<blocks, THREADS, 0, s>>>(p);
    else if (p.m_pad <= 128) gate_topk_kernel<8, THREADS><<<blocks, THREADS, 0, s>>>(p);
    else gate_topk_kernel<16, THREADS><<<blocks, THREADS, 0, s>>>(p);
}

static int gate_token_tile(int64_t T, int n_eb)
{
    return T * n_eb <= kGateSmallTokens ? 16 : T * n_eb >= kGateLargeTokens ? 128 : 64;
}

// How a batch with more than 16 experts goes through the gate.  The order of a logit's sum follows from n_slice, so that
// comes from the batch alone (T, m, d): the same bits whatever the scratch holds.  A batch whose logits the scratch cannot hold
// goes through it in pieces of `chunk` tokens (the token tile of a piece does not show: every tile adds up alike).
struct GatePlan { int n_slice, chunk; };
static GatePlan plan_gate(int T, int m_pad, int d, size_t bytes)
{
    const int n_eb = ceil_div(m_pad, kGateExperts), ksteps = d / 64;
    const int sl = std::max(1, std::min({kGateBlocks / (ceil_div(T, gate_token_tile(T, n_eb)) * n_eb), kGateSlices, ksteps / 2}));
    GatePlan P;
    P.n_slice = ceil_div(ksteps, ceil_div(ksteps, sl));                  // no empty slice
    const int64_t most = (int64_t)(bytes / ((size_t)m_pad * (P.n_slice == 1 ? 4 : 8 * P.n_slice)));
    const int64_t unit = most >= 64 ? 64 : most >= 16 ? 16 : 1;
    P.chunk = most >= T ? T : (int)std::max<int64_t>(most / unit * unit, 1);
    return P;
}

// Logits, and TopK of them unless the routing block takes it (g.topk_idx null).
static hipError_t launch_gate(GateArgs g, const GatePlan& plan, bool topk, hipStream_t s)
{
    const int T = g.T, n_eb = ceil_div(g.m_pad, kGateExperts);
    g.n_slice = plan.n_slice;
    for (int c0 = 0; c0 < T; c0 += plan.chunk) {
        GateArgs p = g;
        p.T = std::min(plan.chunk, T - c0);
        p.t_base = c0;
        p.x = g.x + (size_t)c0 * g.d;
        p.topk_idx = g.topk_idx + (size_t)c0 * g.K;
        p.topk_w = g.topk_w + (size_t)c0 * g.K;
        if (g.near_tie != nullptr) p.near_tie = g.near_tie + c0;
        if (c0 > 0) p.clear_cnt = nullptr;
        const int tile = gate_token_tile(p.T, n_eb), blocks = ceil_div(p.T, tile) * n_eb * p.n_slice;
        if (tile == 16) gate_logits_kernel<1, 1, 1, 4, 3><<<blocks, 256, kGateLds16, s>>>(p);
        else if (tile == 128) gate_logits_kernel<4, 2, 2, 2, 2><<<blocks, 256, kGateLds128, s>>>(p);
        else gate_logits_kernel<2, 2, 2, 2, 2><<<blocks, 256, kGateLds64, s>>>(p);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (!topk) continue;
        if (p.expert_cnt == nullptr) launch_topk<256>(p, s);
        else if (p.n_slice > 1) launch_topk<512>(p, s);     // fewer, larger blocks: each flushes a histogram
        else launch_topk<1024>(p, s);                       // (partial logits need the registers, logits do not)
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

// Whether one block takes TopK and routes the batch: a segment of at most 16 experts, or of at most 64 and 15 entries; of more, as
// long as one CU has the logits ranked before a launch over several would have started.  moe_route with that launch / without, us: 24
// tokens x 15 of 256 experts 24.8 / 24.8, x 16 of 128 20.7 / 20.8, 32 tokens 24.8 / 27.0, 20.9 / 24.6; 32 tokens x 8 of 128 16.9 / 17.1, x 2
// of 128 15.9 / 14.4; 64 tokens x 8 of 128 17.1 / 22.7, x 15 of 256 25.5 / 39.4, x 32 of 128 31 / 60; 64 x 4 of 60 15.8 / 15.6, x 8 of 32
// 15.9 / 14.1.
static bool one_block_routes(const Dims& D)
{
    if (D.n_seg > 1) return false;
    if (D.m_pad == 16 || (D.m_pad <= 64 && D.K <= 15)) return true;
    return D.T <= (D.m_pad <= 128 && D.K <= 15 ? 32 : 24);
}

// The block that takes TopK of a batch of one segment and routes it.
template <bool STREAM>
static hipError_t launch_route_topk(const GateArgs& g, const RowArgs& p, hipStream_t s)
{
    const size_t lds = g.m_pad == 16 ? 0 : (size_t)p.T * (g.m_pad + 16) * 4;     // the logits
    if (g.m_pad == 16) route_rows_kernel<kTopK, 1, STREAM><<<1, 1024, lds, s>>>(p, g);
    else if (g.K + 1 > 16) route_rows_kernel<kTopK, 0, STREAM><<<1, 1024, lds, s>>>(p, g);
    else if (g.m_pad <= 64) route_rows_kernel<kTopK, 4, STREAM><<<1, 1024, lds, s>>>(p, g);
    else if (g.m_pad <= 128) route_rows_kernel<kTopK, 8, STREAM><<<1, 1024, lds, s>>>(p, g);
    else route_rows_kernel<kTopK, 16, STREAM><<<1, 1024, lds, s>>>(p, g);
    return hipGetLastError();
}

hipError_t launch_route(const Dims& D, const bf16_t* x, const void* gate, const float* gate_bias,
                        double threshold, int full_brownout, const RouteBufs& R, bf16_t* gate_split,
                        int32_t* seg_cnt, int32_t* seg_off, void* logits, size_t logit_bytes, const TileJobs& jobs,
                        hipStream_t s)
{
    hipError_t e = ensure_device_init(nullptr);
    if (e != hipSuccess) return e;
    const bool packed = D.gate_format == MOE_GATE_PACKED;
    // At most 16 experts: the gate matrix is fp32 rows in either format, and up to kFewExpertsTokens tokens the
    // plain fp64 gate reads them as they are (larger batches: cut here on every call, 6 us, then the MFMA gate).
    const bool few_fmt = D.m_pad == 16;
    const bool few = few_fmt && D.T <= kFewExpertsTokens;
    // Who makes the row lists: one block that takes TopK of a small batch's logits as well, a block per segment on the whole
    // batch's bitmaps, or beyond kRowSegs segments the count, scan and scatter launches.
    GatePlan plan{1, D.T};
    if (!few_fmt) plan = plan_gate(D.T, D.m_pad, D.d, logit_bytes);
    const bool whole = plan.chunk >= D.T;
    enum { kOneBlock, kFromBits, kFromLists, kThreeLaunches } how = kThreeLaunches;
    if (whole && one_block_routes(D)) how = kOneBlock;
    else if (!few && rows_fit(D.n_seg, D.m) && (whole || plan.chunk % 16 == 0)) how = kFromBits;
    else if (rows_fit(D.n_seg, D.m) && (few || D.n_seg == 1)) how = kFromLists;
    int32_t* counters = how == kThreeLaunches ? R.expert_cnt : nullptr;
    // Preparation: cut an fp32 gate matrix into its pieces (only the MFMA gates need them) and clear the expert
    // counters, if used (the logit kernel of the many-expert gate clears them itself).
    const bool split = !few && (!packed || few_fmt);
    if (split || (few_fmt && counters != nullptr)) {
        ProfScope ps(MOE_STAGE_PREP, s);
        const size_t n = split ? (size_t)D.m_pad * D.d : (size_t)D.m;
        const int blocks = (int)std::min<size_t>((n + 255) / 256, 2048);
        prep_kernel<<<blocks, 256, 0, s>>>(split ? static_cast<const float*>(gate) : nullptr, D.m, D.m_pad, D.d,
                                           split ? reinterpret_cast<unsigned short*>(gate_split) : nullptr, counters);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    GateArgs g;
    g.x = x;
    g.split = split ? reinterpret_cast<const unsigned short*>(gate_split) : static_cast<const unsigned short*>(gate);
    g.bias = gate_bias;
    g.T = D.T; g.d = D.d; g.m = D.m; g.m_pad = D.m_pad; g.K = D.K; g.score_fn = D.score_fn;
    g.topk_idx = R.topk_idx; g.topk_w = R.topk_w; g.near_tie = R.near_tie;
    g.expert_cnt = counters;
    g.n_slice = plan.n_slice; g.clear_cnt = few_fmt ? nullptr : counters;
    g.logits = few_fmt && how != kOneBlock ? nullptr : logits;
    // the bitmaps take the place of the segment counts and offsets, which only the three launches use
    g.bits = how == kFromBits ? reinterpret_cast<unsigned long long*>(seg_cnt) : nullptr;
    g.t_base = 0;
    {
        ProfScope ps(MOE_STAGE_GATE, s);
        if (few) {
            const float* gw = static_cast<const float*>(gate);      // fp32 rows in either gate format
            if (D.m <= 8) gate_small_kernel<8, 1><<<D.T, 256, 0, s>>>(g, gw);
            else gate_small_kernel<16, 1><<<D.T, 256, 0, s>>>(g, gw);
        } else if (few_fmt) {
            // at most 16 experts beyond kFewExpertsTokens tokens
            gate_few_kernel<<<ceil_div(D.T, 16), 512, kGateFewLds, s>>>(g);
        } else {
            if ((e = launch_gate(g, plan, how != kOneBlock, s)) != hipSuccess) return e;
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    RowArgs p;
    p.topk_idx = R.topk_idx; p.topk_w = R.topk_w; p.expert_cnt = R.expert_cnt;
    p.expert_unit = R.expert_unit; p.expert_in_s1 = R.expert_in_s1;
    p.T = D.T; p.K = D.K; p.m = D.m; p.way = D.way; p.G = D.G; p.Ns = D.Ns; p.U = D.U; p.n_seg = D.n_seg;
    p.full = full_brownout; p.threshold = threshold;
    p.lk = 0;
    while ((1 << p.lk) < D.K) ++p.lk;
    p.seg_cnt = seg_cnt; p.seg_off = seg_off; p.unit_cnt = R.unit_cnt; p.unit_off = R.unit_off; p.n_rows = R.n_rows;
    p.row_token = R.row_token; p.row_weight = R.row_weight; p.token_rows = R.token_rows;
    p.expert_cnt_out = R.expert_cnt; p.bits = g.bits;
    p.jobs = jobs;
    if (how != kThreeLaunches) {
        ProfScope ps(MOE_STAGE_COUNT, s);
        auto launch = [&](auto stream) -> hipError_t {
            constexpr bool STREAM = decltype(stream)::value;
            if (how == kOneBlock) return launch_route_topk<STREAM>(g, p, s);
            const size_t lds = (size_t)D.n_seg * bit_pitch(D.m) * 8;
            if (how == kFromBits) route_rows_kernel<kBits, 0, STREAM><<<D.n_seg + 1, 1024, lds, s>>>(p, g);
            else route_rows_kernel<kLists, 0, STREAM><<<D.n_seg + 1, 1024, lds, s>>>(p, g);
            return hipGetLastError();
        };
        return jobs.may_stream() ? launch(std::true_type{}) : launch(std::false_type{});
    }
    {
        ProfScope ps(MOE_STAGE_COUNT, s);
        route_count_kernel<<<D.n_seg, 1024, 0, s>>>(p);
    }
    {
        ProfScope ps(MOE_STAGE_SCAN, s);
        route_scan_kernel<<<ceil_div(D.U, 4), 256, 0, s>>>(p);
    }
    {
        ProfScope ps(MOE_STAGE_SCATTER, s);
        route_scatter_kernel<<<D.n_seg + 1, 256, 0, s>>>(p);
    }
    return hipGetLastError();
}

}  // namespace bmoe

// United-expert distillation (the paper's section "United Expert Model"): the student FFN of a group is
// fitted to the group's teacher FFNs on calibration tokens by minimising the section's MSE equation
//   L = (1/k) sum_i || H_u - H_o^i ||^2   (summed over features, averaged over tokens)
// with full-batch Adam.  The paper gives no optimiser, settings or data; this is the reading documented in
// the header.
//   forward   G = X W1^T, U = X W3^T, A = silu(G) U, Y = A W2^T
//   backward  dY = Y - mean_i Y_i  (the factor 2/n goes into the update), dW2 = dY^T A, dA = dY W2,
//             dG = dA U silu'(G), dU = dA silu(G), dW1 = dG^T X, dW3 = dU^T X
// A step is four launches of one GEMM kernel, over several groups at a time (the groups are independent and one of a small model
// does not fill the chip):
//   kSwiglu    G, U, A and A^T          kResidual  dY, dY^T and the loss        (Y is not stored)
//   kUpdate    kAdam of W2 beside kBackward: dG^T, dU^T (dA is not stored; the loss of the step is summed up on the way)
//   kUpdate    kAdam of W1 and W3, and the new W2 transposed, which the backward pass beside W2's update may not see yet
// kAdam: the gradients stay in registers, masters, moments and the bf16 copies are updated there.
// The contractions over tokens read K-contiguous operands that the earlier epilogues have written transposed.
// Why: with each of these as a pass of its own (64-row GEMM tiles with fp32 results, transposes, SwiGLU, Adam, the loss
// summed by one block) a pass over two groups of 8 and 4 teachers at n = d = 2048, F = 1408 with 8 steps took 56.9 ms,
// 50 of them in the one-block sums and 3.4 in the GEMMs; now 2.85 ms.  Of those a step's four launches take 0.30 ms in a kernel trace
// (kSwiglu 61 us, kResidual 40, kBackward with W2 100, W1 and W3 99; at best 55, 33, 92 and 80; the 484 MB of masters and moments alone are 94 us
// at the rate of a large copy).  With the loads, fragment reads and MFMAs of a k tile one after the other, and W2 updated with W1 and W3, the
// call took 3.37 ms.
#include "internal.h"

#include <algorithm>
#include <type_traits>

namespace bmoe {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float bf_to_f(unsigned short b) { return __uint_as_float(((unsigned)b) << 16); }
__device__ __forceinline__ uint2 pack4(const float (&v)[4]) { return make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])); }

// out[c][r] = in[r][c] (16-bit elements), R and C multiples of 64; blockIdx.z: group
__global__ void __launch_bounds__(256) transpose16_kernel(const unsigned short* __restrict__ in, size_t in_stride,
                                                          unsigned short* __restrict__ out, size_t out_stride, int R, int C)
{
    __shared__ unsigned short tile[64][66];
    in += blockIdx.z * in_stride;
    out += blockIdx.z * out_stride;
    const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    for (int i = ty; i < 64; i += 4) tile[i][tx] = in[(size_t)(r0 + i) * C + c0 + tx];
    __syncthreads();
    for (int i = ty; i < 64; i += 4) out[(size_t)(c0 + i) * R + r0 + tx] = tile[tx][i];
}

__global__ void __launch_bounds__(256) fill_f32_kernel(float* __restrict__ p, size_t n, float v)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

// Sum of a double over the block (256 threads), fixed order; the result is valid in thread 0.
__device__ __forceinline__ double block_sum(double s, double* red)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}

// One batch of b teachers (FFN output rows in half precision, y_stride elements apart): sum over the teachers so
// far in tbar (the first batch starts it, the last one turns it into the mean of k), and per block
// sum_i y_i^2 (last batch: - sum (sum_i y_i)^2 / k, which leaves sum_i |y_i - mean|^2) in fp64.
__global__ void __launch_bounds__(256) teacher_stats_kernel(const unsigned short* __restrict__ y, size_t y_stride, int b,
                                                            float* __restrict__ tbar, size_t n8, int first, int last, int k,
                                                            double* __restrict__ part)
{
    __shared__ double red[4];
    double q = 0.0;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n8; e += (size_t)gridDim.x * 256) {
        float s[8];
        if (first) {
#pragma unroll
            for (int c = 0; c < 8; ++c) s[c] = 0.0f;
        } else {
            const float4 a = reinterpret_cast<const float4*>(tbar)[2 * e], c4 = reinterpret_cast<const float4*>(tbar)[2 * e + 1];
            s[0] = a.x; s[1] = a.y; s[2] = a.z; s[3] = a.w;
            s[4] = c4.x; s[5] = c4.y; s[6] = c4.z; s[7] = c4.w;
        }
        for (int i = 0; i < b; ++i) {
            const f16x8 v = *reinterpret_cast<const f16x8*>(y + i * y_stride + e * 8);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const float f = (float)v[c];
                s[c] += f;
                q += (double)(f * f);                      // the product of two halves is exact in fp32
            }
        }
        if (last) {
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                q -= (double)s[c] * (double)s[c] / (double)k;
                s[c] = s[c] / (float)k;
            }
        }
        reinterpret_cast<float4*>(tbar)[2 * e] = make_float4(s[0], s[1], s[2], s[3]);
        reinterpret_cast<float4*>(tbar)[2 * e + 1] = make_float4(s[4], s[5], s[6], s[7]);
    }
    const double t = block_sum(q, red);
    if (threadIdx.x == 0) part[blockIdx.x] = first ? t : part[blockIdx.x] + t;
}

// out[g] = (offset ? offset[g] : 0) + scale * sum part[g][0..n): one block per group (strides in bytes)
__device__ __forceinline__ float sum_partials(const double* part, int n, float offset, double scale, double* red)
{
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) s += part[i];
    // the teachers' spread is a difference of sums and may round below zero; a comparison, so that NaN stays NaN (fmax would
    // turn the loss of a training run that has diverged into the best one there is)
    const double t = block_sum(s, red) * scale;
    return offset + (float)(t < 0.0 ? 0.0 : t);
}
__global__ void __launch_bounds__(256) sum_partials_kernel(const char* part, size_t part_stride, int n, const char* offset,
                                                           size_t offset_stride, double scale, float* out, size_t out_stride)
{
    __shared__ double red[4];
    const int g = blockIdx.x;
    const float off = offset ? *reinterpret_cast<const float*>(offset + g * offset_stride) : 0.0f;
    const float v = sum_partials(reinterpret_cast<const double*>(part + g * part_stride), n, off, scale, red);
    if (threadIdx.x == 0) out[g * out_stride] = v;
}

// ------------------------------------------------------------------------------------------------
// C = A . B^T (A [M][K], B [N][K], bf16, fp32 accumulators; M, N, K multiples of 64) with an epilogue.
// ------------------------------------------------------------------------------------------------
struct Ref {                                              // a buffer of every group, `stride` bytes apart
    char* p; size_t stride;
    template <typename T> __device__ __forceinline__ T* at(int g) const { return reinterpret_cast<T*>(p + g * stride); }
};
enum { kSwiglu, kResidual, kUpdate };                      // the kernels
enum { kBackward, kAdam, kTranspose };                     // what a job of kUpdate is; kTranspose: r[0] = A transposed, no product
struct DJob {
    int kind;                                              // kUpdate only
    Ref A, B, B1;                                          // B1: kSwiglu only (B = W1, B1 = W3)
    int M, N, K;
    int mt, nt;                                            // tiles of a group
    int chunk;                                             // an XCD's share of the tiles of all groups
    Ref r[4];                                              // see the epilogues
};
struct DGemm {
    DJob job[3];                                           // in the order in which their tiles are handed out
    int n_jobs, groups;
    float gscale, lr, c1, c2;                              // kAdam
    int first, last;                                       // kAdam: no masters or moments yet; none are read again
    Ref part, floor_; int n_part; double lscale; float* hist; size_t hist_stride;   // kBackward: the loss of this step
};

constexpr int kImgPitch = 272;                             // bytes per row of a 128 x 128 bf16 image in LDS
// kAdam: per wave 32 rows x 64 columns of products
constexpr int kAdamRow = 272, kAdamWave = 32 * kAdamRow;
// LDS bytes of a block with tiles of 32 FM rows of A by 32 FN rows of B: two buffers of A rows and three of B rows in the k loop; an
// epilogue's images take their place, and the last 32 bytes are block_sum's.  Two blocks of the smaller tiles share a CU's 160 KiB.
constexpr int dgemm_lds(int fm, int fn) { return (2 * fm + 3 * fn) * 32 * 128; }
static_assert(2 * 128 * kImgPitch <= dgemm_lds(4, 4) - 32 && 4 * kAdamWave <= dgemm_lds(4, 4) && dgemm_lds(4, 4) <= 80 * 1024, "4 x 4");

// Four waves, 16x16x32 MFMA, k tiles of 64: 128 x 128 tiles (64 x 64 a wave), two blocks per CU, or for kSwiglu 256 x 192 (128 x 96 a wave, the
// accumulators in the accumulation registers), one block.  M and N are multiples of 64, so a 64 x 64 wave tile is inside the matrix or outside.
// What bounds the k loop: 128 KiB of fragments and 64 KiB of tiles pass through the LDS per k tile of two blocks, 1536 cycles against 1024
// of MFMAs, if nothing in a wave waits for anything else in it.  So the fragments of the next step of 16 MFMAs are read between the MFMAs of
// this one, and direct global->LDS loads are issued one by one between them (all eight of a k tile in a row, then fragments, then MFMAs,
// over two stages of 64 KiB: 2085 cycles, as long with one block on a CU as with two; now 1780 and 1530).  The
// 80 KiB of a block are two buffers of A rows and three of B rows, so that loads lead by one and two k tiles.  One barrier per k tile, three
// quarters into its first step, when a wave has read its last fragments of tile kt and its loads of tile kt+1 have landed; behind it come
// the A rows of tile kt+2 into the buffer just left, then the B rows of tile kt+3.  Loads past the end of K are clamped to the last
// k tile and never used.  Two groups at n = d = 2048, F = 1408, 128 x 128 tiles in all kernels: kSwiglu 77 -> 65 us, the call with 8 steps 3.37 -> 3.20 ms.
template <int EPI, int FM, int FN>
__global__ void __launch_bounds__(256, FM * FN == 16 ? 2 : 1) distill_gemm_kernel(DGemm p)
{
    static_assert(EPI == kSwiglu || (FM == 4 && FN == 4), "the other epilogues are written for 128 x 128 tiles");
    // rows of A and of B of a tile, its output columns, bytes of the two in a k tile
    constexpr int BM = 32 * FM, BN = 32 * FN, BNC = EPI == kSwiglu ? BN / 2 : BN, kSlabA = BM * 128, kSlabB = BN * 128;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    // block id mod 8 is the XCD: of every job a contiguous range of tiles each, super-tiles of 8 M tiles x all N tiles inside
    int at = blockIdx.x >> 3, jn = 0;
    while (jn + 1 < p.n_jobs && at >= p.job[jn].chunk) at -= p.job[jn++].chunk;
    const DJob& J = p.job[jn];
    const int tiles = J.mt * J.nt, L = (blockIdx.x & 7) * J.chunk + at;
    if (at >= J.chunk || L >= p.groups * tiles) return;
    const int g = L / tiles, tile = L - g * tiles;
    const int gspan = 8 * J.nt, gi = tile / gspan, rem = tile - gi * gspan;
    const int gsz = min(8, J.mt - gi * 8);
    const int nt = rem / gsz, mt = gi * 8 + (rem - nt * gsz);
    const int m0 = mt * BM, n0 = nt * BNC;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int K = J.K;

    // image of R rows x C columns -> out[(row0 + r) * ld + col0 + c], 16 bytes per thread, rows < row_end, columns < col_end
    auto flush = [&](const char* img, int pitch, int R, int C, unsigned short* out, int ld, int row0, int row_end, int col0, int col_end) {
        const int cpr = C >> 3;
        for (int i = tid; i < R * cpr; i += 256) {
            const int r = i / cpr, c = (i - r * cpr) * 8;
            if (row0 + r < row_end && col0 + c < col_end)
                *reinterpret_cast<uint4*>(out + (size_t)(row0 + r) * ld + col0 + c) =
                    *reinterpret_cast<const uint4*>(img + r * pitch + c * 2);
        }
    };
    if (EPI == kUpdate && J.kind == kTranspose) {
        const unsigned short* in = J.A.at<const unsigned short>(g);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = wave * 32 + (i & 3) * 8 + (lane >> 3), c = (i >> 2) * 64 + (lane & 7) * 8;
            if (m0 + r < J.M && n0 + c < J.N) {
                const uint4 v = *reinterpret_cast<const uint4*>(in + (size_t)(m0 + r) * J.N + n0 + c);
                const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    *reinterpret_cast<unsigned short*>(smem + (c + e) * kImgPitch + r * 2) = (unsigned short)(w[e >> 1] >> (16 * (e & 1)));
            }
        }
        __syncthreads();
        flush(smem, kImgPitch, 128, 128, J.r[0].at<unsigned short>(g), J.M, n0, J.N, m0, J.M);
        return;
    }

    // Wave w moves the 8-row groups w, w+4, ... of A and of B; 16-byte chunk c of row r sits in slot c ^ ((r/2)&7) (conflict-free
    // ds_read_b128), a term that is the same for all loads of a lane.  An address is a wave-uniform base and a lane offset.
    const int wave_s = __builtin_amdgcn_readfirstlane(wave);
    const int r8 = lane >> 3, csw = (lane & 7) ^ ((((wave & 1) << 2) + (r8 >> 1)) & 7);
    const unsigned off = (unsigned)(r8 * K * 2 + csw * 16);
    const bf16_t *base_a[FM], *base_b[FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
        base_a[i] = uniform_ptr(J.A.at<const bf16_t>(g) + (size_t)min(m0 + (wave_s + i * 4) * 8, J.M - 8) * K);
#pragma unroll
    for (int i = 0; i < FN; ++i) {
        const int grp = wave_s + i * 4;                   // of 4 FN
        // kSwiglu: the wave tile's 16-column MFMA tiles alternate W1 / W3 of the same 16 columns
        const int half = grp / (2 * FN), j = (grp - half * 2 * FN) >> 1;
        const bool third = EPI == kSwiglu && (j & 1);
        const int col = EPI == kSwiglu ? n0 + half * (BN / 4) + (j >> 1) * 16 + (grp & 1) * 8 : n0 + grp * 8;
        base_b[i] = uniform_ptr((third ? J.B1 : J.B).at<const bf16_t>(g) + (size_t)min(col, J.N - 8) * K);
    }
    const int nk = K >> 6, last = nk - 1;
    auto load_a = [&](int i, int kt) {
        load_lds(reinterpret_cast<const char*>(base_a[i] + (size_t)min(kt, last) * 64) + off,
                 smem + (kt & 1) * kSlabA + (wave_s + i * 4) * 1024);
    };
    auto load_b = [&](int i, int kt, int buf) {
        load_lds(reinterpret_cast<const char*>(base_b[i] + (size_t)min(kt, last) * 64) + off,
                 smem + 2 * kSlabA + buf * kSlabB + (wave_s + i * 4) * 1024);
    };
    const int a_off = (wm * (BM / 2) + (lane & 15)) * 128, b_off = 2 * kSlabA + (wn * (BN / 2) + (lane & 15)) * 128;
    const int swz = ((lane & 15) >> 1) & 7;
    bf16x8 fa[2][FM], fb[2][FN];
    auto read_a = [&](int buf, int half, int i) {
        fa[half][i] = *reinterpret_cast<const bf16x8*>(smem + buf * kSlabA + a_off + i * 2048 + (((half * 4 + (lane >> 4)) ^ swz) << 4));
    };
    auto read_b = [&](int buf, int half, int j) {
        fb[half][j] = *reinterpret_cast<const bf16x8*>(smem + buf * kSlabB + b_off + j * 2048 + (((half * 4 + (lane >> 4)) ^ swz) << 4));
    };
    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // large tiles: the accumulators stay in the accumulation registers
    auto pin = [&]() {
        if constexpr (FM * FN > 16) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) asm volatile("" : "+a"(acc[i][j]));
        }
    };
    pin();
    constexpr int NM = FM * FN, BAR = NM * 3 / 4;         // MFMAs of a step, and the barrier's place in the first step
    // loads of a k tile (A rows of the next but one, then B rows of the one after that), MFMAs from one to the next (from the barrier on), and
    // how many come before the next k tile
    constexpr int LD = FM + FN, GAP = 2 * NM / LD, SL = (2 * NM - BAR + GAP - 1) / GAP;
    static_assert((LD - 1) * GAP < 2 * NM && SL >= FM && SL <= LD && LD <= BAR, "loads end before the next ones begin, reads before the barrier");
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
        for (int i = 0; i < FM; ++i) load_a(i, kt);
#pragma unroll
        for (int i = 0; i < FN; ++i) load_b(i, kt, kt);
    }
#pragma unroll
    for (int i = 0; i < SL - FM; ++i) load_b(i, 2, 2);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(FN + SL));       // tile 0 has landed, the younger loads are in flight
    lds_barrier();
#pragma unroll
    for (int j = 0; j < FN; ++j) read_b(0, 0, j);
#pragma unroll
    for (int i = 0; i < FM; ++i) read_a(0, 0, i);
    __builtin_amdgcn_s_waitcnt(0xC07F);
    int b_cur = 0;                                        // B buffer of tile kt (kt mod 3)
    for (int kt = 0; kt < nk; ++kt) {
        const int a_cur = kt & 1, b_nxt = b_cur == 2 ? 0 : b_cur + 1, b_nn = b_nxt == 2 ? 0 : b_nxt + 1;
#pragma unroll
        for (int st = 0; st < 2; ++st) {
#pragma unroll
            for (int mi = 0; mi < NM; ++mi) {
                if (st == 0 && mi == BAR) {
                    // my reads of tile kt are done (its buffers may be refilled) and my loads of tile kt+1 have landed:
                    // all but the youngest, B rows of tile kt+2
                    __builtin_amdgcn_sched_barrier(0);
                    __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_imm(FN));
                    lds_barrier();
                    __builtin_amdgcn_sched_barrier(0);
                }
                const int i = mi / (2 * FN) * 2 + (mi & 1), j = mi % (2 * FN) >> 1;
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[st][j], fa[st][i], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                constexpr int RG = FM * FN > 16 ? 2 : 1;  // fragments of the next step
                if (mi % RG == 0 && mi / RG < LD) {
                    const int r = mi / RG;
                    if (r < FN) read_b(st == 0 ? b_cur : b_nxt, st ^ 1, r);
                    else read_a(st == 0 ? a_cur : a_cur ^ 1, st ^ 1, r - FN);
                }
                const int l = st == 0 ? mi < BAR ? mi + 2 * NM - BAR : mi - BAR : mi + NM - BAR;       // MFMAs since the barrier
                if (l % GAP == 0 && l / GAP < LD) {
                    if (st == 0 && mi < BAR) load_b(l / GAP - FM, kt + 2, b_nn);
                    else if (l / GAP < FM) load_a(l / GAP, kt + 2);
                    else load_b(l / GAP - FM, kt + 3, b_cur);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_s_waitcnt(0xC07F);           // lgkmcnt(0): the next step's fragments are in registers
            __builtin_amdgcn_sched_barrier(0);
        }
        b_cur = b_nxt;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));             // clamped loads still target this block's LDS
    lds_barrier();                                        // every wave has left the buffers: images go there
    pin();
    double* red = reinterpret_cast<double*>(smem + dgemm_lds(FM, FN) - 32);

    // A lane holds, for row wm*BM/2 + 16 i + (lane & 15) of the tile, the B rows wn*BN/2 + 16 j + 4 (lane >> 4) + 0..3.
    const int r_l = wm * (BM / 2) + (lane & 15), c4 = 4 * (lane >> 4);
    const bool w_in = m0 + wm * 64 < J.M && n0 + wn * 64 < J.N;            // (not kSwiglu)
    // what kResidual and kBackward read, all of it in flight together; a tile outside the matrix reads the first one
    const size_t at0 = w_in ? (size_t)(m0 + r_l) * J.N + n0 + wn * 64 + c4 : (size_t)(lane & 15) * J.N + c4;
    auto fetch = [&](const float* from, f32x4 (&to)[FM][FN]) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) to[i][j] = *reinterpret_cast<const f32x4*>(from + at0 + (size_t)(i * 16) * J.N + j * 16);
    };
    // bf16 results go through LDS: `rows` holds [tile row][tile column], `cols` [tile column][tile row]
    constexpr int kRowPitch = BNC * 2 + 16, kColPitch = BM * 2 + 16;
    auto put_row = [&](char* img, int r, int c, uint2 v) { *reinterpret_cast<uint2*>(img + r * kRowPitch + c * 2) = v; };
    auto put_col = [&](char* img, int r, int c, uint2 v) {
        const unsigned w[2] = {v.x, v.y};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            *reinterpret_cast<unsigned short*>(img + (c + e) * kColPitch + r * 2) = (unsigned short)(w[e >> 1] >> (16 * (e & 1)));
    };
    char* rows = smem;
    char* cols = smem + (EPI == kSwiglu ? BM * kRowPitch : 128 * kImgPitch);
    static_assert(EPI != kSwiglu || BM * kRowPitch + BNC * kColPitch <= dgemm_lds(FM, FN), "both images");

    if constexpr (EPI == kSwiglu) {
        // r: G, U (fp32 [n][F]), A [n][F], A^T [F][n]
        float* G = J.r[0].at<float>(g);
        float* U = J.r[1].at<float>(g);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int jp = 0; jp < FN / 2; ++jp) {
                const f32x4 gv = acc[i][2 * jp], uv = acc[i][2 * jp + 1];
                const int r = r_l + i * 16, c = wn * (BNC / 2) + jp * 16 + c4;
                float a[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] = gv[e] / (1.0f + __expf(-gv[e])) * uv[e];
                put_row(rows, r, c, pack4(a));
                put_col(cols, r, c, pack4(a));
                if (m0 + wm * (BM / 2) + i * 16 < J.M && n0 + wn * (BNC / 2) + jp * 16 < J.N) {
                    const size_t at = (size_t)(m0 + r) * J.N + n0 + c;
                    *reinterpret_cast<f32x4*>(G + at) = gv;
                    *reinterpret_cast<f32x4*>(U + at) = uv;
                }
            }
        __syncthreads();
        flush(rows, kRowPitch, BM, BNC, J.r[2].at<unsigned short>(g), J.N, m0, J.M, n0, J.N);
        flush(cols, kColPitch, BNC, BM, J.r[3].at<unsigned short>(g), J.M, n0, J.N, m0, J.M);
    } else if constexpr (EPI == kResidual) {
        // r: mean teacher output (fp32 [n][d]), dY [n][d], dY^T [d][n] (null: loss only), loss partials [tiles]
        const float* tb = J.r[0].at<const float>(g);
        const bool store = J.r[1].p != nullptr;
        f32x4 ts[FM][FN];
        fetch(tb, ts);
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = r_l + i * 16, c = wn * 64 + j * 16 + c4;
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float df = acc[i][j][e] - ts[i][j][e];
                    v[e] = df;
                    if (w_in) s += (double)df * (double)df;
                }
                if (store) {
                    put_row(rows, r, c, pack4(v));
                    put_col(cols, r, c, pack4(v));
                }
            }
        const double t = block_sum(s, red);               // (its barrier also completes the images)
        if (tid == 0) J.r[3].at<double>(g)[tile] = t;
        if (store) {
            flush(rows, kImgPitch, 128, 128, J.r[1].at<unsigned short>(g), J.N, m0, J.M, n0, J.N);
            flush(cols, kImgPitch, 128, 128, J.r[2].at<unsigned short>(g), J.M, n0, J.N, m0, J.M);
        }
    } else if (J.kind == kBackward) {
        // r: G, U (fp32 [n][F]), dG^T, dU^T [F][n].  dG = dA U sig(G) (1 + G (1 - sig(G))), dU = dA silu(G)
        const float* G = J.r[0].at<const float>(g);
        const float* U = J.r[1].at<const float>(g);
        f32x4 gvs[FM][FN], uvs[FM][FN];
        fetch(G, gvs);
        fetch(U, uvs);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = r_l + i * 16, c = wn * 64 + j * 16 + c4;
                const f32x4 gv = gvs[i][j], uv = uvs[i][j];
                float dg[4], du[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float da = acc[i][j][e], sg = 1.0f / (1.0f + __expf(-gv[e]));
                    dg[e] = da * uv[e] * sg * (1.0f + gv[e] * (1.0f - sg));
                    du[e] = da * gv[e] * sg;
                }
                put_col(rows, r, c, pack4(dg));
                put_col(cols, r, c, pack4(du));
            }
        __syncthreads();
        flush(rows, kImgPitch, 128, 128, J.r[2].at<unsigned short>(g), J.M, n0, J.N, m0, J.M);
        flush(cols, kImgPitch, 128, 128, J.r[3].at<unsigned short>(g), J.M, n0, J.N, m0, J.M);
        if (tile == 0 && p.hist != nullptr) {
            const float l = sum_partials(p.part.at<const double>(g), p.n_part, *p.floor_.at<const float>(g), p.lscale, red);
            if (tid == 0) p.hist[g * p.hist_stride] = l;
        }
    } else {
        // r: master, first and second moment (fp32 [M][N]), the bf16 copy [M][N].
        // Adam with bias correction; the first step starts from the bf16 copy and zero moments.  32 rows x 64 columns of products
        // at a time go through LDS of the wave's own, and a lane works on rows 4 q + (lane >> 4), columns 4 (lane & 15) + 0..3: 256
        // bytes of a row at a time, and the state of the next 16 rows is on its way meanwhile.
        float* W = J.r[0].at<float>(g);
        float* Mo = J.r[1].at<float>(g);
        float* V = J.r[2].at<float>(g);
        unsigned short* wb = J.r[3].at<unsigned short>(g);
        const float beta1 = 0.9f, beta2 = 0.999f, eps = 1e-8f;
        char* own = smem + wave * kAdamWave;
        const int cr = lane >> 4, cc = 4 * (lane & 15);
        const size_t at0 = (size_t)(m0 + wm * 64 + cr) * J.N + n0 + wn * 64 + cc;
        // (the first and the last step by themselves, so that the loads in flight can be counted; behind the last one nothing reads the
        // state, which a run of one step writes all the same)
        auto update = [&](auto first, auto last_step) {
            f32x4 have[4][3], next[4][3];
            auto fetch = [&](int row, f32x4 (&to)[4][3]) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const size_t at = at0 + (size_t)(row + 4 * q) * J.N;
                    if constexpr (decltype(first)::value) {
                        const uint2 b = *reinterpret_cast<const uint2*>(wb + at);
                        to[q][0] = f32x4{bf_to_f(b.x & 0xFFFF), bf_to_f(b.x >> 16), bf_to_f(b.y & 0xFFFF), bf_to_f(b.y >> 16)};
                        to[q][1] = to[q][2] = f32x4{0.f, 0.f, 0.f, 0.f};
                    } else {
                        to[q][0] = *reinterpret_cast<const f32x4*>(W + at);
                        to[q][1] = *reinterpret_cast<const f32x4*>(Mo + at);
                        to[q][2] = *reinterpret_cast<const f32x4*>(V + at);
                    }
                }
            };
            fetch(0, have);
#pragma unroll
            for (int rg = 0; rg < 2; ++rg) {
                if (rg > 0) wave_lds_order();
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        *reinterpret_cast<f32x4*>(own + (i * 16 + (lane & 15)) * kAdamRow + (j * 16 + c4) * 4) = acc[rg * 2 + i][j];
                wave_lds_order();
#pragma unroll
                for (int ps = 0; ps < 2; ++ps) {
                    if (rg * 32 + ps * 16 + 16 < 64) fetch(rg * 32 + ps * 16 + 16, next);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int rl = ps * 16 + 4 * q + cr;
                        const size_t at = at0 + (size_t)(rg * 32 + ps * 16 + 4 * q) * J.N;
                        const f32x4 prod = *reinterpret_cast<const f32x4*>(own + rl * kAdamRow + cc * 4);
                        f32x4 &w = have[q][0], &m = have[q][1], &v = have[q][2];
                        float o[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float gr = prod[e] * p.gscale;
                            m[e] = fmaf(beta1, m[e], (1.0f - beta1) * gr);
                            v[e] = fmaf(beta2, v[e], (1.0f - beta2) * gr * gr);
                            // correctly rounded (the reciprocal and square root that are 1 ulp off would save 2 % of a call)
                            w[e] = w[e] - p.lr * (m[e] * p.c1) / (sqrtf(v[e] * p.c2) + eps);
                            o[e] = w[e];
                        }
                        if constexpr (!decltype(last_step)::value) {
                            *reinterpret_cast<f32x4*>(W + at) = w;
                            *reinterpret_cast<f32x4*>(Mo + at) = m;
                            *reinterpret_cast<f32x4*>(V + at) = v;
                        }
                        *reinterpret_cast<uint2*>(wb + at) = pack4(o);
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int k = 0; k < 3; ++k) have[q][k] = next[q][k];
                }
            }
        };
        if (w_in) {
            if (p.first) update(std::true_type{}, std::false_type{});
            else if (p.last) update(std::false_type{}, std::true_type{});
            else update(std::false_type{}, std::false_type{});
        }
    }
}

template <int EPI, int FM = 4, int FN = 4>
static hipError_t launch_dgemm(DGemm& p, int groups, hipStream_t s)
{
    int slots = 0;
    for (int j = 0; j < p.n_jobs; ++j) {
        DJob& J = p.job[j];
        J.mt = ceil_div(J.M, FM * 32);
        J.nt = ceil_div(J.N, FN * (EPI == kSwiglu ? 16 : 32));
        J.chunk = ceil_div(groups * J.mt * J.nt, 8);
        slots += J.chunk;
    }
    p.groups = groups;
    distill_gemm_kernel<EPI, FM, FN><<<slots * 8, 256, dgemm_lds(FM, FN), s>>>(p);
    return hipGetLastError();
}

// kSwiglu in tiles of 256 x 192 or of 128 x 128: what takes less time by rounds of one or two blocks on a CU.  Epilogue included, a round
// takes so many us (n = 2048, one group, F = 3072 and 2048):
//   K                  64    128    256    512   1024   2048   4096
//   one large tile   18.4   19.0   20.5   24.5   33.5     51     87      17.5 + 1.03 per k tile
//   two small ones   13.8   14.5   15.8   18.8   24.2     40     71      12.5 + 0.87 per k tile
// A last round of small tiles that is not full takes half to all of that: its blocks start before the round in front of it has ended.  Over 350 shapes
// of 128 to 4096 x 128 to 3072, 256 to 4096 tokens, 1 to 8 groups (fitted to 150 of them), a step takes 0.08 % longer than with the better tile each time,
// 3.4 % at most (small ones always 0.52 %; with 48, 37 and, for a last round of up to 256, 27 us at every K, 0.27 %: 3008 tokens, 512 x 1600, 3 groups
// lost 2.3 %).  Two groups of 2048 tokens at 2048 x 1408 are 240 large tiles in 61 us (kernel trace, 54 at best) or 704 small ones in 70 (60).  Per MFMA a large tile
// passes 3/4 of the bytes through the LDS and 7/12 through the L1.  (The other three epilogues lose more as one block on a CU than their loop gains: kResidual
// at 256 x 128 37 -> 39 us, the launch with kBackward at 256 x 192 87 -> 116.)
static bool large_swiglu(int M, int N, int K, int groups, int n_cu)
{
    const int64_t small = (int64_t)groups * ceil_div(M, 128) * ceil_div(N, 64), large = (int64_t)groups * ceil_div(M, 256) * ceil_div(N, 96);
    const int64_t slots = 2 * n_cu, rest = small % slots, kt = K / 64;
    const int64_t rounds = small / slots * 1024 + (rest > 0 ? 512 + 512 * rest / slots : 0);               // in 1/1024, times in 1/100 us
    return (large + n_cu - 1) / n_cu * 1024 * (1750 + 103 * kt) < rounds * (1250 + 87 * kt);
}

template <int EPI, int FM = 4, int FN = 4>
static hipError_t init_dgemm()
{
    return hipFuncSetAttribute(reinterpret_cast<const void*>(distill_gemm_kernel<EPI, FM, FN>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               dgemm_lds(FM, FN));
}

hipError_t init_distill_kernels()
{
    const hipError_t e[] = {init_dgemm<kSwiglu>(), init_dgemm<kSwiglu, 8, 6>(), init_dgemm<kResidual>(), init_dgemm<kUpdate>()};
    for (hipError_t x : e)
        if (x != hipSuccess) return x;
    return hipSuccess;
}

// Groups trained side by side: enough that the smallest of a step's GEMMs gives every CU two blocks, at most 8.
static int distill_groups_at_once(int n, int d, int F, int n_groups)
{
    const int64_t t = std::min((int64_t)ceil_div(n, 128) * ceil_div(F, 128), (int64_t)ceil_div(n, 128) * ceil_div(d, 128));
    return (int)std::max<int64_t>(1, std::min<int64_t>({n_groups, (512 + t - 1) / t, 8}));
}

constexpr int kStatBlocks = 512;                          // most blocks of the teacher statistics

// Buffers of one group (offsets from the group's base) and, behind those of all groups, X^T.
struct DistillLayout {
    size_t W[3], M[3], V[3], w2t, G, U, A, At, dGt, dUt, tbar, dY, dYt, floor_, part, group, xt, total;
};

static DistillLayout distill_layout(int n, int d, int F, int groups)
{
    const size_t dF = (size_t)d * F, nF = (size_t)n * F, nd = (size_t)n * d;
    DistillLayout B;
    size_t o = 0;
    auto take = [&](size_t bytes) { const size_t at = o; o = align_up(o + bytes, 256); return at; };
    for (int q = 0; q < 3; ++q) B.W[q] = take(dF * 4);
    for (int q = 0; q < 3; ++q) B.M[q] = take(dF * 4);
    for (int q = 0; q < 3; ++q) B.V[q] = take(dF * 4);
    B.w2t = take(dF * 2);
    B.G = take(nF * 4);
    B.U = take(nF * 4);
    B.A = take(nF * 2);
    B.At = take(nF * 2);
    B.dGt = take(nF * 2);
    B.dUt = take(nF * 2);
    B.tbar = take(nd * 4);
    B.dY = take(nd * 2);
    B.dYt = take(nd * 2);
    B.floor_ = take(4);
    B.part = take(8 * (size_t)std::max(kStatBlocks, ceil_div(n, 128) * ceil_div(d, 128)));
    B.group = o;
    B.xt = o * groups;
    B.total = B.xt + align_up(nd * 2, 256);
    return B;
}

size_t distill_buffer_bytes(int n, int d, int F, int groups) { return distill_layout(n, d, F, groups).total; }

// Fewer tokens ask for more groups side by side, so the bytes they would take rise and fall with n.  A workspace is sized for
// n and every smaller number: the most that g groups take at the largest n' <= n that asks for them (from t tiles of the
// smallest GEMM: ceil(512 / t) >= g, t (g - 1) < 512).  Beyond kSideBySide bytes the weights and moments are so large that one
// group's kAdam fills the chip by itself (DeepSeek-V3 shape: 2688 blocks and 0.5 GB of state per step).
constexpr size_t kSideBySide = (size_t)1 << 30;
size_t distill_wanted_bytes(int n, int d, int F, int n_groups)
{
    size_t most = distill_buffer_bytes(n, d, F, 1);
    for (int g = 2; g <= std::min(8, n_groups); ++g) {
        const int64_t rows = 511 / ((int64_t)(g - 1) * std::min(ceil_div(F, 128), ceil_div(d, 128)));
        if (rows < 1) break;
        most = std::max(most, std::min(distill_buffer_bytes((int)std::min<int64_t>(n, rows * 128), d, F, g), kSideBySide));
    }
    return most;
}

int distill_groups_that_fit(int n, int d, int F, int n_groups, size_t bytes)
{
    int g = distill_groups_at_once(n, d, F, n_groups);
    while (g > 0 && distill_buffer_bytes(n, d, F, g) > bytes) --g;
    return g;
}

hipError_t launch_teacher_stats(const bf16_t* y_half, int b, bool first, bool last, int k, int n, int d, int F, int g, void* buf,
                                hipStream_t s)
{
    const DistillLayout B = distill_layout(n, d, F, 1);
    char* base = static_cast<char*>(buf) + g * B.group;
    const size_t n8 = (size_t)n * d / 8;
    const int blocks = (int)std::min<size_t>((n8 + 255) / 256, kStatBlocks);
    double* part = reinterpret_cast<double*>(base + B.part);
    teacher_stats_kernel<<<blocks, 256, 0, s>>>(reinterpret_cast<const unsigned short*>(y_half), (size_t)n * d, b,
                                                reinterpret_cast<float*>(base + B.tbar), n8, first, last, k, part);
    if (last)
        sum_partials_kernel<<<1, 256, 0, s>>>(base + B.part, 0, blocks, nullptr, 0, 1.0 / ((double)k * n),
                                              reinterpret_cast<float*>(base + B.floor_), 0);
    return hipGetLastError();
}

// Trains the students of `groups` consecutive groups (w1u, w3u [g][F][d], w2u [g][d][F], bf16, updated in place).
// Their teachers' statistics are in buf (launch_teacher_stats).  hist: [g][steps + 1] or null.
hipError_t distill_groups(const bf16_t* x, int n, int d, int F, int groups, bf16_t* w1u, bf16_t* w3u, bf16_t* w2u, int steps,
                          float lr, float* hist, void* buf, hipStream_t s)
{
    DeviceInfo dev;
    hipError_t e = ensure_device_init(&dev);
    if (e != hipSuccess) return e;
    const DistillLayout B = distill_layout(n, d, F, groups);
    char* base = static_cast<char*>(buf);
    const size_t dF = (size_t)d * F;
    auto ref = [&](size_t off) { return Ref{base + off, B.group}; };
    auto weight = [&](const bf16_t* w) { return Ref{reinterpret_cast<char*>(const_cast<bf16_t*>(w)), dF * 2}; };
    const Ref none{nullptr, 0}, X{reinterpret_cast<char*>(const_cast<bf16_t*>(x)), 0}, Xt{base + B.xt, 0};
    auto us = [](const void* p) { return static_cast<const unsigned short*>(p); };
    auto job = [&](int kind, Ref a, Ref b, Ref b1, int M, int N, int K, Ref r0, Ref r1, Ref r2, Ref r3) {
        DJob j;
        j.kind = kind; j.A = a; j.B = b; j.B1 = b1; j.M = M; j.N = N; j.K = K; j.mt = j.nt = j.chunk = 0;
        j.r[0] = r0; j.r[1] = r1; j.r[2] = r2; j.r[3] = r3;
        return j;
    };
    transpose16_kernel<<<dim3(d / 64, n / 64, 1), 256, 0, s>>>(us(x), 0, reinterpret_cast<unsigned short*>(base + B.xt), 0, n, d);
    if (steps > 0)
        transpose16_kernel<<<dim3(F / 64, d / 64, groups), 256, 0, s>>>(
            us(w2u), dF, reinterpret_cast<unsigned short*>(base + B.w2t), B.group / 2, d, F);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    double b1t = 1.0, b2t = 1.0;
    const int loss_tiles = ceil_div(n, 128) * ceil_div(d, 128);
    for (int t = 0; t <= steps; ++t) {
        const bool train = t < steps;
        if (!train && hist == nullptr) break;
        DGemm p;
        p.gscale = 2.0f / (float)n; p.lr = lr; p.c1 = p.c2 = 1.0f; p.first = t == 0 ? 1 : 0; p.last = t + 1 == steps ? 1 : 0;
        p.part = ref(B.part); p.floor_ = ref(B.floor_); p.n_part = loss_tiles; p.lscale = (double)(1.0f / (float)n);
        p.hist = hist ? hist + t : nullptr; p.hist_stride = steps + 1;
        p.n_jobs = 1;
        p.job[0] = p.job[1] = p.job[2] =
            job(0, X, weight(w1u), weight(w3u), n, F, d, ref(B.G), ref(B.U), ref(B.A), ref(B.At));
        e = large_swiglu(n, F, d, groups, dev.n_cu) ? launch_dgemm<kSwiglu, 8, 6>(p, groups, s) : launch_dgemm<kSwiglu>(p, groups, s);
        if (e != hipSuccess) return e;
        p.job[0] = job(0, ref(B.A), weight(w2u), none, n, d, F, ref(B.tbar), train ? ref(B.dY) : none,
                       train ? ref(B.dYt) : none, ref(B.part));
        if ((e = launch_dgemm<kResidual>(p, groups, s)) != hipSuccess) return e;
        if (!train) {
            sum_partials_kernel<<<groups, 256, 0, s>>>(base + B.part, B.group, loss_tiles, base + B.floor_, B.group, p.lscale,
                                                       p.hist, p.hist_stride);
            return hipGetLastError();
        }
        b1t *= 0.9f;
        b2t *= 0.999f;
        p.c1 = (float)(1.0 / (1.0 - b1t));
        p.c2 = (float)(1.0 / (1.0 - b2t));
        auto adam = [&](int q, Ref a, Ref b, int M, int N, bf16_t* w) {
            return job(kAdam, a, b, none, M, N, n, ref(B.W[q]), ref(B.M[q]), ref(B.V[q]), weight(w));
        };
        // W2 is updated beside the backward pass, which reads W2^T; that follows beside the update of W1 and W3
        p.n_jobs = 2;
        p.job[0] = adam(2, ref(B.dYt), ref(B.At), d, F, w2u);
        p.job[1] = job(kBackward, ref(B.dY), ref(B.w2t), none, n, F, d, ref(B.G), ref(B.U), ref(B.dGt), ref(B.dUt));
        if ((e = launch_dgemm<kUpdate>(p, groups, s)) != hipSuccess) return e;
        p.n_jobs = t + 1 < steps ? 3 : 2;
        p.job[0] = adam(0, ref(B.dGt), Xt, F, d, w1u);
        p.job[1] = adam(1, ref(B.dUt), Xt, F, d, w3u);
        p.job[2] = job(kTranspose, weight(w2u), none, none, d, F, 64, ref(B.w2t), none, none, none);
        if ((e = launch_dgemm<kUpdate>(p, groups, s)) != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_fill_f32(float* p, size_t n, float v, hipStream_t s)
{
    fill_f32_kernel<<<(int)((n + 255) / 256), 256, 0, s>>>(p, n, v);
    return hipGetLastError();
}

}  // namespace bmoe

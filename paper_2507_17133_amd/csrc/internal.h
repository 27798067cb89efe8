// Internal declarations shared by the translation units of libbrownout_moe.so.
// Host-side launchers only; every kernel lives in the .hip file that launches it.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/brownout_moe.h"

namespace bmoe {

typedef __bf16 bf16_t;

constexpr int kMaxExperts = 256;  // m
constexpr int kMaxTopK = 32;      // K
constexpr int kMaxShared = 8;     // N_s
constexpr int kMaxUnits = kMaxExperts + kMaxExperts + kMaxShared;  // U
constexpr int kSegTokens = 64;    // tokens per routing segment (one wavefront)
constexpr int kFewExpertsTokens = 2048;   // at most 16 experts and this many tokens: the fp64 gate (no matrix cores)
constexpr int kMinTileRows = 32;  // smallest GEMM M tile
constexpr int kTailBlocks = 256;  // largest grid of the persistent GEMM whose K-split tail has scratch (one block per CU)

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Measurement switches, read from the environment ONCE (when the library is loaded); all unset in normal use.
struct Tuning {
    int force_bm;      // BROWNOUT_MOE_BM = 32/64/128/256: one tile height for every unit (0: not forced)
    int group_m;       // BROWNOUT_MOE_GM: M tiles per L2 super-tile of the GEMMs (0: 8 for 256-row tiles, else 4)
    int force_ksplit;  // BROWNOUT_MOE_KSPLIT = 1/2/4: K planes of GEMM2 with small tiles (0: not forced)
};
const Tuning& tuning();

// One-time set-up per device: kernel attributes (dynamic LDS sizes), CU count.  Done by moe_init and by
// moe_workspace_size; the launch paths only check that it has happened (and do it if not, which works
// everywhere except under stream capture).
struct DeviceInfo { int n_cu; };
hipError_t ensure_device_init(DeviceInfo* info);
hipError_t init_ffn_kernels();      // ffn.hip
hipError_t init_route_kernels();    // route.hip

// How the rows of the units are cut into GEMM M tiles: one tile height for every unit of a launch, from the expected rows per
// unit on the host, or one of two from the real counts on the device (tiles.h), both taken by the same launch.
struct TilePlan {
    int bm;          // 256, 128, 64 or 32
    int lo = 0;      // 64 (with bm 128) or 32 (64): the height that the table takes unless the taller one saves rounds; 0: none
    int cols1 = 0, cols2 = 0, k1 = 0, k2 = 0;     // with lo: blocks per M tile and k tiles per block of the two GEMMs
    int n_cu = 0;                                 // and the CUs, with 2^32 / n_cu rounded up
    unsigned inv_cu = 0;
};
TilePlan make_tile_plan(int64_t rows_per_unit, bool even);     // even: exactly that many in every unit, else their mean

// Derived sizes of one (config, T) problem.
struct Dims {
    int T, d, F, m, K, way, G, Ns, Fs, U, slots, m_pad, Fmax;
    int score_fn, add_residual, gate_format;
    int64_t row_cap;   // rows the row lists can hold: T*(K+Ns)
    int n_seg;         // routing segments
    int tile_cap;      // entries of one GEMM tile table
    int ksplit;        // K slices of GEMM2 (partial products in separate planes of Y)
    int64_t y_plane;   // elements between two planes of Y
    int tail_blocks;   // fp32 tiles in the scratch of the persistent GEMM's K-split tail (a bound on its grid)
};
Dims make_dims(const moe_config& c, int T);

// Carving of the caller's workspace.  All offsets are multiples of 256 bytes.
struct Workspace {
    size_t topk_idx, topk_w, expert_cnt, expert_unit, expert_in_s1, unit_cnt, unit_off, row_token, row_weight,
        token_rows, n_rows, near_tie;                 // default homes of the moe_route_out fields
    size_t gate_split;                                // [3][m_pad][d] bf16
    size_t seg_cnt, seg_off;                          // [n_seg][U] int32
    size_t route_total;                               // bytes of the pieces above (all that routing alone needs)
    size_t tiles0, tiles1;                            // GEMM tile tables: int32[4] header + int4 entries
    size_t H;                                         // [h_rows][Fmax] bf16
    size_t Y;                                         // [y_rows][d], IEEE half (2 bytes; carried as bf16_t*)
    size_t loss_part;                                 // T*4 bytes: fp64 partial sums of build_united's loss
    size_t partial, partial_bytes;                    // fp32 tiles of GEMM2's K-split tail (256-row tiles, one plane)
    size_t total;
    int64_t h_rows, y_rows;
};
Workspace carve_workspace(const Dims& D);

// Resolved device pointers of the routing artefacts (caller's or workspace's).
struct RouteBufs {
    int32_t* topk_idx; float* topk_w; int32_t* expert_cnt; int32_t* expert_unit; uint8_t* expert_in_s1;
    int32_t* unit_cnt; int32_t* unit_off; int32_t* row_token; float* row_weight; int32_t* token_rows;
    int32_t* n_rows; uint8_t* near_tie;
};

// ---- profiling hooks (api.hip) ----
void prof_begin(int stage, hipStream_t s);
void prof_end(int stage, hipStream_t s);
struct ProfScope {
    int stage; hipStream_t s;
    ProfScope(int st, hipStream_t str) : stage(st), s(str) { prof_begin(stage, s); }
    ~ProfScope() { prof_end(stage, s); }
};

// Between what the lanes of a wave write to LDS and what others of its lanes read there: an order for the compiler, which knows one
// lane's accesses only and may move a load above stores of another type.  The hardware carries out a wave's LDS operations in
// order, so no instruction comes of it.
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Workgroup barrier that orders LDS traffic for the compiler without the vmcnt(0) wait __syncthreads()
// implies: tiles still in flight to LDS (tracked by vmcnt) must stay in flight across it.  Every wave
// waits for the loads it needs (s_waitcnt vmcnt) itself before arriving.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// One direct load: 16 bytes per lane, 1 KiB of LDS from dst on.
template <int POLICY = 0>
__device__ __forceinline__ void load_lds(const void* src, char* dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)dst, 16,
                                     0, POLICY);
}

// s_waitcnt immediates (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8).
__host__ __device__ constexpr int vmcnt_imm(int n) { return (n & 0xF) | ((n >> 4) << 14) | 0x0F70; }       // vmcnt <= n
__host__ __device__ constexpr int vmcnt_lgkm0_imm(int n) { return vmcnt_imm(n) & 0xF0FF; }                 // and lgkmcnt 0

// Tells the compiler that a pointer is the same in every lane (keeps it in scalar registers).
__device__ __forceinline__ const bf16_t* uniform_ptr(const bf16_t* ptr)
{
    const unsigned long long v = reinterpret_cast<unsigned long long>(ptr);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return reinterpret_cast<const bf16_t*>(((unsigned long long)hi << 32) | lo);
}

// two floats -> two bf16 (round to nearest even) in one 32-bit word, first value in the low half
__device__ __forceinline__ unsigned pack_bf16(float lo, float hi)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {lo, hi};
    const bf16x2 b = __builtin_convertvector(v, bf16x2);
    return __builtin_bit_cast(unsigned, b);
}

// ---- routing (route.hip) ----
struct TileJobs;
// gate: fp32 [m][d] (D.gate_format MOE_GATE_FP32; split into gate_split on the way) or the packed pieces
// (MOE_GATE_PACKED; gate_split unused).  logits: scratch of the many-expert gate, at least 64 bytes per expert
// (m_pad).  jobs: GEMM tile tables to build once the unit counts are known (jobs.n == 0: none).
hipError_t launch_route(const Dims& D, const bf16_t* x, const void* gate, const float* gate_bias,
                        double threshold, int full_brownout, const RouteBufs& R, bf16_t* gate_split,
                        int32_t* seg_cnt, int32_t* seg_off, void* logits, size_t logit_bytes, const TileJobs& jobs,
                        hipStream_t s);
hipError_t launch_pack_gate(const float* gate_w, int m, int m_pad, int d, bf16_t* packed, hipStream_t s);

// ---- FFN (ffn.hip) ----
struct FfnWeights { const bf16_t *w1, *w3, *w2; };
// The units of a launch: how many may hold rows, the TopK entries spread over the experts among them, and how many hold
// all T tokens each (shared experts; units on calibration tokens).
struct FfnUnits { int n; int64_t entries; int even; };
// Units of one width: how their rows are cut into M tiles, and the tile table, which the routing kernels or
// launch_tile_tables have written; bm_hi: a height that has a launch of its own (TileJob::bm_hi).
struct FfnProblem { FfnUnits units; int F; TilePlan plan; int bm_hi; int32_t* table; };
// Runs W2(silu(W1 x)*(W3 x)) for the rows of the tiles in the tables of one problem, or of the routed and united units and then the
// shared experts; writes Y[row][d] = FFN(x[gather ? gather[row] : row]) (the row weights are applied by the combine).  Weight
// source of unit u: u<m experts[u]; u<m+G united[u-m]; else shared[u-m-G].  may_stream: TileJobs::may_stream().
hipError_t launch_ffn(const Dims& D, const FfnProblem* problems, int n_problems, const bf16_t* x, const int32_t* gather,
                      const FfnWeights& experts, const FfnWeights& united, const FfnWeights& shared, bf16_t* H, bf16_t* Y,
                      float* partial, bool may_stream, hipStream_t s);
// Tile tables from the unit counts of a route that the caller brings.
hipError_t launch_tile_tables(const int32_t* unit_cnt, const int32_t* unit_off, const TileJobs& jobs, hipStream_t s);
hipError_t launch_combine(const Dims& D, const bf16_t* x, const bf16_t* Y, const int32_t* token_rows,
                          const float* row_weight, bf16_t* out, hipStream_t s);

// ---- united experts (united.hip) ----
hipError_t launch_united_mean(const bf16_t* w, int m, int way, size_t n_elem, bf16_t* u, hipStream_t s);
// Tile table of n_units0 units u0, u0+1, ... and n_units1 units u1, ..., each holding the n rows r*n .. r*n+n-1
// (r: position in that list, + first_slot).
hipError_t launch_uniform_units(int u0, int n_units0, int u1, int n_units1, int first_slot, int n, int bm, int32_t* table,
                                hipStream_t s);
// row_token[r*n + t] = t for `slots` such units.
hipError_t launch_repeat_tokens(int32_t* row_token, int n, int slots, hipStream_t s);
// part[0..blocks) (+)= per-block sums of (yu - yo_i)^2 over b teachers' rows of n elements each; if last,
// *loss = scale * sum of part.  part: kSqdiffBlocks doubles at most.
constexpr int kSqdiffBlocks = 512;
hipError_t launch_sqdiff(const bf16_t* yu, const bf16_t* yo, int b, size_t n, int blocks, bool first, bool last, double scale,
                         double* part, float* loss, hipStream_t s);

// United-expert distillation (distill.hip).  buf: distill_buffer_bytes of device memory for `groups` groups trained
// side by side; one group is enough, distill_wanted_bytes hold as many as keep the chip busy (it grows with n).
hipError_t init_distill_kernels();
size_t distill_buffer_bytes(int n, int d, int F, int groups);
size_t distill_wanted_bytes(int n, int d, int F, int n_groups);
int distill_groups_that_fit(int n, int d, int F, int n_groups, size_t bytes);       // 0: not even one
hipError_t launch_fill_f32(float* p, size_t n, float v, hipStream_t s);
// FFN output rows (half) of b of the k teachers of group g, n*d elements apart; first / last: of the k
hipError_t launch_teacher_stats(const bf16_t* y_half, int b, bool first, bool last, int k, int n, int d, int F, int g, void* buf,
                                hipStream_t s);
hipError_t distill_groups(const bf16_t* x, int n, int d, int F, int groups, bf16_t* w1u, bf16_t* w3u, bf16_t* w2u, int steps,
                          float lr, float* hist, void* buf, hipStream_t s);

// Probes (probe.hip): sustained rate of a pure MFMA loop on the caller's operand bits (operands: 64 KiB of
// bf16, sink: 2 MiB), and of a read-only sweep over buf (sink: 4 bytes).  Both wait for the stream.
hipError_t probe_mfma(const void* operands, void* sink, hipStream_t s, double* tflops);
hipError_t probe_hbm_read(const void* buf, size_t bytes, void* sink, hipStream_t s, double* gbs);

}  // namespace bmoe

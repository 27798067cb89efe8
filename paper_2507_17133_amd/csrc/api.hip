// C ABI of libbrownout_moe.so: argument validation, workspace carving, kernel sequencing, profiling.
#include "internal.h"
#include "tiles.h"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

// Scratch of moe_route_static (callers that cannot allocate): routing work space of a stated, modest size
// that lives in the library's own device image.  In host code this name is only a handle for
// hipGetSymbolAddress; the device address is looked up once per device in ensure_device_init.
constexpr size_t kStaticScratchBytes = (size_t)8 << 20;
// Behind it: room for the gate's logits, with what the routing work space leaves (larger batches go through it in pieces).
constexpr size_t kStaticLogitBytes = (size_t)2 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes + kStaticLogitBytes];

namespace bmoe {

constexpr int kMixedRows = 384;      // expected rows per unit from which 256-row tiles are used
constexpr int kMaxDevices = 64;

static Tuning read_tuning()
{
    Tuning t{0, 0, 0};
    if (const char* e = std::getenv("BROWNOUT_MOE_BM")) {
        const int v = std::atoi(e);
        if (v == 32 || v == 64 || v == 128 || v == 256) t.force_bm = v;
    }
    if (const char* e = std::getenv("BROWNOUT_MOE_GM")) t.group_m = std::max(1, std::min(64, std::atoi(e)));
    if (const char* e = std::getenv("BROWNOUT_MOE_KSPLIT")) {
        const int v = std::atoi(e);
        if (v == 1 || v == 2 || v == 4) t.force_ksplit = v;
    }
    return t;
}
const Tuning& tuning()
{
    static const Tuning t = read_tuning();       // read once, when first asked for
    return t;
}

static std::mutex g_init_mutex;
static bool g_init_done[kMaxDevices] = {false};
static DeviceInfo g_dev_info[kMaxDevices];
static void* g_scratch_ptr[kMaxDevices] = {nullptr};

hipError_t ensure_device_init(DeviceInfo* info)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_init_mutex);
    if (!g_init_done[dev]) {
        (void)tuning();
        if ((e = init_ffn_kernels()) != hipSuccess) return e;
        if ((e = init_route_kernels()) != hipSuccess) return e;
        if ((e = init_distill_kernels()) != hipSuccess) return e;
        int n_cu = 0;
        if ((e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
        void* sp = nullptr;
        if ((e = hipGetSymbolAddress(&sp, HIP_SYMBOL(scratch))) != hipSuccess) return e;
        g_dev_info[dev].n_cu = n_cu;
        g_scratch_ptr[dev] = sp;
        g_init_done[dev] = true;
    }
    if (info) *info = g_dev_info[dev];
    return hipSuccess;
}

static void* static_scratch_of_current_device()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    return g_scratch_ptr[dev];
}

static thread_local std::string g_hip_error;

static moe_status hip_fail(hipError_t e, const char* where)
{
    g_hip_error = std::string(where) + ": " + hipGetErrorString(e);
    (void)hipGetLastError();
    return MOE_ERR_HIP;
}

// GEMM tile height from the rows per unit: `even`, every unit holds that many (calibration tokens, a shared expert), else
// their mean over the experts.  A gate's popular experts hold several times the mean, and every further tile of a
// unit stages its weights again, so a tile is at least one to four times the mean.  Layer forward in us at tiles of 32 / 64
// / 128 rows, Zipf gates: DeepSeek-V3 shape, 16 rows per expert 2919 / 2635 / 2622, 32 rows 4231 / 3497 / 3334; Qwen3 shape,
// 8 rows 222 / 229 / 229, 16 rows 259 / 246 / 247, 64 rows 398 / 339 / 311; uniform gate, Mixtral shape, 16 rows 512 / 531 / 542, 100 rows
// 1073 / 647 / 573.
static int pick_tile_rows(int64_t rows, bool even)
{
    if (tuning().force_bm) return tuning().force_bm;
    if (rows >= kMixedRows) return 256;
    if (rows >= 48) return 128;
    return rows >= (even ? 24 : 12) ? 64 : 32;
}

TilePlan make_tile_plan(int64_t rows, bool even)
{
    TilePlan p;
    p.bm = pick_tile_rows(rows, even);
    return p;
}

// Tile heights of the routed units.  Where all experts together have fewer 256-column blocks than the chip has CUs, weights are
// few and the narrow kernel's time is its own latency: no taller tiles then (64 tokens over 8 experts of 256 x 512: 23.8 us
// at 32 rows, 25.3 at 64).  With many experts whose weights take some k tiles to stream, a GEMM takes as long as its rounds of blocks,
// and those follow from how the gate and brownout fill the units: from 4 rows per expert on the table kernel chooses between 32
// and 64 rows, from 12 on between 64 and 128 (tiles.h; one launch takes either).  Layer forward in us at the lower height, the taller and
// as chosen, skewed gate, then even gate; 2048 x 768, 128 experts: 8 rows per expert without brownout 200 / 207 / 200, 16 rows 230 / 228 /
// 222, 28 rows 250 / 275 / 250; at 0.5 brownout 85 / 69 / 69, 97 / 79 / 79, 106 / 98 / 98; even, at 0.5, 11 rows 149 / 155 / 149, 16 rows 154 /
// 166 / 154, 28 rows 183 / 176 / 175; 2048 x 1408, 60 experts at 0.6: 8 rows 68 / 60 / 61, even 119 / 129 / 119, 17 rows 131 / 147 / 131; DeepSeek-V3
// shape, 8 rows 2084 / 1962 / 1964, 12 rows 2447 / 2388 / 2388, even, at 0.4, 40 rows 3115 / 2967 / 2969.
// With up to 16 experts or less than 1024 columns the mean decides.  There too the other height can be the better one (4096 x 2048, 16
// experts, 8 rows 176 us at 32 rows and 164 at 64; 960 x 2048, 128 experts, 8 rows at 0.5 107 and 92), now and then by as much.
// Shared experts of a width of their own go out with tiles of up to 64 rows only: 250 tokens of the 60-expert shape, 17 rows, 270 at
// 64 and 296 at 128.
constexpr int kBesideTokens = 256;
static TilePlan routed_tile_plan(const Dims& D, int n_cu)
{
    const int64_t entries = (int64_t)D.T * D.K, rows = entries / D.m;
    const bool few = std::min<int64_t>(entries, D.m) * ceil_div(D.F, 128) < n_cu;
    TilePlan p;
    p.bm = pick_tile_rows(rows, few);
    if (few || tuning().force_bm || D.m <= 16 || D.d < 1024) return p;
    const bool beside = D.Ns > 0 && D.Fs != D.F && D.T <= kBesideTokens;
    if (p.bm == 64 && !beside) {
        p.bm = 128;
        p.lo = 64;
    } else if (p.bm == 32 && rows >= 4) {
        p.bm = 64;
        p.lo = 32;
    }
    p.cols1 = ceil_div(D.F, 128); p.k1 = D.d / 64;
    p.cols2 = ceil_div(D.d, 256) * D.ksplit; p.k2 = ceil_div(D.F / 64, D.ksplit);
    p.n_cu = n_cu; p.inv_cu = (unsigned)((((uint64_t)1 << 32) + n_cu - 1) / n_cu);
    return p;
}

// A launch of shared experts alone.  Up to kBesideTokens tokens of few enough 64-row blocks go to the narrow kernel, in one launch
// with the routed units (100 tokens over F = 5632, 44 blocks of 128 rows: layer with its routed experts 157.6 -> 124.7 us; 250
// tokens 285 -> 270), and 256 rows need a tile for every CU (500 tokens at 0.6 brownout: 205 us with them, 156 with 128).
static TilePlan make_shared_plan(const Dims& D, int n_cu)
{
    TilePlan p = make_tile_plan(D.T, true);
    if (tuning().force_bm) return p;
    const int cols = D.Ns * ceil_div(D.Fs, 128);
    if (p.bm == 256 && ceil_div(D.T, 256) * cols < n_cu) p.bm = 128;
    if (p.bm == 128 && D.T <= kBesideTokens && ceil_div(D.T, 64) * cols < n_cu) p.bm = 64;
    return p;
}

// The taller tile that the table kernel may choose instead in a browned-out batch (0: none).  Offered where its blocks fill
// the CUs once if no entry is dropped: the launch that gets no tiles costs 3 to 10 us, which shorter forwards would feel.
// Layer forward in us at 40 / 80 % brownout, tiles of 64, 128 and 256 rows: DeepSeek-V3 shape, 16 rows per expert
// 1079 / 932, 901 / 812, 950 / 821; 32 rows 1613 / 1452, 1216 / 1058, 1144 / 999; 94 rows (128 and 256) 2431 / 2312, 2131 / 1954;
// Qwen3 shape, 250 rows 360 / 331, 354 / 308; with a uniform gate and 30 %, 32 rows 3275, 3372, 3845.
// GEMM2 keeps its planes at either height (the 256-row kernel then does not cut its tail, nor has it scratch for that below 384
// tokens).  Still the better height there: 8 experts of 4096 x 14336 at 30 / 80 % with 128 rows and with the choice of 256, 400
// tokens 530 / 357, 540 / 351, 1021 tokens 1012 / 654, 903 / 570.
static int taller_tile_rows(const Dims& D, int bm, int n_cu)
{
    if (tuning().force_bm) return 0;
    const int64_t rows = (int64_t)D.T * D.K / D.m;
    const int hi = rows >= 20 ? 256 : rows >= 5 ? 128 : 0;
    if (hi <= bm || (int64_t)D.T * D.K / hi * ceil_div(D.F, 128) < n_cu) return 0;
    return hi;
}

// Weights of the units that hold rows, and of the shared experts, beyond which they are streamed past the caches.  Below it one layer called over and
// over would lose what it still finds in the 256 MiB memory-side cache; above it the lines push each other out before they are read again.
// Layer forward in us without and with streaming, one layer over and over, then as many in turn as hold 1.6 GB:
//   37 tokens, 60-expert shape    231 MiB  67.5  77.2   80.3  76.7     4096 x 4096, 128 tokens  192 MiB  61.7  81.0   82.8  80.5
//                                 264 MiB  73.1  78.0   83.7  79.6                              288 MiB  92.9  88.0   93.8  88.1
//                                 280 MiB  82.7  80.4   92.1  85.9     4096 x 4096, 20 tokens   288 MiB  78.6  73.5   82.9  74.5
//                                 297 MiB  92.1  86.3   94.3  87.1     one of 4096 x 14336, 256 tokens (336 MiB) 132.3 124.7 131.6 124.0
//   232 tokens, Qwen3 experts     270 MiB  83.8  89.2   94.4  89.1                              64 tokens        108.9 102.1 106.3 101.1
//                                 288 MiB  95.8  92.1   97.8  92.4     7168 x 2048, 40 tokens   252 MiB  76.4  75.8   79.3  76.4
//                                 306 MiB 111.3 106.0  108.3 102.5                              336 MiB  86.7  78.2   87.0  79.0
// So layers in turn would gain some 5 % below the line too, and one layer alone lose up to 30.  With weights streamed that further tiles read later:
// 7113 tokens of the DeepSeek-V3 shape 8510 -> 10130; in the 256-row kernel, where eight M tiles in a row read the same ones: 8192 of the
// Qwen3 shape 618 -> 649.
constexpr int64_t kKeptBytes = (int64_t)288 << 20;
static int units_to_stream(const Dims& D)
{
    const int64_t left = kKeptBytes - (int64_t)D.Ns * 6 * D.d * D.Fs, unit = (int64_t)6 * D.d * D.F;
    return (int)std::max<int64_t>(0, left / unit + 1);
}

Dims make_dims(const moe_config& c, int T)
{
    Dims D;
    D.T = T; D.d = c.d_model; D.F = c.d_ff; D.m = c.n_experts; D.K = c.top_k; D.way = c.way;
    D.G = ceil_div(c.n_experts, c.way);
    D.Ns = c.n_shared; D.Fs = c.n_shared > 0 ? c.d_ff_shared : 0;
    D.U = D.m + D.G + D.Ns;
    D.slots = D.K + D.Ns;
    D.m_pad = ceil_div(D.m, 16) * 16;
    D.Fmax = D.F > D.Fs ? D.F : D.Fs;
    D.score_fn = c.score_fn; D.add_residual = c.add_residual;
    D.gate_format = c.gate_format;
    D.row_cap = (int64_t)T * D.slots;
    D.n_seg = ceil_div(T, kSegTokens);
    D.tile_cap = (int)(D.row_cap / kMinTileRows) + D.U;
    // GEMM2 has few, long tiles (N = d): split K (at most 4 ways) until about four rounds of blocks fill
    // the 256 CUs; more slices only add prologues and planes for the combine to sum.
    // Planes are partial sums in half precision, so their number does not follow the tile height that the rows of popular
    // experts ask for (routed_tile_rows): it comes from the mean alone, as for even units, and taller tiles keep it.
    const int bm = pick_tile_rows((int64_t)T * D.K / D.m, true);
    const int64_t tiles2 = (D.row_cap / bm + (D.m + D.G) / 2 + D.Ns) * (int64_t)ceil_div(D.d, 256);
    int ks = 1;
    while (ks < 4 && tiles2 * ks < 1024 && (D.F / 64) / (ks * 2) >= 8) ks *= 2;
    if (bm == 256) ks = 1;                                // the persistent kernel cuts its left-over tiles itself
    if (tuning().force_ksplit) ks = tuning().force_ksplit;
    D.ksplit = ks;
    D.y_plane = D.row_cap * (int64_t)D.d;
    const int64_t max_tiles = (D.row_cap / 256 + D.U) * (int64_t)std::max(ceil_div(D.d, 256), ceil_div(D.Fmax, 128));
    D.tail_blocks = (int)std::min<int64_t>(kTailBlocks, (max_tiles + 7) / 8 * 8);
    return D;
}

// Rows of Y the workspace holds: an upper bound of rows x K planes over every batch of at most T tokens, so
// that a workspace sized for T_max serves every smaller batch.  More than one plane is only chosen while
// GEMM2 has few tiles (make_dims): 2 planes need fewer than 1024 tiles of at most 128 rows, 4 planes fewer
// than 512, which bounds the rows such a batch can have.
static int64_t y_rows_bound(const Dims& D)
{
    const int64_t nt_d = ceil_div(D.d, 256);
    const int64_t lim2 = 128 * (1024 / nt_d) + 128, lim4 = 128 * (512 / nt_d) + 128;
    int64_t rows = std::max<int64_t>(D.row_cap, 2 * (int64_t)D.T);
    rows = std::max(rows, 2 * std::min(D.row_cap, lim2));
    rows = std::max(rows, 4 * std::min(D.row_cap, lim4));
    if (tuning().force_ksplit) rows = std::max(rows, D.row_cap * tuning().force_ksplit);
    return rows;
}

// Every piece grows (weakly) with T, so the total does: moe_workspace_size(T_max) covers every T <= T_max.
// The routing pieces come first: carve_route_only() is the prefix moe_route_static needs.
static void carve_route_pieces(const Dims& D, Workspace& W, size_t& o)
{
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, 256); return at; };
    W.topk_idx = take((size_t)D.T * D.K * 4);
    W.topk_w = take((size_t)D.T * D.K * 4);
    W.expert_cnt = take((size_t)D.m * 4);
    W.expert_unit = take((size_t)D.m * 4);
    W.expert_in_s1 = take((size_t)D.m);
    W.unit_cnt = take((size_t)D.U * 4);
    W.unit_off = take((size_t)(D.U + 1) * 4);
    W.row_token = take((size_t)D.row_cap * 4);
    W.row_weight = take((size_t)D.row_cap * 4);
    W.token_rows = take((size_t)D.row_cap * 4);
    W.near_tie = take((size_t)D.T);
    // the pieces of an fp32 gate matrix.  A packed gate of more than 16 experts brings them; with at most 16
    // experts the gate is fp32 rows in either format, cut on the way only beyond kFewExpertsTokens tokens
    const bool no_pieces = D.m_pad == 16 ? D.T <= kFewExpertsTokens : D.gate_format == MOE_GATE_PACKED;
    W.gate_split = take(no_pieces ? 0 : (size_t)3 * D.m_pad * D.d * 2);
    W.seg_cnt = take((size_t)D.n_seg * D.U * 4);
    W.seg_off = take((size_t)D.n_seg * D.U * 4);
    W.n_rows = take(4);
}

Workspace carve_workspace(const Dims& D)
{
    Workspace W;
    size_t o = 0;
    carve_route_pieces(D, W, o);
    W.route_total = o;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, 256); return at; };
    // the first table follows n_rows in its 256 bytes, 16 of them for the flag before the table (TileJobs::may_stream)
    W.tiles0 = W.n_rows + 32;
    o = align_up(W.tiles0 + 16 + (size_t)D.tile_cap * 16, 256);
    W.tiles1 = take(16 + (size_t)D.tile_cap * 16);
    W.h_rows = D.row_cap;
    W.y_rows = y_rows_bound(D);
    // one tile of rows past the end: GEMM2's ragged last tile reads (and discards) whole tiles of H
    W.H = take((size_t)(W.h_rows + 256) * D.Fmax * 2);
    W.Y = take((size_t)W.y_rows * D.d * 2);
    W.loss_part = take((size_t)D.T * 4);
    // K-split tail of the persistent 256-row GEMMs: one fp32 tile per block of their grid.  256-row tiles can
    // occur from kMixedRows tokens on (a shared expert, or one unit holding all calibration tokens).
    W.partial = 0;
    W.partial_bytes = 0;
    if (D.T >= kMixedRows || tuning().force_bm == 256) {
        W.partial_bytes = (size_t)D.tail_blocks * 256 * 256 * 4;
        W.partial = take(W.partial_bytes);
    }
    W.total = o;
    return W;
}

static moe_status check_config(const moe_config* c)
{
    if (!c) return MOE_ERR_INVALID_ARG;
    if (c->gate_format != MOE_GATE_FP32 && c->gate_format != MOE_GATE_PACKED) return MOE_ERR_INVALID_ARG;
    if (c->n_experts < 1 || c->top_k < 1 || c->way < 1 || c->n_shared < 0) return MOE_ERR_INVALID_ARG;
    if (c->top_k > c->n_experts) return MOE_ERR_INVALID_ARG;
    if (c->score_fn != 0 && c->score_fn != 1) return MOE_ERR_INVALID_ARG;
    if (c->add_residual != 0 && c->add_residual != 1) return MOE_ERR_INVALID_ARG;
    if (c->d_model <= 0 || c->d_ff <= 0 || c->d_model % 64 || c->d_ff % 64) return MOE_ERR_SHAPE;
    if (c->n_shared > 0 && (c->d_ff_shared <= 0 || c->d_ff_shared % 64)) return MOE_ERR_SHAPE;
    if (c->n_experts > kMaxExperts || c->top_k > kMaxTopK || c->n_shared > kMaxShared) return MOE_ERR_SHAPE;
    return MOE_OK;
}

static moe_status check_T(const moe_config* c, int32_t T)
{
    if (T <= 0) return MOE_ERR_INVALID_ARG;
    if ((int64_t)T * (c->top_k + c->n_shared) > ((int64_t)1 << 30)) return MOE_ERR_SHAPE;
    // byte offsets into the activations are 32-bit in the 256-row GEMM
    if ((int64_t)T * c->d_model * 2 >= ((int64_t)1 << 32)) return MOE_ERR_UNSUPPORTED;
    return MOE_OK;
}

static bool misaligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

static moe_status check_weights(const moe_ffn_weights* w)
{
    if (!w || !w->w1 || !w->w3 || !w->w2) return MOE_ERR_INVALID_ARG;
    if (misaligned(w->w1) || misaligned(w->w3) || misaligned(w->w2)) return MOE_ERR_ALIGNMENT;
    return MOE_OK;
}

static FfnWeights to_ffn(const moe_ffn_weights* w)
{
    FfnWeights f{nullptr, nullptr, nullptr};
    if (w) {
        f.w1 = static_cast<const bf16_t*>(w->w1);
        f.w3 = static_cast<const bf16_t*>(w->w3);
        f.w2 = static_cast<const bf16_t*>(w->w2);
    }
    return f;
}

template <typename Tp>
static Tp* at(void* ws, size_t off) { return reinterpret_cast<Tp*>(static_cast<char*>(ws) + off); }

static RouteBufs resolve_route(const moe_route_out* o, void* ws, const Workspace& W)
{
    RouteBufs R;
    R.topk_idx = (o && o->topk_idx) ? o->topk_idx : at<int32_t>(ws, W.topk_idx);
    R.topk_w = (o && o->topk_w) ? o->topk_w : at<float>(ws, W.topk_w);
    R.expert_cnt = (o && o->expert_cnt) ? o->expert_cnt : at<int32_t>(ws, W.expert_cnt);
    R.expert_unit = (o && o->expert_unit) ? o->expert_unit : at<int32_t>(ws, W.expert_unit);
    R.expert_in_s1 = (o && o->expert_in_s1) ? o->expert_in_s1 : at<uint8_t>(ws, W.expert_in_s1);
    R.unit_cnt = (o && o->unit_cnt) ? o->unit_cnt : at<int32_t>(ws, W.unit_cnt);
    R.unit_off = (o && o->unit_off) ? o->unit_off : at<int32_t>(ws, W.unit_off);
    R.row_token = (o && o->row_token) ? o->row_token : at<int32_t>(ws, W.row_token);
    R.row_weight = (o && o->row_weight) ? o->row_weight : at<float>(ws, W.row_weight);
    R.token_rows = (o && o->token_rows) ? o->token_rows : at<int32_t>(ws, W.token_rows);
    R.n_rows = (o && o->n_rows) ? o->n_rows : at<int32_t>(ws, W.n_rows);
    R.near_tie = (o && o->near_tie) ? o->near_tie : at<uint8_t>(ws, W.near_tie);
    return R;
}

static moe_status check_route_ptr_alignment(const moe_route_out* o)
{
    const void* ps[] = {o->topk_idx, o->topk_w, o->expert_cnt, o->expert_unit, o->unit_cnt, o->unit_off,
                        o->row_token, o->row_weight, o->token_rows, o->n_rows};
    for (const void* p : ps)
        if (p && (reinterpret_cast<uintptr_t>(p) & 3u)) return MOE_ERR_ALIGNMENT;
    return MOE_OK;
}

// ---------------------------------------------------------------- profiling
struct ProfRecord { int stage; hipEvent_t a, b; };
static unsigned g_prof_mask = 0;
static std::vector<ProfRecord> g_prof_records;
static std::vector<hipEvent_t> g_prof_pool;
static hipEvent_t g_prof_open[MOE_N_STAGES];
static bool g_prof_is_open[MOE_N_STAGES] = {false};
constexpr size_t kProfMaxRecords = 4096 * MOE_N_STAGES;

static hipEvent_t prof_event()
{
    if (!g_prof_pool.empty()) {
        hipEvent_t e = g_prof_pool.back();
        g_prof_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

void prof_begin(int stage, hipStream_t s)
{
    if (!(g_prof_mask & (1u << stage)) || g_prof_records.size() >= kProfMaxRecords) return;
    hipEvent_t e = prof_event();
    if (!e) return;
    (void)hipEventRecord(e, s);
    g_prof_open[stage] = e;
    g_prof_is_open[stage] = true;
}

void prof_end(int stage, hipStream_t s)
{
    if (!g_prof_is_open[stage]) return;
    g_prof_is_open[stage] = false;
    hipEvent_t e = prof_event();
    if (!e) { g_prof_pool.push_back(g_prof_open[stage]); return; }
    (void)hipEventRecord(e, s);
    g_prof_records.push_back(ProfRecord{stage, g_prof_open[stage], e});
}

}  // namespace bmoe

using namespace bmoe;

extern "C" {

const char* moe_status_string(moe_status s)
{
    switch (s) {
        case MOE_OK: return "ok";
        case MOE_ERR_INVALID_ARG: return "invalid argument";
        case MOE_ERR_SHAPE: return "unsupported shape";
        case MOE_ERR_ALIGNMENT: return "misaligned pointer";
        case MOE_ERR_WORKSPACE: return "workspace missing or too small";
        case MOE_ERR_UNSUPPORTED: return "not implemented";
        case MOE_ERR_HIP: return "HIP runtime error";
        default: return "unknown status";
    }
}

const char* moe_last_hip_error(void) { return g_hip_error.c_str(); }

moe_status moe_workspace_size(const moe_config* cfg, int32_t T_max, size_t* bytes)
{
    moe_status st = check_config(cfg);
    if (st != MOE_OK) return st;
    if (!bytes) return MOE_ERR_INVALID_ARG;
    st = check_T(cfg, T_max);
    if (st != MOE_OK) return st;
    *bytes = carve_workspace(make_dims(*cfg, T_max)).total;
    // a caller sizes its workspace before its first launch: take the chance to do the per-device set-up, so
    // that even a first call made under stream capture finds it done (no device, e.g. a CPU-only host: skip)
    if (ensure_device_init(nullptr) != hipSuccess) (void)hipGetLastError();
    return MOE_OK;
}

moe_status moe_init(void)
{
    hipError_t e = ensure_device_init(nullptr);
    return e == hipSuccess ? MOE_OK : hip_fail(e, "moe_init");
}

moe_status moe_gate_packed_size(const moe_config* cfg, size_t* bytes)
{
    moe_status st = check_config(cfg);
    if (st != MOE_OK) return st;
    if (!bytes) return MOE_ERR_INVALID_ARG;
    *bytes = (size_t)3 * (ceil_div(cfg->n_experts, 16) * 16) * cfg->d_model * 2;
    return MOE_OK;
}

moe_status moe_pack_gate(const moe_config* cfg, const float* gate_w, void* packed, size_t packed_bytes, void* stream)
{
    moe_status st = check_config(cfg);
    if (st != MOE_OK) return st;
    if (!gate_w || !packed) return MOE_ERR_INVALID_ARG;
    if (misaligned(gate_w) || misaligned(packed)) return MOE_ERR_ALIGNMENT;
    const int m_pad = ceil_div(cfg->n_experts, 16) * 16;
    if (packed_bytes < (size_t)3 * m_pad * cfg->d_model * 2) return MOE_ERR_WORKSPACE;
    hipError_t e = launch_pack_gate(gate_w, cfg->n_experts, m_pad, cfg->d_model, static_cast<bf16_t*>(packed),
                                    static_cast<hipStream_t>(stream));
    return e == hipSuccess ? MOE_OK : hip_fail(e, "moe_pack_gate");
}

static moe_status check_route_args(const moe_config* cfg, const void* x, int32_t T, const void* gate_w,
                                   const float* gate_bias, double threshold, const moe_route_out* out)
{
    moe_status st = check_config(cfg);
    if (st != MOE_OK) return st;
    st = check_T(cfg, T);
    if (st != MOE_OK) return st;
    if (!x || !gate_w || !out) return MOE_ERR_INVALID_ARG;
    if (!(threshold >= 0.0 && threshold <= 1.0)) return MOE_ERR_INVALID_ARG;
    if (misaligned(x) || misaligned(gate_w) || (gate_bias && (reinterpret_cast<uintptr_t>(gate_bias) & 3u)))
        return MOE_ERR_ALIGNMENT;
    return check_route_ptr_alignment(out);
}

moe_status moe_route(const moe_config* cfg, const void* x, int32_t T, const void* gate_w, const float* gate_bias,
                     double threshold, int32_t use_full_brownout, const moe_route_out* out, void* workspace,
                     size_t workspace_bytes, void* stream)
{
    moe_status st = check_route_args(cfg, x, T, gate_w, gate_bias, threshold, out);
    if (st != MOE_OK) return st;
    const Dims D = make_dims(*cfg, T);
    const Workspace W = carve_workspace(D);
    if (!workspace || workspace_bytes < W.total) return MOE_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return MOE_ERR_ALIGNMENT;
    const RouteBufs R = resolve_route(out, workspace, W);
    hipStream_t s = static_cast<hipStream_t>(stream);
    TileJobs none;
    none.n = none.cap = none.count_units = none.stream_units = 0;
    hipError_t e = launch_route(D, static_cast<const bf16_t*>(x), gate_w, gate_bias, threshold,
                                use_full_brownout ? 1 : 0, R, at<bf16_t>(workspace, W.gate_split),
                                at<int32_t>(workspace, W.seg_cnt), at<int32_t>(workspace, W.seg_off),
                                at<void>(workspace, W.H), W.total - W.H, none, s);
    if (e != hipSuccess) return hip_fail(e, "moe_route");
    return MOE_OK;
}

moe_status moe_route_static(const moe_config* cfg, const void* x, int32_t T, const void* gate_w,
                            const float* gate_bias, double threshold, int32_t use_full_brownout,
                            const moe_route_out* out, void* stream)
{
    moe_status st = check_route_args(cfg, x, T, gate_w, gate_bias, threshold, out);
    if (st != MOE_OK) return st;
    const Dims D = make_dims(*cfg, T);
    Workspace W;
    size_t need = 0;
    carve_route_pieces(D, W, need);
    if (need > kStaticScratchBytes) return MOE_ERR_WORKSPACE;          // beyond the stated maximum
    hipError_t e = ensure_device_init(nullptr);                          // first call on this device: looks the scratch up
    if (e != hipSuccess) return hip_fail(e, "moe_route_static/init");
    void* sp = static_scratch_of_current_device();
    if (!sp) return hip_fail(hipErrorInvalidDevice, "moe_route_static/scratch");
    const RouteBufs R = resolve_route(out, sp, W);
    hipStream_t s = static_cast<hipStream_t>(stream);
    TileJobs none;
    none.n = none.cap = none.count_units = none.stream_units = 0;
    // everything the kernels read from the scratch they write first in the same call (counters are cleared by
    // the first kernel), so what an earlier call left there does not matter
    e = launch_route(D, static_cast<const bf16_t*>(x), gate_w, gate_bias, threshold, use_full_brownout ? 1 : 0, R,
                     at<bf16_t>(sp, W.gate_split), at<int32_t>(sp, W.seg_cnt), at<int32_t>(sp, W.seg_off),
                     at<void>(sp, need), kStaticScratchBytes + kStaticLogitBytes - need, none, s);
    if (e != hipSuccess) return hip_fail(e, "moe_route_static");
    return MOE_OK;
}

moe_status moe_forward(const moe_config* cfg, const void* x, int32_t T, const void* gate_w, const float* gate_bias,
                       const moe_ffn_weights* experts, const moe_ffn_weights* united, const moe_ffn_weights* shared,
                       double threshold, int32_t use_full_brownout, const moe_route_out* route, void* out,
                       void* workspace, size_t workspace_bytes, void* stream)
{
    moe_status st = check_config(cfg);
    if (st != MOE_OK) return st;
    st = check_T(cfg, T);
    if (st != MOE_OK) return st;
    if (!x || !out) return MOE_ERR_INVALID_ARG;
    if (misaligned(x) || misaligned(out)) return MOE_ERR_ALIGNMENT;
    st = check_weights(experts);
    if (st != MOE_OK) return st;
    if (cfg->n_shared > 0) {
        st = check_weights(shared);
        if (st != MOE_OK) return st;
    } else if (shared) {
        return MOE_ERR_INVALID_ARG;
    }
    if (united) {
        st = check_weights(united);
        if (st != MOE_OK) return st;
    }
    if (!route) {
        if (!gate_w) return MOE_ERR_INVALID_ARG;
        if (!(threshold >= 0.0 && threshold <= 1.0)) return MOE_ERR_INVALID_ARG;
        if (misaligned(gate_w) || (gate_bias && (reinterpret_cast<uintptr_t>(gate_bias) & 3u)))
            return MOE_ERR_ALIGNMENT;
        if (!united && threshold < 1.0 && !use_full_brownout) return MOE_ERR_INVALID_ARG;
    } else {
        if (!route->expert_unit || !route->unit_cnt || !route->unit_off || !route->row_token || !route->row_weight ||
            !route->token_rows)
            return MOE_ERR_INVALID_ARG;
        st = check_route_ptr_alignment(route);
        if (st != MOE_OK) return st;
    }
    const Dims D = make_dims(*cfg, T);
    const Workspace W = carve_workspace(D);
    if (!workspace || workspace_bytes < W.total) return MOE_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return MOE_ERR_ALIGNMENT;
    const RouteBufs R = resolve_route(route, workspace, W);
    DeviceInfo dev;
    hipError_t e = ensure_device_init(&dev);
    if (e != hipSuccess) return hip_fail(e, "moe_forward/init");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bf16_t* xb = static_cast<const bf16_t*>(x);
    // How the rows are cut into GEMM tiles: routed + united units by the expected rows per expert; shared units
    // (T rows each) with them when they have the same width, else in a launch of their own.
    const bool split_shared = D.Ns > 0 && D.Fs != D.F;
    TileJobs jobs;
    jobs.n = split_shared ? 2 : 1;
    jobs.cap = D.tile_cap;
    jobs.stream_units = units_to_stream(D);
    jobs.job[0].u_lo = 0; jobs.job[0].u_hi = split_shared ? D.m + D.G : D.U;
    jobs.job[0].plan = routed_tile_plan(D, dev.n_cu);
    jobs.job[0].table = at<int32_t>(workspace, W.tiles0);
    // no more units hold rows than there are TopK entries; the 256-row GEMM does not stream
    const bool may_stream = std::min<int64_t>((int64_t)T * D.K, D.m + D.G) >= jobs.stream_units && jobs.job[0].plan.bm < 256;
    jobs.count_units = may_stream ? D.m + D.G : 0;
    // a threshold of 1 browns nothing out (a route of the caller's may, whatever threshold comes with it)
    jobs.job[0].bm_hi = route || threshold < 1.0 ? taller_tile_rows(D, jobs.job[0].plan.bm, dev.n_cu) : 0;
    jobs.job[0].m = D.m; jobs.job[0].entries = T * D.K;
    jobs.job[1].bm_hi = 0; jobs.job[1].m = 0; jobs.job[1].entries = 0;
    jobs.job[1].u_lo = D.m + D.G; jobs.job[1].u_hi = D.U;
    jobs.job[1].plan = make_shared_plan(D, dev.n_cu);
    jobs.job[1].table = at<int32_t>(workspace, W.tiles1);
    if (!route) {
        e = launch_route(D, xb, gate_w, gate_bias, threshold, use_full_brownout ? 1 : 0, R,
                         at<bf16_t>(workspace, W.gate_split), at<int32_t>(workspace, W.seg_cnt),
                         at<int32_t>(workspace, W.seg_off), at<void>(workspace, W.H), W.total - W.H, jobs, s);
        if (e != hipSuccess) return hip_fail(e, "moe_forward/route");
    } else if ((e = launch_tile_tables(R.unit_cnt, R.unit_off, jobs, s)) != hipSuccess) {
        return hip_fail(e, "moe_forward/tiles");
    }
    const FfnWeights fe = to_ffn(experts), fu = to_ffn(united), fs = to_ffn(shared);
    bf16_t* H = at<bf16_t>(workspace, W.H);
    bf16_t* Y = at<bf16_t>(workspace, W.Y);
    float* partial = W.partial_bytes ? at<float>(workspace, W.partial) : nullptr;
    FfnProblem problems[2];
    for (int j = 0; j < jobs.n; ++j) {
        const TileJob& J = jobs.job[j];
        FfnUnits units{J.u_hi - J.u_lo, 0, 0};
        if (j == 0) units.entries = (int64_t)T * D.K;
        if (j == 1 || !split_shared) units.even = D.Ns;
        problems[j] = FfnProblem{units, j == 0 ? D.F : D.Fs, J.plan, J.bm_hi, J.table};
    }
    e = launch_ffn(D, problems, jobs.n, xb, R.row_token, fe, fu, fs, H, Y, partial, may_stream, s);
    if (e != hipSuccess) return hip_fail(e, "moe_forward/ffn");
    e = launch_combine(D, xb, Y, R.token_rows, R.row_weight, static_cast<bf16_t*>(out), s);
    if (e != hipSuccess) return hip_fail(e, "moe_forward/combine");
    return MOE_OK;
}

moe_status moe_build_united(const moe_config* cfg, const moe_ffn_weights* experts, const moe_ffn_weights_out* united_out,
                            const void* calib_x, int32_t n_calib, float* loss_per_group, void* workspace,
                            size_t workspace_bytes, void* stream)
{
    moe_status st = check_config(cfg);
    if (st != MOE_OK) return st;
    st = check_weights(experts);
    if (st != MOE_OK) return st;
    if (!united_out) return MOE_ERR_INVALID_ARG;
    const moe_ffn_weights united_ro{united_out->w1, united_out->w3, united_out->w2};
    st = check_weights(&united_ro);
    if (st != MOE_OK) return st;
    if (n_calib < 0) return MOE_ERR_INVALID_ARG;
    const bool want_loss = calib_x != nullptr && loss_per_group != nullptr && n_calib > 0;
    if (calib_x && misaligned(calib_x)) return MOE_ERR_ALIGNMENT;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int m = cfg->n_experts, way = cfg->way, G = ceil_div(m, way);
    const size_t n_elem = (size_t)cfg->d_model * cfg->d_ff;
    Dims D;
    Workspace W;
    if (want_loss) {
        st = check_T(cfg, n_calib);
        if (st != MOE_OK) return st;
        D = make_dims(*cfg, n_calib);
        W = carve_workspace(D);
        D.ksplit = 1;          // the loss kernel reads single-plane FFN outputs (the carving does not depend on it)
        if (!workspace || workspace_bytes < W.total) return MOE_ERR_WORKSPACE;
        if (reinterpret_cast<uintptr_t>(workspace) & 255u) return MOE_ERR_ALIGNMENT;
    }
    hipError_t e;
    const void* src[3] = {experts->w1, experts->w3, experts->w2};
    void* dst[3] = {united_out->w1, united_out->w3, united_out->w2};
    for (int k = 0; k < 3; ++k) {
        e = launch_united_mean(static_cast<const bf16_t*>(src[k]), m, way, n_elem, static_cast<bf16_t*>(dst[k]), s);
        if (e != hipSuccess) return hip_fail(e, "moe_build_united/mean");
    }
    if (!want_loss) return MOE_OK;

    const FfnWeights fe = to_ffn(experts), fu = to_ffn(&united_ro), fs{nullptr, nullptr, nullptr};
    const TilePlan plan = make_tile_plan(n_calib, true);
    bf16_t* H = at<bf16_t>(workspace, W.H);
    bf16_t* Yu = at<bf16_t>(workspace, W.Y);
    const size_t nd = (size_t)n_calib * D.d;
    float* partial = W.partial_bytes ? at<float>(workspace, W.partial) : nullptr;
    int32_t* row_token = at<int32_t>(workspace, W.row_token);
    int32_t* tiles = at<int32_t>(workspace, W.tiles0);
    const bf16_t* xb = static_cast<const bf16_t*>(calib_x);
    // The workspace holds the FFN rows of K+N_s units: the student's in the first slot, kept while the teachers go
    // through the others in equal batches (one slot only: the teachers' outputs go to the second plane of Y).
    const int cap = D.slots > 1 ? D.slots - 1 : 1;
    // one block per 2048 elements, at most as many as its piece of the workspace holds partial sums for
    const int sq_blocks = (int)std::min<size_t>({(nd / 8 + 255) / 256, (size_t)kSqdiffBlocks,
                                                 align_up((size_t)n_calib * 4, 256) / 8});
    double* sq_part = at<double>(workspace, W.loss_part);
    if ((e = launch_repeat_tokens(row_token, n_calib, D.slots, s)) != hipSuccess) return hip_fail(e, "moe_build_united/rows");
    auto run_units = [&](int u0, int n0, int u1, int n1, int first_slot, bf16_t* Y) -> hipError_t {
        hipError_t err = launch_uniform_units(u0, n0, u1, n1, first_slot, n_calib, plan.bm, tiles, s);
        if (err != hipSuccess) return err;
        const FfnProblem units{FfnUnits{n0 + n1, 0, n0 + n1}, D.F, plan, 0, tiles};
        return launch_ffn(D, &units, 1, xb, row_token, fe, fu, fs, H, Y, partial, false, s);
    };
    for (int g = 0; g < G; ++g) {
        const int lo = g * way, hi = lo + way < m ? lo + way : m, k = hi - lo;
        const int batches = ceil_div(k, cap);
        if (D.slots == 1) {
            e = run_units(m + g, 1, 0, 0, 0, Yu);
            if (e != hipSuccess) return hip_fail(e, "moe_build_united/student");
        }
        for (int q = 0; q < batches; ++q) {
            const int i0 = lo + (int)((int64_t)k * q / batches), i1 = lo + (int)((int64_t)k * (q + 1) / batches);
            if (D.slots == 1) e = run_units(i0, i1 - i0, 0, 0, 0, Yu + nd);
            else if (q == 0) e = run_units(m + g, 1, i0, i1 - i0, 0, Yu);
            else e = run_units(i0, i1 - i0, 0, 0, 1, Yu);
            if (e != hipSuccess) return hip_fail(e, "moe_build_united/teacher");
            e = launch_sqdiff(Yu, Yu + nd, i1 - i0, nd, sq_blocks, q == 0, q == batches - 1, 1.0 / ((double)k * n_calib),
                              sq_part, loss_per_group + g, s);
            if (e != hipSuccess) return hip_fail(e, "moe_build_united/loss");
        }
    }
    return MOE_OK;
}

// Groups with more than one member (all but a ragged last one, or none): the first ones.
static int trained_groups(int m, int way)
{
    return way == 1 ? 0 : m / way + (m % way > 1 ? 1 : 0);
}

static moe_status check_distill(const moe_config* cfg, int32_t n_calib)
{
    moe_status st = check_config(cfg);
    if (st != MOE_OK) return st;
    if (n_calib <= 0 || n_calib % 64) return MOE_ERR_SHAPE;
    return check_T(cfg, n_calib);
}

moe_status moe_distill_workspace_size(const moe_config* cfg, int32_t n_calib, size_t* bytes)
{
    if (!bytes) return MOE_ERR_INVALID_ARG;
    moe_status st = check_distill(cfg, n_calib);
    if (st != MOE_OK) return st;
    const Dims D = make_dims(*cfg, n_calib);
    *bytes = align_up(carve_workspace(D).total, 256) + distill_wanted_bytes(n_calib, D.d, D.F, trained_groups(D.m, D.way));
    return MOE_OK;
}

moe_status moe_distill_united(const moe_config* cfg, const moe_ffn_weights* experts, const moe_ffn_weights_out* united,
                              const void* calib_x, int32_t n_calib, int32_t steps, float lr, float* loss_history,
                              void* workspace, size_t workspace_bytes, void* stream)
{
    moe_status st = check_distill(cfg, n_calib);
    if (st != MOE_OK) return st;
    st = check_weights(experts);
    if (st != MOE_OK) return st;
    if (!united) return MOE_ERR_INVALID_ARG;
    const moe_ffn_weights united_ro{united->w1, united->w3, united->w2};
    st = check_weights(&united_ro);
    if (st != MOE_OK) return st;
    if (!calib_x || steps < 0 || !(lr >= 0.0f)) return MOE_ERR_INVALID_ARG;
    if (misaligned(calib_x)) return MOE_ERR_ALIGNMENT;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int m = cfg->n_experts, way = cfg->way, G = ceil_div(m, way);
    Dims D = make_dims(*cfg, n_calib);
    const Workspace W = carve_workspace(D);
    D.ksplit = 1;
    const TilePlan plan = make_tile_plan(n_calib, true);
    const size_t fwd_bytes = align_up(W.total, 256);
    // groups trained side by side: as many as keep the chip busy and the workspace holds, one at least
    const int trained = trained_groups(m, way);
    const int at_once = !workspace || workspace_bytes < fwd_bytes ? 0 :
                            distill_groups_that_fit(n_calib, D.d, D.F, trained, workspace_bytes - fwd_bytes);
    if (at_once < 1) return MOE_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return MOE_ERR_ALIGNMENT;
    void* buf = static_cast<char*>(workspace) + fwd_bytes;
    const FfnWeights fe = to_ffn(experts), fu = to_ffn(&united_ro), fs{nullptr, nullptr, nullptr};
    bf16_t* H = at<bf16_t>(workspace, W.H);
    bf16_t* Yo = at<bf16_t>(workspace, W.Y);
    int32_t* tiles = at<int32_t>(workspace, W.tiles0);
    int32_t* row_token = at<int32_t>(workspace, W.row_token);
    float* partial = W.partial_bytes ? at<float>(workspace, W.partial) : nullptr;
    const bf16_t* xb = static_cast<const bf16_t*>(calib_x);
    const size_t dF = (size_t)D.d * D.F;
    bf16_t* wu[3] = {static_cast<bf16_t*>(united->w1), static_cast<bf16_t*>(united->w3), static_cast<bf16_t*>(united->w2)};
    hipError_t e;
    if (trained > 0 && (e = launch_repeat_tokens(row_token, n_calib, D.slots, s)) != hipSuccess)
        return hip_fail(e, "moe_distill_united/rows");
    for (int g0 = 0; g0 < trained; g0 += at_once) {
        const int g1 = std::min(trained, g0 + at_once);
        for (int g = g0; g < g1; ++g) {
            // the teachers' outputs, as many at a time as the workspace holds FFN rows for, and their mean
            const int lo = g * way, hi = lo + way < m ? lo + way : m, k = hi - lo;
            const int batches = ceil_div(k, D.slots);
            for (int q = 0; q < batches; ++q) {
                const int i0 = lo + (int)((int64_t)k * q / batches), i1 = lo + (int)((int64_t)k * (q + 1) / batches);
                const FfnProblem units{FfnUnits{i1 - i0, 0, i1 - i0}, D.F, plan, 0, tiles};
                if ((e = launch_uniform_units(i0, i1 - i0, 0, 0, 0, n_calib, plan.bm, tiles, s)) != hipSuccess ||
                    (e = launch_ffn(D, &units, 1, xb, row_token, fe, fu, fs, H, Yo, partial, false, s)) != hipSuccess)
                    return hip_fail(e, "moe_distill_united/teacher");
                e = launch_teacher_stats(Yo, i1 - i0, q == 0, q == batches - 1, k, n_calib, D.d, D.F, g - g0, buf, s);
                if (e != hipSuccess) return hip_fail(e, "moe_distill_united/mean");
            }
        }
        e = distill_groups(xb, n_calib, D.d, D.F, g1 - g0, wu[0] + g0 * dF, wu[1] + g0 * dF, wu[2] + g0 * dF, steps, lr,
                           loss_history ? loss_history + (size_t)g0 * (steps + 1) : nullptr, buf, s);
        if (e != hipSuccess) return hip_fail(e, "moe_distill_united/train");
    }
    for (int g = trained; g < G; ++g) {
        // a lone member is its own best student: the minimiser (loss 0) is known, nothing to train
        const void* we[3] = {experts->w1, experts->w3, experts->w2};
        for (int q = 0; q < 3; ++q) {
            e = hipMemcpyAsync(wu[q] + g * dF, static_cast<const bf16_t*>(we[q]) + (size_t)g * way * dF, dF * 2,
                               hipMemcpyDeviceToDevice, s);
            if (e != hipSuccess) return hip_fail(e, "moe_distill_united/copy");
        }
        if (loss_history && (e = launch_fill_f32(loss_history + (size_t)g * (steps + 1), steps + 1, 0.0f, s)) != hipSuccess)
            return hip_fail(e, "moe_distill_united/clear");
    }
    return MOE_OK;
}

moe_status moe_probe_mfma(const void* operands, size_t operand_bytes, void* sink, size_t sink_bytes, void* stream,
                          double* tflops)
{
    if (!operands || !sink || !tflops) return MOE_ERR_INVALID_ARG;
    if (operand_bytes < 65536 || sink_bytes < ((size_t)2 << 20)) return MOE_ERR_WORKSPACE;
    if (misaligned(operands) || misaligned(sink)) return MOE_ERR_ALIGNMENT;
    hipError_t e = probe_mfma(operands, sink, static_cast<hipStream_t>(stream), tflops);
    return e == hipSuccess ? MOE_OK : hip_fail(e, "moe_probe_mfma");
}

moe_status moe_probe_hbm_read(const void* buf, size_t bytes, void* sink, size_t sink_bytes, void* stream, double* gbs)
{
    if (!buf || !sink || !gbs) return MOE_ERR_INVALID_ARG;
    if (bytes < ((size_t)1 << 20) || sink_bytes < 4) return MOE_ERR_WORKSPACE;
    if (misaligned(buf) || (reinterpret_cast<uintptr_t>(sink) & 3u)) return MOE_ERR_ALIGNMENT;
    hipError_t e = probe_hbm_read(buf, bytes, sink, static_cast<hipStream_t>(stream), gbs);
    return e == hipSuccess ? MOE_OK : hip_fail(e, "moe_probe_hbm_read");
}

moe_status moe_profile_enable(int32_t stage_mask)
{
    g_prof_mask = (unsigned)stage_mask & ((1u << MOE_N_STAGES) - 1u);
    return MOE_OK;
}

moe_status moe_profile_collect(double* total_ms, int64_t* launches)
{
    if (!total_ms || !launches) return MOE_ERR_INVALID_ARG;
    for (int i = 0; i < MOE_N_STAGES; ++i) { total_ms[i] = 0.0; launches[i] = 0; }
    moe_status st = MOE_OK;
    for (const ProfRecord& r : g_prof_records) {
        float ms = 0.0f;
        hipError_t e = hipEventSynchronize(r.b);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, r.a, r.b);
        if (e != hipSuccess) st = hip_fail(e, "moe_profile_collect");
        else { total_ms[r.stage] += (double)ms; launches[r.stage] += 1; }
        g_prof_pool.push_back(r.a);
        g_prof_pool.push_back(r.b);
    }
    g_prof_records.clear();
    return st;
}

}  // extern "C"

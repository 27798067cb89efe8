// GEMM tile table, built on the device from the unit row counts (shared by the routing kernels, which know
// the counts first, and by the stand-alone table kernel used when the caller brings its own row lists).
//
// int32 header {n_tiles, rows of a tile, 0, 0}, then one int4 {unit, first row, rows, 0} per M tile, units in ascending
// order, tiles of a unit consecutive.  Where weights may be streamed, the word before the first job's header says whether they are.
#pragma once
#include "internal.h"

namespace bmoe {

struct TileJob {
    int u_lo, u_hi;          // units [u_lo, u_hi)
    TilePlan plan;
    int32_t* table;
    int bm_hi;               // a taller tile that may suit a browned-out batch better (0: none), with a launch of its own: the
                             // table holds tiles of one height and says of which, the GEMM launch that has no use for it finds none
    int m, entries;          // bm_hi > 0: experts, TopK entries of the batch
};
struct TileJobs {
    int n;                   // 0, 1 or 2 jobs (routed + united units; shared units of another width)
    int count_units;         // weights are streamed past the caches (ffn.hip) if at least stream_units of the units [0, count_units)
    TileJob job[2];          // hold rows; count_units is 0 where the host knows that fewer do
    int cap;                 // entries a table holds
    int stream_units;
    __host__ __device__ bool may_stream() const { return count_units > 0; }
};

// What a GEMM tile of bm rows counts for in the choice of bm_hi, in twentieths of a 32-row one.  Full tiles alone (DeepSeek-V3 shape, even
// gate, 16384 tokens: 33.9, 20.6, 14.0 and 11.9 ms at 32, 64, 128 and 256 rows) would say 20, 24, 33 and 56, but the batches
// that choose hold ragged ones, and 256 rows win there from fewer saved tiles on: 88 tiles of 128 rows against 57 of 256 (1021 tokens at
// 0.4 brownout) 1216 and 1144 us, 57 against 46 (512 tokens) 901 and 950.  The line, 54 / 38 = 1.42, lies between those two.
__device__ __forceinline__ int tile_cost(int bm) { return bm == 256 ? 54 : bm == 128 ? 38 : bm == 64 ? 27 : 20; }

// Inclusive sum over the lanes of a wavefront: four shifts inside the rows of 16 lanes, then the rows' last lanes passed on (cross-lane
// reads through the LDS crossbar take some 100 cycles a step).
__device__ __forceinline__ int wave_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);       // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);       // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);       // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);       // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);       // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);       // row_bcast:31 into rows 2 and 3
    return v;
}

// Whether tiles of plan.bm rows replace tiles of plan.lo rows, n and n_lo of them.  One block of these kernels fits a CU and streams
// weights, so a GEMM takes as long as its rounds of blocks, whichever of the two heights they have: the taller one pays where it saves
// rounds (GEMM1 streams two matrices), by more than the 4 or 8 % that its own rounds cost.  Where GEMM1 has no round of 128-row
// tiles to fill, those go out half as wide, a block on nearly every CU; 64-row ones do not.
__device__ __forceinline__ bool tall_enough(const TilePlan& p, int n, int n_lo)
{
    if (p.lo == 64 && 2 * n * p.cols1 <= p.n_cu) return true;
    auto rounds = [&](int blocks) { return (long)__umulhi(blocks + p.n_cu - 1, p.inv_cu); };
    auto cost = [&](int tiles) { return 2 * rounds(tiles * p.cols1) * p.k1 + rounds(tiles * p.cols2) * p.k2; };
    const int own = p.lo == 64 ? 12 : 24;
    return (own + 1) * cost(n) <= own * cost(n_lo);
}

// One wavefront builds the table of one job.  cnt[u], off[u]: rows and first row of unit u (global or LDS).
// The tile height comes from the counts where the job leaves a choice: how popular the gate makes its experts decides how full their
// tiles are, and brownout takes the rows of unpopular experts away, so the few units that remain hold many times the T K / m
// the host can go by.  bm_hi only when entries have left their experts (256-row GEMMs may add up in another order), so that a
// batch without brownout takes the same kernels whether or not its caller offers the choice.
__device__ __forceinline__ void build_tile_table(const int* cnt, const int* off, const TileJob& j, int cap, int lane)
{
    const int n_units = j.u_hi - j.u_lo;
    const int per = (n_units + 63) / 64;
    // tiles of plan.bm rows, of the other heights (a power of two all; 1: not offered), rows of the experts: a lane's share
    const int h_lo = max(j.plan.lo, 1), h_hi = max(j.bm_hi, 1);
    auto tiles = [](int rows, int height) { return (rows + height - 1) >> __builtin_ctz(height); };
    int own = 0, lo = 0, hi = 0, rows = 0;
    for (int q = 0; q < per; ++q) {
        const int u = j.u_lo + lane * per + q;
        const int c = u < j.u_hi ? cnt[u] : 0;
        own += tiles(c, j.plan.bm);
        lo += tiles(c, h_lo);
        hi += tiles(c, h_hi);
        rows += u < j.m ? c : 0;
    }
    int bm = j.plan.bm, local = own;
    if (j.plan.lo > 0 || j.bm_hi > 0) {
        auto sum = [](int v) { return __builtin_amdgcn_readlane(wave_scan(v), 63); };
        int n = sum(own);
        if (j.plan.lo > 0) {
            const int n_lo = sum(lo);
            if (!tall_enough(j.plan, n, n_lo)) {
                bm = j.plan.lo;
                local = lo;
                n = n_lo;
            }
        }
        if (j.bm_hi > 0 && sum(rows) < j.entries && (long)sum(hi) * tile_cost(j.bm_hi) <= (long)n * tile_cost(bm)) {
            bm = j.bm_hi;
            local = hi;
        }
    }
    const int incl = wave_scan(local);
    const int total = __builtin_amdgcn_readlane(incl, 63);
    int at = incl - local;
    if (lane == 0) {
        j.table[0] = total < cap ? total : cap;
        j.table[1] = bm; j.table[2] = 0; j.table[3] = 0;
    }
    int4* entries = reinterpret_cast<int4*>(j.table + 4);
    for (int q = 0; q < per; ++q) {
        const int u = j.u_lo + lane * per + q;
        if (u >= j.u_hi) break;
        const int c = cnt[u], o = off[u];
        for (int r = 0; r < c; r += bm) {
            if (at < cap) entries[at] = make_int4(u, o + r, min(bm, c - r), 0);
            ++at;
        }
    }
}

// Wavefront w of a kernel that has the counts: table w, and behind the tables whether weights are streamed (STREAM: where they may be).
template <bool STREAM>
__device__ __forceinline__ void build_tables(const int* cnt, const int* off, const TileJobs& jobs, int w, int lane)
{
    if (w < jobs.n) {
        build_tile_table(cnt, off, jobs.job[w], jobs.cap, lane);
    } else if (STREAM && w == jobs.n && jobs.may_stream()) {
        int active = 0;
        for (int u = lane; u < jobs.count_units; u += 64) active += cnt[u] > 0;
        active = __builtin_amdgcn_readlane(wave_scan(active), 63);
        if (lane == 0) jobs.job[0].table[-1] = active >= jobs.stream_units;
    }
}

}  // namespace bmoe

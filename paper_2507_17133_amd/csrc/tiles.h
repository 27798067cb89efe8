// GEMM tile table, built on the device from the unit row counts (shared by the routing kernels, which know
// the counts first, and by the stand-alone table kernel used when the caller brings its own row lists).
//
// int32 header {n_tiles, rows of a tile, 0, 0}, then one int4 {unit, first row, rows, 0} per M tile, units in ascending
// order, tiles of a unit consecutive.
#pragma once
#include "internal.h"

namespace bmoe {

struct TileJob {
    int u_lo, u_hi;          // units [u_lo, u_hi)
    TilePlan plan;
    int32_t* table;
    int bm_hi;               // a taller tile that may suit a browned-out batch better (0: none): the table holds tiles of one
                             // of the two heights and says of which, the GEMM launch for the other one finds none
    int m, entries;          // bm_hi > 0: experts, TopK entries of the batch
};
struct TileJobs {
    int n;                   // 0, 1 or 2 jobs (routed + united units; shared units of another width)
    TileJob job[2];
    int cap;                 // entries a table holds
};

// Time of one GEMM tile of bm rows, in twentieths of a 32-row one (DeepSeek-V3 shape, tiles full: 20.6 and 14.7 ms for all
// of 16384 tokens at 64 and 128 rows, 10.4 at 256; 1021 tokens at 32 and 64 rows: 2.68 and 1.81).
__device__ __forceinline__ int tile_cost(int bm) { return bm == 256 ? 54 : bm == 128 ? 38 : bm == 64 ? 27 : 20; }

// One wavefront builds the table of one job.  cnt[u], off[u]: rows and first row of unit u (global or LDS).
// The tile height comes from the counts where the job leaves a choice: brownout takes the rows of unpopular experts away,
// and the few units that remain hold many times the T K / m the host can go by.  Taken only when entries have left their
// experts, so that a batch without brownout takes the same kernels whether or not its caller offers the choice.
__device__ __forceinline__ void build_tile_table(const int* cnt, const int* off, const TileJob& j, int cap, int lane)
{
    int bm = j.plan.bm;
    const int n_units = j.u_hi - j.u_lo;
    const int per = (n_units + 63) / 64;
    int local = 0;
    for (int q = 0; q < per; ++q) {
        const int u = j.u_lo + lane * per + q;
        if (u < j.u_hi) local += (cnt[u] + bm - 1) / bm;
    }
    if (j.bm_hi > 0) {
        int hi = 0, rows = 0;
        for (int q = 0; q < per; ++q) {
            const int u = j.u_lo + lane * per + q;
            if (u >= j.u_hi) break;
            hi += (cnt[u] + j.bm_hi - 1) / j.bm_hi;
            if (u < j.m) rows += cnt[u];
        }
        int n_lo = local, n_hi = hi;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            n_lo += __shfl_xor(n_lo, o);
            n_hi += __shfl_xor(n_hi, o);
            rows += __shfl_xor(rows, o);
        }
        const bool taller = rows < j.entries && (long)n_hi * tile_cost(j.bm_hi) <= (long)n_lo * tile_cost(bm);
        if (taller) {
            bm = j.bm_hi;
            local = hi;
        }
    }
    int incl = local;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    int at = incl - local;
    const int total = __shfl(incl, 63);
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

}  // namespace bmoe

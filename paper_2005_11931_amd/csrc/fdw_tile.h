// fdw_tile.h - the small-grid kernel's decomposition and launcher (fdw_tile.hip).
//
// One workgroup of `waves` waves per tile of kWaveSize columns (kTileCols owned) and
// kTileRowsPerWave * waves rows (kTileHalo halo rows above and below); the member table holds
// strips = tile columns, seg_rows = owned rows per tile, waves = blocks = tiles.  Time blocks
// 1..8.
#pragma once

#include "fdw_internal.h"

namespace fdw {

constexpr int kTileRowsPerWave = 4;
constexpr int kTileHalo = kMaxTimeBlock;
constexpr int kTileCols = kWaveSize - 2 * kTileHalo;
static_assert(stores_padding(kTileCols, 2), "the last tile stores the padding that is loaded (both types)");
constexpr int kMaxTileWaves = 16;
constexpr int kMaxAdjTileWaves = 12;  // 4-row waves of the reverse tile: 90 to 150 registers per lane, 168 at most

#ifdef __HIPCC__
// Receiver of every lane in RW rows g0.. of a wave (-1: none): the first of each run of coincident
// receivers, of rows [row_lo, row_hi) and columns [col_lo, col_hi); lane l holds column lane_col + l.
// slot: RW x 64 ints of the wave's own LDS.  Returns whether the rows hold any receiver
// (wave-uniform); rec is defined either way.  The receiver lists are sorted by (row, column).
template <int RW, typename M>
__device__ __forceinline__ bool tile_receivers(const M& m, int g0, int row_lo, int row_hi, int col_lo, int col_hi,
                                               int lane_col, int (*slot)[kWaveSize], int (&rec)[RW])
{
    typedef const __attribute__((address_space(4))) int* Table;
    const Table rowptr = (Table)m.rec_rowptr;
    const Table rcol = (Table)m.rec_col;
    const Table rid = (Table)m.rec_id;
    const int lane = threadIdx.x & (kWaveSize - 1);
#pragma unroll
    for (int i = 0; i < RW; ++i) rec[i] = -1;
    if (m.R <= 0 || row_lo >= row_hi || rowptr[row_lo] >= rowptr[row_hi]) return false;
#pragma unroll
    for (int i = 0; i < RW; ++i) slot[i][lane] = -1;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const int g = g0 + i;
        if (g < row_lo || g >= row_hi) continue;
        const int kb = rowptr[g], ke = rowptr[g + 1];
        for (int k0 = kb; k0 < ke; k0 += kWaveSize) {
            const int k = min(k0 + lane, ke - 1);
            const int col = rcol[k];
            const int prev = (k > kb) ? rcol[k - 1] : -1;
            const int id = rid[k];
            if (k0 + lane < ke && col >= col_lo && col < col_hi && prev != col) slot[i][col - lane_col] = id;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < RW; ++i) rec[i] = slot[i][lane];
    return true;
}
#endif

template <typename T>
hipError_t launch_step_tile(const StepArgs& a, int K, int face_mode, int waves, int grid, hipStream_t s);

// Reverse sweep of a small grid (fdw_adjoint_tile.hip): K <= kTileHalo levels per launch; a.strips
// tile columns, a.seg_rows owned rows per tile, a.waves tiles; no two receivers on one node.
template <typename T>
hipError_t launch_adjoint_tile(const AdjArgs& a, int K, int rows_per_wave, int waves, hipStream_t s);

}  // namespace fdw

// fdw_tile.hip - the leapfrog time block for small grids (Section 2, the explicit scheme of
// eq. (2.1) on the Section 3.3 grid; the same point update as the streaming kernel).
//
// On a grid of a few hundred nodes a side the streaming kernel has too few work items to fill
// the device, and each of them is a long serial chain: one wave walks S + 2K rows through K
// levels.  Here one workgroup owns a tile of 64 columns (48 owned, 8 halo columns on each
// side) and NW * 4 rows (8 halo rows above and below), held in registers: each wave keeps 4
// rows of (u, du) and their face coefficients, and the waves advance the tile level by level
// together, exchanging their edge rows through LDS with one barrier per level.  The halo is
// deep enough for any time block up to 8: after K levels the owned nodes are exact, and they
// are computed with the same operations in the same order as in the streaming kernel, so both
// kernels produce the same bits.  Energy partials: one per tile and level, summed over the
// tile's waves in a fixed order.  Receiver traces are stored from the registers as the levels
// pass (k_record_tile; 384^2 FP64, 64 receivers: 8.0 us per 8-step launch against 23 on the streaming
// kernel).
#include "fdw_stream.h"
#include "fdw_tile.h"

namespace fdw {

namespace {

// v from another lane of the same row of 16 lanes (DPP control CTRL; every source lane exists)
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}
// MODE bit 0: per-step energy partials; bit 1: receiver traces.  FACE: coefficient layout as in
// the streaming kernel.  The body of k_step_tile (MODE 0, 1) and k_record_tile (MODE 2, 3).
template <typename T, int FACE, int MODE>
__device__ __forceinline__ void tile_block(const StepArgs& a, int K)
{
    constexpr bool want_energy = (MODE & 1) != 0;
    constexpr bool want_trace = (MODE & 2) != 0;
    constexpr int RW = kTileRowsPerWave;
    __shared__ T s_edge[2][kMaxTileWaves][2][kWaveSize];  // first / last row of every wave, two levels
    __shared__ double s_e[kMaxTimeBlock][4 * kMaxTileWaves];  // energy of every level and row of 16 lanes

    const int NW = (int)(blockDim.x >> 6);
    const int w = wave_in_block();
    const int lane = threadIdx.x & 63;
    const int gb = (int)blockIdx.x + a.block_offset;
    const int eslot = a.eslot;
    const bool one = a.nmembers == 1;
    const int m = one ? a.first : find_member(a.table, a.first, a.nmembers, gb);
    const MemberDev M = member_copy(member_at(a.table, m, one, offsetof(StepArgs, one)));
    // Every field of the member the prologue needs is read here, before any of them is used, so
    // that all table reads are one round of scalar loads ahead of the plane loads (left to the
    // scheduler they were split into several dependent rounds around the index arithmetic).
    // Both pointers of each pair are read and then selected by the parity.  The grid holds
    // exactly the members' tiles: no tile test.
    const int nx = M.nx, ny = M.ny, ld = M.ld;
    const int strips = M.strips, seg_rows = M.seg_rows, block_base = M.block_base, cur0 = M.cur0;
    void* const u0p = M.u[0];
    void* const u1p = M.u[1];
    void* const d0p = M.d[0];
    void* const d1p = M.d[1];
    void* const hv = M.h;
    void* const hyv = M.hy;
    const double axd = M.ax, ayd = M.ay;
    __builtin_amdgcn_sched_barrier(0);
    const int tile = gb - block_base;

    const int strip = tile % strips;
    const int seg = tile / strips;
    const int cb = strip * kTileCols - kTileHalo + lane;  // grid column of this lane
    // Lanes that start past the grid take 0 whatever the padding holds (checkpoint slots are not cleared);
    // the up to three columns that share a lane vector with the last one are stored (as 0) and loaded.
    const bool lane_live = (cb >= 0) && (cb < nx);
    const bool lane_owned = (cb >= 0) && (cb < ((nx + 3) & ~3)) && (lane >= kTileHalo) && (lane < kTileHalo + kTileCols);
    const T colm = ((cb >= 1) && (cb <= nx - 2)) ? T(1) : T(0);
    const int r0 = seg * seg_rows;
    const int r1 = min(r0 + seg_rows, ny);
    const int g0 = r0 - kTileHalo + w * RW;  // grid row of the wave's first row

    const bool cur = ((cur0 ^ a.parity) & 1) != 0;
    const T* __restrict__ uin = (const T*)(cur ? u1p : u0p);
    const T* __restrict__ din = (const T*)(cur ? d1p : d0p);
    T* __restrict__ uout = (T*)(cur ? u0p : u1p);
    T* __restrict__ dout = (T*)(cur ? d0p : d1p);
    const T* __restrict__ hp = (const T*)hv;
    const T* __restrict__ hyp = (const T*)hyv;
    const T ax = (T)axd, ay = (T)ayd;

    // Rows and columns outside the plane read as 0, as in the streaming kernel: the loads go
    // through buffer resources, whose out-of-range offsets return 0 in hardware.  (A load under
    // a lane test compiles to a branch around it and a wait right after it: fourteen
    // serialised memory latencies before the first level.)  The resources start at the first
    // row the tile reads, so that every offset stays far below 2^31.
    const int jbase = max(r0 - kTileHalo - 1, 0);
    const size_t span = (size_t)(ny - jbase) * ld * sizeof(T);
    const unsigned int nbytes =
        __builtin_amdgcn_readfirstlane((unsigned int)min(span, (size_t)kBufferOutOfRange - 16));
    const size_t base_el = (size_t)jbase * ld;
    const __amdgpu_buffer_rsrc_t ru = plane_rsrc(uniform_ptr(uin + base_el), nbytes);
    const __amdgpu_buffer_rsrc_t rd = plane_rsrc(uniform_ptr(din + base_el), nbytes);
    const __amdgpu_buffer_rsrc_t rh = plane_rsrc(uniform_ptr(hp + base_el), nbytes);
    const __amdgpu_buffer_rsrc_t rhy = plane_rsrc(uniform_ptr((FACE ? hyp : hp) + base_el), nbytes);
    auto at = [&](__amdgpu_buffer_rsrc_t r, int g) -> T {
        const unsigned int off = (lane_live && g >= 0 && g < ny)
                                     ? (unsigned int)((g - jbase) * ld + cb) * (unsigned int)sizeof(T)
                                     : kBufferOutOfRange;
        if constexpr (sizeof(T) == 8) {
            return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
        } else {
            return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
        }
    };

    T u[RW], d[RW], FX[RW], FY[RW];  // FY[i]: face between rows i and i + 1 of the wave
    T FYup;                          // face between the row above the wave and its first row
    if (FACE) {
        // face sums: FX = h1_c + h1_{c+1} in h, FY = h2_r + h2_{r+1} in hy (stored at row r)
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            u[i] = at(ru, g0 + i);
            d[i] = at(rd, g0 + i);
            FX[i] = ax * at(rh, g0 + i);
            FY[i] = ay * at(rhy, g0 + i);
        }
        FYup = ay * at(rhy, g0 - 1);
    } else {
        T hr[RW + 2];  // nodal h of rows g0 - 1 .. g0 + RW
#pragma unroll
        for (int j = 0; j < RW + 2; ++j) hr[j] = at(rh, g0 - 1 + j);
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            u[i] = at(ru, g0 + i);
            d[i] = at(rd, g0 + i);
            FX[i] = ax * (hr[i + 1] + lane_from_right(hr[i + 1]));
            FY[i] = ay * (hr[i + 1] + hr[i + 2]);
        }
        FYup = ay * (hr[0] + hr[1]);
    }

    // Receivers in the wave's owned rows and columns (the first of each run of coincident ones), one
    // id per lane and row, found once per launch while the plane loads are in flight; the level
    // loop then stores, and waits for nothing.
    int rec[RW];
    bool wave_rec = false;
    if constexpr (want_trace) {
        __shared__ int s_slot[kMaxTileWaves][RW][kWaveSize];
        wave_rec = tile_receivers<RW>(M, g0, max(g0, r0), min(g0 + RW, r1), strip * kTileCols,
                                      strip * kTileCols + kTileCols, strip * kTileCols - kTileHalo, s_slot[w], rec);
    }
    GlobalPtr<T> const trace_out = want_trace ? (GlobalPtr<T>)uniform_ptr((T*)M.traces) : nullptr;
    const int64_t trace_row0 = want_trace ? a.ctx_step + M.n_offset + 1 : 0;

    // The halo rows are whole waves (kTileHalo is a multiple of the rows per wave), and rows past the
    // grid hold zeros, which add nothing: a wave's energy terms count or not as a whole.  (A test
    // per row was a branch in every row of every level.)
    static_assert(kTileHalo % RW == 0, "halo rows are whole waves");
    const bool wave_owned = w >= kTileHalo / RW && w < NW - kTileHalo / RW;
    // per-lane energy terms of every level, reduced over the wave once after the last level
    // (the K reductions are then independent and their lane exchanges overlap; reduced level
    // by level they would put six dependent exchanges into every level's critical path)
    double acc[kMaxTimeBlock];
#pragma unroll
    for (int t = 0; t < kMaxTimeBlock; ++t) acc[t] = 0.0;

#pragma unroll
    for (int t = 0; t < kMaxTimeBlock; ++t) {
        if (t >= K) break;
        const int b = t & 1;
        s_edge[b][w][0][lane] = u[0];
        s_edge[b][w][1][lane] = u[RW - 1];
        __syncthreads();
        // the tile's first and last rows see 0 beyond them: only halo rows are affected
        const T above = (w > 0) ? s_edge[b][w - 1][1][lane] : T(0);
        const T below = (w < NW - 1) ? s_edge[b][w + 1][0][lane] : T(0);
        // y flux across the face above each row, carried from row to row:
        // sy = fy_{r+1/2}(u_{r+1} - u_r) - fy_{r-1/2}(u_r - u_{r-1})
        T Gp = FYup * (u[0] - above);
        T eb = T(0);
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const T un = (i < RW - 1) ? u[i + 1] : below;
            const T Gn = FY[i] * (un - u[i]);
            const T F = FX[i] * (lane_from_right(u[i]) - u[i]);
            const T Fl = lane_from_left(F);
            const T sx = F - Fl;
            const T sy = Gn - Gp;
            Gp = Gn;
            const T L = sx + sy;
            const int g = g0 + i;
            T nd = fma_t(L, colm, d[i]);
            if (!((g >= 1) && (g <= ny - 2))) nd = T(0);  // Dirichlet rows (and rows outside the grid)
            const T nu = u[i] + nd;
            if (want_energy) {
                eb = fma_t(nd, nd, eb);
                eb = fma_t(-nu, L, eb);
            }
            u[i] = nu;
            d[i] = nd;
        }
        if constexpr (want_trace) {
            if (wave_rec && trace_row0 + t < M.trace_rows) {
#pragma unroll
                for (int i = 0; i < RW; ++i)
                    if (rec[i] >= 0) trace_out[(trace_row0 + t) * M.R + rec[i]] = u[i];
            }
        }
        if (want_energy) acc[t] = (lane_owned && wave_owned) ? (double)eb : 0.0;
    }

#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const int g = g0 + i;
        if (g >= r0 && g < r1 && lane_owned) {
            const size_t off = (size_t)g * ld + cb;
            uout[off] = u[i];
            dout[off] = d[i];
        }
    }

    if (want_energy) {
        // Sums over lanes, the eight levels together: three exchanges within eight lanes (partner 7 - l,
        // l ^ 2, l ^ 1), each lane passing on the half of its levels that its partner keeps, leave lane l
        // with level l & 7 of its eight lanes; one more adds the other half of the row of 16.
        // (Level by level, each over the whole wave, this took 224 instructions instead of 60; with the
        // test-free energy terms above, 256^2 FP64 with energies 1.06 -> 0.97 us per step.)
        static_assert(kMaxTimeBlock == 8 && kWaveSize == 64, "eight levels over rows of sixteen lanes");
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double keep = (lane & 4) ? acc[j + 4] : acc[j];
            const double pass = (lane & 4) ? acc[j] : acc[j + 4];
            acc[j] = keep + dpp_f64<0x141>(pass);  // row_half_mirror
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const double keep = (lane & 2) ? acc[j + 2] : acc[j];
            const double pass = (lane & 2) ? acc[j] : acc[j + 2];
            acc[j] = keep + dpp_f64<0x4E>(pass);  // quad_perm [2, 3, 0, 1]
        }
        const double keep = (lane & 1) ? acc[1] : acc[0];
        const double pass = (lane & 1) ? acc[0] : acc[1];
        double v = keep + dpp_f64<0xB1>(pass);  // quad_perm [1, 0, 3, 2]
        v += dpp_f64<0x128>(v);                 // row_ror:8
        if ((lane & 8) == 0) s_e[lane & 7][w * 4 + (lane >> 4)] = v;
        __syncthreads();
        // wave 0: lane (level, group) adds every eighth of the 4 NW row sums, then the groups are added
        if (w == 0) {
            const int t = lane & 7;
            double s = 0.0;
            for (int k = lane >> 3; k < 4 * NW; k += 8) s += s_e[t][k];
            s += __shfl_xor(s, 8, 64);
            s += __shfl_xor(s, 16, 64);
            s += __shfl_xor(s, 32, 64);
            if (lane < K) M.epart[((size_t)eslot * kMaxTimeBlock + lane) * M.epart_stride + tile] = s;
        }
    }
}

template <typename T, int FACE, int MODE>
__global__ __launch_bounds__(kWaveSize * kMaxTileWaves) void k_step_tile(StepArgs a, int K)
{
    tile_block<T, FACE, MODE>(a, K);
}
template <typename T, int FACE, int MODE>
__global__ __launch_bounds__(kWaveSize * kMaxTileWaves) void k_record_tile(StepArgs a, int K)
{
    tile_block<T, FACE, MODE>(a, K);
}

template <typename T, int FACE>
hipError_t launch_tile_f(const StepArgs& a, int K, int waves, int grid, hipStream_t s)
{
    const dim3 g(grid), b(kWaveSize * waves);
    if (a.want_trace && a.want_energy)
        hipLaunchKernelGGL((k_record_tile<T, FACE, 3>), g, b, 0, s, a, K);
    else if (a.want_trace)
        hipLaunchKernelGGL((k_record_tile<T, FACE, 2>), g, b, 0, s, a, K);
    else if (a.want_energy)
        hipLaunchKernelGGL((k_step_tile<T, FACE, 1>), g, b, 0, s, a, K);
    else
        hipLaunchKernelGGL((k_step_tile<T, FACE, 0>), g, b, 0, s, a, K);
    return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_step_tile(const StepArgs& a, int K, int face_mode, int waves, int grid, hipStream_t s)
{
    if (K < 1 || K > kMaxTimeBlock || waves < 1 || waves > kMaxTileWaves) return hipErrorInvalidValue;
    return face_mode == 1 ? launch_tile_f<T, 1>(a, K, waves, grid, s) : launch_tile_f<T, 0>(a, K, waves, grid, s);
}
template hipError_t launch_step_tile<float>(const StepArgs&, int, int, int, int, hipStream_t);
template hipError_t launch_step_tile<double>(const StepArgs&, int, int, int, int, hipStream_t);

}  // namespace fdw

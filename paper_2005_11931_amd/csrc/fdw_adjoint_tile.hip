// fdw_adjoint_tile.hip - the reverse (adjoint) sweep for small grids (the discrete adjoint of the
// scheme of Section 2 eq. (2.1); see fdw_adjoint.hip for the recurrences).
//
// On a grid of a few hundred nodes a side the streaming reverse kernel has one or two hundred work
// items, each a wave that walks tens of rows through six levels in sequence: 42 us per launch of
// 6 levels at 384^2 FP64 whatever the grid.  Here, as in the forward tile kernel, one workgroup owns a
// tile of 64 columns (48 owned) and 4 rows per wave (8 halo rows above and below), holds
// (u, du, lambda, mu), the scaled faces and the face products in registers, and advances it up
// to 8 levels with one barrier per level.  A launch then costs the latency of its loads, its
// levels and its stores: 12.2 us per launch of 8 levels at 384^2 FP64 (about 4.5 us of it the levels: two
// waves per SIMD x 4 rows x 30 FP64 instructions, an LDS exchange and a barrier per level).  Whole
// gradients (traced forward and reverse sweep, 500 steps, 384^2 FP64): 5.4 -> 1.44 ms.
//
// The states take the same operations in the same order as in the streaming kernel (same bits).
// The gradient is accumulated per face, S = sum over the levels of w (difference of u)(difference of
// lambda) - one fused multiply-add per face and level - and turned into nodal values once per
// launch: dJ/dh1 += -ax (S_{c+1/2} + S_{c-1/2}), dJ/dh2 likewise in y.
#include "fdw_stream.h"
#include "fdw_tile.h"

#include <hip/hip_runtime.h>

#include <algorithm>

namespace fdw {

namespace {

template <typename T, int RW, int FACE, int SPLIT>
__global__ __launch_bounds__(kWaveSize * (RW == 4 ? kMaxAdjTileWaves : 8)) void k_adjoint_tile(AdjArgs a, int K)
{
    // per wave: two levels x (first and last row of u and of lambda)
    extern __shared__ __align__(16) unsigned char smem[];
    typedef T EdgeRows[4][kWaveSize];
    const int NW = (int)(blockDim.x >> 6);
    EdgeRows* const edge = reinterpret_cast<EdgeRows*>(smem);  // [2][NW]

    const int w = wave_in_block();
    const int lane = threadIdx.x & 63;
    const int tile = (int)blockIdx.x;
    const int nx = a.nx, ny = a.ny, ld = a.ld;
    const int strip = tile % a.strips;
    const int seg = tile / a.strips;
    const int cb = strip * kTileCols - kTileHalo + lane;
    // Lanes that start past the grid take 0 whatever the padding holds (checkpoint slots are not cleared);
    // the up to three columns that share a lane vector with the last one are stored (as 0) and loaded.
    const bool lane_live = (cb >= 0) && (cb < nx);
    const bool lane_owned = (cb >= 0) && (cb < ((nx + 3) & ~3)) && (lane >= kTileHalo) && (lane < kTileHalo + kTileCols);
    const T colm = ((cb >= 1) && (cb <= nx - 2)) ? T(1) : T(0);
    const int r0 = seg * a.seg_rows;
    const int r1 = min(r0 + a.seg_rows, ny);
    const int g0 = r0 - kTileHalo + w * RW;  // grid row of the wave's first row
    const T ax = (T)a.ax, ay = (T)a.ay;
    constexpr bool split = SPLIT != 0;

    // plane reads through buffer resources (rows and columns outside the plane read 0), starting
    // at the first row the tile reads
    const int jbase = max(r0 - kTileHalo - 1, 0);
    const size_t base_el = (size_t)jbase * ld;
    const size_t span = (size_t)(ny - jbase) * ld * sizeof(T);
    const unsigned int nbytes = (unsigned int)min(span, (size_t)kBufferOutOfRange - 16);
    const __amdgpu_buffer_rsrc_t ru = plane_rsrc((const T*)a.uin + base_el, nbytes);
    const __amdgpu_buffer_rsrc_t rd = plane_rsrc((const T*)a.din + base_el, nbytes);
    const __amdgpu_buffer_rsrc_t rl = plane_rsrc((const T*)a.lin + base_el, nbytes);
    const __amdgpu_buffer_rsrc_t rm = plane_rsrc((const T*)a.min + base_el, nbytes);
    const __amdgpu_buffer_rsrc_t rh = plane_rsrc((const T*)a.h + base_el, nbytes);
    const __amdgpu_buffer_rsrc_t rhy = plane_rsrc((const T*)(FACE ? a.hy : a.h) + base_el, nbytes);
    const size_t gspan = (size_t)(ny - jbase) * ld * sizeof(double);
    const unsigned int gbytes = (unsigned int)min(gspan, (size_t)kBufferOutOfRange - 16);
    const __amdgpu_buffer_rsrc_t rg1 = plane_rsrc(a.g1 + base_el, gbytes);
    const __amdgpu_buffer_rsrc_t rg2 = plane_rsrc(a.g2 + base_el, gbytes);
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
    auto at_g = [&](__amdgpu_buffer_rsrc_t r, int g) -> double {
        const unsigned int off = (lane_owned && g >= r0 && g < r1)
                                     ? (unsigned int)((g - jbase) * ld + cb) * (unsigned int)sizeof(double)
                                     : kBufferOutOfRange;
        return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
    };

    T u[RW], d[RW], l[RW], m[RW], FX[RW], FY[RW];  // FY[i]: face between rows i and i + 1 of the wave
    T FYup;                                        // face between the row above the wave and its first row
    if (FACE) {
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            FX[i] = ax * at(rh, g0 + i);
            FY[i] = ay * at(rhy, g0 + i);
        }
        FYup = ay * at(rhy, g0 - 1);
    } else {
        T hr[RW + 2];
#pragma unroll
        for (int j = 0; j < RW + 2; ++j) hr[j] = at(rh, g0 - 1 + j);
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            FX[i] = ax * (hr[i + 1] + lane_from_right(hr[i + 1]));
            FY[i] = ay * (hr[i + 1] + hr[i + 2]);
        }
        FYup = ay * (hr[0] + hr[1]);
    }
    // Accumulator rows: requested with the states, except eight rows of doubles, which do not fit the 256
    // registers of two waves per SIMD through the levels (10 registers spilled, 26 with separate gradients;
    // 400 reverse steps at 700^2: 1.29 -> 1.23 ms, separate gradients 1.51 -> 1.31; 1000^2: 2.28 -> 2.21 and
    // 2.70 -> 2.40).
    constexpr bool late_g = sizeof(T) == 8 && RW == 8;
    double g1[RW], g2[RW];
    auto load_g = [&](int i) {
        g1[i] = at_g(rg1, g0 + i);
        g2[i] = split ? at_g(rg2, g0 + i) : 0.0;
    };
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        u[i] = at(ru, g0 + i);
        d[i] = at(rd, g0 + i);
        l[i] = at(rl, g0 + i);
        m[i] = at(rm, g0 + i);
        if constexpr (!late_g) load_g(i);
    }
    // adjoint sources: every copy of a receiver node (halo included) takes its source, requested one
    // level ahead; no two receivers share a node here.  Lanes without one load 0 (out of range).
    int rec[RW];
    const int col0 = strip * kTileCols - kTileHalo;
    const bool wave_rec = tile_receivers<RW>(a, g0, max(g0, 1), min(g0 + RW, ny - 1), col0, col0 + kWaveSize, col0,
                                             (int (*)[kWaveSize])(smem + (size_t)w * RW * kWaveSize * sizeof(int)), rec);
    __syncthreads();  // the slots share LDS with the edge rows
    unsigned int src_off[RW];
    double src[RW];
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        src_off[i] = (rec[i] >= 0) ? (unsigned int)rec[i] * (unsigned int)sizeof(double) : kBufferOutOfRange;
        src[i] = 0.0;
    }
    auto load_source = [&](int64_t n, int i) {
        const __amdgpu_buffer_rsrc_t rs =
            plane_rsrc(a.trace_grad + max(n, (int64_t)0) * a.R, (unsigned int)a.R * (unsigned int)sizeof(double));
        src[i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)src_off[i], 0, 0));
    };
    if (wave_rec) {
#pragma unroll
        for (int i = 0; i < RW; ++i) load_source(a.n_top - 1, i);
    }

    double SX[RW], SY[RW];
#pragma unroll
    for (int i = 0; i < RW; ++i) SX[i] = SY[i] = 0.0;

    for (int t = 0; t < K; ++t) {
        const int64_t n = a.n_top - 1 - t;  // time of this level's forward state
        EdgeRows* const eb = edge + (t & 1) * NW;
        // u^n = u^{n+1} - du^{n+1}
#pragma unroll
        for (int i = 0; i < RW; ++i) u[i] = fma_t(-d[i], colm, u[i]);
        eb[w][0][lane] = u[0];
        eb[w][1][lane] = u[RW - 1];
        eb[w][2][lane] = l[0];
        eb[w][3][lane] = l[RW - 1];
        __syncthreads();
        const T uab = (w > 0) ? eb[w - 1][1][lane] : T(0);
        const T ube = (w < NW - 1) ? eb[w + 1][0][lane] : T(0);
        const T lab = (w > 0) ? eb[w - 1][3][lane] : T(0);
        const T lbe = (w < NW - 1) ? eb[w + 1][2][lane] : T(0);
        // the start step's term (n = 0, the last level of all) counts half: the sums so far are
        // doubled before it and everything halved after it (both exact)
        if (n == 0) {
#pragma unroll
            for (int i = 0; i < RW; ++i) SX[i] *= 2.0, SY[i] *= 2.0;
        }
        T Gu = FYup * (u[0] - uab);
        T Gl = FYup * (l[0] - lab);
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const T duy = ((i < RW - 1) ? u[i + 1] : ube) - u[i];
            const T dly = ((i < RW - 1) ? l[i + 1] : lbe) - l[i];
            const T dux = lane_from_right(u[i]) - u[i];
            const T dlx = lane_from_right(l[i]) - l[i];
            const T Gun = FY[i] * duy;
            const T Gln = FY[i] * dly;
            const T Fu = FX[i] * dux;
            const T Fl = FX[i] * dlx;
            SX[i] = __builtin_fma((double)dux, (double)dlx, SX[i]);
            SY[i] = __builtin_fma((double)duy, (double)dly, SY[i]);
            const T Lu = (Fu - lane_from_left(Fu)) + (Gun - Gu);
            const T Ll = (Fl - lane_from_left(Fl)) + (Gln - Gl);
            Gu = Gun;
            Gl = Gln;
            const int g = g0 + i;
            T nd = fma_t(-Lu, colm, d[i]);
            T nm = fma_t(Ll, colm, m[i]);
            if (!((g >= 1) && (g <= ny - 2))) nd = nm = T(0);  // Dirichlet rows (and rows outside the grid)
            if (wave_rec) {
                nm += (T)src[i];
                load_source(n - 1, i);
            }
            d[i] = nd;
            m[i] = nm;
            l[i] = fma_t(nm, colm, l[i]);
        }
        if (n == 0) {
#pragma unroll
            for (int i = 0; i < RW; ++i) SX[i] *= 0.5, SY[i] *= 0.5;
        }
    }

    if constexpr (late_g) {
#pragma unroll
        for (int i = 0; i < RW; ++i) load_g(i);
    }
    // y face sums of the row above each wave
    __syncthreads();
    double* const s_y = reinterpret_cast<double*>(smem);  // [NW][64]
    s_y[w * kWaveSize + lane] = SY[RW - 1];
    __syncthreads();
    double Sup = (w > 0) ? s_y[(w - 1) * kWaveSize + lane] : 0.0;
    T* const uout = (T*)a.uout;
    T* const dout = (T*)a.dout;
    T* const lout = (T*)a.lout;
    T* const mout = (T*)a.mout;
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const int g = g0 + i;
        const double gx = SX[i] + lane_from_left(SX[i]);
        const double gy = SY[i] + Sup;
        Sup = SY[i];
        if (g >= r0 && g < r1 && lane_owned) {
            const size_t off = (size_t)g * ld + cb;
            uout[off] = u[i];
            dout[off] = d[i];
            lout[off] = l[i];
            mout[off] = m[i];
            if (split) {
                a.g1[off] = __builtin_fma(-a.ax, gx, g1[i]);
                a.g2[off] = __builtin_fma(-a.ay, gy, g2[i]);
            } else {
                a.g1[off] = g1[i] + __builtin_fma(-a.ay, gy, -a.ax * gx);
            }
        }
    }
}

template <typename T, int FACE, int SPLIT>
hipError_t launch_fs(const AdjArgs& a, int K, int rw, int waves, hipStream_t s)
{
    const int need = waves * kWaveSize * std::max(2 * 4 * (int)sizeof(T), std::max(rw * (int)sizeof(int), (int)sizeof(double)));
    if (rw == 8)
        hipLaunchKernelGGL((k_adjoint_tile<T, 8, FACE, SPLIT>), dim3(a.waves), dim3(kWaveSize * waves), (size_t)need, s, a, K);
    else
        hipLaunchKernelGGL((k_adjoint_tile<T, 4, FACE, SPLIT>), dim3(a.waves), dim3(kWaveSize * waves), (size_t)need, s, a, K);
    return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_adjoint_tile(const AdjArgs& a, int K, int rw, int waves, hipStream_t s)
{
    if (K < 1 || K > kTileHalo || (rw != 4 && rw != 8) || waves < 1 || waves > (rw == 4 ? kMaxAdjTileWaves : 8)) return hipErrorInvalidValue;
    const bool split = a.g2 != a.g1;
    if (a.face) return split ? launch_fs<T, 1, 1>(a, K, rw, waves, s) : launch_fs<T, 1, 0>(a, K, rw, waves, s);
    return split ? launch_fs<T, 0, 1>(a, K, rw, waves, s) : launch_fs<T, 0, 0>(a, K, rw, waves, s);
}
template hipError_t launch_adjoint_tile<float>(const AdjArgs&, int, int, int, hipStream_t);
template hipError_t launch_adjoint_tile<double>(const AdjArgs&, int, int, int, hipStream_t);

}  // namespace fdw

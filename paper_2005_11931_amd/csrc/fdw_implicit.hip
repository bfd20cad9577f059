// fdw_implicit.hip - the implicit scheme of the paper's 2D experiment (Section 3.3: an implicit
// finite-difference scheme whose linear systems are solved by cyclic reduction; Section 4,
// Table 1 times it on a GPU), for gfx950.
//
// Scheme (factorized, alternating-direction form; L1 = d_x(h1 d_x .), L2 = d_y(h2 d_y .) with the
// face coefficients of the explicit solver):
//     (I - s tau^2 L1)(I - s tau^2 L2) w^n = tau^2 (L1 + L2) u^n,
//     du^{n+1} = du^n + w^n,  u^{n+1} = u^n + du^{n+1}    (i.e. u^{n+1} - 2u^n + u^{n-1} = w^n),
// start du^1 = tau u1 + w^0 / 2.  One step is two kernels on grids of up to 1024 rows, four beyond:
//   1. x lines (k_adi_x): the right-hand side tau^2 A u is formed from three rows of u and the row's
//      tridiagonal system (I - s tau^2 L1) z = r is solved, one workgroup per grid row;
//   2. y lines and the update: the columns of z are solved where they lie, without a
//      transposition, and w is added into (du, u) as it is found: one workgroup per strip of whole
//      columns (k_adi_y_strip), or blocks of rows joined by a small system per column
//      (k_adi_y_reduce, k_adi_y_join, k_adi_y_block).
// The line systems are symmetric and strictly diagonally dominant (1 + s tau^2 (f_l + f_r)/d^2 on
// the diagonal against s tau^2 f/d^2 off it), so eliminating needs no pivoting.
//
// What a step moves: x lines read u, hx, hy and write z; y lines read z, hy, u, du and write u, du
// (z and hy twice in blocks): 10 to 12 words per node against 14 when z was transposed, solved,
// transposed back and added by kernels of their own.  Measured per step (before -> now): 256^2 FP64
// 32.4 -> 9.6 us (two latency chains instead of four), 1000 x 1500 FP32 54.7 -> 25.1,
// 1024^2 FP64 60 -> 25.8, 2048^2 FP64 114 -> 79, 4096^2 FP64 448 -> 314, FP32 243 -> 153.
#include "../../include/fdw.h"
#include "fdw_internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

namespace {

// longest line (interior unknowns): in FP64 544 chunks of 8, in FP32 528 chunks of 16 (launch_x)
template <typename T>
constexpr int max_line_unknowns() { return sizeof(T) == 8 ? 4352 : 8448; }
constexpr int kMaxXThreads = 576;  // threads of an x-line workgroup, at most
constexpr int kStripUnknowns = 1024;            // y lines up to here: one kernel (see launch_y)
constexpr int kBlockChunk = 8, kBlockChunks = 8;  // beyond: blocks of 8 chunks of 8 rows
constexpr size_t kAdiAlign = 256;
inline size_t adi_align(size_t v) { return (v + kAdiAlign - 1) / kAdiAlign * kAdiAlign; }
inline int pad64(int n) { return (n + 63) / 64 * 64; }

// ------------------------------------------------------------------------------------------
// Line systems: a_k z_{k-1} + b_k z_k + c_k z_{k+1} = d_k, k = 0..n-1 (unknowns at the interior nodes
// i = k + 1), a_k = -g F_k, c_k = -g F_{k+1}, b_k = 1 + g (F_k + F_{k+1}), F_k the face between
// nodes k and k + 1.  Partition method: a line is split into P chunks of MT unknowns, one per
// thread (the last one padded with identity rows), lo the first unknown of a chunk.
//   1. Downward over rows lo+1 .. lo+MT-1 with z_lo kept as a parameter:
//      z_k = d'_k - a'_k z_lo - c'_k z_{k+1}; carried along, z_{lo+1} = al - be z_lo - ga z_{k+1}.
//   2. Row lo, with z_{lo+1} from its own chunk and z_{lo-1} from the last row of the chunk
//      above, couples z_lo to the first unknowns of the two neighbouring chunks only: a
//      tridiagonal system of P unknowns, one per thread, solved by parallel cyclic reduction in
//      LDS (rows kept with unit diagonal: one division and one barrier per level, every thread
//      busy at every level).
//   3. Upward: the chunk's other unknowns from z_lo and the next chunk's first unknown.
// One division per row, three arrays of MT values per thread (the faces' registers take c').
// Eliminating without pivoting is safe: the systems are strictly diagonally dominant, and so are
// their Schur complements.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// The eliminated rows of a chunk (or of a block of chunks) of unknowns lo .. hi, hi + 1 the first
// unknown of the next one: a0 z_{lo-1} + b0 z_lo + c0 z_{hi+1} = d0, and its last unknown
// z_hi = hd - ha z_lo - hc z_{hi+1}.
template <typename T>
struct Ends {
    T a0, b0, c0, d0, ha, hc, hd;
};

template <typename T, int MT>
struct Chunk {
    T d[MT];       // right-hand sides -> d'
    T f[MT + 1];   // faces F_lo .. F_{lo+MT} -> c' at 1 .. MT-1
    T ap[MT];      // a'

    __device__ __forceinline__ Ends<T> down(int lo, int n, T g)
    {
        T a0, b0, c0, d0;
        // identity rows past the line: no coupling, right-hand side 0
        const T g0 = (lo < n) ? g : T(0);
        a0 = -g0 * f[0];
        b0 = fma_t(g0, f[0] + f[1], T(1));
        c0 = -g0 * f[1];
        d0 = d[0];
        T al, be, ga;
        {
            const T gj = (lo + 1 < n) ? g : T(0);
            const T rr = T(1) / fma_t(gj, f[1] + f[2], T(1));
            al = d[1] = d[1] * rr;
            be = ap[1] = -gj * f[1] * rr;
            ga = f[1] = -gj * f[2] * rr;
        }
#pragma unroll
        for (int j = 2; j < MT; ++j) {
            const T gj = (lo + j < n) ? g : T(0);
            const T a = -gj * f[j];
            const T b = fma_t(gj, f[j] + f[j + 1], T(1));
            const T rr = T(1) / fma_t(-a, f[j - 1], b);
            d[j] = fma_t(-a, d[j - 1], d[j]) * rr;
            ap[j] = -(a * ap[j - 1]) * rr;
            f[j] = -gj * f[j + 1] * rr;
            al = fma_t(-ga, d[j], al);
            be = fma_t(-ga, ap[j], be);
            ga = -(ga * f[j]);
        }
        d0 = fma_t(-c0, al, d0);
        b0 = fma_t(-c0, be, b0);
        c0 = -(c0 * ga);
        return {a0, b0, c0, d0, ap[MT - 1], f[MT - 1], d[MT - 1]};
    }
    // the chunk's solution into d, from its first unknown and the next chunk's first one
    __device__ __forceinline__ void up(T zlo, T znext)
    {
        T z = znext;
#pragma unroll
        for (int j = MT - 1; j >= 1; --j) {
            z = fma_t(-f[j], z, fma_t(-ap[j], zlo, d[j]));
            d[j] = z;
        }
        d[0] = zlo;
    }
};

// First unknown of every chunk: `slots` threads of the workgroup call this with their chunk's
// eliminated row (Chunk::down); thread slot t = p * CW + column holds chunk p of one of CW
// systems, P chunks each.  lds: 6 * slots elements.  Returns z_lo; *znext = z_lo of chunk p + 1.
template <typename T>
__device__ __forceinline__ T solve_firsts(const Ends<T>& k, T* lds, int slots, int t, int p, int P, int CW, T* znext)
{
    T* const A0 = lds;
    T* const C0 = A0 + slots;
    T* const D0 = C0 + slots;
    T* const A1 = D0 + slots;
    T* const C1 = A1 + slots;
    T* const D1 = C1 + slots;
    // last row of each chunk, for the chunk below it
    A1[t] = k.ha;
    C1[t] = k.hc;
    D1[t] = k.hd;
    __syncthreads();
    T a, c, d;
    {
        T ha = T(0), hc = T(0), hd = T(0);
        if (p > 0) ha = A1[t - CW], hc = C1[t - CW], hd = D1[t - CW];
        const T rr = T(1) / fma_t(-k.a0, hc, k.b0);
        a = -(k.a0 * ha) * rr;
        c = k.c0 * rr;
        d = fma_t(-k.a0, hd, k.d0) * rr;
    }
    T *ra = A0, *rc = C0, *rd = D0, *wa = A1, *wc = C1, *wd = D1;
    ra[t] = a;
    rc[t] = c;
    rd[t] = d;
    for (int s = 1; s < P; s *= 2) {
        __syncthreads();
        T am = T(0), cm = T(0), dm = T(0), an = T(0), cn = T(0), dn = T(0);
        if (p >= s) am = ra[t - s * CW], cm = rc[t - s * CW], dm = rd[t - s * CW];
        if (p + s < P) an = ra[t + s * CW], cn = rc[t + s * CW], dn = rd[t + s * CW];
        const T rr = T(1) / fma_t(-c, an, fma_t(-a, cm, T(1)));
        d = fma_t(-c, dn, fma_t(-a, dm, d)) * rr;
        a = -(a * am) * rr;
        c = -(c * cn) * rr;
        wa[t] = a;
        wc[t] = c;
        wd[t] = d;
        T* q;
        q = ra, ra = wa, wa = q;
        q = rc, rc = wc, wc = q;
        q = rd, rd = wd, wd = q;
    }
    __syncthreads();
    *znext = (p + 1 < P) ? rd[t + CW] : T(0);
    return d;
}

struct LineArgs {
    int nx, ny;  // nodes
    int ld;      // pitch of every plane
    int P;       // chunks per line
    int cw;      // y lines: columns per workgroup
    double g;    // s tau^2 / d^2 along the line
    const void* u;
    const void* hx;
    const void* hy;
    void* z;
    double idx2, idy2;  // 1 / dx^2, 1 / dy^2
    double tt;          // tau^2
    // y lines: the update
    void* du;
    void* uo;
    const void* u0;
    const void* u1;
    double tau;
    // y lines in blocks of rows: end rows [7][blocks][ld], first unknowns [blocks][ld]
    void* ends;
    void* firsts;
};

// Workgroups are dispatched round-robin over the 8 XCDs: give each XCD a contiguous range of
// strips, so that the strips sharing the cache lines of a row go through one L2
__device__ __forceinline__ int xcd_block(int b, int nb)
{
    const int xcd = b & 7, per = nb >> 3, rem = nb & 7;
    return xcd * per + min(xcd, rem) + (b >> 3);
}

// LDS index of element k of a staged line: one pad slot per chunk of MT elements, so that
// threads reading the elements of their own chunks spread over the banks
template <int MT>
__device__ __host__ constexpr int lds_pad(int k)
{
    return k + k / MT;
}

// Short chunks (short lines) keep the right-hand sides, the faces and (MT = 4) the reduced system
// in LDS regions of their own, which saves two or three barriers of the latency-bound small grids;
// long ones pass them through one region in turn, so that more workgroups fit on a CU.
template <int MT>
constexpr int x_lds_regions() { return MT == 4 ? 3 : MT == 8 ? 2 : 1; }
inline int x_line_span(int P, int MT) { return P * MT + P + 2; }
// LDS (elements) of an x-line workgroup of `threads` threads
template <int MT>
int x_line_lds_elems(int P, int threads)
{
    const int span = x_line_span(P, MT);
    if (x_lds_regions<MT>() == 3) return 2 * span + 6 * threads;
    return std::max(x_lds_regions<MT>() * span, 6 * threads);
}

// x lines: the right-hand side tau^2 A u of one interior grid row is formed from three rows of u
// and the row's system is solved; one workgroup per row.  Every thread forms the right-hand
// sides of 16 bytes of consecutive nodes at a time.
template <typename T, int MT>
__global__ __launch_bounds__(kMaxXThreads) void k_adi_x(LineArgs A)
{
    extern __shared__ unsigned char smem[];
    constexpr int V = 16 / (int)sizeof(T);
    constexpr int kRegions = x_lds_regions<MT>();
    typedef T Vec __attribute__((ext_vector_type(V)));
    const int n = A.nx - 2;
    const int ld = A.ld;
    const int P = A.P;
    const int NT = (int)blockDim.x;
    const int span = P * MT;  // unknowns of the padded line
    const int tid = (int)threadIdx.x;
    T* const sD = reinterpret_cast<T*>(smem);
    T* const sF = kRegions >= 2 ? sD + span + P + 2 : sD;
    T* const sR = kRegions == 3 ? sF + span + P + 2 : sD;
    const size_t row0 = (size_t)(xcd_block(blockIdx.x, gridDim.x) + 1) * ld;
    const T* u = (const T*)A.u + row0;
    const T* hx = (const T*)A.hx + row0;
    const T* hy = (const T*)A.hy + row0;
    const T idx2 = (T)A.idx2, idy2 = (T)A.idy2, tt = (T)A.tt;
    // tau^2 (A u) in flux form, opposite faces added as pairs (as the explicit solver and the oracle
    // form it; the scalings by 1/dx^2 and 1/dy^2 are products with the reciprocals, which differ
    // from the quotients by rounding only), coalesced, and passed through LDS to the threads whose
    // chunks hold them.  Loads past the line read its last nodes instead and their values are
    // dropped: no branch around a load, so that a thread's loads are in flight together.  The threads cover the nodes 0 .. n; node i holds unknown i - 1 and the face F_i.
    const int last = n / V * V;
    Vec fq[MT / V];
#pragma unroll
    for (int q = 0; q < MT / V; ++q) {
        const int iq = V * (tid + q * NT);
        const int i = min(iq, last);
        const Vec uc = *(const Vec*)(u + i);
        const Vec un = *(const Vec*)(u + i + ld);
        const Vec us = *(const Vec*)(u + i - ld);
        const Vec fe = *(const Vec*)(hx + i);
        const Vec fn = *(const Vec*)(hy + i);
        const Vec fs = *(const Vec*)(hy + i - ld);
        const T ul = u[i - 1], ur = u[i + V], fl = hx[i - 1];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const T ue = (v < V - 1) ? uc[(v + 1) % V] : ur;
            const T uw = (v > 0) ? uc[(v + V - 1) % V] : ul;
            const T fw = (v > 0) ? fe[(v + V - 1) % V] : fl;
            const T east = fe[v] * (ue - uc[v]);
            const T west = fw * (uw - uc[v]);
            const T north = fn[v] * (un[v] - uc[v]);
            const T south = fs[v] * (us[v] - uc[v]);
            const T d = ((east + west) * idx2 + (north + south) * idy2) * tt;
            const int k = iq + v - 1;
            if (k >= 0 && k < n) sD[lds_pad<MT>(k)] = d;
            if (kRegions >= 2 && k < n) sF[lds_pad<MT>(k + 1)] = fe[v];
            fq[q][v] = fe[v];
        }
    }
    __syncthreads();
    const int p = tid;
    const bool act = p < P;
    const int lo = p * MT;
    Chunk<T, MT> ck;
#pragma unroll
    for (int q = 0; q < MT; ++q) ck.d[q] = (lo + q < n) ? sD[lds_pad<MT>(lo + q)] : T(0);
    if (kRegions == 1) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < MT / V; ++q) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const int i = V * (tid + q * NT) + v;
                if (i <= n) sF[lds_pad<MT>(i)] = fq[q][v];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q <= MT; ++q) ck.f[q] = (lo + q <= n) ? sF[lds_pad<MT>(lo + q)] : T(0);
    const Ends<T> e = ck.down(lo, n, (T)A.g);
    if (kRegions < 3) __syncthreads();
    T znext;
    const T zlo = solve_firsts<T>(e, sR, NT, tid, p, P, 1, &znext);
    ck.up(zlo, znext);
    if (kRegions < 3) __syncthreads();
    if (act) {
#pragma unroll
        for (int q = 0; q < MT; ++q) sD[lds_pad<MT>(lo + q)] = ck.d[q];
    }
    __syncthreads();
    T* const z = (T*)A.z + row0 + 1;
#pragma unroll
    for (int q = 0; q < MT; ++q) {
        const int k = tid + q * NT;
        if (k < n) z[k] = sD[lds_pad<MT>(k)];
    }
}

// y lines and the update: one workgroup per A.cw (a power of two) grid columns, thread t holding
// the chunk p = t / cw of column t % cw, so that a row of the strip is read and written in
// segments of cw elements.  The columns need no transposition: a chunk's rows are read by its own
// thread.  Then du = du + w, u = u + du (START: du = tau u1 + w/2, u = u0 + du) on interior nodes.
template <typename T, int MT, bool START>
__global__ __launch_bounds__(1024) void k_adi_y_strip(LineArgs A)
{
    extern __shared__ unsigned char smem[];
    T* const sD = reinterpret_cast<T*>(smem);
    const int n = A.ny - 2;
    const int ld = A.ld;
    const int P = A.P;
    const int t = (int)threadIdx.x;
    const int cw = A.cw;
    const int p = t / cw;
    const int col = xcd_block(blockIdx.x, gridDim.x) * cw + (t & (cw - 1));
    const int lo = p * MT;
    const T* z = (const T*)A.z + col;
    const T* hy = (const T*)A.hy + col;
    Chunk<T, MT> ck;
#pragma unroll
    for (int q = 0; q < MT; ++q) {
        const int k = lo + q;
        const T v = z[(size_t)min(k + 1, n) * ld];
        ck.d[q] = (k < n) ? v : T(0);
    }
#pragma unroll
    for (int q = 0; q <= MT; ++q) {
        const int k = lo + q;
        const T v = hy[(size_t)min(k, n) * ld];
        ck.f[q] = (k <= n) ? v : T(0);
    }
    const Ends<T> e = ck.down(lo, n, (T)A.g);
    // the state is requested before the reduced system's chain of exchanges
    const T* pa = (const T*)(START ? A.u1 : A.du) + col;
    const T* pb = (const T*)(START ? A.u0 : A.uo) + col;
    T va[MT], vb[MT];
#pragma unroll
    for (int q = 0; q < MT; ++q) {
        const size_t r = (size_t)min(lo + q + 1, n) * ld;
        va[q] = pa[r];
        vb[q] = pb[r];
    }
    T znext;
    const T zlo = solve_firsts<T>(e, sD, (int)blockDim.x, t, p, P, cw, &znext);
    ck.up(zlo, znext);
    if (col < 1 || col > A.nx - 2) return;
    const T tau = (T)A.tau;
#pragma unroll
    for (int q = 0; q < MT; ++q) {
        if (lo + q < n) {
            const size_t r = (size_t)(lo + q + 1) * ld + col;
            const T nd = START ? fma_t(tau, va[q], T(0.5) * ck.d[q]) : va[q] + ck.d[q];
            ((T*)A.du)[r] = nd;
            ((T*)A.uo)[r] = vb[q] + nd;
        }
    }
}

// y lines of large grids.  A strip whose whole column fits one workgroup is too narrow there (two
// columns of 4096 FP64 unknowns: 16-byte segments); instead the rows are cut into blocks of W * MT,
// a workgroup takes one block of 64 columns (one wave per chunk of MT rows, full cache lines), and
// the columns' blocks are joined by a small system per column:
//   k_adi_y_reduce eliminates within each block and writes its two end rows;
//   k_adi_y_join   solves for the first unknown of every block (parallel cyclic reduction in LDS);
//   k_adi_y_block  solves the block's unknowns between them and updates (du, u).
// The right-hand side and the faces are read twice instead of being transposed.

// Rows of the chunk-level system inside a block: unknown z_lo of chunk p (1 <= p < W) couples to
// those of chunks p - 1 and p + 1; from the chunks' Ends staged in LDS, [7][W][64].
template <typename T, int W>
__device__ __forceinline__ void put_ends(T* s, int w, int c, const Ends<T>& e)
{
    s[(0 * W + w) * 64 + c] = e.a0;
    s[(1 * W + w) * 64 + c] = e.b0;
    s[(2 * W + w) * 64 + c] = e.c0;
    s[(3 * W + w) * 64 + c] = e.d0;
    s[(4 * W + w) * 64 + c] = e.ha;
    s[(5 * W + w) * 64 + c] = e.hc;
    s[(6 * W + w) * 64 + c] = e.hd;
}
template <typename T, int W>
__device__ __forceinline__ void first_row(const T* s, int p, int c, T& a, T& b, T& cc, T& d)
{
    const T a0 = s[(0 * W + p) * 64 + c];
    a = -(a0 * s[(4 * W + p - 1) * 64 + c]);
    b = fma_t(-a0, s[(5 * W + p - 1) * 64 + c], s[(1 * W + p) * 64 + c]);
    cc = s[(2 * W + p) * 64 + c];
    d = fma_t(-a0, s[(6 * W + p - 1) * 64 + c], s[(3 * W + p) * 64 + c]);
}

template <typename T, int MT>
__device__ __forceinline__ void load_column_chunk(const LineArgs& A, int col, int lo, int n, Chunk<T, MT>& ck)
{
    const T* z = (const T*)A.z + col;
    const T* hy = (const T*)A.hy + col;
#pragma unroll
    for (int q = 0; q < MT; ++q) {
        const int k = lo + q;
        const T v = z[(size_t)min(k + 1, n) * A.ld];
        ck.d[q] = (k < n) ? v : T(0);
    }
#pragma unroll
    for (int q = 0; q <= MT; ++q) {
        const int k = lo + q;
        const T v = hy[(size_t)min(k, n) * A.ld];
        ck.f[q] = (k <= n) ? v : T(0);
    }
}

template <typename T, int MT, int W>
__global__ __launch_bounds__(64 * W) void k_adi_y_reduce(LineArgs A)
{
    __shared__ T s[7 * W * 64];
    const int c = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = A.ny - 2;
    const int col = (int)blockIdx.x * 64 + c;
    const int blk = (int)blockIdx.y;
    const int lo = (blk * W + w) * MT;
    Chunk<T, MT> ck;
    load_column_chunk<T, MT>(A, col, lo, n, ck);
    put_ends<T, W>(s, w, c, ck.down(lo, n, (T)A.g));
    __syncthreads();
    if (w != 0) return;
    // the chunks' first unknowns x_1 .. x_{W-1} eliminated downwards with x_0 as a parameter
    T a, b, cc, d;
    first_row<T, W>(s, 1, c, a, b, cc, d);
    T rr = T(1) / b;
    T pa = a * rr, pc = cc * rr, pd = d * rr;
    T al = pd, be = pa, ga = pc;
#pragma unroll
    for (int p = 2; p < W; ++p) {
        first_row<T, W>(s, p, c, a, b, cc, d);
        rr = T(1) / fma_t(-a, pc, b);
        pd = fma_t(-a, pd, d) * rr;
        pa = -(a * pa) * rr;
        pc = cc * rr;
        al = fma_t(-ga, pd, al);
        be = fma_t(-ga, pa, be);
        ga = -(ga * pc);
    }
    const T c0 = s[(2 * W) * 64 + c];
    const T la = s[(4 * W + W - 1) * 64 + c];
    T* const out = (T*)A.ends + (size_t)blk * A.ld + col;
    const size_t st = (size_t)A.P * A.ld;
    out[0 * st] = s[c];
    out[1 * st] = fma_t(-c0, be, s[(1 * W) * 64 + c]);
    out[2 * st] = -(c0 * ga);
    out[3 * st] = fma_t(-c0, al, s[(3 * W) * 64 + c]);
    out[4 * st] = -(la * pa);
    out[5 * st] = fma_t(-la, pc, s[(5 * W + W - 1) * 64 + c]);
    out[6 * st] = fma_t(-la, pd, s[(6 * W + W - 1) * 64 + c]);
}

// First unknown of every block of every column: thread t holds block t / cw of column t % cw.
template <typename T>
__global__ __launch_bounds__(1024) void k_adi_y_join(LineArgs A)
{
    extern __shared__ unsigned char smem[];
    const int cw = A.cw, t = (int)threadIdx.x;
    const int p = t / cw;
    const int col = (int)blockIdx.x * cw + (t & (cw - 1));
    const size_t at = (size_t)min(p, A.P - 1) * A.ld + col;
    const size_t st = (size_t)A.P * A.ld;
    const T* in = (const T*)A.ends + at;
    const Ends<T> e = {in[0], in[st], in[2 * st], in[3 * st], in[4 * st], in[5 * st], in[6 * st]};
    T znext;
    const T x = solve_firsts<T>(e, reinterpret_cast<T*>(smem), (int)blockDim.x, t, p, A.P, cw, &znext);
    if (p < A.P) ((T*)A.firsts)[at] = x;
}

template <typename T, int MT, int W, bool START>
__global__ __launch_bounds__(64 * W) void k_adi_y_block(LineArgs A)
{
    __shared__ T s[7 * W * 64];
    const int c = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = A.ny - 2;
    const int col = (int)blockIdx.x * 64 + c;
    const int blk = (int)blockIdx.y;
    const int lo = (blk * W + w) * MT;
    Chunk<T, MT> ck;
    load_column_chunk<T, MT>(A, col, lo, n, ck);
    const T* fi = (const T*)A.firsts + (size_t)blk * A.ld + col;
    const T x0 = fi[0];
    const T xw = (blk + 1 < A.P) ? fi[A.ld] : T(0);
    put_ends<T, W>(s, w, c, ck.down(lo, n, (T)A.g));
    __syncthreads();
    // x_1 .. x_{W-1} between the known x_0 and x_W (every wave solves this small system itself)
    T pc[W], x[W + 1];
    x[0] = x0;
    x[W] = xw;
#pragma unroll
    for (int p = 1; p < W; ++p) {
        T a, b, cc, d;
        first_row<T, W>(s, p, c, a, b, cc, d);
        const T rr = T(1) / (p > 1 ? fma_t(-a, pc[p - 1], b) : b);
        x[p] = fma_t(-a, x[p - 1], d) * rr;
        pc[p] = cc * rr;
    }
#pragma unroll
    for (int p = W - 1; p >= 1; --p) x[p] = fma_t(-pc[p], x[p + 1], x[p]);
    T zlo = x[0], znext = x[1];
#pragma unroll
    for (int p = 1; p < W; ++p) {
        if (w == p) zlo = x[p], znext = x[p + 1];
    }
    ck.up(zlo, znext);
    if (col < 1 || col > A.nx - 2) return;
    const T* pa = (const T*)(START ? A.u1 : A.du) + col;
    const T* pb = (const T*)(START ? A.u0 : A.uo) + col;
    T va[MT], vb[MT];
#pragma unroll
    for (int q = 0; q < MT; ++q) {
        const size_t r = (size_t)min(lo + q + 1, n) * A.ld;
        va[q] = pa[r];
        vb[q] = pb[r];
    }
    const T tau = (T)A.tau;
#pragma unroll
    for (int q = 0; q < MT; ++q) {
        if (lo + q < n) {
            const size_t r = (size_t)(lo + q + 1) * A.ld + col;
            const T nd = START ? fma_t(tau, va[q], T(0.5) * ck.d[q]) : va[q] + ck.d[q];
            ((T*)A.du)[r] = nd;
            ((T*)A.uo)[r] = vb[q] + nd;
        }
    }
}

// Faces (means of nodal values, 0 past the last node) and validation statistics of h1, h2:
// red[block] = {min h, max x face, max y face, non-finite count}.
template <typename T>
__global__ __launch_bounds__(256) void k_adi_faces(const T* __restrict__ h1, const T* __restrict__ h2, int nx, int ny,
                                                   int ld, T* __restrict__ hx, T* __restrict__ hy, double* red)
{
    __shared__ double s[4][256];
    double mn = INFINITY, mxx = 0.0, mxy = 0.0, bad = 0.0;
    const int64_t total = (int64_t)nx * ny;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < total; k += (int64_t)gridDim.x * 256) {
        const int j = (int)(k / nx), i = (int)(k % nx);
        const T a = h1[k], b2 = h2[k];
        if (!isfinite((double)a) || !isfinite((double)b2)) bad += 1.0;
        mn = fmin(mn, fmin((double)a, (double)b2));
        const T fx = (i < nx - 1) ? T(0.5) * (a + h1[k + 1]) : T(0);
        const T fy = (j < ny - 1) ? T(0.5) * (b2 + h2[k + nx]) : T(0);
        hx[(size_t)j * ld + i] = fx;
        hy[(size_t)j * ld + i] = fy;
        mxx = fmax(mxx, (double)fx);
        mxy = fmax(mxy, (double)fy);
    }
    s[0][threadIdx.x] = mn;
    s[1][threadIdx.x] = mxx;
    s[2][threadIdx.x] = mxy;
    s[3][threadIdx.x] = bad;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            s[0][threadIdx.x] = fmin(s[0][threadIdx.x], s[0][threadIdx.x + w]);
            s[1][threadIdx.x] = fmax(s[1][threadIdx.x], s[1][threadIdx.x + w]);
            s[2][threadIdx.x] = fmax(s[2][threadIdx.x], s[2][threadIdx.x + w]);
            s[3][threadIdx.x] += s[3][threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int q = 0; q < 4; ++q) red[4 * blockIdx.x + q] = s[q][0];
}

}  // namespace

struct fdw_adi {
    fdw_problem p;
    int nx = 0, ny = 0, ld = 0;
    int64_t N = 0, n = 0;
    double dx = 0, dy = 0, sigma = 0.25;
    hipStream_t stream = nullptr;
    std::string err;
    void *u = nullptr, *du = nullptr, *u0 = nullptr, *u1 = nullptr, *hx = nullptr, *hy = nullptr, *z = nullptr, *ends = nullptr;
    double* red = nullptr;
    // kAdiGraphSteps steps (after the start step) captured once in a hipGraph on a private
    // stream and replayed on `stream`
    hipStream_t cap = nullptr;
    hipGraphExec_t exec = nullptr;
    bool graph_failed = false;
};

namespace {

constexpr int kAdiRedBlocks = 256;

size_t adi_plane(int ld, int rows, int dtype) { return adi_align((size_t)ld * rows * (dtype == FDW_F32 ? 4 : 8)); }

// blocks of rows the y lines are cut into (0: none, the strip kernel runs them)
inline int ends_blocks(int ny)
{
    return ny - 2 > kStripUnknowns ? (ny - 2 + kBlockChunk * kBlockChunks - 1) / (kBlockChunk * kBlockChunks) : 0;
}

int adi_fail(fdw_adi* s, int code, const std::string& msg)
{
    if (s) s->err = msg;
    return code;
}

#define ADICHK(s, expr)                                                                              \
    do {                                                                                             \
        hipError_t e_ = (expr);                                                                      \
        if (e_ != hipSuccess) return adi_fail((s), FDW_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

template <typename T, int MT>
hipError_t launch_x_mt(const fdw_adi* s, LineArgs A, hipStream_t st)
{
    const int n = s->nx - 2;
    A.P = (n + MT - 1) / MT;
    A.g = s->sigma * A.tt * A.idx2;
    const int threads = ((n + 1 + MT - 1) / MT + 63) / 64 * 64;  // the threads' nodes 0 .. n
    hipLaunchKernelGGL((k_adi_x<T, MT>), dim3(s->ny - 2), dim3(threads), (size_t)x_line_lds_elems<MT>(A.P, threads) * sizeof(T),
                       st, A);
    return hipGetLastError();
}
// Chunk length of the x lines.  Short chunks give a line more threads, long ones a smaller reduced
// system: 4 unknowns up to 512 (256^2 FP64: 9.6 us per step against 10.1 with 8), then 8
// (2048^2 FP64: 79.2 us per step, 81.3 with 4, 77.9 with 16; 4096^2 FP64: 314, 322 with 16); 16 for
// the lines that 576 threads of 8 do not cover, which only FP32 has.
template <typename T>
hipError_t launch_x(const fdw_adi* s, const LineArgs& A, hipStream_t st)
{
    const int n = s->nx - 2;
    if (n <= 512) return launch_x_mt<T, 4>(s, A, st);
    if constexpr (max_line_unknowns<T>() + 1 > 8 * kMaxXThreads)
        if (n + 1 > 8 * kMaxXThreads) return launch_x_mt<T, 16>(s, A, st);
    return launch_x_mt<T, 8>(s, A, st);
}

template <typename T, bool START>
hipError_t launch_y_blocks(const fdw_adi* s, LineArgs A, hipStream_t st)
{
    constexpr int MT = kBlockChunk, W = kBlockChunks;
    const int n = s->ny - 2;
    A.g = s->sigma * A.tt * A.idy2;
    A.P = (n + MT * W - 1) / (MT * W);
    A.ends = s->ends;
    A.firsts = (T*)s->ends + (size_t)7 * A.P * A.ld;
    const dim3 gr((s->nx - 1 + 63) / 64, A.P), bl(64 * W);
    hipLaunchKernelGGL((k_adi_y_reduce<T, MT, W>), gr, bl, 0, st, A);
    A.cw = 1;
    while (A.cw < 16 && 2 * A.cw * A.P <= 1024) A.cw *= 2;
    const int jt = (A.P * A.cw + 63) / 64 * 64;
    hipLaunchKernelGGL((k_adi_y_join<T>), dim3((s->nx - 1 + A.cw - 1) / A.cw), dim3(jt), (size_t)6 * jt * sizeof(T), st,
                       A);
    hipLaunchKernelGGL((k_adi_y_block<T, MT, W, START>), gr, bl, 0, st, A);
    return hipGetLastError();
}

template <typename T, int MT, bool START>
hipError_t launch_y_strips(const fdw_adi* s, LineArgs A, hipStream_t st)
{
    const int n = s->ny - 2;
    A.P = (n + MT - 1) / MT;
    A.g = s->sigma * A.tt * A.idy2;
    // columns per workgroup: up to 8 (64-byte FP64 segments), as long as about one workgroup per CU
    // is left (1024^2 FP64: 25.8 us per step with 4 columns, 27.8 with 8, 31.4 with 2)
    A.cw = 1;
    while (A.cw < 8 && 2 * A.cw * A.P <= 1024 && (s->nx - 1) / (2 * A.cw) >= 192) A.cw *= 2;
    const int threads = (A.P * A.cw + 63) / 64 * 64;
    hipLaunchKernelGGL((k_adi_y_strip<T, MT, START>), dim3((s->nx - 1 + A.cw - 1) / A.cw), dim3(threads),
                       (size_t)6 * threads * sizeof(T), st, A);
    return hipGetLastError();
}

// Columns of up to 1024 unknowns go through one kernel that holds a strip's whole columns (strips of
// 1 to 8 columns, launch_y_strips, and one launch is shorter than three: 700^2 FP64 19.8 us
// per step against 24.7 in blocks, 3900 x 1000 FP64 74 against 81); longer ones in blocks of 64
// rows, with full cache lines (500 x 4000 FP64 48 against 66; 1000 x 1500 FP32 25.1 against 31;
// 4096^2 FP64 314 against 644).
template <typename T, bool START>
hipError_t launch_y(const fdw_adi* s, const LineArgs& A, hipStream_t st)
{
    const int n = s->ny - 2;
    if (n > kStripUnknowns) return launch_y_blocks<T, START>(s, A, st);
    return n <= 512 ? launch_y_strips<T, 4, START>(s, A, st) : launch_y_strips<T, 8, START>(s, A, st);
}

// one solve w = B^{-1} tau^2 A u and the update of (du, u), on stream st
template <typename T>
int adi_step(fdw_adi* s, bool start, hipStream_t st)
{
    LineArgs A;
    std::memset(&A, 0, sizeof(A));
    A.nx = s->nx;
    A.ny = s->ny;
    A.ld = s->ld;
    A.u = start ? s->u0 : s->u;  // the start step solves with the initial displacement
    A.hx = s->hx;
    A.hy = s->hy;
    A.z = s->z;
    A.idx2 = 1.0 / (s->dx * s->dx);
    A.idy2 = 1.0 / (s->dy * s->dy);
    A.tt = s->p.tau * s->p.tau;
    A.du = s->du;
    A.uo = s->u;
    A.u0 = s->u0;
    A.u1 = s->u1;
    A.tau = s->p.tau;
    ADICHK(s, launch_x<T>(s, A, st));
    if (start)
        ADICHK(s, (launch_y<T, true>(s, A, st)));
    else
        ADICHK(s, (launch_y<T, false>(s, A, st)));
    return FDW_OK;
}

constexpr int kAdiGraphSteps = 16;

// capture kAdiGraphSteps ordinary steps once (their launches depend on nothing but the solver's
// fixed buffers); on any failure the solver keeps launching step by step
template <typename T>
void adi_capture(fdw_adi* s)
{
    if (!s->cap && hipStreamCreateWithFlags(&s->cap, hipStreamNonBlocking) != hipSuccess) {
        s->cap = nullptr;
        s->graph_failed = true;
        return;
    }
    if (hipStreamBeginCapture(s->cap, hipStreamCaptureModeThreadLocal) != hipSuccess) {
        s->graph_failed = true;
        return;
    }
    int rc = FDW_OK;
    for (int k = 0; k < kAdiGraphSteps && rc == FDW_OK; ++k) rc = adi_step<T>(s, false, s->cap);
    hipGraph_t g = nullptr;
    const hipError_t e = hipStreamEndCapture(s->cap, &g);
    if (rc != FDW_OK || e != hipSuccess || !g || hipGraphInstantiate(&s->exec, g, nullptr, nullptr, 0) != hipSuccess) {
        s->exec = nullptr;
        s->graph_failed = true;
    }
    if (g) hipGraphDestroy(g);
}

template <typename T>
int adi_setup(fdw_adi* s, const void* u0, const void* u1, const void* h1, const void* h2)
{
    const int nx = s->nx, ny = s->ny;
    ADICHK(s, fdw::launch_copy_in<T>(u0, nx, ny, s->u0, s->ld, 1, s->stream));
    ADICHK(s, fdw::launch_copy_in<T>(u1, nx, ny, s->u1, s->ld, 1, s->stream));
    hipLaunchKernelGGL((k_adi_faces<T>), dim3(kAdiRedBlocks), dim3(256), 0, s->stream, (const T*)h1,
                       (const T*)(h2 ? h2 : h1), nx, ny, s->ld, (T*)s->hx, (T*)s->hy, s->red);
    ADICHK(s, hipGetLastError());
    std::vector<double> red(4 * kAdiRedBlocks);
    ADICHK(s, hipMemcpyAsync(red.data(), s->red, red.size() * sizeof(double), hipMemcpyDeviceToHost, s->stream));
    ADICHK(s, hipStreamSynchronize(s->stream));
    double mn = INFINITY, mxx = 0, mxy = 0, bad = 0;
    for (int b = 0; b < kAdiRedBlocks; ++b) {
        mn = std::min(mn, red[4 * b]);
        mxx = std::max(mxx, red[4 * b + 1]);
        mxy = std::max(mxy, red[4 * b + 2]);
        bad += red[4 * b + 3];
    }
    if (bad != 0.0) return adi_fail(s, FDW_EINVAL, "h contains non-finite values");
    const bool allow0 = (s->p.flags & FDW_ALLOW_ZERO_H) != 0;
    if (allow0 ? !(mn >= 0.0) : !(mn > 0.0)) return adi_fail(s, FDW_EINVAL, allow0 ? "h must be >= 0" : "h must be > 0");
    if (s->sigma < 0.25 && !(s->p.flags & FDW_ALLOW_UNSTABLE)) {
        // below sigma = 1/4 the scheme is stable for tau^2 lambda_max (1 - 4 sigma) <= 4 only
        const double tt = s->p.tau * s->p.tau;
        const double bound = tt * (4.0 * mxx / (s->dx * s->dx) + 4.0 * mxy / (s->dy * s->dy)) * (1.0 - 4.0 * s->sigma);
        if (bound > 4.0 * (1.0 + 1e-12)) return adi_fail(s, FDW_ECFL, "time step above the stability bound for sigma < 1/4");
    }
    return FDW_OK;
}

}  // namespace

extern "C" {

size_t fdw_adi_workspace_bytes(const fdw_problem* p)
{
    if (!p || p->nx < 3 || p->ny < 3 || (p->dtype != FDW_F32 && p->dtype != FDW_F64)) return 0;
    const int ld = pad64(p->nx);
    size_t b = 7 * adi_plane(ld, p->ny, p->dtype);   // u, du, u0, u1, hx, hy, z
    b += adi_align((size_t)8 * ends_blocks(p->ny) * ld * (p->dtype == FDW_F32 ? 4 : 8));
    b += adi_align(sizeof(double) * 4 * kAdiRedBlocks);
    return b;
}

int fdw_adi_init(const fdw_problem* p, double sigma, void* workspace, size_t ws_bytes, const void* u0, const void* u1,
                 const void* h1, const void* h2, void* hip_stream, fdw_adi** out)
{
    if (!out) return FDW_EINVAL;
    *out = nullptr;
    if (!p || !workspace || !u0 || !u1 || !h1) return FDW_EINVAL;
    if (((uintptr_t)workspace) % kAdiAlign) return FDW_EINVAL;
    if (!(sigma >= 0.0) || !std::isfinite(sigma)) return FDW_EINVAL;
    if (p->nx < 3 || p->ny < 3 || !(p->x1 > p->x0) || !(p->y1 > p->y0) || !(p->tau > 0.0) || !std::isfinite(p->tau) ||
        !(p->T >= 0.0))
        return FDW_EINVAL;
    const int64_t N = (int64_t)std::llround(p->T / p->tau);
    if (std::fabs((double)N * p->tau - p->T) > 1e-9 * std::max(p->T, p->tau)) return FDW_EINVAL;
    const size_t need = fdw_adi_workspace_bytes(p);
    if (need == 0) return FDW_EINVAL;
    if (ws_bytes < need) return FDW_ENOMEM;
    fdw_adi* s = new fdw_adi();
    s->p = *p;
    s->nx = p->nx;
    s->ny = p->ny;
    s->ld = pad64(p->nx);
    s->N = N;
    s->dx = (p->x1 - p->x0) / (p->nx - 1);
    s->dy = (p->y1 - p->y0) / (p->ny - 1);
    s->sigma = sigma;
    s->stream = (hipStream_t)hip_stream;
    // a line is solved by one workgroup
    const int maxn = (p->dtype == FDW_F32) ? max_line_unknowns<float>() : max_line_unknowns<double>();
    if (std::max(p->nx, p->ny) - 2 > maxn) {
        delete s;
        return FDW_ENOTSUP;
    }
    char* w = (char*)workspace;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        void* q = w + off;
        off += bytes;
        return q;
    };
    const size_t pn = adi_plane(s->ld, s->ny, p->dtype);
    s->u = take(pn);
    s->du = take(pn);
    s->u0 = take(pn);
    s->u1 = take(pn);
    s->hx = take(pn);
    s->hy = take(pn);
    s->z = take(pn);
    s->ends = take(adi_align((size_t)8 * ends_blocks(s->ny) * s->ld * (p->dtype == FDW_F32 ? 4 : 8)));
    s->red = (double*)take(adi_align(sizeof(double) * 4 * kAdiRedBlocks));
    // zero the state, faces and scratch (padding columns and the boundary ring stay 0)
    if (fdw::launch_fill_bytes(workspace, off, s->stream) != hipSuccess) {
        delete s;
        return FDW_EHIP;
    }
    const int rc = (p->dtype == FDW_F32) ? adi_setup<float>(s, u0, u1, h1, h2) : adi_setup<double>(s, u0, u1, h1, h2);
    if (rc) {
        const int code = rc;
        delete s;
        return code;
    }
    *out = s;
    return FDW_OK;
}

int fdw_adi_step_n(fdw_adi* s, int64_t n)
{
    if (!s) return FDW_EINVAL;
    if (n < 0) return adi_fail(s, FDW_EINVAL, "n must be >= 0");
    const bool f32 = s->p.dtype == FDW_F32;
    int64_t k = 0;
    while (k < n) {
        const bool start = s->n == 0;
        if (!start && n - k >= kAdiGraphSteps && !s->graph_failed) {
            // runs of kAdiGraphSteps steps are replayed from a hipGraph (the launch-bound small grids
            // gain most)
            if (!s->exec) f32 ? adi_capture<float>(s) : adi_capture<double>(s);
            if (s->exec) {
                ADICHK(s, hipGraphLaunch(s->exec, s->stream));
                s->n += kAdiGraphSteps;
                k += kAdiGraphSteps;
                continue;
            }
        }
        const int rc = f32 ? adi_step<float>(s, start, s->stream) : adi_step<double>(s, start, s->stream);
        if (rc) return rc;
        s->n += 1;
        k += 1;
    }
    return FDW_OK;
}

int fdw_adi_get_state(fdw_adi* s, void* u, void* du, int64_t* n)
{
    if (!s) return FDW_EINVAL;
    if (n) *n = s->n;
    const bool f32 = s->p.dtype == FDW_F32;
    const void* su = (s->n == 0) ? s->u0 : s->u;
    const void* sd = (s->n == 0) ? nullptr : s->du;
    if (du && !sd) ADICHK(s, fdw::launch_fill_bytes(du, (size_t)s->nx * s->ny * (f32 ? 4 : 8), s->stream));
    auto copy = [&](const void* a, void* to, const void* a1, void* to1) {
        return f32 ? fdw::launch_copy_out<float>(a, s->ld, s->nx, s->ny, to, s->stream, a1, to1)
                   : fdw::launch_copy_out<double>(a, s->ld, s->nx, s->ny, to, s->stream, a1, to1);
    };
    if (u && du && sd)
        ADICHK(s, copy(su, u, sd, du));
    else if (u)
        ADICHK(s, copy(su, u, nullptr, nullptr));
    else if (du && sd)
        ADICHK(s, copy(sd, du, nullptr, nullptr));
    return FDW_OK;
}

int fdw_adi_reset(fdw_adi* s)
{
    if (!s) return FDW_EINVAL;
    s->n = 0;
    return FDW_OK;
}

const char* fdw_adi_last_error(const fdw_adi* s) { return s ? s->err.c_str() : "null context"; }

void fdw_adi_destroy(fdw_adi* s)
{
    if (!s) return;
    if (s->exec) hipGraphExecDestroy(s->exec);
    if (s->cap) hipStreamDestroy(s->cap);
    delete s;
}

}  // extern "C"

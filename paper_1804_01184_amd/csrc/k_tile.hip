// Batched path for problems whose state stays in the caches: several time
// steps per launch, with the whole state of a tile of the grid in registers.
//
// A workgroup of NW waves owns a tile of 64 C columns by NW RW rows of one
// shot; a wave holds RW of its rows, a lane C adjacent columns of each.  The
// tile's fields, model and (adjoint) gradient sums are loaded once, advanced
// T time steps and stored once.  Horizontal differences take the neighbour
// lanes' columns with whole-wave shifts, vertical ones run along the wave's
// own registers; only the rows at a wave's upper and lower edge pass through
// LDS, twice a step, with a barrier each.  What lies outside the tile is
// taken as zero, which is right at the edge of the grid and wrong elsewhere:
// the wrong values move in by 3 nodes a step, so a tile owns (and stores) only
// the nodes at least 3 T nodes from its inner edges, and tiles overlap by
// twice that.
//
// What bounds it: the arithmetic (about 45 instructions a cell and step
// forward, 75 in the adjoint), on the owned and the overlapping cells alike,
// and for the smallest problems the launch itself.  The strip kernels, which
// march down the grid, redo fewer cells but run a chain of dependent rows, a
// row of every wave after the other; they win where the state streams from
// memory, where their smaller traffic counts.
//
// Every update is written with the strip kernels' expressions, so the
// wavefields agree with theirs bit for bit.  (1 / h stays out of the stored
// coefficients for the same reason: beta K / h, rounded, is another medium than
// the forward sweep's beta K, alike at every node of a homogeneous model, and
// the phase error grows with the steps.  Against FP64, 8 shots of 201 x 201,
// 1000 steps, the gradient was off by up to 7.5e-7 with it, 4.3e-7 without.)
#include "wave_dev.h"

#include <hip/hip_ext.h>

namespace fwi {

namespace {

// First node of tile k (a multiple of the axis' unit) and the nodes it owns.
__device__ inline int tile_first(const TileAxis &a, int k)
{
    return a.n == 1 ? 0 : k * a.last / (a.n - 1) / a.unit * a.unit;
}
__device__ inline int tile_lo(const TileAxis &a, int k)
{
    return k == 0 ? 0 : tile_first(a, k) + a.halo;
}
__device__ inline int tile_hi(const TileAxis &a, int k)
{
    return k == a.n - 1 ? a.len : tile_first(a, k + 1) + a.halo;
}

// A lane's columns in its tile.
template <int C>
struct TileLane {
    int lane, wv, j0, row0;     // lane, wave, first column, the wave's first row
    int r_lo, r_hi;             // owned rows
    bool ok[C], pml[C];         // column inside the grid, in the absorbing layer
    unsigned v, vw;             // lane offset of loads and of whole-lane stores
    unsigned vt[C];             // element stores of a lane owning only some columns
    unsigned zf[C], zs[C];      // split offsets on full and middle rows
    bool own[C];                // column owned
    bool xpml;                  // some column of the tile lies in the layer
    bool tail;                  // some lane owns only some of its columns
};

template <int C, int RW>
__device__ inline void tile_lane(const Geo &g, const TileAxis &x, const TileAxis &z, int tx,
                                 int tz, TileLane<C> &w)
{
    w.lane = threadIdx.x & (WAVE - 1);
    w.wv = uni((int)(threadIdx.x / WAVE));
    const int c0 = tile_first(x, tx), lo = tile_lo(x, tx), hi = tile_hi(x, tx);
    w.j0 = c0 + w.lane * C;
    w.row0 = tile_first(z, tz) + w.wv * RW;
    w.r_lo = tile_lo(z, tz);
    w.r_hi = tile_hi(z, tz);
    w.v = w.j0 < g.Nx ? 4u * (unsigned)w.j0 : kOOB;
    const bool whole = w.j0 >= lo && w.j0 + C <= hi;
    w.vw = whole ? w.v : kOOB;
    w.xpml = c0 < g.npml || c0 + WAVE * C > g.Nx - g.npml;
    w.tail = hi % C != 0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int j = w.j0 + c;
        w.ok[c] = j < g.Nx;
        w.own[c] = j >= lo && j < hi;
        w.pml[c] = j < g.npml || j >= g.Nx - g.npml;
        w.vt[c] = !whole && w.own[c] ? 4u * (unsigned)j : kOOB;
        w.zf[c] = w.ok[c] ? 4u * (unsigned)j : kOOB;
        w.zs[c] = !w.ok[c] ? kOOB
                  : j < g.npml ? 4u * (unsigned)j
                  : j >= g.Nx - g.npml ? 4u * (unsigned)(j - (g.Nx - 2 * g.npml)) : kOOB;
    }
}

__device__ inline bool row_pml(const Geo &g, int r) { return r < g.npml || r >= g.Nz - g.npml; }

// Stores a row of the tile's own columns (on: the row is owned; uniform).
template <int C>
__device__ inline void tile_store(rsrc_t r, const TileLane<C> &w, unsigned soff,
                                  const float (&v)[C])
{
    vst<C>(r, w.vw, soff, v);
    if (w.tail) {
#pragma unroll
        for (int c = 0; c + 1 < C; ++c)
            bst(r, w.vt[c], soff, v[c]);
    }
}

// A record's base and size: the resource of one of its rows is made where the
// row is read, with no bytes for a row outside the grid (its loads return 0),
// so that no lane offset has to be selected per row.
struct Base {
    const float *p;
    unsigned bytes;
};
__device__ inline Base base_of(const Recd &r, int s)
{
    return {(const float *)((const char *)r.base + (size_t)s * r.sbytes), r.bytes};
}

// Loads a row (zero outside the grid; ok is uniform).
template <int C>
__device__ inline void tile_load(const Base &b, const TileLane<C> &w, bool ok, unsigned soff,
                                 float (&v)[C])
{
    const rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
        (void *)b.p, (short)0, ok ? (int)(b.bytes + kSlack) : 0, kRsrcWord3);
    vld<C>(r, w.v, soff, v);
#pragma unroll
    for (int c = 1; c < C; ++c)
        v[c] = w.ok[c] ? v[c] : 0.f;
}

// A wave's rows at its edges, for its neighbours: the slots hold, per
// wave, three rows of 64 C columns.
template <int C, int NW>
struct Edge {
    float v[NW][3][C][WAVE];
};
template <int C, int NW>
__device__ inline void edge_put(Edge<C, NW> &e, int wv, int q, int lane, const float (&v)[C])
{
#pragma unroll
    for (int c = 0; c < C; ++c)
        e.v[wv][q][c][lane] = v[c];
}
template <int C, int NW>
__device__ inline void edge_get(const Edge<C, NW> &e, int wv, int q, int lane, float (&v)[C])
{
#pragma unroll
    for (int c = 0; c < C; ++c)
        v[c] = (unsigned)wv < (unsigned)NW ? e.v[wv][q][c][lane] : 0.f;
}

// Block -> (tile column, tile row, shot or group), tile column fastest; each
// XCD receives a contiguous range, so the tiles of a shot share its L2.
struct TileId {
    int tx, tz, s;
};
__device__ inline TileId tile_id(const TileAxis &x, const TileAxis &z)
{
    const int b = uni(xcd_item(blockIdx.x, gridDim.x));
    TileId t;
    t.tx = b % x.n;
    const int r = b / x.n;
    t.tz = r % z.n;
    t.s = r / z.n;
    return t;
}

// ---------------------------------------------------------------- forward

template <int C, int RW, int NW>
__global__ void __launch_bounds__(NW * WAVE) __attribute__((amdgpu_waves_per_eu(8, 8)))
    k_tile_fwd(Geo g, const float *__restrict__ tabs, const float *__restrict__ zpad,
               const float *__restrict__ model, FwdTile a)
{
    __shared__ Edge<C, NW> ep, ev;
    const TileId id = tile_id(a.x, a.z);
    TileLane<C> w;
    tile_lane<C, RW>(g, a.x, a.z, id.tx, id.tz, w);
    const unsigned FB = 4u * (unsigned)g.N;
    const int ZP = g.Nz + 2 * kZPad;
    const Base bM = {model, 3u * FB}, bIn = base_of(a.in, id.s), bOut = base_of(a.out, id.s);
    const rsrc_t rIn = res(bIn.p, bIn.bytes), rOut = res(bOut.p, bOut.bytes);

    float ax[C], btx[C], ahx[C], bhx[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int j = imin(w.j0 + c, g.Nx - 1);
        ax[c] = w.ok[c] ? tabs[j] : 0.f;
        btx[c] = w.ok[c] ? tabs[g.Nx + j] : 0.f;
        ahx[c] = w.ok[c] ? tabs[2 * g.Nx + j] : 0.f;
        bhx[c] = w.ok[c] ? tabs[3 * g.Nx + j] : 0.f;
    }
    // z tables of the wave's rows (zero outside the grid: the padded tables
    // hold zero rows there)
    float az[RW], btz[RW], ahz[RW], bhz[RW];
    cfloat *zt = ctab(zpad) + kZPad;
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int i = imin(w.row0 + r, g.Nz);
        az[r] = zt[i];
        btz[r] = zt[ZP + i];
        ahz[r] = zt[2 * ZP + i];
        bhz[r] = zt[3 * ZP + i];
    }

    // rows -1 .. RW+1 of p and -2 .. RW of vz; the rest rows 0 .. RW-1.  The
    // coefficients are held as the products the updates start with:
    // beta_h bx, beta_h bz, beta_x K, beta_z K
    float P[RW + 3][C], VZ[RW + 3][C], VX[RW][C], PZ[RW][C];
    float BX[RW][C], BZ[RW][C], KX[RW][C], KZ[RW][C];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int i = w.row0 + r;
        const bool ok = i < g.Nz;
        const unsigned rb = rowb(g, i);
        tile_load<C>(bIn, w, ok, rb + 2u * FB, P[r + 1]);
        tile_load<C>(bIn, w, ok, rb + FB, VZ[r + 2]);
        tile_load<C>(bIn, w, ok, rb, VX[r]);
        tile_load<C>(bM, w, ok, rb, KX[r]);
        tile_load<C>(bM, w, ok, rb + FB, BX[r]);
        tile_load<C>(bM, w, ok, rb + 2u * FB, BZ[r]);
#pragma unroll
        for (int c = 0; c < C; ++c)
            PZ[r][c] = 0.f;
        if (ok && (w.xpml || row_pml(g, i))) {
            const ZRow z = zrow(g, i);
#pragma unroll
            for (int c = 0; c < C; ++c)
                PZ[r][c] = bld(rIn, pick(z.full, w.zf[c], w.zs[c]), z.base + 3u * FB);
        }
    }
    // source: its bilinear cell's first row, the cell's weights and K on its
    // two rows
    cint *sij = (cint *)a.src_ij + 2 * id.s;
    cfloat *sw4 = ctab(a.src_w) + 4 * id.s;
    const int srow = sij[0], scol = sij[1];
    const bool src = srow + 1 >= w.row0 && srow < w.row0 + RW;
    float Ka[C], Kb[C];
    tile_load<C>(bM, w, src, rowb(g, srow), Ka);
    tile_load<C>(bM, w, src, rowb(g, srow + 1), Kb);
    cfloat *Q = ctab(a.Q) + (size_t)id.s * (size_t)a.nt + a.n;

#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
        for (int c = 0; c < C; ++c) {
            BX[r][c] = bhx[c] * BX[r][c];
            BZ[r][c] = bhz[r] * BZ[r][c];
            KZ[r][c] = btz[r] * KX[r][c];
            KX[r][c] = btx[c] * KX[r][c];
        }

    for (int j = 0; j < a.T; ++j) {
        const float dq = g.dt * Q[j];
        edge_put<C, NW>(ep, w.wv, 0, w.lane, P[1]);
        edge_put<C, NW>(ep, w.wv, 1, w.lane, P[2]);
        edge_put<C, NW>(ep, w.wv, 2, w.lane, P[RW]);
        __syncthreads();
        edge_get<C, NW>(ep, w.wv - 1, 2, w.lane, P[0]);
        edge_get<C, NW>(ep, w.wv + 1, 0, w.lane, P[RW + 1]);
        edge_get<C, NW>(ep, w.wv + 1, 1, w.lane, P[RW + 2]);
        // vz^{n+1/2} at rows i + 1/2
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int c = 0; c < C; ++c)
                VZ[r + 2][c] = ahz[r] * VZ[r + 2][c] -
                               BZ[r][c] *
                                   (kC1 * (P[r + 2][c] - P[r + 1][c]) + kC2 * (P[r + 3][c] - P[r][c])) *
                                   g.rdz;
        edge_put<C, NW>(ev, w.wv, 0, w.lane, VZ[2]);
        edge_put<C, NW>(ev, w.wv, 1, w.lane, VZ[RW]);
        edge_put<C, NW>(ev, w.wv, 2, w.lane, VZ[RW + 1]);
        // vx^{n+1/2} at columns j + 1/2
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            float dp[C];
            dfwd<C>(P[r + 1], dp);
#pragma unroll
            for (int c = 0; c < C; ++c)
                VX[r][c] = ahx[c] * VX[r][c] - BX[r][c] * dp[c] * g.rdx;
        }
        __syncthreads();
        edge_get<C, NW>(ev, w.wv - 1, 1, w.lane, VZ[0]);
        edge_get<C, NW>(ev, w.wv - 1, 2, w.lane, VZ[1]);
        edge_get<C, NW>(ev, w.wv + 1, 0, w.lane, VZ[RW + 2]);
        // p^{n+1}
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const bool rp = row_pml(g, w.row0 + r);
            float dvx[C];
            dbwd<C>(VX[r], dvx);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float dvz = kC1 * (VZ[r + 2][c] - VZ[r + 1][c]) + kC2 * (VZ[r + 3][c] - VZ[r][c]);
                const float pz = PZ[r][c];
                const float px = ax[c] * (P[r + 1][c] - pz) - KX[r][c] * dvx[c] * g.rdx;
                const float pzn = az[r] * pz - KZ[r][c] * dvz * g.rdz;
                P[r + 1][c] = px + pzn;
                // the split is kept only where the layer has one
                PZ[r][c] = rp || w.pml[c] ? pzn : 0.f;
            }
        }
        if (src) {
            float swa[C], swb[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int dj = w.j0 + c - scol;
                swa[c] = dj == 0 ? dq * sw4[0] : (dj == 1 ? dq * sw4[1] : 0.f);
                swb[c] = dj == 0 ? dq * sw4[2] : (dj == 1 ? dq * sw4[3] : 0.f);
            }
#pragma unroll
            for (int r = 0; r < RW; ++r)
                if ((unsigned)(w.row0 + r - srow) < 2u) {
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        P[r + 1][c] += (w.row0 + r == srow ? Ka[c] : Kb[c]) *
                                       (w.row0 + r == srow ? swa[c] : swb[c]);
                }
        }
        if (a.hist) {
            const rsrc_t rH =
                res(a.hist + (size_t)j * (size_t)a.lvl + (size_t)id.s * (size_t)a.ss, FB);
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                const int i = w.row0 + r;
                if (i >= w.r_lo && i < w.r_hi)
                    tile_store<C>(rH, w, rowb(g, i), P[r + 1]);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int i = w.row0 + r;
        if (i < w.r_lo || i >= w.r_hi)
            continue;
        const unsigned rb = rowb(g, i);
        tile_store<C>(rOut, w, rb, VX[r]);
        tile_store<C>(rOut, w, rb + FB, VZ[r + 2]);
        tile_store<C>(rOut, w, rb + 2u * FB, P[r + 1]);
        if (w.xpml || row_pml(g, i)) {
            const ZRow z = zrow(g, i);
#pragma unroll
            for (int c = 0; c < C; ++c)
                bst(rOut, w.own[c] ? pick(z.full, w.zf[c], w.zs[c]) : kOOB, z.base + 3u * FB,
                    PZ[r][c]);
        }
    }
}

// ---------------------------------------------------------------- adjoint
//
// State on entry to step m (descending): mu, lv = adjoint after step m+1 with
// R^T r^m already added (zero before the first step, m = nt).  Step m:
//   lv_mid = lv + D+(beta K mu),  gb += lv_mid (-beta_h D+ p^m)
//   t = D-(beta_h b lv_mid),  mu' = alpha mu + t + R^T r^{m-1}
//   gK += p^m (mu_x' - alpha_x mu_x) / K,  lv' = alpha_h lv_mid
// The bulk-modulus sensitivity is the sum over steps of mu_x (px^{m+1} -
// alpha_x px^m) + mu_z (pz^{m+1} - alpha_z pz^m) with the terms of each level
// collected (summation by parts in time): px^m meets mu_x' - alpha_x mu_x and
// pz^m the same of mu_z, and both differences are t + R^T r^{m-1}.  So one
// pressure level a step is enough, without its split.  The difference is taken
// of the stored values, rounding included, as in the strip kernels.

template <int C, int RW, int NW>
__global__ void __launch_bounds__(NW * WAVE)
    k_tile_adj(Geo g, const float *__restrict__ tabs, const float *__restrict__ zpad,
               const float *__restrict__ model, AdjTile a)
{
    __shared__ Edge<C, NW> eq, ew;
    __shared__ float inj[NW][RW][C][WAVE];   // R^T r of the step at the tile's nodes
    const TileId id = tile_id(a.x, a.z);
    TileLane<C> w;
    tile_lane<C, RW>(g, a.x, a.z, id.tx, id.tz, w);
    const unsigned FB = 4u * (unsigned)g.N;
    const int ZP = g.Nz + 2 * kZPad;
    const Base bM = {model, 3u * FB};
    const int c0 = tile_first(a.x, id.tx);
#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
        for (int c = 0; c < C; ++c)
            inj[w.wv][r][c][w.lane] = 0.f;

    float ax[C], btx[C], ahx[C], bhx[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int j = imin(w.j0 + c, g.Nx - 1);
        ax[c] = w.ok[c] ? tabs[j] : 0.f;
        btx[c] = w.ok[c] ? tabs[g.Nx + j] : 0.f;
        ahx[c] = w.ok[c] ? tabs[2 * g.Nx + j] : 0.f;
        bhx[c] = w.ok[c] ? tabs[3 * g.Nx + j] : 0.f;
    }
    float az[RW], btz[RW], ahz[RW], bhz[RW];
    cfloat *zt = ctab(zpad) + kZPad;
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int i = imin(w.row0 + r, g.Nz);
        az[r] = zt[i];
        btz[r] = zt[ZP + i];
        ahz[r] = zt[2 * ZP + i];
        bhz[r] = zt[3 * ZP + i];
    }
    // coefficients as the products the step uses: beta_x K, beta_z K, beta_h bx,
    // beta_h bz (formed once every load is under way)
    const int s = id.s;
    const Base bIn = base_of(a.in, s), bOut = base_of(a.out, s);
    const rsrc_t rIn = res(bIn.p, bIn.bytes), rOut = res(bOut.p, bOut.bytes);
    float KX[RW][C], KZ[RW][C], BX[RW][C], BZ[RW][C], gK[RW][C], gX[RW][C], gZ[RW][C];
    float MU[RW][C], MZ[RW][C], LX[RW][C], LZ[RW][C];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int i = w.row0 + r;
        const bool ok = i < g.Nz;
        const unsigned rb = rowb(g, i);
        tile_load<C>(bIn, w, ok, rb + 2u * FB, MU[r]);
        tile_load<C>(bIn, w, ok, rb + FB, LZ[r]);
        tile_load<C>(bIn, w, ok, rb, LX[r]);
        tile_load<C>(bM, w, ok, rb, KX[r]);
        tile_load<C>(bM, w, ok, rb + FB, BX[r]);
        tile_load<C>(bM, w, ok, rb + 2u * FB, BZ[r]);
        if (ok && (w.xpml || row_pml(g, i))) {
            const ZRow z = zrow(g, i);
#pragma unroll
            for (int c = 0; c < C; ++c)
                MZ[r][c] = bld(rIn, pick(z.full, w.zf[c], w.zs[c]), z.base + 3u * FB);
        }
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const bool rp = row_pml(g, w.row0 + r);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            BX[r][c] = bhx[c] * BX[r][c];
            BZ[r][c] = bhz[r] * BZ[r][c];
            KZ[r][c] = btz[r] * KX[r][c];
            KX[r][c] = btx[c] * KX[r][c];
            MZ[r][c] = w.row0 + r < g.Nz && (rp || w.pml[c]) ? MZ[r][c] : MU[r][c];
            gK[r][c] = gX[r][c] = gZ[r][c] = 0.f;
        }
    }

    // injection nodes of the wave's rows (every column)
    cint *rp_ = (cint *)a.rowptr + (size_t)s * (size_t)(g.Nz + 1);
    const int e0 = rp_[imin(w.row0, g.Nz)], e1 = rp_[imin(w.row0 + RW, g.Nz)];

    for (int j = 0; j < a.T; ++j) {
        // R^T r of this step at the wave's nodes, into the LDS image of
        // its rows (each node once; read and cleared below by this wave)
        if (e1 > e0) {
            const float *vals = a.injv + (size_t)j * (size_t)a.nnodes;
            for (int e = e0 + w.lane; e < e1; e += WAVE) {
                const unsigned rc = a.injrc[e];
                const int lc = (int)(rc & 0xffffu) - c0, r = (int)(rc >> 16) - w.row0;
                if ((unsigned)lc < (unsigned)(WAVE * C))
                    inj[w.wv][r][lc % C][lc / C] = vals[e];
            }
        }
        const Base bH = {a.hist - (size_t)j * (size_t)a.lvl + (size_t)s * (size_t)a.ss, FB};
        // p^m rows -1 .. RW+1
        float PN[RW + 3][C];
#pragma unroll
        for (int r = 0; r < RW + 3; ++r) {
            const int i = w.row0 + r - 1;
            tile_load<C>(bH, w, row_ok(g, i), rowb(g, i), PN[r]);
        }
        // q = beta_z K mu_z, rows -1 .. RW+1
        float q[RW + 3][C];
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int c = 0; c < C; ++c)
                q[r + 1][c] = KZ[r][c] * MZ[r][c];
        edge_put<C, NW>(eq, w.wv, 0, w.lane, q[1]);
        edge_put<C, NW>(eq, w.wv, 1, w.lane, q[2]);
        edge_put<C, NW>(eq, w.wv, 2, w.lane, q[RW]);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        edge_get<C, NW>(eq, w.wv - 1, 2, w.lane, q[0]);
        edge_get<C, NW>(eq, w.wv + 1, 0, w.lane, q[RW + 1]);
        edge_get<C, NW>(eq, w.wv + 1, 1, w.lane, q[RW + 2]);
        // lvz_mid at rows i + 1/2, and beta_h bz lvz_mid rows -2 .. RW
        float WZ[RW + 3][C];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const bool ok = w.row0 + r < g.Nz;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float l = LZ[r][c] + (kC1 * (q[r + 2][c] - q[r + 1][c]) +
                                            kC2 * (q[r + 3][c] - q[r][c])) * g.rdz;
                LZ[r][c] = ok ? l : 0.f;
                WZ[r + 2][c] = BZ[r][c] * LZ[r][c];
            }
        }
        edge_put<C, NW>(ew, w.wv, 0, w.lane, WZ[2]);
        edge_put<C, NW>(ew, w.wv, 1, w.lane, WZ[RW]);
        edge_put<C, NW>(ew, w.wv, 2, w.lane, WZ[RW + 1]);
        // lvx_mid, its divergence, and the buoyancy sensitivities
        float dwx[RW][C];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            float qx[C], dqx[C], dpx[C], wx[C];
#pragma unroll
            for (int c = 0; c < C; ++c)
                qx[c] = KX[r][c] * MU[r][c];
            dfwd<C>(qx, dqx);
            dfwd<C>(PN[r + 1], dpx);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float l = LX[r][c] + dqx[c] * g.rdx;
                LX[r][c] = w.ok[c] ? l : 0.f;
                gX[r][c] += LX[r][c] * (-bhx[c] * dpx[c] * g.rdx);
                gZ[r][c] += LZ[r][c] * (-bhz[r] * (kC1 * (PN[r + 2][c] - PN[r + 1][c]) +
                                                   kC2 * (PN[r + 3][c] - PN[r][c])) * g.rdz);
                wx[c] = BX[r][c] * LX[r][c];
            }
            dbwd<C>(wx, dwx[r]);
        }
        __syncthreads();
        edge_get<C, NW>(ew, w.wv - 1, 1, w.lane, WZ[0]);
        edge_get<C, NW>(ew, w.wv - 1, 2, w.lane, WZ[1]);
        edge_get<C, NW>(ew, w.wv + 1, 0, w.lane, WZ[RW + 2]);
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            float v[C];
#pragma unroll
            for (int c = 0; c < C; ++c)
                v[c] = 0.f;
            if (e1 > e0) {
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    v[c] = inj[w.wv][r][c][w.lane];
                    inj[w.wv][r][c][w.lane] = 0.f;
                }
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float dwz = kC1 * (WZ[r + 2][c] - WZ[r + 1][c]) + kC2 * (WZ[r + 3][c] - WZ[r][c]);
                const float t = dwx[r][c] * g.rdx + dwz * g.rdz;
                const float mu = MU[r][c];
                MU[r][c] = ax[c] * mu + t;
                MU[r][c] += v[c];
                gK[r][c] += PN[r + 1][c] * fmaf(-ax[c], mu, MU[r][c]);
                MZ[r][c] = az[r] * MZ[r][c] + t;
                MZ[r][c] += v[c];
                LX[r][c] = ahx[c] * LX[r][c];
                LZ[r][c] = ahz[r] * LZ[r][c];
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int i = w.row0 + r;
        if (i < w.r_lo || i >= w.r_hi)
            continue;
        const unsigned rb = rowb(g, i);
        tile_store<C>(rOut, w, rb, LX[r]);
        tile_store<C>(rOut, w, rb + FB, LZ[r]);
        tile_store<C>(rOut, w, rb + 2u * FB, MU[r]);
        if (w.xpml || row_pml(g, i)) {
            const ZRow z = zrow(g, i);
#pragma unroll
            for (int c = 0; c < C; ++c)
                bst(rOut, w.own[c] ? pick(z.full, w.zf[c], w.zs[c]) : kOOB, z.base + 3u * FB,
                    MZ[r][c]);
        }
    }
    // the shot's partial gradient: this launch's sums (the owned cells of a
    // tile belong to no other)
    const Base bG = {a.gpart + (size_t)id.s * 3u * (size_t)g.N, 3u * FB};
    const rsrc_t rG = res(bG.p, bG.bytes);
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int i = w.row0 + r;
        if (i < w.r_lo || i >= w.r_hi)
            continue;
        const unsigned rb = rowb(g, i);
        float k[C], oK[C], oX[C], oZ[C];
        tile_load<C>(bM, w, true, rb, k);
        tile_load<C>(bG, w, true, rb, oK);
        tile_load<C>(bG, w, true, rb + FB, oX);
        tile_load<C>(bG, w, true, rb + 2u * FB, oZ);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const float rK = k[c] != 0.f ? __builtin_amdgcn_rcpf(k[c]) : 0.f;
            oK[c] = oK[c] + gK[r][c] * rK;
            oX[c] = oX[c] + gX[r][c];
            oZ[c] = oZ[c] + gZ[r][c];
        }
        tile_store<C>(rG, w, rb, oK);
        tile_store<C>(rG, w, rb + FB, oX);
        tile_store<C>(rG, w, rb + 2u * FB, oZ);
    }
}

}  // namespace

void launch_tile_fwd(const Geo &g, const float *tabs, const float *zpad, const float *model,
                     const FwdTile &a, hipStream_t st, hipEvent_t e0, hipEvent_t e1)
{
    const unsigned blocks = (unsigned)(a.x.n * a.z.n) * (unsigned)a.S;
    hipExtLaunchKernelGGL((k_tile_fwd<kTileCols, kTileRows, kTileWaves>), dim3(blocks),
                          dim3(kTileWaves * WAVE), 0, st, e0, e1, 0, g, tabs, zpad, model, a);
}

void launch_tile_adj(const Geo &g, const float *tabs, const float *zpad, const float *model,
                     const AdjTile &a, hipStream_t st, hipEvent_t e0, hipEvent_t e1)
{
    const unsigned blocks = (unsigned)(a.x.n * a.z.n) * (unsigned)a.S;
    hipExtLaunchKernelGGL((k_tile_adj<kTileCols, kTileRows, kTileWaves>), dim3(blocks),
                          dim3(kTileWaves * WAVE), 0, st, e0, e1, 0, g, tabs, zpad, model, a);
}

}  // namespace fwi

// Batched path for problems whose state stays in the caches: several time
// steps per launch, with the whole state of a tile of the grid in registers.
//
// A workgroup of NW waves owns a tile of 64 columns by NW RW rows of one
// shot; a wave holds RW of its rows, a lane one column.  The tile's fields, model and (adjoint) gradient sums are loaded once, advanced
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

// First node of tile k and the nodes it owns.
__device__ inline int tile_first(const TileAxis &a, int k)
{
    return a.n == 1 ? 0 : k * a.last / (a.n - 1);
}
__device__ inline int tile_lo(const TileAxis &a, int k)
{
    return k == 0 ? 0 : tile_first(a, k) + a.halo;
}
__device__ inline int tile_hi(const TileAxis &a, int k)
{
    return k == a.n - 1 ? a.len : tile_first(a, k + 1) + a.halo;
}

// A lane's column in its tile.
struct TileLane {
    int lane, wv, j0, row0;     // lane, wave, column, the wave's first row
    int r_lo, r_hi;             // owned rows
    bool ok, own, pml;          // column inside the grid, owned, in the absorbing layer
    unsigned v, vw;             // lane offset of loads and of stores
    unsigned zf, zs;            // split offsets on full and middle rows
    bool xpml;                  // some column of the tile lies in the layer
};

template <int RW>
__device__ inline void tile_lane(const Geo &g, const TileAxis &x, const TileAxis &z, int tx,
                                 int tz, TileLane &w)
{
    w.lane = threadIdx.x & (WAVE - 1);
    w.wv = uni((int)(threadIdx.x / WAVE));
    const int c0 = tile_first(x, tx), lo = tile_lo(x, tx), hi = tile_hi(x, tx);
    w.j0 = c0 + w.lane;
    w.row0 = tile_first(z, tz) + w.wv * RW;
    w.r_lo = tile_lo(z, tz);
    w.r_hi = tile_hi(z, tz);
    w.xpml = c0 < g.npml || c0 + WAVE > g.Nx - g.npml;
    const int j = w.j0;
    w.ok = j < g.Nx;
    w.own = j >= lo && j < hi;
    w.pml = j < g.npml || j >= g.Nx - g.npml;
    w.v = w.ok ? 4u * (unsigned)j : kOOB;
    w.vw = w.own ? w.v : kOOB;
    w.zf = w.v;
    w.zs = !w.ok ? kOOB
           : j < g.npml ? 4u * (unsigned)j
           : j >= g.Nx - g.npml ? 4u * (unsigned)(j - (g.Nx - 2 * g.npml)) : kOOB;
}

__device__ inline bool row_pml(const Geo &g, int r) { return r < g.npml || r >= g.Nz - g.npml; }

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

// A value of a row (zero outside the grid; ok is uniform).
__device__ inline float tile_load(const Base &b, const TileLane &w, bool ok, unsigned soff)
{
    const rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
        (void *)b.p, (short)0, ok ? (int)(b.bytes + kSlack) : 0, kRsrcWord3);
    return bld(r, w.v, soff);
}

// The horizontal differences of wave_dev.h, one column a lane.
__device__ inline float tile_dfwd(float v)
{
    const float a[1] = {v};
    float d[1];
    dfwd<1>(a, d);
    return d[0];
}
__device__ inline float tile_dbwd(float v)
{
    const float a[1] = {v};
    float d[1];
    dbwd<1>(a, d);
    return d[0];
}

// A wave's rows at its edges, for its neighbours: three rows a wave.
template <int NW>
struct Edge {
    float v[NW][3][WAVE];
    __device__ float get(int wv, int q, int lane) const
    {
        return (unsigned)wv < (unsigned)NW ? v[wv][q][lane] : 0.f;
    }
};

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

template <int RW, int NW>
__global__ void __launch_bounds__(NW * WAVE) __attribute__((amdgpu_waves_per_eu(8, 8)))
    k_tile_fwd(Geo g, const float *__restrict__ tabs, const float *__restrict__ zpad,
               const float *__restrict__ model, FwdTile a)
{
    __shared__ Edge<NW> ep, ev;
    const TileId id = tile_id(a.x, a.z);
    TileLane w;
    tile_lane<RW>(g, a.x, a.z, id.tx, id.tz, w);
    const unsigned FB = 4u * (unsigned)g.N;
    const int ZP = g.Nz + 2 * kZPad;
    const Base bM = {model, 3u * FB}, bIn = base_of(a.in, id.s), bOut = base_of(a.out, id.s);
    const rsrc_t rIn = res(bIn.p, bIn.bytes), rOut = res(bOut.p, bOut.bytes);

    const int jt = imin(w.j0, g.Nx - 1);
    const float ax = w.ok ? tabs[jt] : 0.f, btx = w.ok ? tabs[g.Nx + jt] : 0.f;
    const float ahx = w.ok ? tabs[2 * g.Nx + jt] : 0.f, bhx = w.ok ? tabs[3 * g.Nx + jt] : 0.f;
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
    float P[RW + 3], VZ[RW + 3], VX[RW], PZ[RW];
    float BX[RW], BZ[RW], KX[RW], KZ[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int i = w.row0 + r;
        const bool ok = i < g.Nz;
        const unsigned rb = rowb(g, i);
        P[r + 1] = tile_load(bIn, w, ok, rb + 2u * FB);
        VZ[r + 2] = tile_load(bIn, w, ok, rb + FB);
        VX[r] = tile_load(bIn, w, ok, rb);
        KX[r] = tile_load(bM, w, ok, rb);
        BX[r] = tile_load(bM, w, ok, rb + FB);
        BZ[r] = tile_load(bM, w, ok, rb + 2u * FB);
        PZ[r] = 0.f;
        if (ok && (w.xpml || row_pml(g, i))) {
            const ZRow z = zrow(g, i);
            PZ[r] = bld(rIn, pick(z.full, w.zf, w.zs), z.base + 3u * FB);
        }
    }
    // source: its bilinear cell's first row, the cell's weights and K on its
    // two rows
    cint *sij = (cint *)a.src_ij + 2 * id.s;
    cfloat *sw4 = ctab(a.src_w) + 4 * id.s;
    const int srow = sij[0], scol = sij[1];
    const bool src = srow + 1 >= w.row0 && srow < w.row0 + RW;
    const float Ka = tile_load(bM, w, src, rowb(g, srow));
    const float Kb = tile_load(bM, w, src, rowb(g, srow + 1));
    cfloat *Q = ctab(a.Q) + (size_t)id.s * (size_t)a.nt + a.n;

#pragma unroll
    for (int r = 0; r < RW; ++r) {
        BX[r] = bhx * BX[r];
        BZ[r] = bhz[r] * BZ[r];
        KZ[r] = btz[r] * KX[r];
        KX[r] = btx * KX[r];
    }

    for (int j = 0; j < a.T; ++j) {
        const float dq = g.dt * Q[j];
        ep.v[w.wv][0][w.lane] = P[1];
        ep.v[w.wv][1][w.lane] = P[2];
        ep.v[w.wv][2][w.lane] = P[RW];
        __syncthreads();
        P[0] = ep.get(w.wv - 1, 2, w.lane);
        P[RW + 1] = ep.get(w.wv + 1, 0, w.lane);
        P[RW + 2] = ep.get(w.wv + 1, 1, w.lane);
        // vz^{n+1/2} at rows i + 1/2
#pragma unroll
        for (int r = 0; r < RW; ++r)
            VZ[r + 2] = ahz[r] * VZ[r + 2] -
                        BZ[r] * (kC1 * (P[r + 2] - P[r + 1]) + kC2 * (P[r + 3] - P[r])) * g.rdz;
        ev.v[w.wv][0][w.lane] = VZ[2];
        ev.v[w.wv][1][w.lane] = VZ[RW];
        ev.v[w.wv][2][w.lane] = VZ[RW + 1];
        // vx^{n+1/2} at columns j + 1/2
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const float dp = tile_dfwd(P[r + 1]);
            VX[r] = ahx * VX[r] - BX[r] * dp * g.rdx;
        }
        __syncthreads();
        VZ[0] = ev.get(w.wv - 1, 1, w.lane);
        VZ[1] = ev.get(w.wv - 1, 2, w.lane);
        VZ[RW + 2] = ev.get(w.wv + 1, 0, w.lane);
        // p^{n+1}
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const bool rp = row_pml(g, w.row0 + r);
            const float dvx = tile_dbwd(VX[r]);
            const float dvz = kC1 * (VZ[r + 2] - VZ[r + 1]) + kC2 * (VZ[r + 3] - VZ[r]);
            const float pz = PZ[r];
            const float px = ax * (P[r + 1] - pz) - KX[r] * dvx * g.rdx;
            const float pzn = az[r] * pz - KZ[r] * dvz * g.rdz;
            P[r + 1] = px + pzn;
            // the split is kept only where the layer has one
            PZ[r] = rp || w.pml ? pzn : 0.f;
        }
        if (src) {
            const int dj = w.j0 - scol;
            const float swa = dj == 0 ? dq * sw4[0] : (dj == 1 ? dq * sw4[1] : 0.f);
            const float swb = dj == 0 ? dq * sw4[2] : (dj == 1 ? dq * sw4[3] : 0.f);
#pragma unroll
            for (int r = 0; r < RW; ++r)
                if ((unsigned)(w.row0 + r - srow) < 2u)
                    P[r + 1] += (w.row0 + r == srow ? Ka : Kb) *
                                (w.row0 + r == srow ? swa : swb);
        }
        if (a.hist) {
            const rsrc_t rH =
                res(a.hist + (size_t)j * (size_t)a.lvl + (size_t)id.s * (size_t)a.ss, FB);
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                const int i = w.row0 + r;
                if (i >= w.r_lo && i < w.r_hi)
                    bst(rH, w.vw, rowb(g, i), P[r + 1]);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int i = w.row0 + r;
        if (i < w.r_lo || i >= w.r_hi)
            continue;
        const unsigned rb = rowb(g, i);
        bst(rOut, w.vw, rb, VX[r]);
        bst(rOut, w.vw, rb + FB, VZ[r + 2]);
        bst(rOut, w.vw, rb + 2u * FB, P[r + 1]);
        if (w.xpml || row_pml(g, i)) {
            const ZRow z = zrow(g, i);
            bst(rOut, w.own ? pick(z.full, w.zf, w.zs) : kOOB, z.base + 3u * FB, PZ[r]);
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

template <int RW, int NW>
__global__ void __launch_bounds__(NW * WAVE)
    k_tile_adj(Geo g, const float *__restrict__ tabs, const float *__restrict__ zpad,
               const float *__restrict__ model, AdjTile a)
{
    __shared__ Edge<NW> eq, ew;
    __shared__ float inj[NW][RW][WAVE];   // R^T r of the step at the tile's nodes
    const TileId id = tile_id(a.x, a.z);
    TileLane w;
    tile_lane<RW>(g, a.x, a.z, id.tx, id.tz, w);
    const unsigned FB = 4u * (unsigned)g.N;
    const int ZP = g.Nz + 2 * kZPad;
    const Base bM = {model, 3u * FB};
    const int c0 = tile_first(a.x, id.tx);
#pragma unroll
    for (int r = 0; r < RW; ++r)
        inj[w.wv][r][w.lane] = 0.f;

    const int jt = imin(w.j0, g.Nx - 1);
    const float ax = w.ok ? tabs[jt] : 0.f, btx = w.ok ? tabs[g.Nx + jt] : 0.f;
    const float ahx = w.ok ? tabs[2 * g.Nx + jt] : 0.f, bhx = w.ok ? tabs[3 * g.Nx + jt] : 0.f;
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
    float KX[RW], KZ[RW], BX[RW], BZ[RW], gK[RW], gX[RW], gZ[RW];
    float MU[RW], MZ[RW], LX[RW], LZ[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int i = w.row0 + r;
        const bool ok = i < g.Nz;
        const unsigned rb = rowb(g, i);
        MU[r] = tile_load(bIn, w, ok, rb + 2u * FB);
        LZ[r] = tile_load(bIn, w, ok, rb + FB);
        LX[r] = tile_load(bIn, w, ok, rb);
        KX[r] = tile_load(bM, w, ok, rb);
        BX[r] = tile_load(bM, w, ok, rb + FB);
        BZ[r] = tile_load(bM, w, ok, rb + 2u * FB);
        if (ok && (w.xpml || row_pml(g, i))) {
            const ZRow z = zrow(g, i);
            MZ[r] = bld(rIn, pick(z.full, w.zf, w.zs), z.base + 3u * FB);
        }
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const bool rp = row_pml(g, w.row0 + r);
        BX[r] = bhx * BX[r];
        BZ[r] = bhz[r] * BZ[r];
        KZ[r] = btz[r] * KX[r];
        KX[r] = btx * KX[r];
        MZ[r] = w.row0 + r < g.Nz && (rp || w.pml) ? MZ[r] : MU[r];
        gK[r] = gX[r] = gZ[r] = 0.f;
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
                if ((unsigned)lc < (unsigned)WAVE)
                    inj[w.wv][r][lc] = vals[e];
            }
        }
        const Base bH = {a.hist - (size_t)j * (size_t)a.lvl + (size_t)s * (size_t)a.ss, FB};
        // p^m rows -1 .. RW+1
        float PN[RW + 3];
#pragma unroll
        for (int r = 0; r < RW + 3; ++r) {
            const int i = w.row0 + r - 1;
            PN[r] = tile_load(bH, w, row_ok(g, i), rowb(g, i));
        }
        // q = beta_z K mu_z, rows -1 .. RW+1
        float q[RW + 3];
#pragma unroll
        for (int r = 0; r < RW; ++r)
            q[r + 1] = KZ[r] * MZ[r];
        eq.v[w.wv][0][w.lane] = q[1];
        eq.v[w.wv][1][w.lane] = q[2];
        eq.v[w.wv][2][w.lane] = q[RW];
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        q[0] = eq.get(w.wv - 1, 2, w.lane);
        q[RW + 1] = eq.get(w.wv + 1, 0, w.lane);
        q[RW + 2] = eq.get(w.wv + 1, 1, w.lane);
        // lvz_mid at rows i + 1/2, and beta_h bz lvz_mid rows -2 .. RW
        float WZ[RW + 3];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const bool ok = w.row0 + r < g.Nz;
            const float l =
                LZ[r] + (kC1 * (q[r + 2] - q[r + 1]) + kC2 * (q[r + 3] - q[r])) * g.rdz;
            LZ[r] = ok ? l : 0.f;
            WZ[r + 2] = BZ[r] * LZ[r];
        }
        ew.v[w.wv][0][w.lane] = WZ[2];
        ew.v[w.wv][1][w.lane] = WZ[RW];
        ew.v[w.wv][2][w.lane] = WZ[RW + 1];
        // lvx_mid, its divergence, and the buoyancy sensitivities
        float dwx[RW];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const float qx = KX[r] * MU[r], dqx = tile_dfwd(qx), dpx = tile_dfwd(PN[r + 1]);
            const float l = LX[r] + dqx * g.rdx;
            LX[r] = w.ok ? l : 0.f;
            gX[r] += LX[r] * (-bhx * dpx * g.rdx);
            gZ[r] += LZ[r] * (-bhz[r] * (kC1 * (PN[r + 2] - PN[r + 1]) +
                                         kC2 * (PN[r + 3] - PN[r])) * g.rdz);
            dwx[r] = tile_dbwd(BX[r] * LX[r]);
        }
        __syncthreads();
        WZ[0] = ew.get(w.wv - 1, 1, w.lane);
        WZ[1] = ew.get(w.wv - 1, 2, w.lane);
        WZ[RW + 2] = ew.get(w.wv + 1, 0, w.lane);
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            float v = 0.f;
            if (e1 > e0) {
                v = inj[w.wv][r][w.lane];
                inj[w.wv][r][w.lane] = 0.f;
            }
            const float dwz = kC1 * (WZ[r + 2] - WZ[r + 1]) + kC2 * (WZ[r + 3] - WZ[r]);
            const float t = dwx[r] * g.rdx + dwz * g.rdz;
            const float mu = MU[r];
            MU[r] = ax * mu + t;
            MU[r] += v;
            gK[r] += PN[r + 1] * fmaf(-ax, mu, MU[r]);
            MZ[r] = az[r] * MZ[r] + t;
            MZ[r] += v;
            LX[r] = ahx * LX[r];
            LZ[r] = ahz[r] * LZ[r];
        }
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int i = w.row0 + r;
        if (i < w.r_lo || i >= w.r_hi)
            continue;
        const unsigned rb = rowb(g, i);
        bst(rOut, w.vw, rb, LX[r]);
        bst(rOut, w.vw, rb + FB, LZ[r]);
        bst(rOut, w.vw, rb + 2u * FB, MU[r]);
        if (w.xpml || row_pml(g, i)) {
            const ZRow z = zrow(g, i);
            bst(rOut, w.own ? pick(z.full, w.zf, w.zs) : kOOB, z.base + 3u * FB, MZ[r]);
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
        const float k = tile_load(bM, w, true, rb), oK = tile_load(bG, w, true, rb);
        const float oX = tile_load(bG, w, true, rb + FB);
        const float oZ = tile_load(bG, w, true, rb + 2u * FB);
        const float rK = k != 0.f ? __builtin_amdgcn_rcpf(k) : 0.f;
        bst(rG, w.vw, rb, oK + gK[r] * rK);
        bst(rG, w.vw, rb + FB, oX + gX[r]);
        bst(rG, w.vw, rb + 2u * FB, oZ + gZ[r]);
    }
}

}  // namespace

void launch_tile_fwd(const Geo &g, const float *tabs, const float *zpad, const float *model,
                     const FwdTile &a, hipStream_t st, hipEvent_t e0, hipEvent_t e1)
{
    const unsigned blocks = (unsigned)(a.x.n * a.z.n) * (unsigned)a.S;
    hipExtLaunchKernelGGL((k_tile_fwd<kTileRows, kTileWaves>), dim3(blocks),
                          dim3(kTileWaves * WAVE), 0, st, e0, e1, 0, g, tabs, zpad, model, a);
}

void launch_tile_adj(const Geo &g, const float *tabs, const float *zpad, const float *model,
                     const AdjTile &a, hipStream_t st, hipEvent_t e0, hipEvent_t e1)
{
    const unsigned blocks = (unsigned)(a.x.n * a.z.n) * (unsigned)a.S;
    hipExtLaunchKernelGGL((k_tile_adj<kTileRows, kTileWaves>), dim3(blocks),
                          dim3(kTileWaves * WAVE), 0, st, e0, e1, 0, g, tabs, zpad, model, a);
}

}  // namespace fwi

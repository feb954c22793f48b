// Batched path: every launch covers every shot of the model, for one time
// step (k_fwd, k_adj) or two (k_fwd2, k_adj2: the intermediate state stays
// on chip).
//
// Each wave64 owns a strip of consecutive columns and a band of rows, and
// marches down the band one row at a time.  A lane holds C adjacent columns
// (C = 1, 2 or 4), read and written with one 4C-byte buffer access, so the
// per-row scalar work and the memory instructions are shared by C cells.
// The strip is 64 C columns wide, of which ceil(3 / C) lanes on each side
// are halo (the stencil reaches 3 columns through the two half steps).  The
// vertical parts of the stencils live in per-lane register windows (the
// rows above and below the current one); the horizontal parts take the
// neighbouring lane's edge columns with DPP wave shifts, so the kernels need
// no barriers and share nothing between waves (k_adj2 keeps what waits for
// its second step in LDS words of the lane's own).  Velocity and pressure
// half-steps are fused: the new velocities of a row are formed and consumed
// by the new pressure of the same row in registers, so every wavefield value
// is read once and written once per step (ping-pong buffers, since
// neighbouring strips and bands still read the old level).
//
// A wave advances SPG shots of the same model together, row by row: the
// model coefficients of a row are read once for all of them, and in the
// adjoint kernel the gradient contributions of the SPG shots are summed in
// registers and added to the group's partial gradient once per row.  The
// shot count of a launch is padded to a multiple of SPG with all-zero shots
// (no source, no receivers), so every group is full.
//
// The loads of row i+1 are issued before the arithmetic and the stores of
// row i into one of two alternating register sets, so their latency overlaps
// a row of work and no register copies (which would wait for them) are
// needed.  The adjoint reads the values it needs only at the end of a row
// (the partial gradient) into a single set, issued at the start of the row
// before the next row's loads.  Loads are unconditional: rows outside the
// grid or past the band are read through an out-of-range lane offset, which
// returns zero without touching memory, so the memory counters see the same
// sequence on every row.
//
// Receiver sampling is a separate small launch, and the receivers' sums of the
// adjoint source (R^T r) are staged per node by one, up to 64 steps at a time.  The
// kernels only add or write the nodes listed for their strip and row: k_adj
// and k_adj2 add the staged sums to the new adjoint pressure, and k_fwd2 writes
// the receiver nodes of an intermediate level that is only sampled, for a node
// sampling launch after it.
// Workgroups are numbered so that each XCD receives a contiguous range of
// waves (neighbouring strips, the shot groups of a band and neighbouring
// bands share its L2).
#include "wave_dev.h"

#include <hip/hip_ext.h>
#include <type_traits>

namespace fwi {

namespace {

constexpr int NTHR = 256;  // 4 independent waves per workgroup

// Strip geometry for C columns per lane and a stencil reach of R columns
// (3 for one time step, 6 for two).
template <int C, int R = HALO>
struct Lanes {
    static constexpr int HL = (R + C - 1) / C;      // halo lanes on each side
    static constexpr int W = (WAVE - 2 * HL) * C;   // output columns per strip
};

template <int C>
struct WaveGeo {
    int lane, j0;         // lane and its first column
    bool colok[C];        // column inside the grid
    unsigned vcol;        // lane byte offset for loads, kOOB if its first column is outside
    unsigned vcolw;       // for whole-lane stores: kOOB unless an output lane fully inside
    unsigned vtail[C];    // element stores of the output lane holding the last column
    unsigned zf[C], zs[C];    // split offsets on full rows / middle rows (loads)
    unsigned zfw[C], zsw[C];  // the same for stores
    bool colpml[C];       // column inside the absorbing layer
    int i0, i1;           // owned rows [i0, i1)
    int s0;               // shots [s0, s0 + SPG)
    int strip, band, grp;
};

template <int C, int R = HALO>
__device__ inline bool wave_geo(const Geo &g, const Sweep &sw, WaveGeo<C> &w)
{
    constexpr int HL = Lanes<C, R>::HL, W = Lanes<C, R>::W;
    w.lane = threadIdx.x & (WAVE - 1);
    // wave index, made provably uniform so that everything derived from it
    // (rows, shots, buffer resources) lives in scalar registers
    int wid = uni(xcd_item(blockIdx.x, gridDim.x) * (NTHR / WAVE) + (int)(threadIdx.x / WAVE));
    if (wid >= sw.nwaves)
        return false;
    // strip fastest, then shot group, then band: the groups of a band run
    // together, so the model rows they all read are shared in L2
    w.strip = wid % sw.nstrips;
    int rest = wid / sw.nstrips;
    w.grp = rest % sw.ngroups;
    w.band = rest / sw.ngroups;
    w.j0 = w.strip * W + (w.lane - HL) * C;
    const bool outl = w.lane >= HL && w.lane < WAVE - HL;
    const bool in0 = w.j0 >= 0 && w.j0 < g.Nx;
    const bool whole = in0 && w.j0 + C - 1 < g.Nx;
    w.vcol = in0 ? 4u * (unsigned)w.j0 : kOOB;
    w.vcolw = outl && whole ? w.vcol : kOOB;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int j = w.j0 + c;
        w.colok[c] = j >= 0 && j < g.Nx;
        w.colpml[c] = j < g.npml || j >= g.Nx - g.npml;
        w.vtail[c] = outl && in0 && !whole && w.colok[c] ? 4u * (unsigned)j : kOOB;
        unsigned side = kOOB;
        if (w.colok[c] && j < g.npml)
            side = 4u * (unsigned)j;
        else if (w.colok[c] && j >= g.Nx - g.npml)
            side = 4u * (unsigned)(j - (g.Nx - 2 * g.npml));
        w.zf[c] = w.colok[c] ? 4u * (unsigned)j : kOOB;
        w.zs[c] = side;
        w.zfw[c] = outl ? w.zf[c] : kOOB;
        w.zsw[c] = outl ? side : kOOB;
    }
    w.i0 = w.band * sw.H;
    w.i1 = imin(w.i0 + sw.H, g.Nz);
    w.s0 = w.grp * sw.spg;
    return true;
}

// Whole-lane store plus the element stores of the lane holding the last
// grid column (on = false drops both).
template <int C>
__device__ inline void vst_row(rsrc_t r, const WaveGeo<C> &w, bool on, unsigned soff,
                               const float (&v)[C])
{
    vst<C>(r, on ? w.vcolw : kOOB, soff, v);
#pragma unroll
    for (int c = 0; c + 1 < C; ++c)
        bst(r, on ? w.vtail[c] : kOOB, soff, v[c]);
}

// Zero the elements past the last grid column (they were read from the
// next row or past the field and feed horizontal differences).
template <int C>
__device__ inline void mask_cols(const WaveGeo<C> &w, float (&v)[C])
{
#pragma unroll
    for (int c = 1; c < C; ++c)
        v[c] = w.colok[c] ? v[c] : 0.f;
}

// Split element offsets of row i for loads (live = false: none) and stores.
template <int C>
__device__ inline void zoffs(const WaveGeo<C> &w, const ZRow &z, bool live, unsigned (&o)[C])
{
#pragma unroll
    for (int c = 0; c < C; ++c)
        o[c] = live ? pick(z.full, w.zf[c], w.zs[c]) : kOOB;
}
template <int C>
__device__ inline void zoffs_w(const WaveGeo<C> &w, const ZRow &z, unsigned (&o)[C])
{
#pragma unroll
    for (int c = 0; c < C; ++c)
        o[c] = pick(z.full, w.zfw[c], w.zsw[c]);
}

// One resource for the records of shots [s0, s0 + SPG): shot s0 + k sits
// k * sbytes bytes after the first (uniform offset skoff).
__device__ inline rsrc_t grp_res(const Recd &r, int s0, int spg)
{
    return res((const float *)((const char *)r.base + (size_t)s0 * r.sbytes),
               (unsigned)(spg - 1) * r.sbytes + r.bytes);
}
__device__ inline unsigned skoff(const Recd &r, int k) { return (unsigned)k * r.sbytes; }

// Lane offsets of the loads of row r: the lane offset, or kOOB where the row
// (r, r+1, r+3) lies outside the grid or r lies past the band.
struct RowOff {
    unsigned o0, o1, o3;
};
template <int C>
__device__ inline RowOff row_off(const Geo &g, const WaveGeo<C> &w, int r)
{
    const bool live = r < w.i1;
    RowOff o;
    o.o0 = live ? w.vcol : kOOB;
    o.o1 = live && r + 1 < g.Nz ? w.vcol : kOOB;
    o.o3 = live && r + 3 < g.Nz ? w.vcol : kOOB;
    return o;
}

// x tables of the lane's columns (alpha, beta at nodes, alpha_h, beta_h at
// half nodes); zero outside the grid.
template <int C>
struct XTab {
    float ax[C], btx[C], ahx[C], bhx[C];
};
template <int C>
__device__ inline void xtab(const Geo &g, const float *__restrict__ tabs, const WaveGeo<C> &w,
                            XTab<C> &t)
{
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int jc = imin(imax(w.j0 + c, 0), g.Nx - 1);
        const bool ok = w.colok[c];
        t.ax[c] = ok ? tabs[jc] : 0.f;
        t.btx[c] = ok ? tabs[g.Nx + jc] : 0.f;
        t.ahx[c] = ok ? tabs[2 * g.Nx + jc] : 0.f;
        t.bhx[c] = ok ? tabs[3 * g.Nx + jc] : 0.f;
    }
}

// ---------------------------------------------------------------- forward

template <int SPG, int C>
struct FRow {
    float K[C], bx[C], bz1[C];                              // K, bx at r; bz at r+1
    float p3[SPG][C], vz1[SPG][C], vx[SPG][C], pz[SPG][C];  // p at r+3, vz at r+1, vx, split at r
};

template <int SPG, int C>
__global__ void __launch_bounds__(NTHR)
    k_fwd(Geo g, const float *__restrict__ tabs, const float *model, const SweepTables *T, int S,
          Sweep sw, FwdStep a)
{
    WaveGeo<C> w;
    if (!wave_geo<C>(g, sw, w))
        return;
    XTab<C> xt;
    xtab<C>(g, tabs, w, xt);
    // z tables: alpha, beta at nodes, alpha_h, beta_h at half nodes
    cfloat *zaz = ctab(tabs + 4 * g.Nx), *zbz = zaz + g.Nz;
    cfloat *zahz = zbz + g.Nz, *zbhz = zahz + g.Nz;
    const unsigned FB = 4u * (unsigned)g.N;
    const rsrc_t rM = res(model, 3u * FB);   // K, bx, bz at 0, FB, 2 FB
    const unsigned rowN = 4u * (unsigned)g.Nx;
    const rsrc_t rPin = grp_res(a.pin, w.s0, SPG), rVin = grp_res(a.vin, w.s0, SPG);
    const rsrc_t rPout = grp_res(a.pout, w.s0, SPG), rVout = grp_res(a.vout, w.s0, SPG);

    float P[SPG][4][C];   // pressure rows i .. i+3
    float VZ[SPG][3][C];  // new vz rows i-2 .. i
    // source: first row of its bilinear cell and this lane's injection
    // weights dt Q w / (dx dz) on that row and the next
    int srow[SPG];
    float swa[SPG][C], swb[SPG][C];
#pragma unroll
    for (int k = 0; k < SPG; ++k) {
        const int s = w.s0 + k;
        srow[k] = -8;
#pragma unroll
        for (int c = 0; c < C; ++c)
            swa[k][c] = swb[k][c] = 0.f;
        if (s < S) {
            const int2 sij = T->src_ij[s];
            const float4 sw4 = T->src_w[s];
            const float dq = g.dt * a.Q[(long long)s * T->nt + a.n];
            srow[k] = uni(sij.x);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int dj = w.j0 + c - sij.y;
                swa[k][c] = dj == 0 ? dq * sw4.x : (dj == 1 ? dq * sw4.y : 0.f);
                swb[k][c] = dj == 0 ? dq * sw4.z : (dj == 1 ? dq * sw4.w : 0.f);
            }
        }
        const unsigned op = skoff(a.pin, k), ovz = FB + skoff(a.vin, k);
        float pr[6][C];
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const int r = w.i0 - 3 + q;
            vld<C>(rPin, row_ok(g, r) ? w.vcol : kOOB, row_ok(g, r) ? rowb(g, r) + op : 0u, pr[q]);
            mask_cols<C>(w, pr[q]);
        }
        // vz at rows i0-2 .. i0 from p rows r-1 .. r+2
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int r = w.i0 - 2 + q;
            const bool ok = row_ok(g, r);
            const unsigned rb = ok ? rowb(g, r) : 0u, vo = ok ? w.vcol : kOOB;
            float bz[C], vz[C];
            vld<C>(rM, vo, rb + 2u * FB, bz);
            vld<C>(rVin, vo, rb + ovz, vz);
            const float ahz = ok ? zahz[r] : 0.f, bhz = ok ? zbhz[r] : 0.f;
#pragma unroll
            for (int c = 0; c < C; ++c)
                VZ[k][q][c] = ahz * vz[c] -
                              bhz * bz[c] *
                                  (kC1 * (pr[q + 2][c] - pr[q + 1][c]) + kC2 * (pr[q + 3][c] - pr[q][c])) *
                                  g.rdz;
        }
        vst_row<C>(rVout, w, true, rowb(g, w.i0) + FB + skoff(a.vout, k), VZ[k][2]);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            P[k][0][c] = pr[3][c];
            P[k][1][c] = pr[4][c];
            P[k][2][c] = pr[5][c];
            P[k][3][c] = 0.f;
        }
    }

    auto load_row = [&](int r, FRow<SPG, C> &b) {
        const unsigned rb = rowb(g, r);
        const RowOff o = row_off<C>(g, w, r);
        const ZRow z = zrow(g, r);
        unsigned oz[C];
        zoffs<C>(w, z, r < w.i1, oz);
        vld<C>(rM, o.o0, rb, b.K);
        vld<C>(rM, o.o0, rb + FB, b.bx);
        vld<C>(rM, o.o1, rb + rowN + 2u * FB, b.bz1);
#pragma unroll
        for (int k = 0; k < SPG; ++k) {
            const unsigned kp = skoff(a.pin, k), kv = skoff(a.vin, k);
            vld<C>(rPin, o.o3, rb + 3u * rowN + kp, b.p3[k]);
            vld<C>(rVin, o.o1, rb + rowN + FB + kv, b.vz1[k]);
            vld<C>(rVin, o.o0, rb + kv, b.vx[k]);
#pragma unroll
            for (int c = 0; c < C; ++c)
                b.pz[k][c] = bld(rPin, oz[c], z.base + FB + kp);
        }
    };

    auto row = [&](int i, FRow<SPG, C> &b) {
        const unsigned rb = rowb(g, i);
        const bool rn = row_ok(g, i + 1);
        const float ahz1 = rn ? zahz[i + 1] : 0.f, bhz1 = rn ? zbhz[i + 1] : 0.f;
        const float az = zaz[i], btz = zbz[i];
        const ZRow z = zrow(g, i);
        unsigned zw[C];
        zoffs_w<C>(w, z, zw);
        const bool more = i + 1 < w.i1;   // this wave owns vz row i+1
#pragma unroll
        for (int k = 0; k < SPG; ++k) {
            mask_cols<C>(w, b.p3[k]);
            float vzn[C], vxn[C], dp[C], pn[C], pzn[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                P[k][3][c] = b.p3[k][c];
                // vz at row (i+1) + 1/2
                vzn[c] = ahz1 * b.vz1[k][c] -
                         bhz1 * b.bz1[c] *
                             (kC1 * (P[k][2][c] - P[k][1][c]) + kC2 * (P[k][3][c] - P[k][0][c])) * g.rdz;
            }
            // vx at (i, j + 1/2)
            dfwd<C>(P[k][0], dp);
#pragma unroll
            for (int c = 0; c < C; ++c)
                vxn[c] = xt.ahx[c] * b.vx[k][c] - xt.bhx[c] * b.bx[c] * dp[c] * g.rdx;
            // pressure at n+1 (the split is zero where the layer has none,
            // and alpha = 1, beta = dt there)
            float dvx[C];
            dbwd<C>(vxn, dvx);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float dvz = kC1 * (VZ[k][2][c] - VZ[k][1][c]) + kC2 * (vzn[c] - VZ[k][0][c]);
                const float pz = b.pz[k][c];
                const float px = xt.ax[c] * (P[k][0][c] - pz) - xt.btx[c] * b.K[c] * dvx[c] * g.rdx;
                pzn[c] = az * pz - btz * b.K[c] * dvz * g.rdz;
                pn[c] = px + pzn[c];
            }
            if ((unsigned)(i - srow[k]) < 2u) {
#pragma unroll
                for (int c = 0; c < C; ++c)
                    pn[c] += b.K[c] * (i == srow[k] ? swa[k][c] : swb[k][c]);
            }
            const unsigned kv = skoff(a.vout, k), kp = skoff(a.pout, k);
            vst_row<C>(rVout, w, true, rb + kv, vxn);
            vst_row<C>(rVout, w, more, rb + rowN + FB + kv, vzn);
            vst_row<C>(rPout, w, true, rb + kp, pn);
#pragma unroll
            for (int c = 0; c < C; ++c)
                bst(rPout, zw[c], z.base + FB + kp, pzn[c]);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                VZ[k][0][c] = VZ[k][1][c];
                VZ[k][1][c] = VZ[k][2][c];
                VZ[k][2][c] = vzn[c];
                P[k][0][c] = P[k][1][c];
                P[k][1][c] = P[k][2][c];
                P[k][2][c] = P[k][3][c];
            }
        }
    };

    FRow<SPG, C> A, B;
    load_row(w.i0, A);
    for (int i = w.i0;;) {
        load_row(i + 1, B);
        row(i, A);
        if (++i >= w.i1)
            break;
        load_row(i + 1, A);
        row(i, B);
        if (++i >= w.i1)
            break;
    }
}

// Per-row uniform values of 64 consecutive rows, one row a lane: the z damping
// tables (zero outside the grid) and the packed receiver-node entries of the
// wave's shots.  A row's values are read out with v_readlane: scalar loads
// return out of order, so a wait for a table value would also wait for the
// node entries prefetched with it, which miss the caches on every row.
template <int NW>
struct RowLanes {
    int base;              // row of lane 0
    float az, bz, ahz, bhz;
    unsigned win[NW];
    __device__ float at(float v, int r) const
    {
        return __builtin_bit_cast(
            float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), r - base));
    }
    __device__ unsigned node(int k, int r) const
    {
        return (unsigned)__builtin_amdgcn_readlane((int)win[k], r - base);
    }
    // Rows [r, r + 64) (clamped to the tables' padding).  node_row(k): entry of
    // row 0 of the wave's k-th shot and strip, row_stride entries a row.
    template <typename F>
    __device__ void load(const Geo &g, const float *zpad, int r, int lane, int lo, int hi, F node_row,
                         int row_stride)
    {
        base = r;
        const int ZP = g.Nz + 2 * kZPad;
        const int i = imin(imax(r + lane, -kZPad), g.Nz + kZPad - 1);
        const float *z = zpad + kZPad + i;
        az = z[0];
        bz = z[ZP];
        ahz = z[2 * ZP];
        bhz = z[3 * ZP];
        const int n = imin(imax(r + lane, lo), hi);
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const unsigned *q = node_row(k);
            win[k] = q ? q[(long long)n * row_stride] : 0u;
        }
        // (used here, so that the wait for them stays in this branch of the row
        // loop: at its end it would wait for the next row's loads on every row)
        asm volatile("" ::"v"(az), "v"(bz), "v"(ahz), "v"(bhz));
#pragma unroll
        for (int k = 0; k < NW; ++k)
            asm volatile("" ::"v"(win[k]));
    }
};

// A run of 64 receiver nodes of one shot and strip, one a lane: their grid
// columns and a value each.  A strip's nodes lie in row order, so a wave marching
// down its band reads a run every 64 nodes.
struct NodeLanes {
    int base = 0, end = 0;   // node indices [base, end) held
    int col;
    float val;
    __device__ void load(const int *cols, const float *vals, int first, int lane)
    {
        base = first;
        end = first + WAVE;
        col = cols[first + lane];
        val = vals[first + lane];
        asm volatile("" ::"v"(col), "v"(val));   // (wait here, as RowLanes::load)
    }
};

// ------------------------------------------------------- forward, two steps
//
// Steps n -> n+1 -> n+2 in one pass: the wave computes step n+1 on rows
// [i0-3, i1+3) of its band (the second step needs p^{n+1} three rows and
// three columns beyond its own rows and columns, so strips carry a 6-column
// halo and step-one rows run three ahead), keeps step n+1's velocities,
// split and model in three-row delay lines and its pressure in a window,
// and computes step n+2 three rows behind.  Only p^{n+1} of the intermediate
// level is written, to the `mid` record (the pressure history the adjoint
// reads, which needs no split); the intermediate velocities never leave
// registers, so two steps cost one read and one write of the state.

template <int SPG, int C>
__global__ void __launch_bounds__(NTHR)
    k_fwd2(Geo g, const float *__restrict__ tabs, const float *model, const SweepTables *T, int S,
           Sweep sw, FwdStep2 a)
{
    WaveGeo<C> w;
    if (!wave_geo<C, 2 * HALO>(g, sw, w))
        return;
    XTab<C> xt;
    xtab<C>(g, tabs, w, xt);
    const unsigned FB = 4u * (unsigned)g.N;
    const rsrc_t rM = res(model, 3u * FB);
    const rsrc_t rPin = grp_res(a.pin, w.s0, SPG), rVin = grp_res(a.vin, w.s0, SPG);
    const rsrc_t rPmid = grp_res(a.pmid, w.s0, SPG);
    const rsrc_t rPout = grp_res(a.pout, w.s0, SPG), rVout = grp_res(a.vout, w.s0, SPG);
    // row byte offset of row r plus `extra`, or 0 when row r is outside the
    // grid (its lane offset is then kOOB)
    auto rofs = [&](int r, unsigned extra) -> unsigned {
        return row_ok(g, r) ? rowb(g, r) + extra : 0u;
    };
    const int t0 = w.i0 - 3;
    // z tables and, where the intermediate level is only sampled, its nodes
    // (rows without nodes and padding shots hold 0)
    cfloat *zaz = ctab(a.zpad) + kZPad, *zbz = zaz + g.Nz + 2 * kZPad;
    cfloat *zahz = zbz + g.Nz + 2 * kZPad, *zbhz = zahz + g.Nz + 2 * kZPad;
    int nbase[SPG];   // first node of the wave's strip
#pragma unroll
    for (int k = 0; k < SPG; ++k)
        nbase[k] = a.midw == 1 && w.s0 + k < S ? ((cint *)a.nptr)[(w.s0 + k) * sw.nstrips + w.strip] : 0;

    float P1[SPG][4][C];    // p^n rows t .. t+3
    float VZ1[SPG][3][C];   // vz^{n+1/2} rows t-2 .. t
    float P2[SPG][3][C];    // p^{n+1} rows t-3 .. t-1
    float VZ2[SPG][3][C];   // vz^{n+3/2} rows r-2 .. r (r = t-3)
    float DVZ[SPG][3][C];   // vz^{n+1/2} rows t-2 .. t (made at t-3 .. t-1)
    float DVX[SPG][3][C];   // vx^{n+1/2} rows t-3 .. t-1
    float DPZ[SPG][3][C];   // pz^{n+1} rows t-3 .. t-1
    float DK[3][C], DBX[3][C], DBZ[3][C];   // K, bx rows t-3 .. t-1; bz rows t-2 .. t
    int srow[SPG];
    float swa[2][SPG][C], swb[2][SPG][C];   // source weights of steps n and n+1
#pragma unroll
    for (int k = 0; k < SPG; ++k) {
        const int s = w.s0 + k;
        srow[k] = -8;
#pragma unroll
        for (int c = 0; c < C; ++c)
            swa[0][k][c] = swb[0][k][c] = swa[1][k][c] = swb[1][k][c] = 0.f;
        if (s < S) {
            const int2 sij = T->src_ij[s];
            const float4 sw4 = T->src_w[s];
            srow[k] = uni(sij.x);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float dq = g.dt * a.Q[(long long)s * T->nt + a.n + h];
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const int dj = w.j0 + c - sij.y;
                    swa[h][k][c] = dj == 0 ? dq * sw4.x : (dj == 1 ? dq * sw4.y : 0.f);
                    swb[h][k][c] = dj == 0 ? dq * sw4.z : (dj == 1 ? dq * sw4.w : 0.f);
                }
            }
        }
        const unsigned op = skoff(a.pin, k), ovz = FB + skoff(a.vin, k);
        float pr[6][C];
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const int r = t0 - 3 + q;
            vld<C>(rPin, row_ok(g, r) ? w.vcol : kOOB, rofs(r, op), pr[q]);
            mask_cols<C>(w, pr[q]);
        }
        // vz^{n+1/2} at rows t0-2 .. t0
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int r = t0 - 2 + q;
            const bool ok = row_ok(g, r);
            const unsigned vo = ok ? w.vcol : kOOB;
            float bz[C], vz[C];
            vld<C>(rM, vo, rofs(r, 2u * FB), bz);
            vld<C>(rVin, vo, rofs(r, ovz), vz);
            const float ahz = zahz[r], bhz = zbhz[r];
#pragma unroll
            for (int c = 0; c < C; ++c)
                VZ1[k][q][c] = ahz * vz[c] -
                               bhz * bz[c] *
                                   (kC1 * (pr[q + 2][c] - pr[q + 1][c]) + kC2 * (pr[q + 3][c] - pr[q][c])) *
                                   g.rdz;
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            P1[k][0][c] = pr[3][c];
            P1[k][1][c] = pr[4][c];
            P1[k][2][c] = pr[5][c];
            P1[k][3][c] = 0.f;
#pragma unroll
            for (int q = 0; q < 3; ++q)
                P2[k][q][c] = VZ2[k][q][c] = DVZ[k][q][c] = DVX[k][q][c] = DPZ[k][q][c] = 0.f;
        }
    }
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int c = 0; c < C; ++c)
            DK[q][c] = DBX[q][c] = DBZ[q][c] = 0.f;

    // step-one loads of row t (p at t+3, vz at t+1, vx and split at t,
    // K and bx at t, bz at t+1); rows outside the grid read zero
    auto load_row = [&](int t, FRow<SPG, C> &b) {
        const bool live = t < w.i1 + 3;
        const bool ok0 = live && row_ok(g, t), ok1 = live && row_ok(g, t + 1);
        const bool ok3 = live && row_ok(g, t + 3);
        const unsigned o0 = ok0 ? w.vcol : kOOB, o1 = ok1 ? w.vcol : kOOB;
        const unsigned o3 = ok3 ? w.vcol : kOOB;
        const ZRow z = zrow(g, ok0 ? t : 0);
        unsigned oz[C];
        zoffs<C>(w, z, ok0, oz);
        vld<C>(rM, o0, rofs(t, 0u), b.K);
        vld<C>(rM, o0, rofs(t, FB), b.bx);
        vld<C>(rM, o1, rofs(t + 1, 2u * FB), b.bz1);
#pragma unroll
        for (int k = 0; k < SPG; ++k) {
            const unsigned kp = skoff(a.pin, k), kv = skoff(a.vin, k);
            vld<C>(rPin, o3, rofs(t + 3, kp), b.p3[k]);
            vld<C>(rVin, o1, rofs(t + 1, FB + kv), b.vz1[k]);
            vld<C>(rVin, o0, rofs(t, kv), b.vx[k]);
#pragma unroll
            for (int c = 0; c < C; ++c)
                b.pz[k][c] = bld(rPin, oz[c], z.base + FB + kp);
        }
    };

    auto row = [&](int t, FRow<SPG, C> &b) {
        const bool okt = row_ok(g, t);
        const bool rp1 = t < g.npml || t >= g.Nz - g.npml;   // row t in the layer
        const float ahz1 = zahz[t + 1], bhz1 = zbhz[t + 1];
        const float az1 = zaz[t], btz1 = zbz[t];
        const bool mid_on = t >= w.i0 && t < w.i1;   // this wave owns p^{n+1} row t
        const int r = t - 3;                          // step-two row
        const bool two = t >= w.i0;                   // step two runs (r >= i0 - 3)
        const bool full = r >= w.i0;                  // step two on an owned row
        const bool rn = row_ok(g, r + 1);
        const float ahz2 = zahz[r + 1], bhz2 = zbhz[r + 1];
        const float az2 = zaz[r], btz2 = zbz[r];
        const ZRow z2 = zrow(g, full ? r : 0);
        unsigned zw2[C];
        zoffs_w<C>(w, z2, zw2);
        const unsigned rb1 = okt ? rowb(g, t) : 0u, rb2 = full ? rowb(g, r) : 0u;
        const unsigned rbz = (r + 1 >= w.i0 && r + 1 < w.i1) ? rowb(g, r + 1) : 0u;
        const bool vz_on = r + 1 >= w.i0 && r + 1 < w.i1;   // owns vz row r+1
#pragma unroll
        for (int k = 0; k < SPG; ++k) {
            mask_cols<C>(w, b.p3[k]);
            // ---- step one at row t
            float vzn[C], vxn[C], dp[C], pn[C], pzn[C], dvx[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                P1[k][3][c] = b.p3[k][c];
                vzn[c] = ahz1 * b.vz1[k][c] -
                         bhz1 * b.bz1[c] *
                             (kC1 * (P1[k][2][c] - P1[k][1][c]) + kC2 * (P1[k][3][c] - P1[k][0][c])) * g.rdz;
            }
            dfwd<C>(P1[k][0], dp);
#pragma unroll
            for (int c = 0; c < C; ++c)
                vxn[c] = xt.ahx[c] * b.vx[k][c] - xt.bhx[c] * b.bx[c] * dp[c] * g.rdx;
            dbwd<C>(vxn, dvx);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float dvz = kC1 * (VZ1[k][2][c] - VZ1[k][1][c]) + kC2 * (vzn[c] - VZ1[k][0][c]);
                const float pz = b.pz[k][c];
                const float px = xt.ax[c] * (P1[k][0][c] - pz) - xt.btx[c] * b.K[c] * dvx[c] * g.rdx;
                pzn[c] = az1 * pz - btz1 * b.K[c] * dvz * g.rdz;
                pn[c] = px + pzn[c];
            }
            if ((unsigned)(t - srow[k]) < 2u) {
#pragma unroll
                for (int c = 0; c < C; ++c)
                    pn[c] += b.K[c] * (t == srow[k] ? swa[0][k][c] : swb[0][k][c]);
            }
            // p^{n+1} past the last grid column must read zero in step two's
            // horizontal differences
            mask_cols<C>(w, pn);
            if (a.midw == 0) {
                vst_row<C>(rPmid, w, mid_on, rb1 + skoff(a.pmid, k), pn);
            } else if (a.midw == 1 && mid_on) {
                // only the receiver nodes of the row that this strip owns
                const unsigned ie = w.s0 + k < S ? ((cuint *)a.nwin)[((size_t)(w.s0 + k) * (size_t)g.Nz + (size_t)t) * (size_t)sw.nstrips + (size_t)w.strip] : 0u;
                const int first = nbase[k] + (int)(ie >> 9), last = first + (int)(ie & 511u);
                for (int e = first; e < last; ++e) {
                    const int j = ((cint *)a.ncol)[e];
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        if (w.j0 + c == j)
                            a.nodes[e] = pn[c];
                }
            }
            // ---- step two at row r = t-3 (p^{n+1} rows r .. r+3 = P2, pn)
            if (two) {
                float vz2[C];
#pragma unroll
                for (int c = 0; c < C; ++c)
                    vz2[c] = rn ? ahz2 * DVZ[k][0][c] -
                                      bhz2 * DBZ[0][c] *
                                          (kC1 * (P2[k][2][c] - P2[k][1][c]) + kC2 * (pn[c] - P2[k][0][c])) *
                                          g.rdz
                                : 0.f;
                const unsigned kv = skoff(a.vout, k), kp = skoff(a.pout, k);
                if (full) {
                    float dp2[C], vx2[C], dvx2[C], p2[C], pz2[C];
                    dfwd<C>(P2[k][0], dp2);
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        vx2[c] = xt.ahx[c] * DVX[k][0][c] - xt.bhx[c] * DBX[0][c] * dp2[c] * g.rdx;
                    dbwd<C>(vx2, dvx2);
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const float dvz = kC1 * (VZ2[k][2][c] - VZ2[k][1][c]) + kC2 * (vz2[c] - VZ2[k][0][c]);
                        const float pz = DPZ[k][0][c];
                        const float px =
                            xt.ax[c] * (P2[k][0][c] - pz) - xt.btx[c] * DK[0][c] * dvx2[c] * g.rdx;
                        pz2[c] = az2 * pz - btz2 * DK[0][c] * dvz * g.rdz;
                        p2[c] = px + pz2[c];
                    }
                    if ((unsigned)(r - srow[k]) < 2u) {
#pragma unroll
                        for (int c = 0; c < C; ++c)
                            p2[c] += DK[0][c] * (r == srow[k] ? swa[1][k][c] : swb[1][k][c]);
                    }
                    vst_row<C>(rVout, w, true, rb2 + kv, vx2);
                    vst_row<C>(rPout, w, true, rb2 + kp, p2);
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        bst(rPout, zw2[c], z2.base + FB + kp, pz2[c]);
                }
                vst_row<C>(rVout, w, vz_on, rbz + FB + kv, vz2);
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    VZ2[k][0][c] = VZ2[k][1][c];
                    VZ2[k][1][c] = VZ2[k][2][c];
                    VZ2[k][2][c] = vz2[c];
                }
            }
            // ---- shift the windows and delay lines
#pragma unroll
            for (int c = 0; c < C; ++c) {
                P2[k][0][c] = P2[k][1][c];
                P2[k][1][c] = P2[k][2][c];
                P2[k][2][c] = pn[c];
                DVZ[k][0][c] = DVZ[k][1][c];
                DVZ[k][1][c] = DVZ[k][2][c];
                DVZ[k][2][c] = vzn[c];
                DVX[k][0][c] = DVX[k][1][c];
                DVX[k][1][c] = DVX[k][2][c];
                DVX[k][2][c] = vxn[c];
                DPZ[k][0][c] = DPZ[k][1][c];
                DPZ[k][1][c] = DPZ[k][2][c];
                // the split is kept only where the layer has one (elsewhere
                // the one-step path reads it as zero); carrying the computed
                // value would round the interior differently
                DPZ[k][2][c] = rp1 || w.colpml[c] ? pzn[c] : 0.f;
                VZ1[k][0][c] = VZ1[k][1][c];
                VZ1[k][1][c] = VZ1[k][2][c];
                VZ1[k][2][c] = vzn[c];
                P1[k][0][c] = P1[k][1][c];
                P1[k][1][c] = P1[k][2][c];
                P1[k][2][c] = P1[k][3][c];
            }
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            DK[0][c] = DK[1][c];
            DK[1][c] = DK[2][c];
            DK[2][c] = b.K[c];
            DBX[0][c] = DBX[1][c];
            DBX[1][c] = DBX[2][c];
            DBX[2][c] = b.bx[c];
            DBZ[0][c] = DBZ[1][c];
            DBZ[1][c] = DBZ[2][c];
            DBZ[2][c] = b.bz1[c];
        }
    };

    FRow<SPG, C> A, B;
    const int tend = w.i1 + 3;   // step-one rows [t0, tend)
    load_row(t0, A);
    for (int t = t0;;) {
        load_row(t + 1, B);
        row(t, A);
        if (++t >= tend)
            break;
        load_row(t + 1, A);
        row(t, B);
        if (++t >= tend)
            break;
    }
}

// ---------------------------------------------------------------- adjoint
//
// Step m (descending from nt) on entry: mu, lv = adjoint after step m+1 with
// R^T r^m already added to the pressure components (all zero at m = nt).  Main
// pressure field = mu_px; split field = mu_pz in the absorbing layer
// (elsewhere mu_pz = mu_px).
//   lv_mid = nu_v + D+(beta K mu_p)                       (T2 transposed)
//   gbx += lvx_mid * (-bhx Dx+ p^m),  gbz likewise
//   t = D-(beta_h b lv_mid);  mu_p' = alpha mu_p + t + R^T r^{m-1};
//   lv' = alpha_h lv_mid                                  (T1^T)
//   gK  += p^m (mu_px' - alpha_x mu_px) / K
// The bulk-modulus sensitivity of the discrete scheme is the sum over steps of
// mu_x (px^{m+1} - alpha_x px^m) + mu_z (pz^{m+1} - alpha_z pz^m).  Collecting
// the terms of each level (summation by parts in time; the field is zero before
// the first step and the adjoint after the last), px^m meets mu_x' - alpha_x
// mu_x and pz^m meets mu_z' - alpha_z mu_z, which are the same t + R^T r^{m-1}.
// So a step needs the pressure of one level and no split.  At smooth-1001 (64
// shots of 1081 x 1081) that took two of five pressure reads and four of six
// split reads per shot and row out of the two-step kernel.  The difference is
// taken of the stored values: with t + R^T r^{m-1} the sum misses the rounding of
// mu'.  Error of the K gradient against FP64, over 60 problems of 10 000 to 3
// million nodes, as a multiple of that of the direct sum: 0.996 on average and 1.39
// at most with the difference, 1.018 and 1.28 with t (single shots are the worst:
// the running sum carries the boundary term p^m mu of the parts).
// Outside the layer the split forms reduce to the unsplit ones (alpha = 1,
// pz = 0).

// One shot's part of an adjoint step at output row i (the update above).
// Ring slots S0 .. S3 of MU, MZ, PN hold rows i .. i+3 of mu_px, mu_pz and
// p^m, bK rows i .. i+3 of beta_z K, and WZ rows i-2 .. i+1 of
// beta_h bz lvz_mid (slot S3 receives row i+1 here).  Adds the shot's buoyancy
// sensitivities (gbx at row i, gbz at row i+1) to accX, accZ, and returns the
// new adjoint state of row i without R^T r^{m-1} (lvz of row i+1).  Both adjoint kernels call it, so one step rounds the same way in
// either.
template <int C>
struct AdjOut {
    float opx[C], opz[C], ovx[C], ovz[C];   // mu_px, mu_pz, lvx at row i; lvz at row i+1
};

template <int C, int S0, int S1, int S2, int S3>
__device__ inline void adj_shot(const Geo &g, const XTab<C> &xt, const WaveGeo<C> &w, bool rn,
                                float ahz1, float bhz1, float az, const float (&bK)[4][C],
                                const float (&K0)[C], const float (&MU)[4][C],
                                const float (&MZ)[4][C], const float (&PN)[4][C],
                                float (&WZ)[4][C], const float (&lvz1)[C], const float (&lvx)[C],
                                const float (&bx)[C], const float (&bz1)[C], float (&accX)[C],
                                float (&accZ)[C], AdjOut<C> &o)
{
    float lvzm[C], qx[C], dqx[C], dpx[C], lvxm[C], wx[C], dwx[C], t[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        // lvz_mid at row (i+1): D+z of beta_z K mu_pz
        const float q0 = bK[0][c] * MZ[S0][c], q1 = bK[1][c] * MZ[S1][c];
        const float q2 = bK[2][c] * MZ[S2][c], q3 = bK[3][c] * MZ[S3][c];
        lvzm[c] = rn ? lvz1[c] + (kC1 * (q2 - q1) + kC2 * (q3 - q0)) * g.rdz : 0.f;
        accZ[c] += lvzm[c] * (-bhz1 * (kC1 * (PN[S2][c] - PN[S1][c]) +
                                       kC2 * (PN[S3][c] - PN[S0][c])) * g.rdz);
        WZ[S3][c] = bhz1 * bz1[c] * lvzm[c];
        // lvx_mid at row i: D+x of beta_x K mu_px
        qx[c] = xt.btx[c] * K0[c] * MU[S0][c];
    }
    dfwd<C>(qx, dqx);
    dfwd<C>(PN[S0], dpx);
#pragma unroll
    for (int c = 0; c < C; ++c) {
        lvxm[c] = w.colok[c] ? lvx[c] + dqx[c] * g.rdx : 0.f;
        accX[c] += lvxm[c] * (-xt.bhx[c] * dpx[c] * g.rdx);
        wx[c] = xt.bhx[c] * bx[c] * lvxm[c];
    }
    dbwd<C>(wx, dwx);
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const float dwz = kC1 * (WZ[S2][c] - WZ[S1][c]) + kC2 * (WZ[S3][c] - WZ[S0][c]);
        t[c] = dwx[c] * g.rdx + dwz * g.rdz;
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
        o.opx[c] = xt.ax[c] * MU[S0][c] + t[c];
        o.opz[c] = az * MZ[S0][c] + t[c];
        o.ovx[c] = xt.ahx[c] * lvxm[c];
        o.ovz[c] = ahz1 * lvzm[c];
    }
}

// R^T r of a step at the receiver nodes of one row that lie in the wave's
// window (ie: the packed range of AdjNodes, counted from node nbase), added to
// the row's new adjoint pressure.  The lanes holding the row's nodes push them
// to the lanes holding their columns, all at once; the others push 0 to lane 0,
// a halo lane that no result depends on.  (Taken one by one with v_readlane they
// set the length of the waves that hold receivers: us a pair of steps, before and
// after, 63 shots of 511 x 189 with 349 receivers 135 and 103, 40 of 367 x 250 with
// 289 93 and 71, 40 of 481 x 481 with 360 166 and 158.)
template <int C>
__device__ inline void add_nodes(const AdjNodes &nd, const float *val, NodeLanes &nl, int nbase,
                                 unsigned ie, int lane, int col0, float (&mu)[C])
{
    const int last = nbase + (int)(ie >> 9) + (int)(ie & 511u);
    for (int e = nbase + (int)(ie >> 9); e < last;) {
        if (e < nl.base || e >= nl.end)
            nl.load(nd.col, val, e, lane);
        const int n = imin(last, nl.end) - e;
        const bool in = (unsigned)(lane - (e - nl.base)) < (unsigned)n;
        const int j = nl.col - col0;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const bool on = in && (C == 1 || j % C == c);
            mu[c] += __builtin_bit_cast(
                float, __builtin_amdgcn_ds_permute(on ? j / C * 4 : 0,
                                                   on ? __builtin_bit_cast(int, nl.val) : 0));
        }
        e += n;
    }
}

template <int SPG, int C>
struct ARow {   // loads needed early in the row (double buffered)
    float K3[C], bx[C], bz1[C];                 // K at r+3, bx at r, bz at r+1
    float mu3[SPG][C], mz3[SPG][C], pn3[SPG][C];  // mu_px, split mu_pz, p^n at r+3
    float lvz1[SPG][C], lvx[SPG][C];            // lvz at r+1, lvx at r
    unsigned inj[SPG];                          // receiver nodes of row r (packed)
};
template <int C>
struct ALate {  // loads needed at the end of the row (single set)
    float gK[C], gX[C], gZ1[C];                 // partials at r (gbz at r+1)
};

template <int SPG, int C>
__global__ void __launch_bounds__(NTHR)
    k_adj(Geo g, const float *__restrict__ tabs, const float *model, Sweep sw, AdjStep a)
{
    WaveGeo<C> w;
    if (!wave_geo<C>(g, sw, w))
        return;
    XTab<C> xt;
    xtab<C>(g, tabs, w, xt);
    // z tables: alpha, beta at nodes, alpha_h, beta_h at half nodes
    const float *__restrict__ zaz = tabs + 4 * g.Nx, *__restrict__ zbz = zaz + g.Nz;
    const float *__restrict__ zahz = zbz + g.Nz, *__restrict__ zbhz = zahz + g.Nz;
    const unsigned FB = 4u * (unsigned)g.N;
    const unsigned rowN = 4u * (unsigned)g.Nx;
    const rsrc_t rM = res(model, 3u * FB);                                  // K, bx, bz
    const rsrc_t rG = res(a.gpart + (long long)w.grp * 3 * g.N, 3u * FB);  // gK, gbx, gbz
    const rsrc_t rLin = grp_res(a.lin, w.s0, SPG), rLout = grp_res(a.lout, w.s0, SPG);
    const rsrc_t rPn = grp_res(a.pn, w.s0, SPG);
    cuint *injwin = (cuint *)a.nd.win;
    const int ZP = g.Nz + 2 * kZPad;
    NodeLanes nl[SPG];
    int nbase[SPG];   // first node of the wave's strip
#pragma unroll
    for (int k = 0; k < SPG; ++k)
        nbase[k] = injwin ? ((cint *)a.nd.ptr)[(w.s0 + k) * sw.nstrips + w.strip] : 0;
    auto rowpml = [&](int r) { return r < g.npml || r >= g.Nz - g.npml; };
    auto btz_at = [&](int r) -> float { return row_ok(g, r) ? zbz[r] : 0.f; };
    // mu_pz of shot k at row r (zero outside the grid)
    auto muz_at = [&](int k, int r, float (&o)[C]) {
        const bool ok = row_ok(g, r);
        const unsigned kl = skoff(a.lin, k);
        float mx[C];
        vld<C>(rLin, ok ? w.vcol : kOOB, ok ? rowb(g, r) + 2u * FB + kl : 0u, mx);
        const ZRow z = zrow(g, ok ? r : 0);
        unsigned oz[C];
        zoffs<C>(w, z, ok, oz);
        const bool rp = rowpml(r);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const float mz = bld(rLin, oz[c], z.base + 3u * FB + kl);
            o[c] = rp || w.colpml[c] ? mz : mx[c];
        }
    };

    // Row windows are rings of 4 slots: at phase R = (i - i0) mod 4 the row
    // of logical index q sits in slot (q + R) & 3, so moving down a row
    // re-labels the slots instead of copying them (the row loop is unrolled
    // four times, one phase each).
    float KW[4][C];         // K rows i .. i+3
    float MU[SPG][4][C];    // mu_px rows i .. i+3
    float MZ[SPG][4][C];    // mu_pz rows i .. i+3
    float PN[SPG][4][C];    // p^n rows i .. i+3
    float WZ[SPG][4][C];    // beta_h bz lvz_mid rows i-2 .. i+1

    float Kr[6][C], btzr[6], wzr[3][C];
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const int r = w.i0 - 3 + q;
        const bool ok = row_ok(g, r);
        vld<C>(rM, ok ? w.vcol : kOOB, ok ? rowb(g, r) : 0u, Kr[q]);
        btzr[q] = btz_at(r);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int r = w.i0 - 2 + q;
        const bool ok = row_ok(g, r);
        float bz[C];
        vld<C>(rM, ok ? w.vcol : kOOB, ok ? rowb(g, r) + 2u * FB : 0u, bz);
        const float bhz = ok ? zbhz[r] : 0.f;
#pragma unroll
        for (int c = 0; c < C; ++c)
            wzr[q][c] = bhz * bz[c];
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
        KW[0][c] = Kr[3][c];
        KW[1][c] = Kr[4][c];
        KW[2][c] = Kr[5][c];
        KW[3][c] = 0.f;
    }
    const float bhz0 = zbhz[w.i0], ahz0 = zahz[w.i0];
    float accZ0[C];
#pragma unroll
    for (int c = 0; c < C; ++c)
        accZ0[c] = 0.f;
#pragma unroll
    for (int k = 0; k < SPG; ++k) {
        const unsigned kl = skoff(a.lin, k), kn = skoff(a.pn, k);
        float qz[6][C], pnr[4][C];
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const int r = w.i0 - 3 + q;
            float mz[C];
            muz_at(k, r, mz);
#pragma unroll
            for (int c = 0; c < C; ++c)
                qz[q][c] = Kr[q][c] * btzr[q] * mz[c];
            if (q >= 3) {
#pragma unroll
                for (int c = 0; c < C; ++c)
                    MZ[k][q - 3][c] = mz[c];
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = w.i0 - 1 + q;
            const bool ok = row_ok(g, r);
            vld<C>(rPn, ok ? w.vcol : kOOB, ok ? rowb(g, r) + kn : 0u, pnr[q]);
            mask_cols<C>(w, pnr[q]);
        }
        // lvz_mid at rows i0-2 .. i0 (zero outside the grid)
        float l[3][C];
#pragma unroll
        for (int c = 0; c < C; ++c)
            WZ[k][3][c] = 0.f;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int r = w.i0 - 2 + q;
            const bool ok = row_ok(g, r);
            float lz[C];
            vld<C>(rLin, ok ? w.vcol : kOOB, ok ? rowb(g, r) + FB + kl : 0u, lz);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                l[q][c] = ok ? lz[c] + (kC1 * (qz[q + 2][c] - qz[q + 1][c]) +
                                        kC2 * (qz[q + 3][c] - qz[q][c])) * g.rdz
                             : 0.f;
                WZ[k][q][c] = wzr[q][c] * l[q][c];
            }
        }
        float lo[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            accZ0[c] += l[2][c] * (-bhz0 * (kC1 * (pnr[2][c] - pnr[1][c]) + kC2 * (pnr[3][c] - pnr[0][c])) * g.rdz);
            lo[c] = ahz0 * l[2][c];
        }
        vst_row<C>(rLout, w, true, rowb(g, w.i0) + FB + skoff(a.lout, k), lo);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int r = w.i0 + q;
            const bool ok = row_ok(g, r);
            vld<C>(rLin, ok ? w.vcol : kOOB, ok ? rowb(g, r) + 2u * FB + kl : 0u, MU[k][q]);
#pragma unroll
            for (int c = 0; c < C; ++c)
                PN[k][q][c] = pnr[q + 1][c];
        }
#pragma unroll
        for (int c = 0; c < C; ++c)
            MU[k][3][c] = MZ[k][3][c] = PN[k][3][c] = 0.f;
    }
    {
        const unsigned o = rowb(g, w.i0) + 2u * FB;
        float gz[C];
        vld<C>(rG, w.vcolw, o, gz);
#pragma unroll
        for (int c = 0; c < C; ++c)
            if (c + 1 < C) {
                const float t = bld(rG, w.vtail[c], o);
                gz[c] = w.vtail[c] != kOOB ? t : gz[c];
            }
#pragma unroll
        for (int c = 0; c < C; ++c)
            gz[c] += accZ0[c];
        vst_row<C>(rG, w, true, o, gz);
    }

    auto load_row = [&](int r, ARow<SPG, C> &b) {
        const unsigned rb = rowb(g, r);
        const RowOff o = row_off<C>(g, w, r);
        const bool live = r < w.i1;
        // split element offsets of row r+3 (kOOB where it has no split)
        const ZRow z3 = zrow(g, r + 3);
        unsigned oz3[C];
        zoffs<C>(w, z3, live && r + 3 < g.Nz, oz3);
        vld<C>(rM, o.o3, rb + 3u * rowN, b.K3);
        vld<C>(rM, o.o0, rb + FB, b.bx);
        vld<C>(rM, o.o1, rb + rowN + 2u * FB, b.bz1);
#pragma unroll
        for (int k = 0; k < SPG; ++k) {
            const unsigned kl = skoff(a.lin, k), kn = skoff(a.pn, k);
            vld<C>(rLin, o.o3, rb + 3u * rowN + 2u * FB + kl, b.mu3[k]);
#pragma unroll
            for (int c = 0; c < C; ++c)
                b.mz3[k][c] = bld(rLin, oz3[c], z3.base + 3u * FB + kl);
            vld<C>(rPn, o.o3, rb + 3u * rowN + kn, b.pn3[k]);
            vld<C>(rLin, o.o1, rb + rowN + FB + kl, b.lvz1[k]);
            vld<C>(rLin, o.o0, rb + kl, b.lvx[k]);
            // (rows and padding shots without nodes hold 0)
            b.inj[k] = injwin ? injwin[((size_t)(w.s0 + k) * (size_t)ZP + (size_t)(r + kZPad)) *
                                           (size_t)sw.nstrips + (size_t)w.strip]
                              : 0u;
        }
    };
    // end-of-row values of row i (issued before the next row's loads)
    auto load_late = [&](int i, ALate<C> &t) {
        const unsigned rb = rowb(g, i);
        const bool more = i + 1 < w.i1;
        // partial gradient: this wave's output columns only (the lane
        // holding the last column reads its elements one by one)
        vld<C>(rG, w.vcolw, rb, t.gK);
        vld<C>(rG, w.vcolw, rb + FB, t.gX);
        vld<C>(rG, more ? w.vcolw : kOOB, rb + rowN + 2u * FB, t.gZ1);
#pragma unroll
        for (int c = 0; c + 1 < C; ++c) {
            const float a0 = bld(rG, w.vtail[c], rb), a1 = bld(rG, w.vtail[c], rb + FB);
            const float a2 = bld(rG, more ? w.vtail[c] : kOOB, rb + rowN + 2u * FB);
            const bool tl = w.vtail[c] != kOOB;
            t.gK[c] = tl ? a0 : t.gK[c];
            t.gX[c] = tl ? a1 : t.gX[c];
            t.gZ1[c] = tl ? a2 : t.gZ1[c];
        }
    };

    auto row = [&](auto phase, int i, ARow<SPG, C> &b, const ALate<C> &t) {
        constexpr int R = decltype(phase)::value;
        constexpr int S0 = R & 3, S1 = (1 + R) & 3, S2 = (2 + R) & 3, S3 = (3 + R) & 3;
        const unsigned rb = rowb(g, i);
        const bool rn = row_ok(g, i + 1);
        const bool more = i + 1 < w.i1;   // this wave owns lvz / gbz row i+1
        const float ahz1 = rn ? zahz[i + 1] : 0.f, bhz1 = rn ? zbhz[i + 1] : 0.f;
        const float az = zaz[i];
        const float bt0 = btz_at(i), bt1 = btz_at(i + 1), bt2 = btz_at(i + 2), bt3 = btz_at(i + 3);
        const bool rp3 = rowpml(i + 3);
        const ZRow z = zrow(g, i);
        unsigned zw[C];
        zoffs_w<C>(w, z, zw);
        float numK[C], accX[C], accZ[C], bK[4][C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            KW[S3][c] = b.K3[c];
            numK[c] = accX[c] = accZ[c] = 0.f;
            bK[0][c] = KW[S0][c] * bt0;
            bK[1][c] = KW[S1][c] * bt1;
            bK[2][c] = KW[S2][c] * bt2;
            bK[3][c] = KW[S3][c] * bt3;
        }
#pragma unroll
        for (int k = 0; k < SPG; ++k) {
            mask_cols<C>(w, b.pn3[k]);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                MU[k][S3][c] = b.mu3[k][c];
                MZ[k][S3][c] = rp3 || w.colpml[c] ? b.mz3[k][c] : b.mu3[k][c];
                PN[k][S3][c] = b.pn3[k][c];
            }
            AdjOut<C> o;
            adj_shot<C, S0, S1, S2, S3>(g, xt, w, rn, ahz1, bhz1, az, bK, KW[S0], MU[k], MZ[k],
                                        PN[k], WZ[k], b.lvz1[k], b.lvx[k], b.bx, b.bz1, accX,
                                        accZ, o);
            if (b.inj[k] != 0u)
                add_nodes<C>(a.nd, a.injv, nl[k], nbase[k], b.inj[k], w.lane, w.j0 - w.lane * C, o.opx);
#pragma unroll
            for (int c = 0; c < C; ++c)
                numK[c] += PN[k][S0][c] * fmaf(-xt.ax[c], MU[k][S0][c], o.opx[c]);
            const unsigned ko = skoff(a.lout, k);
            vst_row<C>(rLout, w, true, rb + 2u * FB + ko, o.opx);
#pragma unroll
            for (int c = 0; c < C; ++c)
                bst(rLout, zw[c], z.base + 3u * FB + ko, o.opz[c]);
            vst_row<C>(rLout, w, true, rb + ko, o.ovx);
            vst_row<C>(rLout, w, more, rb + rowN + FB + ko, o.ovz);
        }
        // one reciprocal per row for the bulk-modulus sensitivity (1 ulp)
        float gk[C], gx[C], gz[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const float rK = KW[S0][c] != 0.f ? __builtin_amdgcn_rcpf(KW[S0][c]) : 0.f;
            gk[c] = t.gK[c] + numK[c] * rK;
            gx[c] = t.gX[c] + accX[c];
            gz[c] = t.gZ1[c] + accZ[c];
        }
        vst_row<C>(rG, w, true, rb, gk);
        vst_row<C>(rG, w, true, rb + FB, gx);
        vst_row<C>(rG, w, more, rb + rowN + 2u * FB, gz);
    };

    ARow<SPG, C> A, B;
    ALate<C> L;
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    using P2 = std::integral_constant<int, 2>;
    using P3 = std::integral_constant<int, 3>;
    load_row(w.i0, A);
    for (int i = w.i0;;) {
        load_late(i, L);
        load_row(i + 1, B);
        row(P0{}, i, A, L);
        if (++i >= w.i1)
            break;
        load_late(i, L);
        load_row(i + 1, A);
        row(P1{}, i, B, L);
        if (++i >= w.i1)
            break;
        load_late(i, L);
        load_row(i + 1, B);
        row(P2{}, i, A, L);
        if (++i >= w.i1)
            break;
        load_late(i, L);
        load_row(i + 1, A);
        row(P3{}, i, B, L);
        if (++i >= w.i1)
            break;
    }
}

// ------------------------------------------------------- adjoint, two steps
//
// Adjoint steps m and m-1 in one pass, the reverse counterpart of k_fwd2.
// Step A (adjoint step m) runs on rows [i0-3, i1+3) of the band with a
// 6-column halo; step B (adjoint step m-1) follows three rows behind, on
// rows [i0-3, i1) (its first three rows only fill its windows, their
// results are dropped).  Step A's new adjoint state never leaves the chip:
// its pressure rows feed step B's windows, and its velocities, the model
// rows and p^n reach step B through four-slot rings read three rows later.
// Each step adds R^T r of the level below it, staged per receiver node by an
// earlier launch, to its new pressure at the nodes in the wave's window.
// Step A's sensitivities on the wave's own rows wait three rows and are added
// to the group's partial gradient before step B's, each with the one-step
// kernel's expression, so the pair rounds exactly as two one-step launches.
//
// What bounds it is the memory path of each CU (L1 misses in flight against
// their latency, about 4.3 TB/s moved), so the bytes and requests count: one
// pressure level a step without its split, the receivers' sums staged 64 steps
// at a time instead of a launch a pair, and four shots a wave, which read the
// model and read and write the partial gradient once.  Four shots fit the 256
// registers of two waves a SIMD (three with two shots) because the values that
// wait three rows sit in LDS.  us per launch on one and the same buffer, before
// and after: 958 and 886 (64 shots of 1081 x 1081, 4 shots a wave, 91 rows),
// 1865 and 1590 (32 of 2081 x 2081; 4, 64), 172 and 158 (40 of 481 x 481; 2,
// 20); 18 + 10 f + 18 / SPG bytes a cell-step became 16 + 4 f + 18 / SPG, f the
// layer's share of the cells.

template <int SPG, int C>
struct A2Row {   // loads of iteration t (double buffered)
    float K3[C], bx[C], bz1[C];                   // K at t+3, bx at t, bz at t+1
    float mu3[SPG][C], mz3[SPG][C], pn3[SPG][C];  // mu_px, mu_pz, p^m at t+3
    float lvz1[SPG][C], lvx[SPG][C];              // lvz at t+1, lvx at t
    float pm[SPG][C];                             // p^{m-1} at t
};

template <int SPG, int C>
__global__ void __launch_bounds__(NTHR) __attribute__((amdgpu_waves_per_eu(C > 1 ? 1 : SPG == 1 ? 4 : SPG == 2 ? 3 : 2)))
    k_adj2(Geo g, const float *__restrict__ tabs, const float *model, Sweep sw, AdjStep2 a)
{
    WaveGeo<C> w;
    if (!wave_geo<C, 2 * HALO>(g, sw, w))
        return;
    XTab<C> xt;
    xtab<C>(g, tabs, w, xt);
    // z tables and receiver nodes of 64 rows (rows and padding shots without
    // nodes hold 0)
    RowLanes<SPG> rl;
    auto node_row = [&](int k) -> const unsigned * {
        return a.nd.win + ((size_t)(w.s0 + k) * (size_t)(g.Nz + 2 * kZPad) + kZPad) *
                              (size_t)sw.nstrips + w.strip;
    };
    rl.load(g, a.zpad, w.i0 - 6, w.lane, -kZPad, g.Nz + kZPad - 1, node_row, sw.nstrips);
    NodeLanes nlA[SPG], nlB[SPG];
    int nbase[SPG];   // first node of the wave's strip
#pragma unroll
    for (int k = 0; k < SPG; ++k)
        nbase[k] = ((cint *)a.nd.ptr)[(w.s0 + k) * sw.nstrips + w.strip];
    const unsigned FB = 4u * (unsigned)g.N;
    const rsrc_t rM = res(model, 3u * FB);                                  // K, bx, bz
    const rsrc_t rG = res(a.gpart + (long long)w.grp * 3 * g.N, 3u * FB);  // gK, gbx, gbz
    const rsrc_t rLin = grp_res(a.lin, w.s0, SPG), rLout = grp_res(a.lout, w.s0, SPG);
    // the two pressure levels of the group: p^{m-1} at 0, p^m at lvl bytes
    const rsrc_t rP = res((const float *)((const char *)a.pm1.base + (size_t)w.s0 * a.pm1.sbytes),
                          a.lvl + (unsigned)(SPG - 1) * a.pm1.sbytes + a.pm1.bytes);
    const unsigned LN = a.lvl;
    auto rowpml = [&](int r) { return r < g.npml || r >= g.Nz - g.npml; };
    // byte offset of row r plus `extra`, 0 for rows outside the grid (whose
    // lane offsets are then kOOB)
    auto rofs = [&](int r, unsigned extra) -> unsigned {
        return row_ok(g, r) ? rowb(g, r) + extra : 0u;
    };
    auto vo = [&](bool ok) -> unsigned { return ok ? w.vcol : kOOB; };
    // mu_pz of shot k at row r (zero outside the grid)
    auto muz_at = [&](int k, int r, float (&o)[C]) {
        const bool ok = row_ok(g, r);
        const unsigned kl = skoff(a.lin, k);
        float mx[C];
        vld<C>(rLin, vo(ok), rofs(r, 2u * FB + kl), mx);
        const ZRow z = zrow(g, ok ? r : 0);
        unsigned oz[C];
        zoffs<C>(w, z, ok, oz);
        const bool rp = rowpml(r);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const float mz = bld(rLin, oz[c], z.base + 3u * FB + kl);
            o[c] = rp || w.colpml[c] ? mz : mx[c];
        }
    };

    const int tA0 = w.i0 - 3, tend = w.i1 + 3;   // step-A rows [tA0, tend)

    // Delay rings, in LDS (each lane its own words): slot R holds the values of
    // iteration t, slot R + 1 those of iteration t - 3.  Of each shot A's lvx
    // (row t) and lvz (row t+1); bx (t) and bz (t+1); A's gK numerator, gbx (t)
    // and gbz (t+1).
    constexpr int RX = 0, RZ = SPG, RBX = 2 * SPG, RBZ = RBX + 1, RNK = RBX + 2, RAX = RBX + 3,
                  RAZ = RBX + 4, RN = RBX + 5;
    __shared__ float ring[NTHR / WAVE][4][RN][C][WAVE];
    auto &D = ring[threadIdx.x / WAVE];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int n = 0; n < RN; ++n)
#pragma unroll
            for (int c = 0; c < C; ++c)
                D[q][n][c][w.lane] = 0.f;

    // Windows (rings of 4 slots relabelled by the phase R = (t - tA0) mod 4,
    // as in k_adj): step A's rows t .. t+3 (WZA: t-2 .. t+1), step B's rows
    // r .. r+3 (WZB: r-2 .. r+1) with r = t-3.  Delay rings: slot R holds
    // the value of iteration t, slot R+1 that of iteration t-3.
    float KA[4][C], KB[4][C];
    float MUA[SPG][4][C], MZA[SPG][4][C], PNA[SPG][4][C], WZA[SPG][4][C];
    float MUB[SPG][4][C], MZB[SPG][4][C], PMB[SPG][4][C], WZB[SPG][4][C];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int c = 0; c < C; ++c) {
            KB[q][c] = 0.f;
#pragma unroll
            for (int k = 0; k < SPG; ++k)
                MUB[k][q][c] = MZB[k][q][c] = PMB[k][q][c] = WZB[k][q][c] = 0.f;
        }

    // step A's windows at its first row tA0 (k_adj's start of a band)
    {
        float Kr[6][C], btzr[6], wzr[3][C];
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const int r = tA0 - 3 + q;
            vld<C>(rM, vo(row_ok(g, r)), rofs(r, 0u), Kr[q]);
            btzr[q] = rl.at(rl.bz, r);
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int r = tA0 - 2 + q;
            float bz[C];
            vld<C>(rM, vo(row_ok(g, r)), rofs(r, 2u * FB), bz);
            const float bhz = rl.at(rl.bhz, r);
#pragma unroll
            for (int c = 0; c < C; ++c)
                wzr[q][c] = bhz * bz[c];
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            KA[0][c] = Kr[3][c];
            KA[1][c] = Kr[4][c];
            KA[2][c] = Kr[5][c];
            KA[3][c] = 0.f;
        }
#pragma unroll
        for (int k = 0; k < SPG; ++k) {
            const unsigned kl = skoff(a.lin, k), kn = skoff(a.pm1, k);
            float qz[6][C], pnr[4][C];
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                float mz[C];
                muz_at(k, tA0 - 3 + q, mz);
#pragma unroll
                for (int c = 0; c < C; ++c)
                    qz[q][c] = Kr[q][c] * btzr[q] * mz[c];
                if (q >= 3) {
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        MZA[k][q - 3][c] = mz[c];
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = tA0 - 1 + q;
                vld<C>(rP, vo(row_ok(g, r)), rofs(r, LN + kn), pnr[q]);
                mask_cols<C>(w, pnr[q]);
            }
#pragma unroll
            for (int c = 0; c < C; ++c)
                WZA[k][3][c] = 0.f;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const int r = tA0 - 2 + q;
                const bool ok = row_ok(g, r);
                float lz[C];
                vld<C>(rLin, vo(ok), rofs(r, FB + kl), lz);
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const float l = ok ? lz[c] + (kC1 * (qz[q + 2][c] - qz[q + 1][c]) +
                                                  kC2 * (qz[q + 3][c] - qz[q][c])) * g.rdz
                                       : 0.f;
                    WZA[k][q][c] = wzr[q][c] * l;
                }
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const int r = tA0 + q;
                vld<C>(rLin, vo(row_ok(g, r)), rofs(r, 2u * FB + kl), MUA[k][q]);
#pragma unroll
                for (int c = 0; c < C; ++c)
                    PNA[k][q][c] = pnr[q + 1][c];
            }
#pragma unroll
            for (int c = 0; c < C; ++c)
                MUA[k][3][c] = MZA[k][3][c] = PNA[k][3][c] = 0.f;
        }
    }

    auto load_row = [&](int t, A2Row<SPG, C> &b) {
        const bool live = t < tend;
        const bool ok0 = live && row_ok(g, t), ok1 = live && row_ok(g, t + 1);
        const bool ok3 = live && row_ok(g, t + 3);
        const ZRow z3 = zrow(g, ok3 ? t + 3 : 0);
        unsigned oz3[C];
        zoffs<C>(w, z3, ok3, oz3);
        vld<C>(rM, vo(ok3), rofs(t + 3, 0u), b.K3);
        vld<C>(rM, vo(ok0), rofs(t, FB), b.bx);
        vld<C>(rM, vo(ok1), rofs(t + 1, 2u * FB), b.bz1);
#pragma unroll
        for (int k = 0; k < SPG; ++k) {
            const unsigned kl = skoff(a.lin, k), kp = skoff(a.pm1, k);
            vld<C>(rLin, vo(ok3), rofs(t + 3, 2u * FB + kl), b.mu3[k]);
#pragma unroll
            for (int c = 0; c < C; ++c)
                b.mz3[k][c] = bld(rLin, oz3[c], z3.base + 3u * FB + kl);
            vld<C>(rP, vo(ok3), rofs(t + 3, LN + kp), b.pn3[k]);
            vld<C>(rLin, vo(ok1), rofs(t + 1, FB + kl), b.lvz1[k]);
            vld<C>(rLin, vo(ok0), rofs(t, kl), b.lvx[k]);
            vld<C>(rP, vo(ok0), rofs(t, kp), b.pm[k]);
        }
    };
    // values needed late in iteration t (issued before the next row's loads)
    auto load_late = [&](int t, ALate<C> &L) {
        const int r = t - 3;
        const bool own = r >= w.i0 && r < w.i1, ownz = r + 1 >= w.i0 && r + 1 < w.i1;
        // partial gradient of step B's row: this wave's output columns only
        // (the lane holding the last column reads its elements one by one)
        const unsigned gk = own ? w.vcolw : kOOB, gz = ownz ? w.vcolw : kOOB;
        const unsigned ob = own ? rowb(g, r) : 0u, obz = ownz ? rowb(g, r + 1) : 0u;
        vld<C>(rG, gk, ob, L.gK);
        vld<C>(rG, gk, ob + FB, L.gX);
        vld<C>(rG, gz, obz + 2u * FB, L.gZ1);
#pragma unroll
        for (int c = 0; c + 1 < C; ++c) {
            const float a0 = bld(rG, own ? w.vtail[c] : kOOB, ob);
            const float a1 = bld(rG, own ? w.vtail[c] : kOOB, ob + FB);
            const float a2 = bld(rG, ownz ? w.vtail[c] : kOOB, obz + 2u * FB);
            const bool tl = w.vtail[c] != kOOB;
            L.gK[c] = tl ? a0 : L.gK[c];
            L.gX[c] = tl ? a1 : L.gX[c];
            L.gZ1[c] = tl ? a2 : L.gZ1[c];
        }
    };

    auto row = [&](auto phase, int t, A2Row<SPG, C> &b, const ALate<C> &L) {
        constexpr int R = decltype(phase)::value;
        constexpr int S0 = R & 3, S1 = (1 + R) & 3, S2 = (2 + R) & 3, S3 = (3 + R) & 3;
        // ---- step A (adjoint step n) at row t
        const bool okt = row_ok(g, t), rnA = row_ok(g, t + 1);
        if (t + 3 - rl.base >= WAVE)
            rl.load(g, a.zpad, t - 3, w.lane, -kZPad, g.Nz + kZPad - 1, node_row, sw.nstrips);
        const float ahz1A = rl.at(rl.ahz, t + 1), bhz1A = rl.at(rl.bhz, t + 1);
        const float azA = rl.at(rl.az, t);
        const float bt0 = rl.at(rl.bz, t), bt1 = rl.at(rl.bz, t + 1);
        const float bt2 = rl.at(rl.bz, t + 2), bt3 = rl.at(rl.bz, t + 3);
        const bool rp3 = rowpml(t + 3), rpt = rowpml(t);
        // ---- step B (adjoint step n-1) at row r
        const int r = t - 3;
        const bool runB = t >= w.i0;                          // r >= i0 - 3
        const bool own = r >= w.i0;                           // (r < i1 always)
        const bool ownz = r + 1 >= w.i0 && r + 1 < w.i1;      // owns lvz / gbz row r+1
        const bool rnB = row_ok(g, r + 1);
        const float ahz1B = rl.at(rl.ahz, r + 1), bhz1B = rl.at(rl.bhz, r + 1);
        const float azB = rl.at(rl.az, r);
        const float bu0 = rl.at(rl.bz, r), bu1 = rl.at(rl.bz, r + 1);
        const float bu2 = rl.at(rl.bz, r + 2), bu3 = bt0;
        const unsigned rbB = own ? rowb(g, r) : 0u, rbZ = ownz ? rowb(g, r + 1) : 0u;
        const ZRow zB = zrow(g, own ? r : 0);
        unsigned zwB[C];
        zoffs_w<C>(w, zB, zwB);
        float numA[C], axA[C], azA_[C], bKA[4][C];
        float numB[C], axB[C], azB_[C], bKB[4][C];
        float dly[RN][C];   // iteration t - 3
#pragma unroll
        for (int n = 0; n < RN; ++n)
#pragma unroll
            for (int c = 0; c < C; ++c)
                dly[n][c] = D[S1][n][c][w.lane];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            KA[S3][c] = b.K3[c];
            KB[S3][c] = KA[S0][c];   // K at row t = r+3
            numA[c] = axA[c] = azA_[c] = numB[c] = axB[c] = azB_[c] = 0.f;
            bKA[0][c] = KA[S0][c] * bt0;
            bKA[1][c] = KA[S1][c] * bt1;
            bKA[2][c] = KA[S2][c] * bt2;
            bKA[3][c] = KA[S3][c] * bt3;
            bKB[0][c] = KB[S0][c] * bu0;
            bKB[1][c] = KB[S1][c] * bu1;
            bKB[2][c] = KB[S2][c] * bu2;
            bKB[3][c] = KB[S3][c] * bu3;
        }
#pragma unroll
        for (int k = 0; k < SPG; ++k) {
            mask_cols<C>(w, b.pn3[k]);
            mask_cols<C>(w, b.pm[k]);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                MUA[k][S3][c] = b.mu3[k][c];
                MZA[k][S3][c] = rp3 || w.colpml[c] ? b.mz3[k][c] : b.mu3[k][c];
                PNA[k][S3][c] = b.pn3[k][c];
            }
            AdjOut<C> oA;
            adj_shot<C, S0, S1, S2, S3>(g, xt, w, rnA, ahz1A, bhz1A, azA, bKA, KA[S0], MUA[k],
                                        MZA[k], PNA[k], WZA[k], b.lvz1[k], b.lvx[k], b.bx, b.bz1,
                                        axA, azA_, oA);
            // step A's new state as step B's input: zero outside the grid
            float mA[C];
#pragma unroll
            for (int c = 0; c < C; ++c)
                mA[c] = okt && w.colok[c] ? oA.opx[c] : 0.f;
            const unsigned ieA = rl.node(k, t);
            if (ieA != 0u)
                add_nodes<C>(a.nd, a.injA, nlA[k], nbase[k], ieA, w.lane, w.j0 - w.lane * C, mA);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                numA[c] += PNA[k][S0][c] * fmaf(-xt.ax[c], MUA[k][S0][c], mA[c]);
                const bool in = okt && w.colok[c];
                MUB[k][S3][c] = mA[c];
                MZB[k][S3][c] = rpt || w.colpml[c] ? (in ? oA.opz[c] : 0.f) : mA[c];
                PMB[k][S3][c] = b.pm[k][c];
            }
            if (runB) {
                AdjOut<C> oB;
                adj_shot<C, S0, S1, S2, S3>(g, xt, w, rnB, ahz1B, bhz1B, azB, bKB, KB[S0],
                                            MUB[k], MZB[k], PMB[k], WZB[k], dly[RZ + k],
                                            dly[RX + k], dly[RBX], dly[RBZ], axB, azB_, oB);
                const unsigned ieB = own && a.injB ? rl.node(k, r) : 0u;
                if (ieB != 0u)
                    add_nodes<C>(a.nd, a.injB, nlB[k], nbase[k], ieB, w.lane, w.j0 - w.lane * C, oB.opx);
#pragma unroll
                for (int c = 0; c < C; ++c)
                    numB[c] += PMB[k][S0][c] * fmaf(-xt.ax[c], MUB[k][S0][c], oB.opx[c]);
                const unsigned ko = skoff(a.lout, k);
                vst_row<C>(rLout, w, own, rbB + 2u * FB + ko, oB.opx);
#pragma unroll
                for (int c = 0; c < C; ++c)
                    bst(rLout, own ? zwB[c] : kOOB, zB.base + 3u * FB + ko, oB.opz[c]);
                vst_row<C>(rLout, w, own, rbB + ko, oB.ovx);
                vst_row<C>(rLout, w, ownz, rbZ + FB + ko, oB.ovz);
            }
            // step A's values for step B three rows later
#pragma unroll
            for (int c = 0; c < C; ++c) {
                D[S0][RX + k][c][w.lane] = okt && w.colok[c] ? oA.ovx[c] : 0.f;
                D[S0][RZ + k][c][w.lane] = rnA && w.colok[c] ? oA.ovz[c] : 0.f;
            }
        }
        if (runB) {
            // step A's sensitivities at row r, then step B's, as two one-step
            // launches add them (one reciprocal per row, 1 ulp)
            float gk[C], gx[C], gz[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float rK = KB[S0][c] != 0.f ? __builtin_amdgcn_rcpf(KB[S0][c]) : 0.f;
                gk[c] = L.gK[c] + dly[RNK][c] * rK;
                gk[c] = gk[c] + numB[c] * rK;
                gx[c] = L.gX[c] + dly[RAX][c];
                gx[c] = gx[c] + axB[c];
                gz[c] = L.gZ1[c] + dly[RAZ][c];
                gz[c] = gz[c] + azB_[c];
            }
            vst_row<C>(rG, w, own, rbB, gk);
            vst_row<C>(rG, w, own, rbB + FB, gx);
            vst_row<C>(rG, w, ownz, rbZ + 2u * FB, gz);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            D[S0][RNK][c][w.lane] = numA[c];
            D[S0][RAX][c][w.lane] = axA[c];
            D[S0][RAZ][c][w.lane] = azA_[c];
            D[S0][RBX][c][w.lane] = b.bx[c];
            D[S0][RBZ][c][w.lane] = b.bz1[c];
        }
    };

    A2Row<SPG, C> A, B;
    ALate<C> L;
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    using P2 = std::integral_constant<int, 2>;
    using P3 = std::integral_constant<int, 3>;
    load_row(tA0, A);
    for (int t = tA0;;) {
        load_late(t, L);
        load_row(t + 1, B);
        row(P0{}, t, A, L);
        if (++t >= tend)
            break;
        load_late(t, L);
        load_row(t + 1, A);
        row(P1{}, t, B, L);
        if (++t >= tend)
            break;
        load_late(t, L);
        load_row(t + 1, B);
        row(P2{}, t, A, L);
        if (++t >= tend)
            break;
        load_late(t, L);
        load_row(t + 1, A);
        row(P3{}, t, B, L);
        if (++t >= tend)
            break;
    }
}

inline unsigned blocks_of(const Sweep &sw)
{
    return (unsigned)((sw.nwaves + NTHR / WAVE - 1) / (NTHR / WAVE));
}

// The start / stop events (may be null) take the dispatch's own start and
// end times.
template <int SPG, int C>
void launch_f(const Geo &g, const float *tabs, const float *model, const SweepTables *T, int S,
              const Sweep &sw, const FwdStep &a, hipStream_t st, hipEvent_t e0, hipEvent_t e1)
{
    hipExtLaunchKernelGGL((k_fwd<SPG, C>), dim3(blocks_of(sw)), dim3(NTHR), 0, st, e0, e1, 0, g,
                          tabs, model, T, S, sw, a);
}
template <int SPG, int C>
void launch_f2(const Geo &g, const float *tabs, const float *model, const SweepTables *T, int S,
               const Sweep &sw, const FwdStep2 &a, hipStream_t st, hipEvent_t e0, hipEvent_t e1)
{
    hipExtLaunchKernelGGL((k_fwd2<SPG, C>), dim3(blocks_of(sw)), dim3(NTHR), 0, st, e0, e1, 0, g,
                          tabs, model, T, S, sw, a);
}
template <int SPG, int C>
void launch_a(const Geo &g, const float *tabs, const float *model, const Sweep &sw,
              const AdjStep &a, hipStream_t st, hipEvent_t e0, hipEvent_t e1)
{
    hipExtLaunchKernelGGL((k_adj<SPG, C>), dim3(blocks_of(sw)), dim3(NTHR), 0, st, e0, e1, 0, g,
                          tabs, model, sw, a);
}

template <int SPG, int C>
void launch_a2(const Geo &g, const float *tabs, const float *model, const Sweep &sw,
               const AdjStep2 &a, hipStream_t st, hipEvent_t e0, hipEvent_t e1)
{
    hipExtLaunchKernelGGL((k_adj2<SPG, C>), dim3(blocks_of(sw)), dim3(NTHR), 0, st, e0, e1, 0, g,
                          tabs, model, sw, a);
}

// Waves of `kern` that the current device holds at once: its workgroups per
// compute unit (from its register and LDS use) times the compute units, or
// 0 when the runtime cannot tell.
template <typename Kern>
int resident_waves(Kern kern)
{
    int blocks = 0, dev = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, kern, NTHR, 0) != hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return blocks * (NTHR / WAVE) * cus;
}

}  // namespace

int resident_waves2(int spg, int cols)
{
    switch (cols * 16 + spg) {
    case 16 + 1: return resident_waves(k_fwd2<1, 1>);
    case 16 + 2: return resident_waves(k_fwd2<2, 1>);
    case 32 + 1: return resident_waves(k_fwd2<1, 2>);
    case 32 + 2: return resident_waves(k_fwd2<2, 2>);
    case 64 + 1: return resident_waves(k_fwd2<1, 4>);
    }
    return 0;
}

// Instantiated (shots per group, columns per lane) pairs of the two-step
// adjoint kernel.
bool adj2_supported(int spg, int cols)
{
    return cols == 1 ? (spg == 1 || spg == 2 || spg == 4) : (cols == 2 && (spg == 1 || spg == 2));
}

// Instantiated (shots per group, columns per lane) pairs of the two-step
// forward kernel.
bool fused2_supported(int spg, int cols)
{
    return (spg == 1 || spg == 2) && (cols == 1 || cols == 2 || (cols == 4 && spg == 1));
}

// Instantiated (shots per group, columns per lane) pairs.
bool fused_supported(int spg, int cols)
{
    switch (cols) {
    case 1: return spg == 1 || spg == 2 || spg == 4 || spg == 8;
    case 2: return spg == 1 || spg == 2 || spg == 4;
    case 4: return spg == 1 || spg == 2;
    }
    return false;
}

int strip_cols(int cols, int steps)
{
    if (steps == 2) {
        switch (cols) {
        case 2: return Lanes<2, 2 * HALO>::W;
        case 4: return Lanes<4, 2 * HALO>::W;
        default: return Lanes<1, 2 * HALO>::W;
        }
    }
    switch (cols) {
    case 2: return Lanes<2>::W;
    case 4: return Lanes<4>::W;
    default: return Lanes<1>::W;
    }
}

Sweep sweep_of(const Geo &g, int S, int band_rows, int spg, int cols, int steps)
{
    Sweep sw;
    sw.H = band_rows;
    sw.spg = spg;
    sw.cols = cols;
    const int W = strip_cols(cols, steps);
    sw.nstrips = (g.Nx + W - 1) / W;
    sw.nbands = (g.Nz + band_rows - 1) / band_rows;
    sw.ngroups = (S + spg - 1) / spg;
    sw.nwaves = sw.nstrips * sw.nbands * sw.ngroups;
    return sw;
}

#define FWI_DISPATCH(fn, ...)                                                   \
    switch (sw.cols * 16 + sw.spg) {                                            \
    case 16 + 1: fn<1, 1>(__VA_ARGS__); break;                                  \
    case 16 + 2: fn<2, 1>(__VA_ARGS__); break;                                  \
    case 16 + 4: fn<4, 1>(__VA_ARGS__); break;                                  \
    case 16 + 8: fn<8, 1>(__VA_ARGS__); break;                                  \
    case 32 + 1: fn<1, 2>(__VA_ARGS__); break;                                  \
    case 32 + 2: fn<2, 2>(__VA_ARGS__); break;                                  \
    case 32 + 4: fn<4, 2>(__VA_ARGS__); break;                                  \
    case 64 + 1: fn<1, 4>(__VA_ARGS__); break;                                  \
    case 64 + 2: fn<2, 4>(__VA_ARGS__); break;                                  \
    default: break;                                                             \
    }

void launch_fused_fwd(const Geo &g, const float *tabs, const float *model,
                      const SweepTables *T, int S, const Sweep &sw, const FwdStep &a,
                      hipStream_t st, hipEvent_t e0, hipEvent_t e1)
{
    FWI_DISPATCH(launch_f, g, tabs, model, T, S, sw, a, st, e0, e1)
}

void launch_fused_fwd2(const Geo &g, const float *tabs, const float *model,
                       const SweepTables *T, int S, const Sweep &sw, const FwdStep2 &a,
                       hipStream_t st, hipEvent_t e0, hipEvent_t e1)
{
    switch (sw.cols * 16 + sw.spg) {
    case 16 + 1: launch_f2<1, 1>(g, tabs, model, T, S, sw, a, st, e0, e1); break;
    case 16 + 2: launch_f2<2, 1>(g, tabs, model, T, S, sw, a, st, e0, e1); break;
    case 32 + 1: launch_f2<1, 2>(g, tabs, model, T, S, sw, a, st, e0, e1); break;
    case 32 + 2: launch_f2<2, 2>(g, tabs, model, T, S, sw, a, st, e0, e1); break;
    case 64 + 1: launch_f2<1, 4>(g, tabs, model, T, S, sw, a, st, e0, e1); break;
    default: break;
    }
}

void launch_fused_adj2(const Geo &g, const float *tabs, const float *model, const Sweep &sw,
                       const AdjStep2 &a, hipStream_t st, hipEvent_t e0, hipEvent_t e1)
{
    switch (sw.cols * 16 + sw.spg) {
    case 16 + 1: launch_a2<1, 1>(g, tabs, model, sw, a, st, e0, e1); break;
    case 16 + 2: launch_a2<2, 1>(g, tabs, model, sw, a, st, e0, e1); break;
    case 16 + 4: launch_a2<4, 1>(g, tabs, model, sw, a, st, e0, e1); break;
    case 32 + 1: launch_a2<1, 2>(g, tabs, model, sw, a, st, e0, e1); break;
    case 32 + 2: launch_a2<2, 2>(g, tabs, model, sw, a, st, e0, e1); break;
    default: break;
    }
}

void launch_fused_adj(const Geo &g, const float *tabs, const float *model, const Sweep &sw,
                      const AdjStep &a, hipStream_t st, hipEvent_t e0, hipEvent_t e1)
{
    FWI_DISPATCH(launch_a, g, tabs, model, sw, a, st, e0, e1)
}

}  // namespace fwi

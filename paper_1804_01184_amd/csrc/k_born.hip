// Born modelling of schemes I and II in the frequency domain: Green
// function tables of the homogeneous reference medium, the single-scattering
// sum and its adjoint (the gradient in the inverse contrasts), the reduced
// 2x2 Hessian of a point scatterer, and the maps between parameter contrasts
// and inverse contrasts.
//
// Reference operator L0 = w^2/K0 + div (1/rho0) grad with L0 G0 = -delta and
// time dependence exp(-i w t): G0(r) = (i rho0/4) H0(k r), k = w sqrt(rho0/K0),
// grad_x G0(|x - y|) = -(i rho0 k/4) H1(k r) (x - y)/r, H_n = J_n + i Y_n the
// Hankel functions of the first kind.  Born term (section "Modelling and
// Inversion"): dA sum_c [w^2/K0 Gr Gs xi_{1/K} - (1/rho0) (Grx Gsx + Grz Gsz)
// xi_{1/rho}], Gr = G0(x_r; x_c), Gs = G0(x_c; x_s), gradients with respect
// to the cell position x_c.
//
// Tables are complex FP32 (re, im) in [F][C][P] order: for frequency f and
// cell c, the values of all points p are contiguous.  The Hankel functions
// are evaluated in FP64.
#include "fwi2d_internal.h"

#include <algorithm>
#include <atomic>

namespace fwi {

namespace {

constexpr double kPi = 3.14159265358979323846;

__device__ inline void cmac(float2 &acc, float2 a, float2 b)
{
    acc.x = fmaf(a.x, b.x, acc.x);
    acc.x = fmaf(-a.y, b.y, acc.x);
    acc.y = fmaf(a.x, b.y, acc.y);
    acc.y = fmaf(a.y, b.x, acc.y);
}

// H0 and H1 of the first kind, FP64, by polynomials fitted (interpolation at
// Chebyshev nodes in 50-digit arithmetic) to the smooth parts of the functions
// (Abramowitz & Stegun 9.1.10-9.1.13 and 9.2.5-9.2.10), with q = z^2:
//  z <= 8: J0 = kJ0(q), J1 = z kJ1(q), Y0 = (2/pi) ln(z/2) J0 + kY0(q),
//          Y1 = (2/pi) ln(z/2) J1 - 2/(pi z) + z kY1(q);
//  beyond: with t = 64/q, H0 = sqrt(2/(pi z)) (kP0(t) + i kQ0(t)/z) e^{i(z -
//          pi/4)}, H1 the same with kP1, kQ1 and 3 pi/4.
// The fits hold to 4e-13.  kSin, kCos: (sin r / r - 1) / r^2 and (cos r - 1 +
// r^2/2) / r^4 in r^2 on |r| <= pi/4; kAtanh: (atanh s / s - 1) / s^2 in s^2 for
// the logarithm of a number in [sqrt(1/2), sqrt(2)].
struct HankelFits {
    double j0[14];
    double j1[13];
    double y0[14];
    double y1[13];
    double p0[8];
    double q0[8];
    double p1[8];
    double q1[8];
    double sin[6];
    double cos[6];
    double atanh[7];
};

// Not const: the evaluation reads the coefficients with scalar loads, as scalar
// operands of the multiply-adds.  Folded into the code each would cost two
// vector moves, or, hoisted, two vector registers.
__constant__ HankelFits kHankelFits = {
    // j0
    {
        0.9999999999999572043, -0.24999999999973782578, 0.015624999999733470806,
        -0.00043402777767097507023, 6.7816840054270305896e-6, -6.7816837473309711815e-8,
        4.709500514671600133e-10, -2.4027949215353595835e-12, 9.3854789987930326262e-15,
        -2.8955704111326555279e-17, 7.2165659298467443337e-20, -1.4619900035641834196e-22,
        2.2916232939754155663e-25, -2.1572475316340808821e-28},
    // j1
    {
        0.49999999999992488639, -0.062499999999603210955, 0.0026041666663190563466,
        -0.00005425347210246335148, 6.7816838131915695578e-7, -5.6514010654425559235e-9,
        3.3639148438873005429e-11, -1.5016822309942907482e-13, 5.2121314499462638237e-16,
        -1.443437545998798192e-18, 3.2172429633435731951e-21, -5.502789423709497323e-24,
        5.6110340657238926651e-27},
    // y0
    {
        0.36746690519668789215, 0.067288216792300682914, -0.0091791055207200690225,
        0.00034707870821628387703, -6.5024433166199339449e-6, 7.3659137111036989289e-8,
        -5.6149081110198401634e-10, 3.0832547273758600763e-12, -1.2790137344919944897e-14,
        4.150497425842241877e-17, -1.0799648959402175201e-19, 2.2689972911032069787e-22,
        -3.6608996610966444043e-25, 3.5163693313010823991e-28},
    // y1
    {
        0.024578509506537139641, 0.026769238140771144964, -0.0018061615847086134648,
        0.000047702192492997437319, -6.9341784126636405219e-7, 6.4380742801699146213e-9,
        -4.1635927937762061729e-11, 1.98668016056152811e-13, -7.2867028061173489042e-16,
        2.1141510222845600483e-18, -4.8997388290641789349e-21, 8.6427197945358487798e-24,
        -9.0030089590404234719e-27},
    // p0
    {
        0.99999999999994500632, -0.0010986328054246964598, 0.000027380731218344226662,
        -2.1826361458224328399e-6, 3.5653580416357752692e-7, -8.8784284458752349479e-8,
        2.2779968314839150533e-8, -3.4847854195629241764e-9},
    // q0
    {
        -0.12499999999965337459, 0.0011444091350653774757, -0.000055445324997359559167,
        6.582591018335405075e-6, -1.4177993431358785477e-6, 4.2391321045424295295e-7,
        -1.20507062055868782e-7, 1.9422201870656740034e-8},
    // p1
    {
        1.0000000000000594474, 0.0018310546798520035145, -0.000035203828536838568742,
        2.5796093876226302928e-6, -4.0437007550875756549e-7, 9.8499853783403413323e-8,
        -2.4999275865222461659e-8, 3.8049125847715505426e-9},
    // q1
    {
        0.37499999999962687244, -0.001602172803530637258, 0.00006776664917162284443,
        -7.5959349964801027881e-6, 1.5861085097058607519e-6, -4.6621640070498607782e-7,
        1.3141200534002729273e-7, -2.1094092541175852538e-8},
    // sin
    {
        -0.16666666666666664498, 0.0083333333333308269303, -0.00019841269836575642768,
        2.7557316008147241632e-6, -2.5051112268671621888e-8, 1.5916725966176020443e-10},
    // cos
    {
        0.04166666666666666531, -0.0013888888888887321196, 0.000024801587298651250119,
        -2.7557317212671384338e-7, 2.0876134021649628009e-9, -1.1381754511224291529e-11},
    // atanh
    {
        0.33333333333333350761, 0.19999999999943257228, 0.14285714315895303417,
        0.11111105098130762589, 0.090914783874292007506, 0.076647481537395702497,
        0.073218370965616570338},
};

typedef const HankelFits __attribute__((address_space(4))) *FitsPtr;

typedef const double __attribute__((address_space(4))) *CoefPtr;

// The polynomial with M coefficients c at x.
template <int M>
__device__ inline double poly(CoefPtr c, double x)
{
    // left to itself the compiler copies each c to vector registers (two moves)
    // to accumulate into it
    double v;
    asm("v_mov_b64 %0, %1" : "=v"(v) : "s"(c[M - 1]));
#pragma unroll
    for (int i = M - 2; i >= 0; --i) {
        double u;
        asm("v_fma_f64 %0, %1, %2, %3" : "=v"(u) : "v"(v), "v"(x), "s"(c[i]));
        v = u;
    }
    return v;
}

// 1 / sqrt(x), x > 0: the hardware's estimate and one step of third order.
__device__ inline double rsqrt_pos(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// ln x of a normal x > 0; -inf at 0, NaN below.
__device__ inline double log_pos(FitsPtr fit, double x)
{
    double m = __builtin_amdgcn_frexp_mant(x);
    int e = __builtin_amdgcn_frexp_exp(x);
    const bool low = m < 0.70710678118654752;
    m = low ? m + m : m;
    e = low ? e - 1 : e;
    const double d = m + 1.0;
    double rd = __builtin_amdgcn_rcp(d);
    rd = fma(fma(-d, rd, 1.0), rd, rd);
    rd = fma(fma(-d, rd, 1.0), rd, rd);
    const double s = (m - 1.0) * rd, w = s * s;
    const double l =
        fma((double)e, 0.69314718055994530942, 2.0 * fma(s * w, poly<7>(fit->atanh, w), s));
    return x > 0.0 ? l : (x == 0.0 ? -__builtin_inf() : __builtin_nan(""));
}

// H0 and H1 at z = k r: rz = 1 / z, lz = (2/pi) ln(z/2), az = sqrt(2/(pi z)).  The
// reduction of z - pi/4 holds to 2^50; beyond, where a double z no longer
// carries a phase, it is only kept in range.
__device__ inline void hankel01(FitsPtr fit, double z, double rz, double lz, double az,
                                double2 &h0, double2 &h1)
{
    if (fabs(z) <= 8.0) {
        const double q = z * z;
        const double j0 = poly<14>(fit->j0, q), j1 = z * poly<13>(fit->j1, q);
        const double y0 = poly<14>(fit->y0, q), y1 = poly<13>(fit->y1, q);
        h0 = make_double2(j0, fma(lz, j0, y0));
        h1 = make_double2(j1, fma(lz, j1, fma(z, y1, -(2.0 / kPi) * rz)));
        return;
    }
    const double t = 64.0 * rz * rz;
    // z - pi/4 = n pi/2 + r, |r| <= pi/4, with pi/2 and pi/4 in two parts; adding
    // and taking off 1.5 x 2^52 rounds to n and leaves n mod 4 in the low bits
    const double zc = fmin(z, 0x1p50);
    const double u = fma(zc, 2.0 / kPi, -0.5) + 0x1.8p52, n = u - 0x1.8p52;
    const int quadrant = __double2loint(u);
    double r = fma(-n, 0x1.921fb54442d18p+0, zc) - 0x1.921fb54442d18p-1;
    r -= fma(n, 0x1.1a62633145c07p-54, 0x1.1a62633145c07p-55);
    const double w = r * r;
    const double sn = fma(r * w, poly<6>(fit->sin, w), r);
    const double cs = fma(w * w, poly<6>(fit->cos, w), fma(-0.5, w, 1.0));
    const double s1 = quadrant & 1 ? cs : sn, c1 = quadrant & 1 ? -sn : cs;
    const double amp = __hiloint2double(__double2hiint(az) ^ ((quadrant & 2) << 30),
                                        __double2loint(az));
    const double s = amp * s1, c = amp * c1;
    const double P0 = poly<8>(fit->p0, t), Q0 = poly<8>(fit->q0, t) * rz;
    const double P1 = poly<8>(fit->p1, t), Q1 = poly<8>(fit->q1, t) * rz;
    // e^{i(z - 3 pi/4)} = -i e^{i(z - pi/4)}
    h0 = make_double2(P0 * c - Q0 * s, P0 * s + Q0 * c);
    h1 = make_double2(P1 * s + Q1 * c, Q1 * s - P1 * c);
}

// One entry a thread for a run of frequencies: the distance, its logarithm and
// its roots serve all of them.  Entries are taken in the order of the table
// (cell by cell, points contiguous), so that a wave's store is 512 contiguous
// bytes and k r, and with it the branch of the Hankel evaluation, varies
// little across it.  Tiles of 64 cells x 32 points through LDS, and waves of 8
// x 8 or 4 x 16 entries, share fewer branches but write parts of 64-byte
// pieces: as fast at 360 points, 1.3 to 1.6 times as long at 100 and 211.
// grid: x, z = pieces of 256 entries, y = runs of frequencies.
//
// What bounds it is the FP64 rate: at 401^2 cells, 400 points, 4 frequencies
// (6.2 GB) 1.40 ms, 4.1 ms with the term-by-term series and one entry and
// frequency at a time that this replaces; writing alone would take 0.95 ms.
constexpr int kGreenRun = 64;   // frequencies in a run at most

__global__ __launch_bounds__(256) void k_born_green(int F, int frun, int C, int P,
                                                    const float *omega, const float *cells,
                                                    const float *pts, double slow, double rho0,
                                                    float2 *G, float2 *Gx, float2 *Gz)
{
    __shared__ double4 wave[kGreenRun];   // k, 1/k, (2/pi) ln(k/2), sqrt(2/(pi k))
    FitsPtr fit = (FitsPtr)&kHankelFits;
    const int f0 = (int)blockIdx.y * frun, f1 = min(f0 + frun, F);
    if (f0 + (int)threadIdx.x < f1) {
        const double k = (double)omega[f0 + threadIdx.x] * slow;
        wave[threadIdx.x] = make_double4(k, 1.0 / k, (2.0 / kPi) * log_pos(fit, 0.5 * k),
                                         0.79788456080286535588 * rsqrt_pos(k));
    }
    __syncthreads();
    const long long e0 = ((long long)blockIdx.z * gridDim.x + blockIdx.x) * 256;
    const long long cb = e0 / P;
    const unsigned t = (unsigned)(e0 - cb * P) + threadIdx.x;
    const long long c = cb + t / (unsigned)P, q = t % (unsigned)P;
    if (c >= C)
        return;
    const double dx = (double)cells[2 * c] - (double)pts[2 * q];
    const double dz = (double)cells[2 * c + 1] - (double)pts[2 * q + 1];
    const double r2 = dx * dx + dz * dz;
    const double rr = rsqrt_pos(r2), r = r2 * rr, rs = rsqrt_pos(r);
    const double ux = dx * rr, uz = dz * rr;
    const double lr = (1.0 / kPi) * log_pos(fit, r2);
    const double a = 0.25 * rho0;
    long long at = ((long long)f0 * C + c) * P + q;
    for (int f = f0; f < f1; ++f, at += (long long)C * P) {
        asm volatile("" : "+s"(fit));   // read anew for each frequency, not held across
        const double4 k = wave[f - f0];
        double2 h0, h1;
        hankel01(fit, k.x * r, k.y * rr, k.z + lr, k.w * rs, h0, h1);
        // G = (i rho0/4)(J0 + i Y0); grad = (rho0 k/4)(Y1 - i J1) (x - y)/r
        float2 g = make_float2((float)(-a * h0.y), (float)(a * h0.x));
        const double b = a * k.x, by = b * h1.y, bj = -b * h1.x;
        float2 gx = make_float2((float)(by * ux), (float)(bj * ux));
        float2 gz = make_float2((float)(by * uz), (float)(bj * uz));
        if (!(r2 > 0.0))
            g = gx = gz = make_float2(0.f, 0.f);
        G[at] = g;
        if (Gx) {
            Gx[at] = gx;
            Gz[at] = gz;
        }
    }
}

// Cells staged per step of the data kernel.
constexpr int kCB = 16;

// Partial Born sums of one frequency over a range of cells:
// part[split][f][s][r] = sum_{c in range} aK xiK[c] Gr Gs + cR xiR[c] (Grx Gsx + Grz Gsz)
// with aK = w_f^2 dA / K0, cR = -dA / rho0.  One lane per receiver; the
// source-side values of a chunk of kCB cells (and the cell coefficients) sit
// in LDS and are read by every lane at the same address.
// grid: x = receiver tiles of blockDim.x, y = source chunks of TS,
// z = f * nsplit + split.
template <int TS>
__global__ __launch_bounds__(512) void k_born_data(int F, int S, int R, int C, int nsplit,
                                                   int cells_per_split, const float *omega,
                                                   float dA_K0, float cR, const float *xiK,
                                                   const float *xiR, const float2 *Gs,
                                                   const float2 *Gsx, const float2 *Gsz,
                                                   const float2 *Gr, const float2 *Grx,
                                                   const float2 *Grz, float2 *part)
{
    __shared__ float2 sB[3][kCB][TS];
    __shared__ float sK[kCB], sR[kCB];
    const int f = blockIdx.z / nsplit;
    const int split = blockIdx.z % nsplit;
    const int s0 = blockIdx.y * TS;
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = r < R;
    const int rr = live ? r : R - 1;
    const int c_begin = split * cells_per_split;
    const int c_end = min(C, c_begin + cells_per_split);
    const float w = omega[f];
    const float aK = w * w * dA_K0;
    const long long fC = (long long)f * C;

    float2 acc[TS];
#pragma unroll
    for (int s = 0; s < TS; ++s)
        acc[s] = make_float2(0.f, 0.f);

    for (int c0 = c_begin; c0 < c_end; c0 += kCB) {
        const int nc = min(kCB, c_end - c0);
        __syncthreads();
        for (int e = threadIdx.x; e < kCB * TS; e += blockDim.x) {
            const int cc = e / TS, s = e % TS;
            float2 v0 = make_float2(0.f, 0.f), v1 = v0, v2 = v0;
            if (cc < nc && s0 + s < S) {
                const long long o = (fC + c0 + cc) * S + s0 + s;
                v0 = Gs[o];
                v1 = Gsx[o];
                v2 = Gsz[o];
            }
            sB[0][cc][s] = v0;
            sB[1][cc][s] = v1;
            sB[2][cc][s] = v2;
        }
        if (threadIdx.x < kCB) {
            const int cc = threadIdx.x;
            sK[cc] = cc < nc ? aK * xiK[c0 + cc] : 0.f;
            sR[cc] = cc < nc ? cR * xiR[c0 + cc] : 0.f;
        }
        __syncthreads();
        for (int cc = 0; cc < nc; ++cc) {
            const long long o = (fC + c0 + cc) * R + rr;
            const float2 g = Gr[o], gx = Grx[o], gz = Grz[o];
            const float k = sK[cc], q = sR[cc];
            const float2 a0 = make_float2(k * g.x, k * g.y);
            const float2 a1 = make_float2(q * gx.x, q * gx.y);
            const float2 a2 = make_float2(q * gz.x, q * gz.y);
#pragma unroll
            for (int s = 0; s < TS; ++s) {
                cmac(acc[s], a0, sB[0][cc][s]);
                cmac(acc[s], a1, sB[1][cc][s]);
                cmac(acc[s], a2, sB[2][cc][s]);
            }
        }
    }
    if (!live)
        return;
    float2 *out = part + ((long long)split * F + f) * S * R;
#pragma unroll
    for (int s = 0; s < TS; ++s)
        if (s0 + s < S)
            out[(long long)(s0 + s) * R + r] = acc[s];
}

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4f8 __attribute__((ext_vector_type(4), aligned(8)));   // two float2 of a table
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// Three bf16 parts of a pair of FP32 values, one pair in a register (x below):
// x = h + m + l to 24 bits and more, each the rest's nearest bf16.  Sums of
// products on the bf16 matrix cores take the six products h h, h m, m h, m m,
// h l, l h; the dropped ones are within 2^-24 of the product, the size of an FP32
// rounding of it.  Against FP64 sums over the same tables the data are off by 1.3
// to 2.3e-7 at 9 to 53 sources (FP32 matrix instructions: 1.3 to 4.9e-7), the
// gradients by 0.5 to 3.7e-7 (0.6 to 4.4e-7).  The range is narrower than FP32's:
// below about 2^-110 the low parts fall under the smallest bf16 and vanish, and an
// infinite value gives NaN (inf - inf).
struct Split3 {
    unsigned h, m, l;
};

__device__ inline unsigned bf16_pair(float x, float y)
{
    typedef float v2f __attribute__((ext_vector_type(2)));
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){x, y}, v2bf));
}

__device__ inline Split3 split3(float x, float y)
{
    Split3 s;
    s.h = bf16_pair(x, y);
    x -= __uint_as_float(s.h << 16);
    y -= __uint_as_float(s.h & 0xffff0000u);
    s.m = bf16_pair(x, y);
    x -= __uint_as_float(s.m << 16);
    y -= __uint_as_float(s.m & 0xffff0000u);
    s.l = bf16_pair(x, y);
    return s;
}

// A matrix operand of v_mfma_f32_16x16x32_bf16 in parts [h, m, l]: 4 pairs a
// lane.  Lane l holds row (or column) l % 16 and 8 of 32 k, which of them is for
// the caller to choose, the same for both operands; D[4 (l / 16) + v][l % 16] is
// left in register v of lane l.
struct Frag3 {
    uint4 part[3];
};

__device__ inline Frag3 frag3(const Split3 (&p)[4])
{
    Frag3 f;
    f.part[0] = make_uint4(p[0].h, p[1].h, p[2].h, p[3].h);
    f.part[1] = make_uint4(p[0].m, p[1].m, p[2].m, p[3].m);
    f.part[2] = make_uint4(p[0].l, p[1].l, p[2].l, p[3].l);
    return f;
}

// (re, -im) and (im, re) of pairs (re, im).
__device__ inline uint4 conj_form(uint4 u)
{
    const unsigned n = 0x80000000u;
    return make_uint4(u.x ^ n, u.y ^ n, u.z ^ n, u.w ^ n);
}

__device__ inline uint4 swap_form(uint4 u)
{
    return make_uint4(__builtin_amdgcn_alignbit(u.x, u.x, 16),
                      __builtin_amdgcn_alignbit(u.y, u.y, 16),
                      __builtin_amdgcn_alignbit(u.z, u.z, 16),
                      __builtin_amdgcn_alignbit(u.w, u.w, 16));
}

__device__ inline v4f mfma_bf16(uint4 a, uint4 b, v4f d)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a),
                                                   __builtin_bit_cast(v8bf, b), d, 0, 0, 0);
}

// The six products, the small ones first: part of the first operand, of the second.
constexpr int kProducts = 6;
constexpr int kProdA[kProducts] = {2, 0, 1, 1, 0, 0}, kProdB[kProducts] = {0, 2, 1, 0, 1, 0};

// The same partial sums on the matrix cores: per frequency and cell range,
// D[r][s] = sum_k A[k][r] B[k][s] with k running over (table, cell) and
// complex entries, A = receiver table, B = coefficient x source table, both in
// three bf16 parts.  A complex product is two real ones over k = (cell, re / im
// part): Re D = sum ar br - ai bi, Im D = sum ar bi + ai br, so that the
// receiver side comes in two forms, (ar, -ai) and (ai, ar).
// A wave computes 32 receivers x 16 NS sources from chunks of 16 cells; a lane
// reads two neighbouring receivers at once (rows of two tiles) at four cells.
// The four waves of a block take consecutive receiver groups of one (frequency,
// cell range, source group) and share, per chunk, the source side in LDS (two
// buffers).  The next chunk is loaded while one is computed.  Blocks are
// remapped so that those of one cell range run on one XCD.
//
// Reading the tables and the matrix instructions bound it together: at three
// source tiles a chunk is 12 KB and 216 instructions of 16 cycles a wave (432 of
// 32 cycles with FP32 operands, which alone were the bound).  401^2 cells, 40 x
// 360 pairs, 16 frequencies (24.8 GB of tables): 5.9 ms, 10.5 ms with FP32
// operands; 4.4 ms with the first of the six products alone.  16 receivers a
// wave, for three or four waves a SIMD, take 6.9 to 8.0 ms; splitting one tile
// between the products of another, 6.2 to 6.5 ms.
// Cells per chunk of the matrix-core data kernel.
constexpr int kDCH = 16;

template <int NS, bool PAIRS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_born_data_mfma(
    int F, int S, int R, int C, int nsplit, int cells_per_split, int sgroups, int nrg,
    long long nblocks, const float *omega, float dA_K0, float cR, const float *xiK,
    const float *xiR, const float2 *Gs, const float2 *Gsx, const float2 *Gsz, const float2 *Gr,
    const float2 *Grx, const float2 *Grz, float2 *part)
{
    constexpr int SW = 16 * NS;
    constexpr int kItems = 3 * 4 * SW;   // (table, four cells, source) staged per chunk
    constexpr int NST = (kItems + 255) / 256;
    __shared__ uint4 sB[2][3][3][4][SW];   // [buffer][table][part][cell % 4][source]
    const long long per = (nblocks + 7) / 8;
    const long long w = (long long)(blockIdx.x % 8) * per + blockIdx.x / 8;
    if (w >= nblocks)
        return;
    const int bpr = (nrg + 3) / 4;
    const int rb = (int)(w % bpr);
    long long fsg = w / bpr;
    const int sg = (int)(fsg % sgroups);
    fsg /= sgroups;
    const int split = (int)(fsg % nsplit);
    const int f = (int)(fsg / nsplit);
    const int rg = rb * 4 + (int)(threadIdx.x >> 6);
    // a wave past the last receiver group still stages and waits with the
    // others; it computes and stores nothing
    const bool active = rg < nrg;
    const int l = threadIdx.x & 63;
    const int li = l & 15, kk = l >> 4;
    // the last group is moved back to end with the last receiver; below 32
    // receivers (PAIRS false) rows past the end repeat the last one
    const int r_first = (active ? rg : 0) * 32, r0 = max(0, min(r_first, R - 32)), s0 = sg * SW;
    const int ra = min(r0 + 2 * li, R - 1), rb1 = min(ra + 1, R - 1);
    const int c_begin = split * cells_per_split;
    const int c_end = min(C, c_begin + cells_per_split);
    const float wf = omega[f];
    const float aK = wf * wf * dA_K0;
    const long long fC = (long long)f * C;
    v4f dre[2][NS], dim[2][NS];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < NS; ++b) {
            dre[a][b] = v4f{0.f, 0.f, 0.f, 0.f};
            dim[a][b] = v4f{0.f, 0.f, 0.f, 0.f};
        }
    v4f av[3][4];           // [table][cell / 4]: two receivers, re and im
    float2 stg[NST][4];
    float sq[NST][4];
    // this thread's items of the source side: a table and a source (a column
    // past the last one repeats it and is not stored) at cells 4 j + ig
    const float2 *ib[NST];
    const float *ix[NST];
    float ic[NST];
    int ig[NST];
#pragma unroll
    for (int i = 0; i < NST; ++i) {
        const int e = min((int)threadIdx.x + 256 * i, kItems - 1), t = e / (4 * SW);
        ib[i] = (t == 0 ? Gs : (t == 1 ? Gsx : Gsz)) + (fC + c_begin) * S + min(s0 + e % SW, S - 1);
        ix[i] = (t == 0 ? xiK : xiR) + c_begin;
        ic[i] = t == 0 ? aK : cR;
        ig[i] = e / SW % 4;
    }
    // offsets of this lane's cells 4 j + kk of the chunk at CN, the last cell
    // again past the end
    long long off[4];
#define CHUNK_OFFSETS(CN)                                                                  \
    _Pragma("unroll") for (int j = 0; j < 4; ++j)                                          \
        off[j] = (long long)min(4 * j + kk, c_end - 1 - (CN)) * R;
    // receiver table T of the chunk at CN
#define LOAD_TABLE(CN, T)                                                                  \
    {                                                                                      \
        const float2 *base = ((T) == 0 ? Gr : ((T) == 1 ? Grx : Grz)) + (fC + (CN)) * R;   \
        _Pragma("unroll") for (int j = 0; j < 4; ++j)                                      \
        {                                                                                  \
            const float2 *row = base + off[j];                                             \
            if (PAIRS) {                                                                   \
                av[T][j] = *(const v4f8 *)(row + ra);                                      \
            } else {                                                                       \
                const float2 u = row[ra], v = row[rb1];                                    \
                av[T][j] = v4f{u.x, u.y, v.x, v.y};                                        \
            }                                                                              \
        }                                                                                  \
    }
    // this thread's share of the chunk's source side; cells past the end have
    // coefficient 0
#define LOAD_STAGE(CN)                                                                     \
    _Pragma("unroll") for (int i = 0; i < NST; ++i)                                        \
    {                                                                                      \
        if (256 * (i + 1) <= kItems || (int)threadIdx.x < kItems - 256 * i) {              \
            const int last = c_end - 1 - (CN);                                             \
            const float2 *B = ib[i] + (long long)((CN) - c_begin) * S;                     \
            const float *x = ix[i] + ((CN) - c_begin);                                     \
            _Pragma("unroll") for (int j = 0; j < 4; ++j)                                  \
            {                                                                              \
                const int g = 4 * j + ig[i], k = min(g, last);                             \
                stg[i][j] = B[(long long)k * S];                                           \
                sq[i][j] = (g <= last ? ic[i] : 0.f) * x[k];                               \
            }                                                                              \
        }                                                                                  \
    }
#define STORE_STAGE(BUF)                                                                   \
    _Pragma("unroll") for (int i = 0; i < NST; ++i)                                        \
    {                                                                                      \
        const int e = (int)threadIdx.x + 256 * i;                                          \
        if (256 * (i + 1) <= kItems || e < kItems) {                                       \
            const int t = e / (4 * SW), g = e / SW % 4, s = e % SW;                        \
            const Split3 p0 = split3(sq[i][0] * stg[i][0].x, sq[i][0] * stg[i][0].y);      \
            const Split3 p1 = split3(sq[i][1] * stg[i][1].x, sq[i][1] * stg[i][1].y);      \
            const Split3 p2 = split3(sq[i][2] * stg[i][2].x, sq[i][2] * stg[i][2].y);      \
            const Split3 p3 = split3(sq[i][3] * stg[i][3].x, sq[i][3] * stg[i][3].y);      \
            sB[BUF][t][0][g][s] = make_uint4(p0.h, p1.h, p2.h, p3.h);                      \
            sB[BUF][t][1][g][s] = make_uint4(p0.m, p1.m, p2.m, p3.m);                      \
            sB[BUF][t][2][g][s] = make_uint4(p0.l, p1.l, p2.l, p3.l);                      \
        }                                                                                  \
    }
    if (c_begin < c_end) {
        LOAD_STAGE(c_begin)
        CHUNK_OFFSETS(c_begin)
        LOAD_TABLE(c_begin, 0)
        LOAD_TABLE(c_begin, 1)
        LOAD_TABLE(c_begin, 2)
    }
    int buf = 0;
    for (int c0 = c_begin; c0 < c_end; c0 += kDCH, buf ^= 1) {
        // a buffer is written two chunks after its last readers, who have
        // passed the barrier between
        STORE_STAGE(buf)
        __syncthreads();
        // the next chunk (this one again after the last) is loaded while this
        // one is computed, each receiver table once it has been split
        const int cn = c0 + kDCH < c_end ? c0 + kDCH : c0;
        LOAD_STAGE(cn)
        CHUNK_OFFSETS(cn)
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            Frag3 fre[2], fim[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const Split3 p[4] = {split3(av[t][0][2 * a], av[t][0][2 * a + 1]),
                                     split3(av[t][1][2 * a], av[t][1][2 * a + 1]),
                                     split3(av[t][2][2 * a], av[t][2][2 * a + 1]),
                                     split3(av[t][3][2 * a], av[t][3][2 * a + 1])};
                fim[a] = frag3(p);
                fre[a] = fim[a];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    fre[a].part[k] = conj_form(fim[a].part[k]);
                    fim[a].part[k] = swap_form(fim[a].part[k]);
                }
            }
            LOAD_TABLE(cn, t)
            if (active) {
#pragma unroll
                for (int b = 0; b < NS; ++b) {
                    uint4 g[3];
#pragma unroll
                    for (int k = 0; k < 3; ++k)
                        g[k] = sB[buf][t][k][kk][16 * b + li];
#pragma unroll
                    for (int k = 0; k < kProducts; ++k)
#pragma unroll
                        for (int a = 0; a < 2; ++a) {
                            dre[a][b] = mfma_bf16(fre[a].part[kProdA[k]], g[kProdB[k]], dre[a][b]);
                            dim[a][b] = mfma_bf16(fim[a].part[kProdA[k]], g[kProdB[k]], dim[a][b]);
                        }
                }
            }
        }
    }
#undef CHUNK_OFFSETS
#undef LOAD_TABLE
#undef LOAD_STAGE
#undef STORE_STAGE
    if (!active)
        return;
    float2 *out = part + ((long long)split * F + f) * S * R;
#pragma unroll
    for (int b = 0; b < NS; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const int r = r0 + 2 * (4 * kk + v) + a, sc = s0 + 16 * b + li;
                if (r >= r_first && r < R && sc < S)
                    out[(long long)sc * R + r] = make_float2(dre[a][b][v], dim[a][b][v]);
            }
}

// d[f][s][r] = spec[f] (Gd[f][s][r] + sum_split part[split][f][s][r]);
// Gd may be null (scattered data only).
__global__ __launch_bounds__(256) void k_born_finish(long long n, int SR, int nsplit,
                                                     const float2 *spec, const float2 *Gd,
                                                     const float2 *part, float2 *d)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        float2 v = Gd ? Gd[i] : make_float2(0.f, 0.f);
#pragma unroll 8
        for (int k = 0; k < nsplit; ++k) {
            const float2 p = part[(long long)k * n + i];
            v.x += p.x;
            v.y += p.y;
        }
        const float2 sp = spec[i / SR];
        d[i] = make_float2(sp.x * v.x - sp.y * v.y, sp.x * v.y + sp.y * v.x);
    }
}

// Receivers per chunk of the matrix-core gradient kernel.
constexpr int kGRC = 16;

// Receiver of pair j of lane group kk in a chunk: two neighbours at a time.
__device__ inline int grad_receiver(int kk, int j)
{
    return 8 * (j / 2) + 2 * kk + j % 2;
}

// The weights W[s][r] = conj(resid[f][s][r]) spec[f] of the gradient sums as
// first matrix operands (rows: 16 sources; k: 16 receivers, (wr, wi)) in three
// bf16 parts: Wf[f][source group][receiver chunk][source tile][part][lane].
// Zero past the last source and receiver.
__global__ __launch_bounds__(256) void k_born_weights(long long n, int S, int R, int sgroups,
                                                      int ns, int nchunk, const float2 *spec,
                                                      const float2 *resid, uint4 *Wf)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const int l = (int)(i % 64), li = l & 15, kk = l >> 4;
        long long k = i / 64;
        const int b = (int)(k % ns);
        k /= ns;
        const int ch = (int)(k % nchunk);
        k /= nchunk;
        const int sg = (int)(k % sgroups);
        const int f = (int)(k / sgroups);
        const int s = (sg * ns + b) * 16 + li;
        const float2 sp = spec[f];
        Split3 p[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = ch * kGRC + grad_receiver(kk, j);
            float2 q = make_float2(0.f, 0.f);
            if (s < S && r < R) {
                q = resid[((long long)f * S + s) * R + r];
                q = make_float2(q.x * sp.x + q.y * sp.y, q.x * sp.y - q.y * sp.x);
            }
            p[j] = split3(q.x, q.y);
        }
        uint4 *out = Wf + (i / 64 * 3) * 64 + l;
        const Frag3 w = frag3(p);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            out[64 * k] = w.part[k];
    }
}

// The gradient sums on the matrix cores.  Per frequency and table,
// U_t[s][c] = sum_r W[s][r] A_t[c][r] is a complex product with k over
// (receiver, re / im part), in three bf16 parts as in k_born_data_mfma: D[s][c]
// with the weights as the first operand (rows: 16 sources) and the receiver
// table as the second (columns: 16 cells).  A block takes 64 cells, 16 a wave; a
// lane reads its cell's rows, two neighbouring receivers at once, straight from
// the tables, and the weights of a chunk of 16 receivers go through LDS (two
// buffers, in the forms of the real and of the imaginary part), once for the
// block and its three tables.  The next chunk, across source groups and
// frequencies, is loaded while one is computed.  The epilogue of a frequency
// and source group adds Re sum_s Gs_t[c][s] U_t[s][c] per lane; the four lane
// groups holding one cell are summed at the end.
// grid: x = blocks of 64 cells, y = frequency ranges.
//
// Bound as the data kernel is: at the sizes named there 6.4 ms, 10.2 ms with FP32
// operands, 5.3 ms with one product of the six.  Three waves a SIMD take 7.9 ms
// (at one source tile, without spills, 5 % more than two), tables loaded two
// chunks ahead 6.6 ms.
template <int NS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_born_grad_mfma(
    int F, int S, int R, int C, int freqs_per_split, int sgroups, const float *omega,
    const uint4 *Wf, const float2 *Gs, const float2 *Gsx, const float2 *Gsz, const float2 *Gr,
    const float2 *Grx, const float2 *Grz, float *partK, float *partR)
{
    constexpr int kWords = NS * 3 * 64;   // operand words of a chunk, one form
    constexpr int NW = (kWords + 255) / 256;
    __shared__ uint4 sW[2][2][kWords];   // [buffer][real, imaginary][tile, part, lane]
    const int wave = (int)(threadIdx.x >> 6), l = (int)(threadIdx.x & 63);
    const int li = l & 15, kk = l >> 4;
    const int c = blockIdx.x * 64 + wave * 16 + li;
    const bool live = c < C;
    const int cl = live ? c : C - 1;
    const int f_begin = blockIdx.y * freqs_per_split;
    const int f_end = min(F, f_begin + freqs_per_split);
    const int nchunk = (R + kGRC - 1) / kGRC;
    float accK = 0.f, accR = 0.f, acc[3] = {0.f, 0.f, 0.f};

    v4f av[3][2];   // [table][receiver pair]
    uint4 rw[NW];
    auto load_weights = [&](const uint4 *W) {
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const int e = (int)threadIdx.x + 256 * k;
            rw[k] = W[e < kWords ? e : 0];
        }
    };
    auto load_tables = [&](int f, int ch) {
        const long long row = ((long long)f * C + cl) * R;
        const int r0 = ch * kGRC;
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const float2 *A = (t == 0 ? Gr : (t == 1 ? Grx : Grz)) + row;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int r = r0 + grad_receiver(kk, 2 * h);
                if (r0 + kGRC <= R) {
                    av[t][h] = *(const v4f8 *)(A + r);
                } else {
                    const float2 u = A[min(r, R - 1)], v = A[min(r + 1, R - 1)];
                    av[t][h] = v4f{u.x, u.y, v.x, v.y};
                }
            }
        }
    };
    v4f dre[3][NS], dim[3][NS];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int b = 0; b < NS; ++b) {
            dre[t][b] = v4f{0.f, 0.f, 0.f, 0.f};
            dim[t][b] = v4f{0.f, 0.f, 0.f, 0.f};
        }
    int f = f_begin, sg = 0, ch = 0, buf = 0;
    const uint4 *W = Wf + (long long)f_begin * sgroups * nchunk * kWords;
    if (f < f_end) {
        load_weights(W);
        load_tables(f, 0);
    }
    while (f < f_end) {
        // a buffer is written two chunks after its last readers, who have
        // passed the barrier between
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const int e = (int)threadIdx.x + 256 * k;
            if (e < kWords) {
                sW[buf][0][e] = conj_form(rw[k]);
                sW[buf][1][e] = swap_form(rw[k]);
            }
        }
        __syncthreads();
        Frag3 tab[3];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            Split3 p[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                p[j] = split3(av[t][j / 2][2 * (j % 2)], av[t][j / 2][2 * (j % 2) + 1]);
            tab[t] = frag3(p);
        }
        // the next chunk; this one again after the last
        int fn = f, sn = sg, cn = ch + 1;
        if (cn == nchunk) {
            cn = 0;
            if (++sn == sgroups) {
                sn = 0;
                ++fn;
            }
        }
        const bool more = fn < f_end;
        W += more ? kWords : 0;
        load_weights(W);
        load_tables(more ? fn : f, more ? cn : ch);
#pragma unroll
        for (int b = 0; b < NS; ++b) {
            uint4 wre[3], wim[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                wre[k] = sW[buf][0][(b * 3 + k) * 64 + l];
                wim[k] = sW[buf][1][(b * 3 + k) * 64 + l];
            }
#pragma unroll
            for (int k = 0; k < kProducts; ++k)
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    dre[t][b] = mfma_bf16(wre[kProdA[k]], tab[t].part[kProdB[k]], dre[t][b]);
                    dim[t][b] = mfma_bf16(wim[kProdA[k]], tab[t].part[kProdB[k]], dim[t][b]);
                }
        }
        if (cn == 0) {   // the last chunk of this frequency and source group
            const int s0 = sg * 16 * NS;
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const float2 *brow =
                    (t == 0 ? Gs : (t == 1 ? Gsx : Gsz)) + ((long long)f * C + cl) * S;
#pragma unroll
                for (int b = 0; b < NS; ++b) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int s = s0 + 16 * b + 4 * kk + v;
                        if (s < S) {
                            const float2 g = brow[s];
                            acc[t] = fmaf(g.x, dre[t][b][v], acc[t]);
                            acc[t] = fmaf(-g.y, dim[t][b][v], acc[t]);
                        }
                    }
                    dre[t][b] = v4f{0.f, 0.f, 0.f, 0.f};
                    dim[t][b] = v4f{0.f, 0.f, 0.f, 0.f};
                }
            }
            if (sn == 0) {
                const float w = omega[f];
                accK = fmaf(w * w, acc[0], accK);
                accR += acc[1] + acc[2];
                acc[0] = acc[1] = acc[2] = 0.f;
            }
        }
        f = fn;
        sg = sn;
        ch = cn;
        buf ^= 1;
    }
    // lanes li, li + 16, li + 32, li + 48 hold the same cell
    accK += __shfl_xor(accK, 16);
    accK += __shfl_xor(accK, 32);
    accR += __shfl_xor(accR, 16);
    accR += __shfl_xor(accR, 32);
    if (kk == 0 && live) {
        partK[(long long)blockIdx.y * C + c] = accK;
        partR[(long long)blockIdx.y * C + c] = accR;
    }
}

// gK[c] = dA/K0 sum_split partK, gR[c] = -dA/rho0 sum_split partR.
__global__ __launch_bounds__(256) void k_born_grad_finish(int C, int nsplit, float dA_K0,
                                                          float cR, const float *partK,
                                                          const float *partR, float *gK,
                                                          float *gR)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= C)
        return;
    float a = 0.f, b = 0.f;
    for (int k = 0; k < nsplit; ++k) {
        a += partK[(long long)k * C + c];
        b += partR[(long long)k * C + c];
    }
    gK[c] = dA_K0 * a;
    gR[c] = cR * b;
}

// d(xi_{1/K}, xi_{1/rho}) / d(xa, xb) at zero contrast; rows (1/K, 1/rho).
__host__ __device__ inline void linear_map(int param, float A[2][2])
{
    // K = rho Vp^2 and Ip = rho Vp linearised (Table 2)
    const float m[5][4] = {{-1.f, 0.f, 0.f, -1.f},   // K, rho
                           {-2.f, -1.f, 0.f, -1.f},  // Vp, rho
                           {-2.f, 1.f, 0.f, -1.f},   // Ip, rho
                           {-1.f, -1.f, 1.f, -1.f},  // Vp, Ip
                           {1.f, 0.f, 0.f, 1.f}};    // 1/K, 1/rho
    A[0][0] = m[param][0];
    A[0][1] = m[param][1];
    A[1][0] = m[param][2];
    A[1][1] = m[param][3];
}

// Scheme II: the exact inverse contrasts of a model m0 (1 + x) in a
// homogeneous background, and their derivatives.  With u = 1 + xa,
// v = 1 + xb: K-rho K/K0 = u, rho/rho0 = v; Vp-rho K/K0 = u^2 v; Ip-rho
// K/K0 = u^2 / v; Vp-Ip K/K0 = u v, rho/rho0 = v / u; 1/K-1/rho identity.
__device__ inline void exact_map(int param, float xa, float xb, float &xk, float &xr,
                                 float J[2][2])
{
    const float u = 1.f + xa, v = 1.f + xb;
    const float iu = 1.f / u, iv = 1.f / v;
    switch (param) {
    case 0:  // K, rho
        xk = iu - 1.f;
        xr = iv - 1.f;
        J[0][0] = -iu * iu; J[0][1] = 0.f;
        J[1][0] = 0.f;      J[1][1] = -iv * iv;
        break;
    case 1:  // Vp, rho: 1/K ~ u^-2 v^-1
        xk = iu * iu * iv - 1.f;
        xr = iv - 1.f;
        J[0][0] = -2.f * iu * iu * iu * iv; J[0][1] = -iu * iu * iv * iv;
        J[1][0] = 0.f;                      J[1][1] = -iv * iv;
        break;
    case 2:  // Ip, rho: 1/K ~ v u^-2
        xk = v * iu * iu - 1.f;
        xr = iv - 1.f;
        J[0][0] = -2.f * v * iu * iu * iu; J[0][1] = iu * iu;
        J[1][0] = 0.f;                     J[1][1] = -iv * iv;
        break;
    case 3:  // Vp, Ip: 1/K ~ (u v)^-1, 1/rho ~ u / v
        xk = iu * iv - 1.f;
        xr = u * iv - 1.f;
        J[0][0] = -iu * iu * iv; J[0][1] = -iu * iv * iv;
        J[1][0] = iv;            J[1][1] = -u * iv * iv;
        break;
    default:  // 1/K, 1/rho
        xk = xa;
        xr = xb;
        J[0][0] = 1.f; J[0][1] = 0.f;
        J[1][0] = 0.f; J[1][1] = 1.f;
        break;
    }
}

__global__ __launch_bounds__(256) void k_born_contrasts(int scheme, int param, long long n,
                                                        const float *xa, const float *xb,
                                                        float *xk, float *xr)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const float a = xa[i], b = xb[i];
        float J[2][2], k, r;
        if (scheme == 1) {
            linear_map(param, J);
            k = J[0][0] * a + J[0][1] * b;
            r = J[1][0] * a + J[1][1] * b;
        } else {
            exact_map(param, a, b, k, r, J);
        }
        xk[i] = k;
        xr[i] = r;
    }
}

__global__ __launch_bounds__(256) void k_born_chain(int scheme, int param, long long n,
                                                    const float *xa, const float *xb,
                                                    const float *gK, const float *gR,
                                                    float *ga, float *gb)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        float J[2][2], k, r;
        if (scheme == 1)
            linear_map(param, J);
        else
            exact_map(param, xa[i], xb[i], k, r, J);
        const float p = gK[i], q = gR[i];
        ga[i] = J[0][0] * p + J[1][0] * q;
        gb[i] = J[0][1] * p + J[1][1] * q;
    }
}

// Reduced Hessian of a point scatterer (section "Point-scatterer Analysis"):
// H = sum_f |S_f|^2 sum_{s,r} conj(W) W^T with W = A^T (w^2/K0 Gr Gs,
// -(1/rho0)(Grx Gsx + Grz Gsz)), A the scheme-I map of `param`.  Tables at
// the scatterer: sources [F][S], receivers [F][R].  One block of 256 lanes,
// FP64 accumulation, fixed-order reduction; out [2][2] complex (re, im).
__global__ __launch_bounds__(256) void k_born_hessian(int F, int S, int R, const float *omega,
                                                      const float2 *spec, double rK0,
                                                      double rrho0, const float2 *Gs,
                                                      const float2 *Gsx, const float2 *Gsz,
                                                      const float2 *Gr, const float2 *Grx,
                                                      const float2 *Grz, int param, float *out)
{
    __shared__ double red[4][256];
    double h00 = 0.0, h11 = 0.0, h01r = 0.0, h01i = 0.0;
    const long long n = (long long)F * S * R;
    for (long long i = threadIdx.x; i < n; i += blockDim.x) {
        const int r = (int)(i % R);
        const int s = (int)((i / R) % S);
        const int f = (int)(i / ((long long)R * S));
        const long long os = (long long)f * S + s, orr = (long long)f * R + r;
        const double w = omega[f];
        const double sp2 = (double)spec[f].x * spec[f].x + (double)spec[f].y * spec[f].y;
        const float2 a = Gr[orr], b = Gs[os];
        const double aK = w * w * rK0;
        const double wkr = aK * ((double)a.x * b.x - (double)a.y * b.y);
        const double wki = aK * ((double)a.x * b.y + (double)a.y * b.x);
        const float2 ax = Grx[orr], bx = Gsx[os], az = Grz[orr], bz = Gsz[os];
        const double wrr = -rrho0 * ((double)ax.x * bx.x - (double)ax.y * bx.y +
                                     (double)az.x * bz.x - (double)az.y * bz.y);
        const double wri = -rrho0 * ((double)ax.x * bx.y + (double)ax.y * bx.x +
                                     (double)az.x * bz.y + (double)az.y * bz.x);
        h00 += sp2 * (wkr * wkr + wki * wki);
        h11 += sp2 * (wrr * wrr + wri * wri);
        // conj(W_K) W_R
        h01r += sp2 * (wkr * wrr + wki * wri);
        h01i += sp2 * (wkr * wri - wki * wrr);
    }
    red[0][threadIdx.x] = h00;
    red[1][threadIdx.x] = h11;
    red[2][threadIdx.x] = h01r;
    red[3][threadIdx.x] = h01i;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int k = 0; k < 4; ++k)
                red[k][threadIdx.x] += red[k][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        // H_ab in the (1/K, 1/rho) basis: [[h00, h01], [conj h01, h11]]
        const double Hr[2][2] = {{red[0][0], red[2][0]}, {red[2][0], red[1][0]}};
        const double Hi[2][2] = {{0.0, red[3][0]}, {-red[3][0], 0.0}};
        float A[2][2];
        linear_map(param, A);
        for (int i = 0; i < 2; ++i)
            for (int j = 0; j < 2; ++j) {
                double re = 0.0, im = 0.0;
                for (int a = 0; a < 2; ++a)
                    for (int b = 0; b < 2; ++b) {
                        re += (double)A[a][i] * A[b][j] * Hr[a][b];
                        im += (double)A[a][i] * A[b][j] * Hi[a][b];
                    }
                out[2 * (2 * i + j)] = (float)re;
                out[2 * (2 * i + j) + 1] = (float)im;
            }
    }
}

int grid_for(long long n, int block)
{
    long long b = (n + block - 1) / block;
    return (int)std::max(1LL, std::min(b, 8192LL));
}

}  // namespace

void launch_born_green(int F, int C, int P, const float *omega, const float *cells,
                       const float *pts, double K0, double rho0, float *G, float *Gx, float *Gz,
                       hipStream_t st)
{
    const long long n = (long long)F * C * P;
    if (n <= 0)
        return;
    const long long pieces = ((long long)C * P + 255) / 256;
    // All frequencies in one run where the pieces alone fill the chip (8 resident
    // workgroups on each of 256 compute units) twice over, shorter runs below.
    const int runs = (int)std::min<long long>(F, (4095 + pieces) / pieces);
    const int frun = std::min((F + runs - 1) / runs, kGreenRun);
    const int nz = (int)((pieces + (1 << 22) - 1) >> 22);
    const dim3 grid((unsigned)((pieces + nz - 1) / nz), (unsigned)((F + frun - 1) / frun),
                    (unsigned)nz);
    hipLaunchKernelGGL(k_born_green, grid, dim3(256), 0, st, F, frun, C, P, omega, cells, pts,
                       std::sqrt(rho0 / K0), rho0, (float2 *)G, (float2 *)Gx, (float2 *)Gz);
}

// Source chunk width of the vector-FMA data kernel (below 9 sources): the
// smallest instantiated width covering S.
static int born_ts(int S)
{
    const int opts[] = {1, 2, 4, 8};
    for (int t : opts)
        if (t >= S)
            return t;
    return 8;
}

// Resident 256-thread blocks per CU of the matrix-core data kernel with NS
// source tiles (set by its register count), from the runtime's occupancy
// calculator; 4 if the query fails.
static int data_mfma_blocks_per_cu(int ns)
{
    static std::atomic<int> cache[5] = {0, 0, 0, 0, 0};
    if (ns < 1 || ns > 4)
        return 4;
    if (cache[ns].load(std::memory_order_relaxed) == 0) {
        int n = 0;
        hipError_t e = hipErrorInvalidValue;
        switch (ns) {
        case 1: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_born_data_mfma<1, true>, 256, 0); break;
        case 2: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_born_data_mfma<2, true>, 256, 0); break;
        case 3: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_born_data_mfma<3, true>, 256, 0); break;
        case 4: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_born_data_mfma<4, true>, 256, 0); break;
        }
        cache[ns].store((e == hipSuccess && n > 0) ? n : 4, std::memory_order_relaxed);
    }
    return cache[ns].load(std::memory_order_relaxed);
}

// Shortest cell range, over one round, that the matrix-core data kernel is split
// to: every range pays for filling its pipeline and writes its partial sums, which
// the finishing kernel reads (121^2 cells, 10 x 100 pairs, 15 frequencies: 150,
// 133, 119, 118 us at 64, 128, 256, 512; always 8 rounds: 264).
constexpr long long kRangeCells = 256;

BornSplit born_data_split(int F, int S, int R, int C)
{
    BornSplit b;
    b.ts = born_ts(S);
    // matrix cores for the data from 9 sources: below, both read the tables near
    // the memory rate and the vector kernel's chunk of 8 wastes less than a
    // 16-wide tile (201^2 cells, 200 receivers, 16 frequencies, vector and
    // matrix: 588 and 612 us at 4 sources, 602 and 645 at 8).  The gradient is on
    // the matrix cores for any number (one source, 401^2 cells, 360 receivers:
    // 4.1 ms, 8.5 with the vector kernel that there was)
    b.ns = S >= 9 ? std::min(4, (S + 15) / 16) : 0;
    b.gns = S >= 1 ? std::min(4, (S + 15) / 16) : 0;
    b.gsgroups = b.gns ? (S + 16 * b.gns - 1) / (16 * b.gns) : 0;
    int step = kCB;
    long long base;
    long long target;
    if (b.ns) {
        b.nrg = (R + 31) / 32;
        b.sgroups = (S + 16 * b.ns - 1) / (16 * b.ns);
        base = (long long)F * b.sgroups * b.nrg;       // waves per cell range
        target = 0;   // set below
        b.block = 256;
        b.rtiles = b.schunks = 0;
    } else {
        const int nw = std::max(1, std::min(8, (R + 63) / 64));
        b.block = 64 * nw;
        b.rtiles = (R + b.block - 1) / b.block;
        b.schunks = (S + b.ts - 1) / b.ts;
        base = (long long)F * b.rtiles * b.schunks;   // blocks per cell range
        target = 2048;
        b.nrg = b.sgroups = 0;
    }
    const int max_split = std::max(1, (C + step - 1) / step);
    long long want = base > 0 ? (target + base - 1) / base : 1;
    if (b.ns && base > 0) {
        // whole rounds of resident blocks (256 CUs x the blocks of 4 waves
        // that fit one CU at this kernel's register count), rounded down so that
        // the last round is full rather than nearly empty: 8, or fewer where the
        // ranges would get short
        const long long slots = 256LL * data_mfma_blocks_per_cu(b.ns);
        const long long per_range = std::max(1LL, base / b.nrg * ((b.nrg + 3) / 4));
        const long long rounds =
            std::max(1LL, std::min(8LL, C / kRangeCells * per_range / slots));
        want = std::max(1LL, rounds * slots / per_range);
    }
    b.nsplit = (int)std::max(1LL, std::min<long long>(want, max_split));
    if (C == 0)
        b.nsplit = 0;
    int per = b.nsplit ? (C + b.nsplit - 1) / b.nsplit : 0;
    per = (per + kCB - 1) / kCB * kCB;
    b.cells_per_split = per;
    if (per > 0)
        b.nsplit = (C + per - 1) / per;
    // gradient: blocks of 64 cells x frequency splits, about 8192 in all, 16
    // rounds of the 2 blocks that fit one CU (4096 and 16384: within 2 %);
    // each block's frequencies are summed in registers
    b.cblocks = (C + 63) / 64;
    const long long gtarget = 8192;
    const long long gw = b.cblocks > 0 ? (gtarget + b.cblocks - 1) / b.cblocks : 1;
    b.fsplit = (int)std::max(1LL, std::min<long long>(gw, std::max(F, 1)));
    b.freqs_per_split = F > 0 ? (F + b.fsplit - 1) / b.fsplit : 0;
    if (F > 0)
        b.fsplit = (F + b.freqs_per_split - 1) / b.freqs_per_split;
    return b;
}

size_t born_grad_wt_offset(const BornSplit &b, int C)
{
    return ((size_t)2 * std::max(b.fsplit, 1) * C * sizeof(float) + 255) / 256 * 256;
}

size_t born_grad_wt_bytes(const BornSplit &b, int F, int R)
{
    return (size_t)F * b.gsgroups * ((R + kGRC - 1) / kGRC) * b.gns * 3 * 64 * sizeof(uint4);
}

template <int NS>
static void data_mfma(const BornSplit &b, int F, int S, int R, int C, const float *omega,
                      float dA_K0, float cR, const float *xiK, const float *xiR,
                      const float2 *Gs, const float2 *Gsx, const float2 *Gsz, const float2 *Gr,
                      const float2 *Grx, const float2 *Grz, float2 *part, hipStream_t st)
{
    const long long nblocks = (long long)F * b.nsplit * b.sgroups * ((b.nrg + 3) / 4);
    const long long grid = (nblocks + 7) / 8 * 8;
    const auto kernel = R >= 32 ? k_born_data_mfma<NS, true> : k_born_data_mfma<NS, false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(256), 0, st, F, S, R, C, b.nsplit,
                       b.cells_per_split, b.sgroups, b.nrg, nblocks, omega, dA_K0, cR, xiK, xiR,
                       Gs, Gsx, Gsz, Gr, Grx, Grz, part);
}

template <int TS>
static void data_ts(const BornSplit &b, int F, int S, int R, int C, const float *omega,
                    float dA_K0, float cR, const float *xiK, const float *xiR, const float2 *Gs,
                    const float2 *Gsx, const float2 *Gsz, const float2 *Gr, const float2 *Grx,
                    const float2 *Grz, float2 *part, hipStream_t st)
{
    hipLaunchKernelGGL(k_born_data<TS>, dim3(b.rtiles, b.schunks, F * b.nsplit), dim3(b.block),
                       0, st, F, S, R, C, b.nsplit, b.cells_per_split, omega, dA_K0, cR, xiK,
                       xiR, Gs, Gsx, Gsz, Gr, Grx, Grz, part);
}

void launch_born_data(const BornSplit &b, int F, int S, int R, int C, const float *omega,
                      const float *spec, double K0, double rho0, double dA, const float *xiK,
                      const float *xiR, const float *Gs, const float *Gsx, const float *Gsz,
                      const float *Gr, const float *Grx, const float *Grz, const float *Gd,
                      float *d, float *part, hipStream_t st)
{
    const long long n = (long long)F * S * R;
    if (n <= 0)
        return;
    const float dA_K0 = (float)(dA / K0), cR = (float)(-dA / rho0);
    auto g2 = [](const float *p) { return (const float2 *)p; };
    if (b.nsplit > 0 && b.ns > 0) {
#define BORN_MFMA(N)                                                                       \
    case N:                                                                                \
        data_mfma<N>(b, F, S, R, C, omega, dA_K0, cR, xiK, xiR, g2(Gs), g2(Gsx), g2(Gsz),  \
                     g2(Gr), g2(Grx), g2(Grz), (float2 *)part, st);                        \
        break;
        switch (b.ns) { BORN_MFMA(1) BORN_MFMA(2) BORN_MFMA(3) BORN_MFMA(4) }
#undef BORN_MFMA
    } else if (b.nsplit > 0) {
#define BORN_DATA(T)                                                                       \
    case T:                                                                                \
        data_ts<T>(b, F, S, R, C, omega, dA_K0, cR, xiK, xiR, g2(Gs), g2(Gsx), g2(Gsz),    \
                   g2(Gr), g2(Grx), g2(Grz), (float2 *)part, st);                          \
        break;
        switch (b.ts) {
            BORN_DATA(1) BORN_DATA(2) BORN_DATA(4) BORN_DATA(8)
        }
#undef BORN_DATA
    }
    hipLaunchKernelGGL(k_born_finish, dim3(grid_for(n, 256)), dim3(256), 0, st, n, S * R,
                       b.nsplit, g2(spec), g2(Gd), (const float2 *)part, (float2 *)d);
}

void launch_born_gradient(const BornSplit &b, int F, int S, int R, int C, const float *omega,
                          const float *spec, double K0, double rho0, double dA,
                          const float *resid, const float *Gs, const float *Gsx,
                          const float *Gsz, const float *Gr, const float *Grx, const float *Grz,
                          float *gK, float *gR, float *part, hipStream_t st)
{
    if (C <= 0)
        return;
    const float dA_K0 = (float)(dA / K0), cR = (float)(-dA / rho0);
    float *partK = part, *partR = part + (long long)std::max(b.fsplit, 1) * C;
    if (F <= 0 || S <= 0 || R <= 0) {
        launch_fill(gK, C, 0.f, st);
        launch_fill(gR, C, 0.f, st);
        return;
    }
    auto g2 = [](const float *p) { return (const float2 *)p; };
    uint4 *Wf = (uint4 *)((char *)part + born_grad_wt_offset(b, C));
    const int nchunk = (R + kGRC - 1) / kGRC;
    const long long n = (long long)F * b.gsgroups * nchunk * b.gns * 64;
    hipLaunchKernelGGL(k_born_weights, dim3(grid_for(n, 256)), dim3(256), 0, st, n, S, R,
                       b.gsgroups, b.gns, nchunk, g2(spec), g2(resid), Wf);
#define BORN_GMFMA(N)                                                                      \
    case N:                                                                                \
        hipLaunchKernelGGL(k_born_grad_mfma<N>, dim3(b.cblocks, b.fsplit), dim3(256), 0, st, \
                           F, S, R, C, b.freqs_per_split, b.gsgroups, omega, Wf, g2(Gs),     \
                           g2(Gsx), g2(Gsz), g2(Gr), g2(Grx), g2(Grz), partK, partR);        \
        break;
    switch (b.gns) { BORN_GMFMA(1) BORN_GMFMA(2) BORN_GMFMA(3) BORN_GMFMA(4) }
#undef BORN_GMFMA
    hipLaunchKernelGGL(k_born_grad_finish, dim3((C + 255) / 256), dim3(256), 0, st, C, b.fsplit,
                       dA_K0, cR, partK, partR, gK, gR);
}

void launch_born_contrasts(int scheme, int param, long long n, const float *xa, const float *xb,
                           float *xk, float *xr, hipStream_t st)
{
    if (n <= 0)
        return;
    hipLaunchKernelGGL(k_born_contrasts, dim3(grid_for(n, 256)), dim3(256), 0, st, scheme, param,
                       n, xa, xb, xk, xr);
}

void launch_born_chain(int scheme, int param, long long n, const float *xa, const float *xb,
                       const float *gK, const float *gR, float *ga, float *gb, hipStream_t st)
{
    if (n <= 0)
        return;
    hipLaunchKernelGGL(k_born_chain, dim3(grid_for(n, 256)), dim3(256), 0, st, scheme, param, n,
                       xa, xb, gK, gR, ga, gb);
}

void launch_born_hessian(int F, int S, int R, const float *omega, const float *spec, double K0,
                         double rho0, const float *Gs, const float *Gsx, const float *Gsz,
                         const float *Gr, const float *Grx, const float *Grz, int param,
                         float *H, hipStream_t st)
{
    auto g2 = [](const float *p) { return (const float2 *)p; };
    hipLaunchKernelGGL(k_born_hessian, dim3(1), dim3(256), 0, st, F, S, R, omega, g2(spec),
                       1.0 / K0, 1.0 / rho0, g2(Gs), g2(Gsx), g2(Gsz), g2(Gr), g2(Grx), g2(Grz),
                       param, H);
}

}  // namespace fwi

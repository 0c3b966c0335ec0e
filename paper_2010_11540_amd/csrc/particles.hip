// Particle-side kernels of libscpic for gfx950: the fused particle pass
// (gather + kick, push, cloud-in-cell deposit into an LDS tile of the charge
// grid) in its four- and six-dimensional forms, with the long-bunch line
// density or the B-spline field, single-beam and batched; and the copy
// between split and interleaved field layouts.
//
// Compiled with -ffp-contract=off: every FP64 expression below is evaluated
// as written, each operation correctly rounded, so the cell index, the
// fixed-point weights and a linear push are bit-identical to the same IEEE
// sums evaluated anywhere else.  The thick elements, which have no
// bit-identical counterpart, use explicit fused multiply-adds.
#include <algorithm>
#include <climits>
#include <type_traits>
#include <vector>

#include "scpic_internal.h"

#pragma clang fp contract(off)

namespace scpic {
namespace {

constexpr int kWave = 64;

// Cell (i, j) holding the particle and its bilinear fractions of Sec. IV-A
// rounded to 12 bits per axis, a and b of 4096; the fixed-point weights of the
// nodes (i,j), (i+1,j), (i,j+1), (i+1,j+1) are (4096-a)(4096-b), a(4096-b),
// (4096-a)b and ab, summing to exactly 2^24.
struct Cic {
    int i, j, a, b;
};

// Keeps a uniform value in vector registers.  A pass has more uniform values
// alive in its particle loop than scalar registers (the compiler then parks
// them in lanes of a vector register and reads each back by an instruction of
// its own), and vector registers to spare: one workgroup of 1024 threads has a
// compute unit to itself, 128 registers per lane.
__device__ __forceinline__ double in_vector(double v)
{
    asm("" : "+v"(v));
    return v;
}

// The grid's geometry as cic() uses it.
struct GridCells {
    double x_min, y_min, inv_dx, inv_dy, nx1, ny1;
    static __device__ __forceinline__ GridCells of(const GridGeom &g)
    {
        return {g.x_min, g.y_min, g.inv_dx, g.inv_dy, (double)(g.nx - 1), (double)(g.ny - 1)};
    }
};

// False when the particle is outside [0, nx-1) x [0, ny-1) in node units (or
// NaN); c is then undefined.
__device__ __forceinline__ bool cic(const GridCells &g, double x, double y, Cic &c)
{
    const double tx = (x - g.x_min) * g.inv_dx;
    const double ty = (y - g.y_min) * g.inv_dy;
    if (!((tx >= 0.0) & (tx < g.nx1) & (ty >= 0.0) & (ty < g.ny1))) return false;
    cell_fraction(tx, c.i, c.a);
    cell_fraction(ty, c.j, c.b);
    return true;
}

template <typename TE>
struct Vec2;
template <>
struct Vec2<double> {
    using type = double2;
};
template <>
struct Vec2<float> {
    using type = float2;
};

// The four weights as TE, in units of 2^-24 (products of integers up to 2^12:
// exact).
template <typename TE>
struct Weights {
    TE w00, w10, w01, w11;
    __device__ __forceinline__ explicit Weights(const Cic &c)
    {
        const TE a = (TE)c.a, b = (TE)c.b;
        const TE a0 = (TE)kFracOne - a, b0 = (TE)kFracOne - b;
        w00 = a0 * b0;
        w10 = a * b0;
        w01 = a0 * b;
        w11 = a * b;
    }
    // of a value at the four nodes, in node order
    __device__ __forceinline__ TE sum(TE u00, TE u10, TE u01, TE u11) const
    {
        return w00 * u00 + w10 * u10 + w01 * u01 + w11 * u11;
    }
};

// The (Ex, Ey) of a cell's four nodes: node (i, j) at byte off of e, row the
// bytes from row i to i+1.
template <typename V>
struct CellField {
    V e00, e10, e01, e11;
    __device__ __forceinline__ void load(const V *e, uint32_t off, uint32_t row)
    {
        const char *p = reinterpret_cast<const char *>(e);
        const V *r0 = reinterpret_cast<const V *>(p + off);
        const V *r1 = reinterpret_cast<const V *>(p + (off + row));
        e00 = r0[0];
        e01 = r0[1];
        e10 = r1[0];
        e11 = r1[1];
    }
};

// Potential at the particle times 2^24 from its four nodes, weighted as the field.
template <typename TE>
__device__ __forceinline__ TE gather_scalar(const TE *u, int l00, int row, const Cic &c)
{
    return Weights<TE>(c).sum(u[l00], u[l00 + row], u[l00 + 1], u[l00 + row + 1]);
}

// Field at (x, y) in cell c (c.i, c.j from cic()) from the bicubic B-spline
// surface of the node potential u (nodes -1..nx by -1..ny):
//   phi = sum_{m,n} u[i+m-1][j+n-1] B_m(tx) B_n(ty),  E = -grad phi,
// with the uniform cubic basis B_m on the exact cell fractions (not the
// 12-bit ones of the deposit); rows are contracted first.  v: the potential on
// the cell's 4 x 4 nodes.
template <typename TE>
struct SplineNodes {
    TE v[4][4];
    // base: node (i-1, j-1), row: the distance from row to row
    __device__ __forceinline__ void load(const TE *base, int row)
    {
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int n = 0; n < 4; ++n) v[m][n] = base[m * row + n];
    }
};

template <typename TE>
__device__ __forceinline__ void bspline_field(const GridGeom &g, const SplineNodes<TE> &u,
                                              double x, double y, const Cic &c, TE &fx, TE &fy)
{
    const TE tx = (TE)((x - g.x_min) * g.inv_dx - (double)c.i);
    const TE ty = (TE)((y - g.y_min) * g.inv_dy - (double)c.j);
    TE bx[4], dbx[4], by[4], dby[4];
    auto basis = [](TE t, TE *b, TE *db) {
        const TE v = TE(1) - t, t2 = t * t;
        b[0] = v * v * v * TE(1.0 / 6.0);
        b[1] = (TE(3) * t2 * t - TE(6) * t2 + TE(4)) * TE(1.0 / 6.0);
        b[2] = (TE(-3) * t2 * t + TE(3) * t2 + TE(3) * t + TE(1)) * TE(1.0 / 6.0);
        b[3] = t2 * t * TE(1.0 / 6.0);
        db[0] = -v * v * TE(0.5);
        db[1] = (TE(3) * t2 - TE(4) * t) * TE(0.5);
        db[2] = (TE(-3) * t2 + TE(2) * t + TE(1)) * TE(0.5);
        db[3] = t2 * TE(0.5);
    };
    basis(tx, bx, dbx);
    basis(ty, by, dby);
    TE sx = 0, sy = 0;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const TE r = u.v[m][0] * by[0] + u.v[m][1] * by[1] + u.v[m][2] * by[2] + u.v[m][3] * by[3];
        const TE d =
            u.v[m][0] * dby[0] + u.v[m][1] * dby[1] + u.v[m][2] * dby[2] + u.v[m][3] * dby[3];
        sx = sx + dbx[m] * r;
        sy = sy + bx[m] * d;
    }
    fx = -sx * (TE)g.inv_dx;
    fy = -sy * (TE)g.inv_dy;
}

// Node k of the line and the particle's two fixed-point line weights
// (4096 - a at k, a at k + 1): t = (sigma - z_min)(1/dz), k = floor(t),
// a = floor((t - k) 4096 + 0.5), the one-dimensional form of cic().  False
// outside [0, nz - 1) in node units (or NaN); c is then undefined.
struct LineCic {
    int k, a;
};

__device__ __forceinline__ bool line_cic(const LineSpec &L, double sg, LineCic &c)
{
    const double t = (sg - L.z_min) * L.inv_dz;
    if (!((t >= 0.0) & (t < (double)(L.nz - 1)))) return false;
    cell_fraction(t, c.k, c.a);
    return true;
}

// One element applied to one particle (Sec. III): v <- M v for the linear
// maps, evaluated row by row left to right; the thin sextupole is the kick
// step of the split thick-sextupole integrator (Sec. III-C).
__device__ __forceinline__ void apply_element(int kind, const double *__restrict__ m, double &x,
                                              double &px, double &y, double &py)
{
    const double X = x, PX = px, Y = y, PY = py;
    if (kind == SCPIC_EL_LIN2X2) {
        x = m[0] * X + m[1] * PX;
        px = m[2] * X + m[3] * PX;
        y = m[4] * Y + m[5] * PY;
        py = m[6] * Y + m[7] * PY;
    } else if (kind == SCPIC_EL_LIN4X4) {
        x = m[0] * X + m[1] * PX + m[2] * Y + m[3] * PY;
        px = m[4] * X + m[5] * PX + m[6] * Y + m[7] * PY;
        y = m[8] * X + m[9] * PX + m[10] * Y + m[11] * PY;
        py = m[12] * X + m[13] * PX + m[14] * Y + m[15] * PY;
    } else if (kind == SCPIC_EL_SEXT_THIN) {
        const double k2l = m[0];
        px = PX - 0.5 * k2l * (X * X - Y * Y);
        py = PY + k2l * X * Y;
    }
}

// The thick elements below carry no bit-exactness contract (their reference
// evaluates other, equivalent formulas), so they use fused multiply-adds.

// sin and cos (HYP false) or sinh and cosh (HYP true) of phi0 + d from their
// values s0, c0 at phi0 and the Taylor series of the functions of d through
// d^11 and d^10 in Horner form (for |d| <= 1/16 the omitted terms are below
// 1e-19 of the result).
template <bool HYP>
__device__ __forceinline__ void shift_angle(double d, double s0, double c0, double &s, double &c)
{
    const double t = HYP ? d * d : -(d * d);
    double ps = fma(t, 1.0 / 39916800.0, 1.0 / 362880.0);
    ps = fma(t, ps, 1.0 / 5040.0);
    ps = fma(t, ps, 1.0 / 120.0);
    ps = fma(t, ps, 1.0 / 6.0);
    double pc = fma(t, 1.0 / 3628800.0, 1.0 / 40320.0);
    pc = fma(t, pc, 1.0 / 720.0);
    pc = fma(t, pc, 1.0 / 24.0);
    pc = fma(t, pc, 0.5);
    const double sd = fma(d * t, ps, d);
    const double cd = fma(t, pc, 1.0);
    s = fma(s0, cd, c0 * sd);
    c = HYP ? fma(c0, cd, s0 * sd) : fma(c0, cd, -(s0 * sd));
}

// One transverse plane of the thick quadrupole (Sec. III-B): u' = q p_u and
// p_u' = -K u with q = 1 - p_sigma (K = k1 for x, -k1 for y).  With C the
// plane's cos or cosh of its angle and sw = (sin or sinh)/sqrt(|K| q), the flow
// over L is u <- u C + q p_u sw, p_u <- p_u C - K u sw.  Returns the integral of
// p_u^2 over the element from the plane's invariant E = q p_u^2 + K u^2: since
// d(u p_u)/ds = 2 q p_u^2 - E, it is (E L + u(L) p_u(L) - u(0) p_u(0)) / (2 q);
// half_q = 1 / (2 q).
__device__ __forceinline__ double quad_plane(double &u, double &pu, double K, double q, double L,
                                             double C, double sw, double half_q)
{
    const double u0 = u, p0 = pu;
    u = fma(u0, C, q * p0 * sw);
    pu = fma(p0, C, -(K * u0 * sw));
    const double inv = fma(q * p0, p0, K * u0 * u0);
    return fma(inv, L, fma(u, pu, -(u0 * p0))) * half_q;
}

// Per-particle quantities every thick element of a pass shares: q = 1 - p_sigma,
// sqrt(q) and 1/sqrt(q).
struct Chroma {
    double psg, q, sq, isq;
};

__device__ __forceinline__ Chroma chroma(double psg)
{
    Chroma k;
    k.psg = psg;
    k.q = 1.0 - psg;
    // 1/sqrt(q) from the hardware estimate and two Newton steps (each about
    // doubles the correct bits), then sqrt(q) = q / sqrt(q): within a unit or
    // two of the last place, in a third of the instructions of a correctly
    // rounded square root and division (the thick elements carry no
    // bit-exactness contract; q <= 0 gives NaN either way)
    double y = __builtin_amdgcn_rsq(k.q);
    const double hq = -0.5 * k.q;
    y = y * fma(hq * y, y, 1.5);
    y = y * fma(hq * y, y, 1.5);
    k.isq = y;
    k.sq = k.q * y;
    return k;
}

// Thick quadrupole with chromatic focusing (Sec. III-B).  Both planes turn by
// phi = sqrt(|k1| q) L = phi0 sqrt(q): trigonometric functions in the
// focusing plane, hyperbolic in the other.  The host supplies phi0 and the
// four functions at phi0 (m[3..7]) and 1/sqrt|k1| (m[8]); a particle's
// functions follow from the offset d = phi - phi0 = phi0 (sqrt(q) - 1) by the
// addition formulas, with the series of the functions of d for |d| <= 1/16
// (any momentum spread of a real beam) and beyond that the series of d / 2^h
// doubled h times (the relative error grows about as 2^h units of rounding:
// 2^-46 at |d| = 64).  Then
//   sigma += p_sigma L / gamma0^2 - (1/2) int (px^2 + py^2) ds.
__device__ __forceinline__ void quad_thick(const double *__restrict__ m, double &x, double &px,
                                           double &y, double &py, double &sg, const Chroma &k)
{
    const double k1 = m[0], L = m[1], ig2 = m[2];
    const double q = k.q;
    double ix, iy;
    if (k1 == 0.0) {
        ix = px * px * L;
        iy = py * py * L;
        x = fma(q * px, L, x);
        y = fma(q * py, L, y);
    } else {
        const double phi0 = m[3], d = phi0 * (k.sq - 1.0);
        double s, c, sh, ch;
        if (fabs(d) <= 0.0625) {
            shift_angle<false>(d, m[4], m[5], s, c);
            shift_angle<true>(d, m[6], m[7], sh, ch);
        } else {
            // halve d into the series' range, double the angle back up, then
            // add phi0 (bounded: an infinite d ends in NaN, not a hang)
            int h = 0;
            double dh = d;
            while (h < 40 && fabs(dh) > 0.0625) {
                dh *= 0.5;
                ++h;
            }
            shift_angle<false>(dh, 0.0, 1.0, s, c);
            shift_angle<true>(dh, 0.0, 1.0, sh, ch);
            for (int r = 0; r < h; ++r) {
                const double s2 = 2.0 * s * c, c2 = fma(2.0 * c, c, -1.0);
                const double sh2 = 2.0 * sh * ch, ch2 = fma(2.0 * ch, ch, -1.0);
                s = s2;
                c = c2;
                sh = sh2;
                ch = ch2;
            }
            const double s0 = m[4], c0 = m[5], sh0 = m[6], ch0 = m[7];
            const double ns = fma(s0, c, c0 * s), nc = fma(c0, c, -(s0 * s));
            const double nsh = fma(sh0, ch, ch0 * sh), nch = fma(ch0, ch, sh0 * sh);
            s = ns;
            c = nc;
            sh = nsh;
            ch = nch;
        }
        const double iw = m[8] * k.isq;  // 1 / sqrt(|k1| q)
        const double half_q = 0.5 * k.isq * k.isq;
        if (k1 > 0.0) {
            ix = quad_plane(x, px, k1, q, L, c, s * iw, half_q);
            iy = quad_plane(y, py, -k1, q, L, ch, sh * iw, half_q);
        } else {
            ix = quad_plane(x, px, k1, q, L, ch, sh * iw, half_q);
            iy = quad_plane(y, py, -k1, q, L, c, s * iw, half_q);
        }
    }
    sg = sg + fma(k.psg * ig2, L, -0.5 * (ix + iy));
}

// One element applied to one particle in six dimensions (Sec. III): the
// four-dimensional elements as above (sigma, p_sigma untouched), the thick
// quadrupole with chromatic focusing (Sec. III-B), whose path length is
//   sigma += p_sigma L / gamma0^2 - (1/2) int (px^2 + py^2) ds,
// and the thick sextupole (Sec. III-C) as n symmetric products of the exact
// flows of H0 = (px^2 + py^2)(1 - p_sigma)/2 + p_sigma^2/(2 gamma0^2) and of
// V = k2 (x^3 - 3 x y^2)/6 over the step h = L/n:
//   H0 (a h), V (h/2), H0 (c h), V (h/2), H0 (a h),  c = 1/sqrt 3, a = (1 - c)/2.
// k2 = 0 takes the drift in one step; m[4] and m[5] are drift lengths the
// host folded into the first and last H0 flow, m[6..9] the step lengths it
// derived (the same for every particle).  p_sigma is constant in every
// element.
__device__ __forceinline__ void apply_element6(int kind, const double *__restrict__ m, double &x,
                                               double &px, double &y, double &py, double &sg,
                                               const Chroma &k)
{
    if (kind == SCPIC_EL_QUAD_THICK) {
        quad_thick(m, x, px, y, py, sg, k);
    } else if (kind == SCPIC_EL_SEXT_THICK && m[0] == 0.0) {
        // no sextupole field: the split composes to the exact drift of H0
        // over the whole length m[1] + m[4] + m[5], which the host put in m[6]
        const double L = m[6];
        sg = fma(fma(-0.5 * px, px, fma(-0.5 * py, py, k.psg * m[2])), L, sg);
        x = fma(px * k.q, L, x);
        y = fma(py * k.q, L, y);
    } else if (kind == SCPIC_EL_SEXT_THICK) {
        // the step h = m[1] / n and the split's a h, c h, k2 h / 2, computed
        // by the host in m[6..9]
        const int n = (int)m[3];
        const double dsg = k.psg * m[2];
        const double ta = m[7], tc = m[8], tv = m[9];
        auto drift = [&](double t) {
            x = fma(px * k.q, t, x);
            y = fma(py * k.q, t, y);
            sg = fma(fma(-0.5 * px, px, fma(-0.5 * py, py, dsg)), t, sg);
        };
        auto kick = [&]() {
            const double X = x, Y = y;
            px = fma(-0.5 * tv, fma(X, X, -(Y * Y)), px);
            py = fma(tv * X, Y, py);
        };
        // folded drifts (host side) lengthen the first and the last H0 flow
        const double lead = m[4], tail = m[5];
        for (int i = 0; i < n; ++i) {
            drift(i == 0 ? ta + lead : ta);
            kick();
            drift(tc);
            kick();
            drift(i == n - 1 ? ta + tail : ta);
        }
    } else {
        apply_element(kind, m, x, px, y, py);
    }
}

// Reductions over the 64 lanes of a wave with DPP row operations (no LDS
// traffic): the two quad permutations and the half-row and row mirrors leave
// every lane of a row of 16 holding its row's result; row broadcast 15 folds
// row 0 into row 1 and row 2 into row 3, row broadcast 31 folds row 1 into
// rows 2 and 3, so lane 63 holds the wave's result.  Rows a step does not
// write keep their value (the identity of the step's operation).
template <typename Op>
__device__ __forceinline__ int wave_reduce(int v, int identity, Op op)
{
    v = op(v, __builtin_amdgcn_update_dpp(identity, v, 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
    v = op(v, __builtin_amdgcn_update_dpp(identity, v, 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
    v = op(v, __builtin_amdgcn_update_dpp(identity, v, 0x141, 0xF, 0xF, false));  // row_half_mirror
    v = op(v, __builtin_amdgcn_update_dpp(identity, v, 0x140, 0xF, 0xF, false));  // row_mirror
    v = op(v, __builtin_amdgcn_update_dpp(identity, v, 0x142, 0xA, 0xF, false));  // row_bcast:15
    v = op(v, __builtin_amdgcn_update_dpp(identity, v, 0x143, 0xC, 0xF, false));  // row_bcast:31
    return __builtin_amdgcn_readlane(v, kWave - 1);
}

// Two 16-bit values in one register: cell indices (i in the low half, j in
// the high one) whose minima and maxima take one instruction for both.
using Pair = unsigned short __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pair_min(uint32_t u, uint32_t v)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(Pair, u),
                                                                  __builtin_bit_cast(Pair, v)));
}
__device__ __forceinline__ uint32_t pair_max(uint32_t u, uint32_t v)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(Pair, u),
                                                                  __builtin_bit_cast(Pair, v)));
}
__device__ __forceinline__ uint32_t wave_pair_min(uint32_t v)
{
    return (uint32_t)wave_reduce((int)v, -1, [](int a, int b) { return (int)pair_min(a, b); });
}
__device__ __forceinline__ uint32_t wave_pair_max(uint32_t v)
{
    return (uint32_t)wave_reduce((int)v, 0, [](int a, int b) { return (int)pair_max(a, b); });
}
// t / w for 0 <= t < 2^16 and 1 <= w <= 2^16: the float product with the
// rounded reciprocal is within 0.01 of the quotient, so one integer step
// either way makes it exact.
__device__ __forceinline__ int div_small(int t, int w, float inv_w)
{
    int r = (int)((float)t * inv_w);
    r -= (r * w > t) ? 1 : 0;
    r += ((r + 1) * w <= t) ? 1 : 0;
    return r;
}

// A rectangle of grid nodes held in LDS: rows i0..i0+h-1, columns
// j0..j0+w-1, row-major with row length w.
struct Box {
    int i0, j0, h, w;
    // nodes (i, j) to (i + SPAN, j + SPAN) lie inside, for a cell the four
    // nodes with SPAN 1 (h and w are at least SPAN)
    template <int SPAN = 1>
    __device__ __forceinline__ bool holds_cell(int i, int j) const
    {
        return ((uint32_t)(i - i0) < (uint32_t)(h - SPAN)) &
               ((uint32_t)(j - j0) < (uint32_t)(w - SPAN));
    }
    __device__ __forceinline__ int at(int i, int j) const { return (i - i0) * w + (j - j0); }
};

// Cells of the charge tile around a known box grown by `margin` cells and
// rounded to 4-column chunks, before any shrinking to a budget.
__device__ __forceinline__ int tile_cells(const GridGeom &g, const BlockHeader &h, int margin)
{
    const int i0 = max(0, h.i0 - margin), i1 = min(g.nx - 1, h.i1 + margin);
    const int j0 = max(0, h.j0 - margin) & ~3, j1 = min(g.ny - 1, h.j1 + margin) | 3;
    return (i1 - i0 + 1) * (j1 - j0 + 1);
}

constexpr int kTileMargin = 12;  // cells around the previous box (particles move)

// Charge tile of a workgroup: the bounding box of its previous deposit grown
// by `margin` cells (the particles move between steps), rounded to 4-column
// chunks, clamped to the grid and to the LDS budget; the whole grid when no
// previous box is known and the grid fits; else as much of the grid's centre
// as fits.  Cells outside the tile go to the global carry grid instead.
__device__ __forceinline__ Box charge_tile(const GridGeom &g, const BlockHeader &h, size_t budget,
                                           int margin)
{
    const int cap_cells = (int)min(budget / sizeof(uint32_t), (size_t)INT_MAX);
    Box t;
    const bool known = h.i0 >= 0 && h.i0 <= h.i1 && h.j0 >= 0 && h.j0 <= h.j1 && h.i1 < g.nx &&
                       h.j1 < g.ny;
    if (!known && g.nx * g.ny <= cap_cells) {
        t.i0 = 0;
        t.j0 = 0;
        t.h = g.nx;
        t.w = g.ny;
        return t;
    }
    int i0, i1, j0, j1;
    if (known) {
        i0 = max(0, h.i0 - margin);
        i1 = min(g.nx - 1, h.i1 + margin);
        j0 = max(0, h.j0 - margin);
        j1 = min(g.ny - 1, h.j1 + margin);
    } else {
        i0 = 0;
        i1 = g.nx - 1;
        j0 = 0;
        j1 = g.ny - 1;
    }
    j0 &= ~3;
    j1 |= 3;  // ny is a multiple of 4, so j1 stays inside the grid
    int w = j1 - j0 + 1, hgt = i1 - i0 + 1;
    // shrink symmetrically (rows first, then 4-column chunks) to the budget
    while (hgt * w > cap_cells && hgt > 2) {
        ++i0;
        if (hgt * w > cap_cells && hgt > 3) --i1;
        hgt = i1 - i0 + 1;
    }
    while (hgt * w > cap_cells && w > 8) {
        j0 += 4;
        w -= 4;
        if (hgt * w > cap_cells && w > 8) w -= 4;
    }
    t.i0 = i0;
    t.j0 = j0;
    t.h = hgt;
    t.w = w;
    return t;
}

// What the lanes of a pass hold of one particle between its load and its use.
struct Loaded {
    double x, px, y, py, sg, psg;
    float w;
    uint8_t lost;
};

// Waits for the loads issued so far (not for LDS).  A block that few waves
// enter and that loads registers waits inside, so that the code after it, which
// every wave runs, need not wait for memory on its account.
__device__ __forceinline__ void wait_loads()
{
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt 0, expcnt and lgkmcnt any
}

// The particle, counted from p0, of this lane in a wave's round of 64 from p0
// on (p0 < n): its own, or the last one for a lane past it.
__device__ __forceinline__ uint32_t round_lane(int64_t left)
{
    const uint32_t last = left < kWave ? (uint32_t)left - 1u : kWave - 1u;
    return min((uint32_t)threadIdx.x & (kWave - 1u), last);
}

// The particles of a wave's round of 64 from p0 on, `left` of them: the addresses are the
// arrays' uniform pointers at p0 (scalar registers) plus the lane's byte
// offset.  Every lane loads (round_lane), and the flags and weights are not
// looked at here, which would wait for the loads.  Without a
// lost array the flag loads some byte that the caller ignores, so that the
// number of loads in flight does not depend on a branch; FLAG_BRANCH: it branches
// (the passes in step, which wait for all their loads anyway: without a lost array
// a deposit of 6e6 40.4 -> 39.7 us, with one tracks of 8e6 on 128^2 2.37 -> 2.29 ms
// per 20 steps; a push alone 71.3 -> 73.7).
template <bool SIX, bool NT, bool FLAG_BRANCH = false>
__device__ __forceinline__ Loaded load_particles(const ParticlePtrs &P, int64_t p0, int64_t left,
                                                 bool weights)
{
    const uint32_t lane = round_lane(left);
    const uint8_t *lost = P.lost ? P.lost + p0 : reinterpret_cast<const uint8_t *>(P.x + p0);
    Loaded v;
    v.w = 1.0f;
    if (weights) v.w = (P.w + p0)[lane];
    if constexpr (NT) {
        v.x = __builtin_nontemporal_load(P.x + p0 + lane);
        v.px = __builtin_nontemporal_load(P.px + p0 + lane);
        v.y = __builtin_nontemporal_load(P.y + p0 + lane);
        v.py = __builtin_nontemporal_load(P.py + p0 + lane);
    } else {
        v.x = (P.x + p0)[lane];
        v.px = (P.px + p0)[lane];
        v.y = (P.y + p0)[lane];
        v.py = (P.py + p0)[lane];
    }
    if constexpr (SIX) {
        v.sg = (P.sigma + p0)[lane];
        v.psg = (P.psigma + p0)[lane];
    }
    v.lost = 0;
    if (!FLAG_BRANCH || P.lost) v.lost = lost[lane];
    return v;
}

// Stores lane l's value at p[l], p the round's first particle (uniform): a store
// to a buffer of `bytes` bytes, which an empty buffer (0) drops without a branch.
template <bool NT>
__device__ __forceinline__ void store_lane(double *p, uint32_t lane, double v, int bytes)
{
    using Words = uint32_t __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(
        __builtin_bit_cast(Words, v),
        __builtin_amdgcn_make_buffer_rsrc(p, (short)0, bytes, 0x00020000),
        (int)(lane * sizeof(double)), 0, NT ? 2 : 0);  // 2: non-temporal
}

// Adds a particle's four weights to the workgroup's tile, where l is the tile
// cell of node (i, j) and row the tile's row length.  A 32-bit cell wraps
// after 2^32 units (256 particles on one node); the atomic's old value shows
// the wrap and the lost 2^32 goes to the carry grid (cg: node (i, j) there).
// All four atomics issue before any check.  (Atomics without a returned value,
// the tile's sum against 2^24 per particle at the end and a second deposit
// where it fell short were no faster: 30.1 and 29.7 us per step at 1e6
// particles.)
__device__ __forceinline__ void deposit_cell(uint32_t *lq, int l, int row,
                                             unsigned long long *carry, int cg, int ny,
                                             const Cic &c)
{
    const uint32_t a = (uint32_t)c.a, b = (uint32_t)c.b;
    const uint32_t a0 = kFracOne - a, b0 = kFracOne - b;
    const uint32_t w00 = __umul24(a0, b0), w10 = __umul24(a, b0), w01 = __umul24(a0, b),
                   w11 = __umul24(a, b);
    const uint32_t o00 = atomicAdd(&lq[l], w00);
    const uint32_t o10 = atomicAdd(&lq[l + row], w10);
    const uint32_t o01 = atomicAdd(&lq[l + 1], w01);
    const uint32_t o11 = atomicAdd(&lq[l + row + 1], w11);
    if (o00 + w00 < o00) atomicAdd(&carry[cg], 1ull << 32);
    if (o10 + w10 < o10) atomicAdd(&carry[cg + ny], 1ull << 32);
    if (o01 + w01 < o01) atomicAdd(&carry[cg + 1], 1ull << 32);
    if (o11 + w11 < o11) atomicAdd(&carry[cg + ny + 1], 1ull << 32);
}

// The fused particle pass.  Wave w of workgroup bid of the nblk of a launch
// walks its rounds of 64 particles from bid * blockDim.x + 64 w on in steps of
// T = nblk * blockDim.x: consecutive lanes take consecutive particles, so
// every SoA load and store is coalesced.  The loads of the next round (of the
// one after next in the streamed form) are issued in each round.  Memory
// operations complete in order, so a gather from the L2 issued behind them waits
// for memory: with the whole grid as the tile, where every lane gathers the field
// from the L2, they come after it; in the other forms, where nearly every lane
// gathers from LDS, before.  (Behind them all the same: the gathers of lanes
// outside the staged box, the B-spline nodes of the whole-grid form, the line's
// tables and potential.)  For the compiler to count on that order the cached forms
// that kick or deposit have no common load or store behind a branch: a spare lane
// of a wave's last round repeats the last particle, which is another lane's of the
// same wave (the same instructions load and store it for both), but for its
// deposit, and a frozen particle stores its old coordinates (unless its whole wave
// is frozen: the stores are then dropped).
// For each particle:
//   KICK     gather the node field at the particle with the deposit weights
//            and kick px, py by kappa * w_p * E (w_p = 1 without weights);
//            a particle found outside the domain is marked lost and frozen;
//   push     through els (uniform, read from the kernel arguments);
//   DEPOSIT  add the particle's four weights to the workgroup's LDS tile of
//            the charge grid (nodes outside the tile: global atomics on the
//            carry grid); particles outside the domain are marked lost.
// With WHOLE (whole_tile, the host's rule) the whole grid is the tile and
// gathers read the L2-resident field: the set-up then needs nothing of the
// previous pass's box and no field staging, only the zeroing of the tile.
// Otherwise the tile covers the box the workgroup's
// previous deposit recorded (its header; a workgroup owns the same particles
// at every step of a track), and that box of the field (of the potential under
// the four-dimensional B-spline gather), which holds every node the kick gathers
// from, is staged in LDS beside the tile when it fits.
// At the end each workgroup writes the bounding box of its tile cells to its
// slice of the partials (no global atomics).
//
// What bounds it: the L2 traffic of the gathers (with every lane gathering
// from one line, 1e6 particles on 128^2 took 28.3 us per step instead of 31.7:
// hence the box staged in LDS), about 8 us of set-up, flush and launch, and
// from there the last-level cache (a round of 2.6e5 particles adds 2.3 us, 7.3
// TB/s).  The order of its memory operations, the resident map, the cells by
// one conversion and the box moved by direct loads together: 18.0 -> 15.5 us
// at 1e6 particles (FP64), the 64-beam scan 222 -> 195 us per step.
//
// FIRST: the kind of the pass's first element when the caller knows it to be a
// linear map (0: any elements).  The map's matrix then stays in registers for
// the whole pass; read inside the particle loop, its kind and its parameters were
// two dependent scalar loads per round, which nothing hid (a later element's
// parameters come from LDS, its kind from a scalar load).
//
// The streamed form is bound by memory.  With workgroups of 1024 threads it does
// best in step (STEP): each wave waits for all its loads before it uses the field,
// also one that gathers from LDS alone, branches around the loads of its last
// rounds and keeps no element in registers.  5e6 particles on 128^2, us a pass:
// 71.2 with the wait left to the waves that gather from the L2, 65.5 in step
// (FP64), 72.3 and 64.3 (mixed); 8e6, one 2x2 map a segment, 107 with the map in
// registers, 101 without.  Whole tracks of 20 steps: 5e6 on 128^2 1740 -> 1600 us
// FP64, 1760 -> 1560 mixed; 8e6 2465 -> 2290; 1e7 on 256^2 5.73 -> 5.46 ms; the
// 64-beam scan, two turns, 6.21 -> 5.85 ms FP64, 5.67 -> 5.44 mixed; the KV beam of
// 1e7 on 256^2, mixed, 2.93 -> 2.83-2.94.  With fewer threads, which have to hide
// the latency themselves, it is the ordered form: 5e6 with 512 threads 2.00 ms in
// step, 1.53 ordered, with 256 2.98 and 1.99.
//
// MODE is a set of flags (0: four-dimensional).  1: the particles carry sigma
// and p_sigma and els may hold thick elements; sigma is loaded and stored with
// the transverse coordinates.  2: six-dimensional, with the long-bunch line
// density (Sec. IV): the kick is scaled by lambda/lambda_peak at the particle's sigma
// and p_sigma takes the longitudinal kick -gamma0 kappa phi lambda'/lambda_peak
// (both tables and the node potential phi from the last solve, interpolated
// with the particle's line and transverse weights); the deposit adds the
// particle's two line weights (the one-dimensional form of the charge
// assignment) to an LDS histogram flushed to the workgroup's row of
// line.partial.  A particle outside the line is lost like one outside the grid.
// 4: the kick's field is the analytic gradient of the bicubic B-spline surface
// of the node potential (Sec. IV-C), ef then pointing at the potential on
// nodes -1..nx by -1..ny.
// 8: the four transverse coordinates are streamed with non-temporal loads and
// stores (particle arrays far larger than the last-level cache, which they
// would only churn; smaller ones stay cached between passes).  16: WHOLE.
// 32: STEP.
// The body is shared by the single-beam kernel and the batched one: bid is
// the workgroup's index among the nblk workgroups working on beam P (its
// slice of the partials and its header).
template <typename TE, bool KICK, bool DEPOSIT, int MODE, int FIRST>
__device__ __forceinline__ void pass_body(const ParticlePtrs &P, const GridGeom &g,
                                          const TE *__restrict__ ef, double kappa,
                                          const PassElements &els, const DepositTarget &dep,
                                          unsigned lds_bytes, int bid, int nblk,
                                          const LineSpec &line)
{
    using V = typename Vec2<TE>::type;
    constexpr bool LINE = (MODE & 2) != 0;
    constexpr bool SIX = (MODE & 1) != 0 || LINE;
    constexpr bool BSPL = (MODE & 4) != 0;
    constexpr bool NT = (MODE & 8) != 0;
    constexpr bool WHOLE = (MODE & 16) != 0;
    constexpr bool STEP = (MODE & 32) != 0;
    static_assert(!WHOLE || DEPOSIT, "the tile is the depositing passes'");
    static_assert(!NT || !SIX, "the streamed pass is four-dimensional");
    static_assert(!STEP || (NT && (KICK || DEPOSIT)), "in step: streamed passes that use LDS");
    static_assert(!FIRST || (!SIX && !STEP), "a resident first element is four-dimensional");
    extern __shared__ __align__(16) unsigned char lds_all[];
    // A pass that uses LDS reads its elements' parameters from there (one
    // broadcast read per value) but for a resident first element: read into
    // scalar registers, they would displace the loop's other uniform values.
    constexpr bool EL_LDS = SIX || KICK || DEPOSIT;
    // LDS: [element parameters (four-dimensional passes)][line histogram
    // (MODE 2)][charge tile][staged field box].  The histogram counts in 32
    // bits: a workgroup adds 4096 per particle and the host launches no
    // workgroup with more than 2^20 particles.
    const unsigned el_bytes =
        EL_LDS && !SIX && els.n_el > (FIRST ? 1 : 0) ? (unsigned)els.n_el * 128u : 0u;
    const unsigned line_bytes = LINE ? ((unsigned)line.nz * 4u + 15u) & ~15u : 0u;
    uint32_t *lh = reinterpret_cast<uint32_t *>(lds_all);
    unsigned char *const lds = lds_all + el_bytes + line_bytes;
    lds_bytes -= el_bytes + line_bytes;
    __shared__ int s_box[4];
    __shared__ int s_count;
    __shared__ double s_el6[SIX ? kMaxPassElements * 16 : 1];
    static_assert(sizeof(s_el6) + 256 <= kPassStaticLds, "static LDS beyond the reserved share");
    double *const s_el = SIX ? s_el6 : reinterpret_cast<double *>(lds_all);
    const GridCells gc = GridCells::of(g);
    const int n_el = els.n_el;
    const int64_t T = (int64_t)nblk * blockDim.x;
    int64_t p0 = (int64_t)bid * blockDim.x +
                 kWave * __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const bool weights = KICK && !LINE && P.w;

    // first round's loads go out before the LDS set-up
    Loaded cur;
    if (p0 < P.n) cur = load_particles<SIX, false>(P, p0, P.n - p0, weights);

    BlockHeader hd;
    hd.i0 = -1;
    hd.i1 = -2;
    hd.j0 = -1;
    hd.j1 = -2;
    if ((KICK || DEPOSIT) && !WHOLE) hd = dep.header[bid];
    // The kick stages the field over the previous box (every node it gathers
    // from) when that box fits in LDS beside the charge tile: (Ex, Ey) of the
    // box's nodes, or the potential on them and one node around (box indices
    // count from node -1 then).  The staging moves units of 16 bytes (4 for the
    // float potential, whose rows are not aligned to more), kUnitNodes nodes
    // each: the box's columns are rounded out to whole units (a row of nodes,
    // ny or ny + 2 of them, holds whole units), and 64 units of slack follow.
    using S = std::conditional_t<BSPL, TE, V>;
    constexpr int kUnitBytes = sizeof(S) == 4 ? 4 : 16;
    constexpr int kUnitNodes = kUnitBytes / (int)sizeof(S);
    constexpr int kSpan = BSPL ? 3 : 1;  // nodes a cell needs beyond its first, per axis
    const bool known = hd.i0 >= 0 && hd.i0 <= hd.i1 && hd.j0 >= 0 && hd.j0 <= hd.j1 &&
                       hd.i1 < g.nx && hd.j1 < g.ny;
    Box fbox{0, 0, kSpan, kSpan};
    if (known) {
        const int around = BSPL ? 2 : 0;
        const int j0 = hd.j0 & ~(kUnitNodes - 1), j1 = (hd.j1 + around) | (kUnitNodes - 1);
        fbox = Box{hd.i0, j0, hd.i1 + around - hd.i0 + 1, j1 - j0 + 1};
    }
    constexpr size_t kSlack = 64 * kUnitBytes;
    // Not in the six-dimensional pass under the B-spline gather, which is bound by
    // instruction issue and short of registers: staged or not, 1e6 particles on
    // 100^2 take 905 us per 20 steps (FP64), and where only the box's centre fits
    // the two ways to gather cost more than they save (256^2, 1e6: 1261 us staged,
    // 1172 not; mixed 1187 and 1084; 2.5e6, FP64, 2175 and 1980).
    constexpr bool STAGE = KICK && !WHOLE && !(SIX && BSPL);
    const size_t field_bytes =
        (STAGE && known) ? (size_t)fbox.h * fbox.w * sizeof(S) + kSlack : 0;
    // LDS layout: [charge tile][staged field box and slack]
    Box tile{0, 0, 1, 1};
    size_t tile_bytes = 0;
    if constexpr (DEPOSIT) {
        // the widest margin (12, 8, 4 or 0 cells) that leaves room for the
        // field box; 12 when none does
        int margin = kTileMargin;
        if (field_bytes) {
            int m = kTileMargin;
            while (m >= 0 &&
                   sizeof(uint32_t) * (size_t)tile_cells(g, hd, m) + field_bytes > lds_bytes)
                m -= 4;
            if (m >= 0) margin = m;
        }
        tile = WHOLE ? Box{0, 0, g.nx, g.ny} : charge_tile(g, hd, lds_bytes, margin);
        tile_bytes = sizeof(uint32_t) * (size_t)tile.h * tile.w;
    }
    uint32_t *lq = reinterpret_cast<uint32_t *>(lds);
    S *le = reinterpret_cast<S *>(lds + tile_bytes);
    Box ebox{0, 0, kSpan, kSpan};
    bool staged = false;
    if constexpr (KICK) {
        staged = field_bytes && field_bytes + tile_bytes <= (size_t)lds_bytes;
        if (staged) ebox = fbox;
        if (field_bytes && !staged && tile_bytes + kSlack < (size_t)lds_bytes) {
            // The whole box does not fit beside the tile: stage its centre, as
            // much as fits (the box's edges hold only the tails of the
            // distribution; a particle outside the staged part gathers from
            // L2).  From half of the nodes on; the streamed form, whose L2 and
            // loads in order are the busier, from an eighth on.  Whole tracks
            // with and without the centre, Gaussian beams in FP64: 8.8e6
            // particles on 128^2 (streamed) 7.67 and 10.65 ms, 5e6 on 256^2
            // (streamed) 6.64 and 6.67, 1.5e6 on 256^2 2.35 and 2.21.
            const int64_t room = (int64_t)(((size_t)lds_bytes - tile_bytes - kSlack) / sizeof(S));
            if ((NT ? 8 : 2) * room >= (int64_t)fbox.h * fbox.w) {
                int i0 = fbox.i0, i1 = fbox.i0 + fbox.h - 1, j0 = fbox.j0, j1 = fbox.j0 + fbox.w - 1;
                while ((int64_t)(i1 - i0 + 1) * (j1 - j0 + 1) > room) {
                    // trim the longer side, one node (one unit) at each end
                    if (i1 - i0 >= j1 - j0) {
                        ++i0;
                        --i1;
                    } else {
                        j0 += kUnitNodes;
                        j1 -= kUnitNodes;
                    }
                }
                staged = i1 - i0 >= kSpan && j1 - j0 >= kSpan;
                if (staged) ebox = Box{i0, j0, i1 - i0 + 1, j1 - j0 + 1};
            }
        }
        if (staged) {
            // A wave moves 64 units at a time straight to consecutive LDS (lane
            // l to slot l; lanes past the box repeat its last unit into the
            // slack): every load is in flight at once and none passes through
            // a register.
            const S *ev = reinterpret_cast<const S *>(ef);
            const int row = BSPL ? g.ny + 2 : g.ny;
            const int wu = ebox.w / kUnitNodes, units = ebox.h * wu;
            const float inv_w = 1.0f / (float)wu;
            const int lane = (int)threadIdx.x & (kWave - 1);
            for (int t0 = kWave * __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
                 t0 < units; t0 += (int)blockDim.x) {
                const int t = min(t0 + lane, units - 1);
                const int r = div_small(t, wu, inv_w);
                const S *src = ev + (ebox.i0 + r) * row + ebox.j0 + (t - r * wu) * kUnitNodes;
                auto *from = (const __attribute__((address_space(1))) void *)(uintptr_t)src;
                auto *to = (__attribute__((address_space(3))) void *)(le + t0 * kUnitNodes);
                if constexpr (kUnitBytes == 16)
                    __builtin_amdgcn_global_load_lds(from, to, 16, 0, 0);
                else
                    __builtin_amdgcn_global_load_lds(from, to, 4, 0, 0);
            }
        }
    }
    if constexpr (DEPOSIT) {
        const int n4 = tile.h * tile.w / 4;  // tile.w is a multiple of 4
        uint4 *q4 = reinterpret_cast<uint4 *>(lq);
        for (int t = threadIdx.x; t < n4; t += blockDim.x) q4[t] = make_uint4(0, 0, 0, 0);
        if constexpr (LINE)
            for (int t = threadIdx.x; t < line.nz; t += blockDim.x) lh[t] = 0u;
        if (threadIdx.x == 0) {
            s_box[0] = INT_MAX;
            s_box[1] = -1;
            s_box[2] = INT_MAX;
            s_box[3] = -1;
            s_count = 0;
        }
    }
    if (SIX || el_bytes)
        for (int t = threadIdx.x; t < n_el * 16; t += blockDim.x)
            s_el[t] = els.p[t >> 4][t & 15];
    // the resident first element, in vector registers (40 production steps, twice:
    // 2.25 ms, in scalar registers 2.27, mixed 2.11 and 2.15) but under the B-spline
    // gather, which needs them for its nodes (25 steps twice, 1.76 and 1.58 ms,
    // mixed 1.44 and 1.48), and for a streamed 4x4 map, where they do not suffice
    // (40 bytes of scratch per lane, 5e6 particles on 128^2 87 us a pass and 71)
    double m0[16] = {};
    if constexpr (FIRST == SCPIC_EL_LIN2X2 || FIRST == SCPIC_EL_LIN4X4)
#pragma unroll
        for (int k = 0; k < (FIRST == SCPIC_EL_LIN4X4 ? 16 : 8); ++k)
            m0[k] = BSPL || (NT && FIRST == SCPIC_EL_LIN4X4) ? els.p[0][k] : in_vector(els.p[0][k]);
    wait_loads();  // the first round and the staged field
    if (KICK || DEPOSIT || SIX) __syncthreads();

    const bool moves = KICK || n_el > 0;
    // the kick's weights and the charge of a node are in units of 2^-24
    constexpr double kUnit = 1.0 / kChargeOne;
    uint32_t lo = 0xffffffffu, hi = 0;  // lowest and highest cell touched, i | j << 16
    int cnt = 0;                        // particles deposited by the wave
    // The streamed form keeps two rounds in flight ahead of the one worked on
    // (its loads come from memory, not the last-level cache).
    Loaded ahead;
    if (NT && p0 < P.n)
        ahead = load_particles<SIX, true, STEP>(
            P, p0 + T < P.n ? p0 + T : p0, p0 + T < P.n ? P.n - p0 - T : 1, weights);
    const bool has_lost = P.lost != nullptr;
    for (; p0 < P.n; p0 += T) {
        const uint32_t lane = round_lane(P.n - p0);
        bool act = (cur.lost == 0) | !has_lost;
        // the last rounds have nothing to load: every lane loads one particle
        const bool more = p0 + (NT ? 2 : 1) * T < P.n;
        const int64_t pn = more ? p0 + (NT ? 2 : 1) * T : p0, left = more ? P.n - pn : 1;
        Loaded next;
        // a push alone has one or two rounds and branches around the last one's
        // (1e6 particles 10.0 -> 9.2 us), and so does the form in step (a
        // deposit of 8e6 106 -> 96 us)
        if constexpr (!WHOLE)
            if ((!STEP && (KICK || DEPOSIT)) || more)
                next = load_particles<SIX, NT, STEP>(P, pn, left, weights);
        // the gathers
        Cic ck;
        LineCic lck;
        bool in = false;
        CellField<V> ev;
        SplineNodes<TE> us;
        if constexpr (KICK) {
            in = act && cic(gc, cur.x, cur.y, ck) && (!LINE || line_cic(line, cur.sg, lck));
            if constexpr (BSPL) {
                if constexpr (!WHOLE) {
                    const bool near =
                        STAGE && in && staged && ebox.template holds_cell<kSpan>(ck.i, ck.j);
                    if (near) us.load(le + ebox.at(ck.i, ck.j), ebox.w);
                    if (in && !near) us.load(ef + ck.i * (g.ny + 2) + ck.j, g.ny + 2);
                }
            } else {
                const V *ge = reinterpret_cast<const V *>(ef);
                const uint32_t row = (uint32_t)sizeof(V) * (uint32_t)g.ny;
                if constexpr (WHOLE) {
                    if (in) ev.load(ge, (uint32_t)sizeof(V) * (uint32_t)(ck.i * g.ny + ck.j), row);
                } else {
                    const bool near = in && staged && ebox.template holds_cell<kSpan>(ck.i, ck.j);
                    if (near)
                        ev.load(le, (uint32_t)sizeof(V) * (uint32_t)ebox.at(ck.i, ck.j),
                                (uint32_t)sizeof(V) * (uint32_t)ebox.w);
                    if (in && !near) {
                        ev.load(ge, (uint32_t)sizeof(V) * (uint32_t)(ck.i * g.ny + ck.j), row);
                        if constexpr (!STEP) wait_loads();
                    }
                }
            }
        }
        if constexpr (WHOLE) next = load_particles<SIX, NT>(P, pn, left, weights);
        double x = cur.x, px = cur.px, y = cur.y, py = cur.py, sg = cur.sg, psg = cur.psg;
        if constexpr (KICK) {
            if (in) {
                TE fx, fy;
                if constexpr (BSPL) {
                    if constexpr (WHOLE) us.load(ef + ck.i * (g.ny + 2) + ck.j, g.ny + 2);
                    bspline_field(g, us, x, y, ck, fx, fy);
                } else {
                    const Weights<TE> w(ck);
                    fx = w.sum(ev.e00.x, ev.e10.x, ev.e01.x, ev.e11.x);
                    fy = w.sum(ev.e00.y, ev.e10.y, ev.e01.y, ev.e11.y);
                }
                if constexpr (LINE) {
                    const double w1 = (double)lck.a, w0 = 4096.0 - w1;
                    const double wl = (w0 * line.lw[lck.k] + w1 * line.lw[lck.k + 1]) / 4096.0;
                    const double dl = (w0 * line.ld[lck.k] + w1 * line.ld[lck.k + 1]) / 4096.0;
                    const TE fp = gather_scalar(reinterpret_cast<const TE *>(line.phi),
                                                (ck.i + 1) * (g.ny + 2) + ck.j + 1, g.ny + 2, ck);
                    const double k = kappa * wl * kUnit;
                    px = px + k * (double)fx;
                    py = py + k * (double)fy;
                    psg = psg - line.gamma0 * kappa * ((double)fp * kUnit) * dl;
                } else {
                    // (kappa 2^-24) w E: the power of two may go anywhere
                    const double k0 = BSPL ? kappa : kappa * kUnit;
                    const double k = weights ? k0 * (double)cur.w : k0;
                    px = px + k * (double)fx;
                    py = py + k * (double)fy;
                }
            } else if (act && has_lost) {
                (P.lost + p0)[lane] = 1;
                act = false;
            }
        }
        bool hit = false;
        if (act) {
            if constexpr (SIX) {
                const Chroma ck = chroma(psg);
                for (int e = 0; e < n_el; ++e)
                    apply_element6(els.kind[e], s_el + 16 * e, x, px, y, py, sg, ck);
            } else if constexpr (FIRST != 0) {
                apply_element(FIRST, m0, x, px, y, py);
                for (int e = 1; e < n_el; ++e)
                    apply_element(els.kind[e], s_el + 16 * e, x, px, y, py);
            } else {
                for (int e = 0; e < n_el; ++e)
                    apply_element(els.kind[e], EL_LDS ? s_el + 16 * e : els.p[e], x, px, y, py);
            }
            if constexpr (DEPOSIT) {
                Cic c;
                LineCic lc;
                const bool inside = cic(gc, x, y, c) && (!LINE || line_cic(line, sg, lc));
                hit = inside & ((threadIdx.x & (kWave - 1)) == lane);
                if (hit) {
                    if constexpr (LINE) {
                        atomicAdd(&lh[lc.k], (uint32_t)(kFracOne - lc.a));
                        atomicAdd(&lh[lc.k + 1], (uint32_t)lc.a);
                    }
                    if (WHOLE || tile.holds_cell(c.i, c.j)) {
                        deposit_cell(lq, tile.at(c.i, c.j), tile.w, dep.carry,
                                     c.i * g.ny + c.j, g.ny, c);
                        const uint32_t cell = (uint32_t)c.i | (uint32_t)c.j << 16;
                        lo = pair_min(lo, cell);
                        hi = pair_max(hi, cell);
                    } else {
                        const uint32_t a = (uint32_t)c.a, b = (uint32_t)c.b;
                        const uint32_t a0 = kFracOne - a, b0 = kFracOne - b;
                        unsigned long long *cg = dep.carry + (c.i * g.ny + c.j);
                        atomicAdd(cg, (unsigned long long)(a0 * b0));
                        atomicAdd(cg + g.ny, (unsigned long long)(a * b0));
                        atomicAdd(cg + 1, (unsigned long long)(a0 * b));
                        atomicAdd(cg + g.ny + 1, (unsigned long long)(a * b));
                    }
                } else if (has_lost & !inside) {
                    (P.lost + p0)[lane] = 1;
                }
            }
        }
        // A wave of frozen particles only stores nothing.  One with a moving particle
        // stores all of its lanes' (whole lines; a frozen particle its old values):
        // 8e6 particles on 128^2, one in two frozen at random, take 2.5 ms per 20
        // steps, lane by lane they took 3.4.  The buffer's size makes the choice,
        // not a branch, in front of which every wave would wait for its loads in
        // flight (40 production steps, twice, mixed: 2.10 and 2.21 ms); a push
        // alone, of few rounds, branches.  With all particles frozen, per 20
        // steps: 1e6 on 128^2 0.45 -> 0.39 ms, 8e6 2.15 -> 1.15; a push of 8e6
        // 97 -> 39 us.
        const bool any = __any(act);
        if (moves && (KICK || DEPOSIT || any)) {
            // the kick changes only the momenta; the elements move the
            // particle (a kick-only pass writes px and py alone)
            const bool shifts = FIRST != 0 || n_el > 0;
            const int bytes = any ? (int)(kWave * sizeof(double)) : 0;
            if (shifts) {
                store_lane<NT>(P.x + p0, lane, x, bytes);
                store_lane<NT>(P.y + p0, lane, y, bytes);
            }
            store_lane<NT>(P.px + p0, lane, px, bytes);
            store_lane<NT>(P.py + p0, lane, py, bytes);
            if constexpr (SIX)
                if (shifts) store_lane<false>(P.sigma + p0, lane, sg, bytes);
            if constexpr (LINE && KICK) store_lane<false>(P.psigma + p0, lane, psg, bytes);
        }
        if constexpr (DEPOSIT) {
            cnt += __popcll(__ballot(hit));
        }
        if constexpr (NT) {
            cur = ahead;
            ahead = next;
        } else {
            cur = next;
        }
    }

    if constexpr (DEPOSIT) {
        // combine the waves' boxes and counts, then copy the box of tile cells
        // to this workgroup's slice of the partials in 16-byte chunks (the
        // extra cells of the end chunks are zero and masked by the reader)
        lo = wave_pair_min(lo);
        hi = wave_pair_max(hi);
        if ((threadIdx.x & (kWave - 1)) == 0 && cnt) {
            if (lo <= hi) {  // some cell of the tile (else lo is still all ones)
                atomicMin(&s_box[0], (int)(lo & 0xffffu));
                atomicMax(&s_box[1], (int)(hi & 0xffffu) + 1);
                atomicMin(&s_box[2], (int)(lo >> 16));
                atomicMax(&s_box[3], (int)(hi >> 16) + 1);
            }
            atomicAdd(&s_count, cnt);
        }
        __syncthreads();
        if constexpr (LINE)
            for (int t = threadIdx.x; t < line.nz; t += blockDim.x)
                line.partial[(size_t)bid * line.nz + t] = (unsigned long long)lh[t];
        const int i0 = s_box[0], i1 = s_box[1], j0 = s_box[2], j1 = s_box[3];
        if (i0 <= i1) {
            const int c0 = j0 >> 2, nch = (j1 >> 2) - c0 + 1;
            const int total = (i1 - i0 + 1) * nch;
            const float inv_nch = 1.0f / (float)nch;
            for (int t = threadIdx.x; t < total; t += blockDim.x) {
                const int r = div_small(t, nch, inv_nch);
                const int i = i0 + r, cc = c0 + (t - r * nch);
                const uint4 v = *reinterpret_cast<const uint4 *>(lq + tile.at(i, 4 * cc));
                reinterpret_cast<uint4 *>(dep.partial +
                                          ((size_t)i * dep.max_blocks + bid) * g.ny)[cc] = v;
            }
        }
        if (threadIdx.x == 0) {
            BlockHeader h;
            h.i0 = i0;
            h.i1 = i1;
            h.j0 = j0;
            h.j1 = j1;
            h.count = s_count;
            h.pad = 0;
            h.rows = i0 <= i1 ? (uint32_t)i0 | (uint32_t)i1 << 16 : 0xffffu;
            h.cols = i0 <= i1 ? (uint32_t)j0 | (uint32_t)j1 << 16 : 0xffffu;
            dep.header[bid] = h;
        }
    }
}

// FORM: 0, 8 (streamed, four-dimensional passes only), 40 (streamed and in step)
// or 16 (the whole grid as the tile, depositing passes only).  FIRST: the pass's
// first element, when it is a linear map (four-dimensional passes only, not in
// step).
template <typename TE, bool KICK, bool DEPOSIT, bool SIX, int FORM = 0, int FIRST = 0>
__global__ void __launch_bounds__(1024)
    k_pass(ParticlePtrs P, GridGeom g, const TE *__restrict__ ef, double kappa,
           PassElements els, DepositTarget dep, unsigned lds_bytes)
{
    pass_body<TE, KICK, DEPOSIT, (SIX ? 1 : 0) | FORM, FIRST>(
        P, g, ef, kappa, els, dep, lds_bytes, (int)blockIdx.x, (int)gridDim.x, LineSpec{});
}

// The pass with the B-spline field (phi: the node potential on nodes -1..nx
// by -1..ny).
template <typename TE, bool KICK, bool DEPOSIT, bool SIX, int FORM = 0, int FIRST = 0>
__global__ void __launch_bounds__(1024)
    k_pass_bspline(ParticlePtrs P, GridGeom g, const TE *__restrict__ phi, double kappa,
                   PassElements els, DepositTarget dep, unsigned lds_bytes)
{
    pass_body<TE, KICK, DEPOSIT, 4 | (SIX ? 1 : 0) | FORM, FIRST>(
        P, g, phi, kappa, els, dep, lds_bytes, (int)blockIdx.x, (int)gridDim.x, LineSpec{});
}

// The pass of a long bunch with its line density (six-dimensional).
template <typename TE, bool KICK, bool DEPOSIT, int FORM = 0>
__global__ void __launch_bounds__(1024)
    k_pass_line(ParticlePtrs P, GridGeom g, const TE *__restrict__ ef, double kappa,
                PassElements els, DepositTarget dep, unsigned lds_bytes, LineSpec line)
{
    pass_body<TE, KICK, DEPOSIT, 2 | FORM, 0>(P, g, ef, kappa, els, dep, lds_bytes, (int)blockIdx.x,
                                       (int)gridDim.x, line);
}

// A pointer read from a table in memory, known to point to global memory (the
// compiler otherwise takes it for one that might point to LDS, whose accesses
// both memory counters must wait for).
template <typename T>
__device__ __forceinline__ T *global_memory(T *p)
{
    return (T *)(__attribute__((address_space(1))) T *)(uintptr_t)p;
}

// One pass over every beam of a batch: workgroup -> beam from the batch's
// table, then the same body on that beam's particles, grid, field and
// partials with its own kick strength and elements (steps[beam]).
template <typename TE, bool KICK, bool DEPOSIT, bool SIX, int FORM = 0, int FIRST = 0>
__global__ void __launch_bounds__(1024)
    k_pass_batched(BatchLaunch b, ParticlePtrs all, const BatchStep *__restrict__ steps,
                   unsigned lds_bytes)
{
    const int k = b.pass_inst[blockIdx.x];
    // copies: a reference into the table would be read again after every store
    const BatchInstance I = b.inst[k];
    const double kappa = steps[k].kappa;
    DepositTarget dep;
    dep.partial = global_memory(I.dep.partial);
    dep.header = global_memory(I.dep.header);
    dep.carry = global_memory(I.dep.carry);
    dep.max_blocks = I.dep.max_blocks;
    ParticlePtrs P;
    P.x = all.x + I.p0;
    P.px = all.px + I.p0;
    P.y = all.y + I.p0;
    P.py = all.py + I.p0;
    P.sigma = all.sigma ? all.sigma + I.p0 : nullptr;
    P.psigma = all.psigma ? all.psigma + I.p0 : nullptr;
    P.w = all.w ? all.w + I.p0 : nullptr;
    P.lost = all.lost ? all.lost + I.p0 : nullptr;
    P.n = I.n;
    P.stream = (FORM & 8) != 0;
    pass_body<TE, KICK, DEPOSIT, (SIX ? 1 : 0) | FORM, FIRST>(
        P, I.g, global_memory((const TE *)I.ef), kappa, steps[k].els, dep, lds_bytes,
        (int)blockIdx.x - I.pass_block0, I.pass_blocks, LineSpec{});
}

// Between two node arrays (ex, ey) and the internal interleaved layout ef
// (Ex, Ey per node), in either direction.
template <typename TE, bool TO_INTERLEAVED>
__global__ void __launch_bounds__(256)
    k_interleave(TE *__restrict__ ex, TE *__restrict__ ey, TE *__restrict__ ef, int ncell)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < ncell) {
        if (TO_INTERLEAVED) {
            ef[2 * c] = ex[c];
            ef[2 * c + 1] = ey[c];
        } else {
            ex[c] = ef[2 * c];
            ey[c] = ef[2 * c + 1];
        }
    }
}

// Dynamic LDS budgets of the four- and six-dimensional passes (the latter
// keep their element parameters in static LDS); set by prepare_pass_kernels.
size_t g_lds_limit = 0, g_lds_limit6 = 0;
template <bool SIX>
size_t lds_budget()
{
    return SIX ? g_lds_limit6 : g_lds_limit;
}

template <typename TE, bool KICK, bool DEPOSIT, bool SIX, int FORM = 0, int FIRST = 0>
hipError_t launch_pass_t(hipStream_t s, const ParticlePtrs &p, const GridGeom &g, const void *ef,
                         double kappa, const PassElements &els, const DepositTarget &dep,
                         int blocks, int threads)
{
    const size_t lds = (KICK || DEPOSIT) ? lds_budget<SIX>() : 0;
    hipLaunchKernelGGL((k_pass<TE, KICK, DEPOSIT, SIX, FORM, FIRST>), dim3(blocks), dim3(threads),
                       lds, s, p, g, (const TE *)ef, kappa, els, dep, (unsigned)lds);
    return hipGetLastError();
}

template <typename TE, bool KICK, bool DEPOSIT, bool SIX, int FORM = 0, int FIRST = 0>
hipError_t launch_pass_bspline_t(hipStream_t s, const ParticlePtrs &p, const GridGeom &g,
                                 const void *phi, double kappa, const PassElements &els,
                                 const DepositTarget &dep, int blocks, int threads)
{
    const size_t lds = lds_budget<SIX>();
    hipLaunchKernelGGL((k_pass_bspline<TE, KICK, DEPOSIT, SIX, FORM, FIRST>), dim3(blocks),
                       dim3(threads), lds, s, p, g, (const TE *)phi, kappa, els, dep,
                       (unsigned)lds);
    return hipGetLastError();
}

template <typename TE, bool KICK, bool DEPOSIT, int FORM = 0>
hipError_t launch_pass_line_t(hipStream_t s, const ParticlePtrs &p, const GridGeom &g,
                              const void *ef, double kappa, const PassElements &els,
                              const DepositTarget &dep, int blocks, int threads,
                              const LineSpec &line)
{
    hipLaunchKernelGGL((k_pass_line<TE, KICK, DEPOSIT, FORM>), dim3(blocks), dim3(threads),
                       g_lds_limit6, s, p, g, (const TE *)ef, kappa, els, dep,
                       (unsigned)g_lds_limit6, line);
    return hipGetLastError();
}

template <typename TE, bool KICK, bool DEPOSIT, bool SIX, int FORM = 0, int FIRST = 0>
hipError_t launch_pass_batched_t(hipStream_t s, const BatchLaunch &b, const ParticlePtrs &all,
                                 const BatchStep *steps, int blocks, int threads)
{
    const size_t lds = (KICK || DEPOSIT) ? lds_budget<SIX>() : 0;
    hipLaunchKernelGGL((k_pass_batched<TE, KICK, DEPOSIT, SIX, FORM, FIRST>), dim3(blocks),
                       dim3(threads), lds, s, b, all, steps, (unsigned)lds);
    return hipGetLastError();
}

// Calls f with the integral constants of a pass's form and, for the passes of
// a steady turn, of its resident first element (none in step).
template <typename F>
hipError_t with_form(bool whole, bool stream, int threads, F &&f)
{
    if (whole) return f(std::integral_constant<int, 16>{});
    if (stream && threads >= 1024) return f(std::integral_constant<int, 40>{});
    if (stream) return f(std::integral_constant<int, 8>{});
    return f(std::integral_constant<int, 0>{});
}
template <int FORM, typename F>
hipError_t with_first(int first, F &&f)
{
    if constexpr (FORM != 40) {
        if (first == SCPIC_EL_LIN2X2) return f(std::integral_constant<int, SCPIC_EL_LIN2X2>{});
        if (first == SCPIC_EL_LIN4X4) return f(std::integral_constant<int, SCPIC_EL_LIN4X4>{});
    }
    return f(std::integral_constant<int, 0>{});
}

// The kernels of one form that use LDS.
template <typename TE, int FORM, int FIRST>
void steady_kernels_of(std::vector<const void *> &out)
{
    if constexpr (FORM != 40 || FIRST == 0) {
        out.push_back((const void *)k_pass<TE, true, true, false, FORM, FIRST>);
        out.push_back((const void *)k_pass_batched<TE, true, true, false, FORM, FIRST>);
    }
    if constexpr (!(FORM & 8))
        out.push_back((const void *)k_pass_bspline<TE, true, true, false, FORM, FIRST>);
}
template <typename TE, int FORM>
void form_kernels_of(std::vector<const void *> &four, std::vector<const void *> &six)
{
    steady_kernels_of<TE, FORM, 0>(four);
    steady_kernels_of<TE, FORM, SCPIC_EL_LIN2X2>(four);
    steady_kernels_of<TE, FORM, SCPIC_EL_LIN4X4>(four);
    four.push_back((const void *)k_pass<TE, false, true, false, FORM>);
    four.push_back((const void *)k_pass_batched<TE, false, true, false, FORM>);
    if constexpr (FORM != 16) {
        four.push_back((const void *)k_pass<TE, true, false, false, FORM>);
        four.push_back((const void *)k_pass_batched<TE, true, false, false, FORM>);
    }
    if constexpr (!(FORM & 8)) {
        six.push_back((const void *)k_pass<TE, true, true, true, FORM>);
        six.push_back((const void *)k_pass<TE, false, true, true, FORM>);
        six.push_back((const void *)k_pass_batched<TE, true, true, true, FORM>);
        six.push_back((const void *)k_pass_batched<TE, false, true, true, FORM>);
        six.push_back((const void *)k_pass_bspline<TE, true, true, true, FORM>);
        six.push_back((const void *)k_pass_line<TE, true, true, FORM>);
        six.push_back((const void *)k_pass_line<TE, false, true, FORM>);
    }
    if constexpr (FORM == 0) {
        four.push_back((const void *)k_pass_bspline<TE, true, false, false>);
        six.push_back((const void *)k_pass<TE, true, false, true>);
        six.push_back((const void *)k_pass_batched<TE, true, false, true>);
        six.push_back((const void *)k_pass_bspline<TE, true, false, true>);
        six.push_back((const void *)k_pass_line<TE, true, false>);
    }
}

}  // namespace

bool has_thick(const PassElements &els)
{
    for (int e = 0; e < els.n_el; ++e)
        if (els.kind[e] == SCPIC_EL_QUAD_THICK || els.kind[e] == SCPIC_EL_SEXT_THICK) return true;
    return false;
}

int first_linear(const PassElements &els)
{
    if (els.n_el < 1) return 0;
    return els.kind[0] == SCPIC_EL_LIN2X2 || els.kind[0] == SCPIC_EL_LIN4X4 ? els.kind[0] : 0;
}

// Allow the passes the dynamic LDS they use (beyond the default limit): the
// device's per-workgroup LDS (lds_per_workgroup) minus the kernels' static
// LDS, at most 256 bytes for the four-dimensional passes and kPassStaticLds
// for the six-dimensional ones.  Called once per context, outside any stream
// capture.
hipError_t prepare_pass_kernels(size_t lds_per_workgroup)
{
    g_lds_limit = lds_per_workgroup - 256;
    g_lds_limit6 = lds_per_workgroup - kPassStaticLds;
    std::vector<const void *> four, six;
    form_kernels_of<double, 0>(four, six);
    form_kernels_of<double, 8>(four, six);
    form_kernels_of<double, 16>(four, six);
    form_kernels_of<double, 40>(four, six);
    form_kernels_of<float, 0>(four, six);
    form_kernels_of<float, 8>(four, six);
    form_kernels_of<float, 16>(four, six);
    form_kernels_of<float, 40>(four, six);
    for (const void *k : four) {
        hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)g_lds_limit);
        if (e != hipSuccess) return e;
    }
    for (const void *k : six) {
        hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)g_lds_limit6);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Whether a depositing pass takes the whole grid as its tile: when it fits in
// LDS and each of the nblk * threads lanes has few particles.  The other form's
// set-up (the header's read, then the field box moved into LDS) is about 1 us
// and its gathers then take no part in the L2's traffic.
// Four dimensions, tracks of 32 steps, FP64, us whole and staged at 1, 2, 3 and 4
// particles per lane: a Gaussian beam on 128^2 692, 712; 804, 799; 874, 819; 953,
// 873; on 200^2, where its box does not fit, 1015, 1116; 1107, 1164; 1181, 1207;
// 1277, 1309; a KV beam, whose box always fits, on 128^2 637, 652; 731, 719; 827,
// 775; 940, 880; on 200^2 909, 897; 1012, 955; 1111, 988; 1225, 1074.  The size
// alone does not say whether the box will fit, so the line at two is between the
// two beams'.
// The six-dimensional passes are bound by instruction issue and hide the gathers:
// the thick ring, 10 steps, at 8, 16, 24 and 32 per lane on 128^2 666, 683; 1155,
// 1188; 1937, 1688; 2360, 2209; on 200^2 750, 775; 1255, 1298; 2230, 2196; 2874,
// 2806; with the line density 772, 768 at 8, 1277, 1250 at 16 and 3275, 2784 at 32;
// under the B-spline gather the two forms, neither of which stages its box, are
// within 1 % from 8 to 32.  Four dimensions under the B-spline gather, four per
// lane: the staged box takes 33.9 us per step in FP64 (36.9 with the same pass
// gathering from the L2) and 31.2 in the mixed form (31.1).
bool whole_tile(const GridGeom &g, int64_t n, int nblk, int threads, bool six, size_t other_lds)
{
    const int64_t most_per_lane = six ? 16 : 2;
    return sizeof(uint32_t) * (size_t)g.nx * g.ny + other_lds <= pass_lds(six) &&
           n <= most_per_lane * nblk * threads;
}

namespace {

template <typename TE>
hipError_t launch_pass_of(hipStream_t s, const ParticlePtrs &p, const GridGeom &g, bool kick,
                          const void *ef, double kappa, const PassElements &els, bool deposit,
                          const DepositTarget &dep, int blocks, int threads, const LineSpec *line,
                          const void *phi)
{
    const bool six = has_thick(els) || (line && (kick || deposit));
    // LDS of the element parameters and the line histogram beside the tile
    const size_t other = sizeof(els.p) + (line ? 4 * (size_t)line->nz + 16 : 0);
    const bool whole = deposit && whole_tile(g, p.n, blocks, threads, six, other);
    if (phi && kick) {
        if (!deposit)
            return six ? launch_pass_bspline_t<TE, true, false, true>(s, p, g, phi, kappa, els, dep,
                                                                      blocks, threads)
                       : launch_pass_bspline_t<TE, true, false, false>(s, p, g, phi, kappa, els,
                                                                       dep, blocks, threads);
        return with_form(whole, false, threads, [&](auto form) {
            constexpr int FORM = decltype(form)::value;
            if constexpr (!(FORM & 8)) {
                if (six)
                    return launch_pass_bspline_t<TE, true, true, true, FORM>(
                        s, p, g, phi, kappa, els, dep, blocks, threads);
                return with_first<FORM>(first_linear(els), [&](auto first) {
                    return launch_pass_bspline_t<TE, true, true, false, FORM,
                                                 decltype(first)::value>(s, p, g, phi, kappa, els,
                                                                         dep, blocks, threads);
                });
            }
            return hipErrorInvalidValue;
        });
    }
    if (line && (kick || deposit)) {
        if (!deposit)
            return launch_pass_line_t<TE, true, false>(s, p, g, ef, kappa, els, dep, blocks,
                                                       threads, *line);
        return with_form(whole, false, threads, [&](auto form) {
            constexpr int FORM = decltype(form)::value;
            if constexpr (!(FORM & 8))
                return kick ? launch_pass_line_t<TE, true, true, FORM>(s, p, g, ef, kappa, els, dep,
                                                                       blocks, threads, *line)
                            : launch_pass_line_t<TE, false, true, FORM>(
                                  s, p, g, ef, kappa, els, dep, blocks, threads, *line);
            return hipErrorInvalidValue;
        });
    }
    if (!deposit) {
        if (six)
            return kick ? launch_pass_t<TE, true, false, true>(s, p, g, ef, kappa, els, dep, blocks,
                                                               threads)
                        : launch_pass_t<TE, false, false, true>(s, p, g, ef, kappa, els, dep,
                                                                blocks, threads);
        return with_form(false, p.stream, threads, [&](auto form) {
            constexpr int FORM = decltype(form)::value;
            if constexpr (FORM != 16)
                return kick ? launch_pass_t<TE, true, false, false, FORM>(s, p, g, ef, kappa, els,
                                                                          dep, blocks, threads)
                            : launch_pass_t<TE, false, false, false, FORM & 31>(
                                  s, p, g, ef, kappa, els, dep, blocks, threads);
            return hipErrorInvalidValue;
        });
    }
    return with_form(whole, p.stream && !six, threads, [&](auto form) {
        constexpr int FORM = decltype(form)::value;
        if constexpr (!(FORM & 8))
            if (six)
                return kick ? launch_pass_t<TE, true, true, true, FORM>(s, p, g, ef, kappa, els,
                                                                        dep, blocks, threads)
                            : launch_pass_t<TE, false, true, true, FORM>(s, p, g, ef, kappa, els,
                                                                         dep, blocks, threads);
        if (!kick)
            return launch_pass_t<TE, false, true, false, FORM>(s, p, g, ef, kappa, els, dep, blocks,
                                                               threads);
        return with_first<FORM>(first_linear(els), [&](auto first) {
            return launch_pass_t<TE, true, true, false, FORM, decltype(first)::value>(
                s, p, g, ef, kappa, els, dep, blocks, threads);
        });
    });
}

template <typename TE>
hipError_t launch_pass_batched_of(hipStream_t s, const BatchLaunch &b, const ParticlePtrs &all,
                                  const BatchStep *steps, bool kick, bool deposit,
                                  const BatchPassForm &f, int blocks, int threads)
{
    if (!deposit) {
        if (f.six)
            return kick ? launch_pass_batched_t<TE, true, false, true>(s, b, all, steps, blocks,
                                                                       threads)
                        : launch_pass_batched_t<TE, false, false, true>(s, b, all, steps, blocks,
                                                                        threads);
        return with_form(false, all.stream, threads, [&](auto form) {
            constexpr int FORM = decltype(form)::value;
            if constexpr (FORM != 16)
                return kick ? launch_pass_batched_t<TE, true, false, false, FORM>(
                                  s, b, all, steps, blocks, threads)
                            : launch_pass_batched_t<TE, false, false, false, FORM & 31>(
                                  s, b, all, steps, blocks, threads);
            return hipErrorInvalidValue;
        });
    }
    return with_form(f.whole, all.stream && !f.six, threads, [&](auto form) {
        constexpr int FORM = decltype(form)::value;
        if constexpr (!(FORM & 8))
            if (f.six)
                return kick ? launch_pass_batched_t<TE, true, true, true, FORM>(s, b, all, steps,
                                                                                blocks, threads)
                            : launch_pass_batched_t<TE, false, true, true, FORM>(s, b, all, steps,
                                                                                 blocks, threads);
        if (!kick)
            return launch_pass_batched_t<TE, false, true, false, FORM>(s, b, all, steps, blocks,
                                                                       threads);
        return with_first<FORM>(f.first, [&](auto first) {
            return launch_pass_batched_t<TE, true, true, false, FORM, decltype(first)::value>(
                s, b, all, steps, blocks, threads);
        });
    });
}

}  // namespace

hipError_t launch_pass(hipStream_t s, const ParticlePtrs &p, const GridGeom &g, bool kick,
                       bool mixed, const void *ef, double kappa, const PassElements &els,
                       bool deposit, const DepositTarget &dep, int blocks, int threads,
                       const LineSpec *line, const void *bspline_phi)
{
    if (blocks <= 0) return hipSuccess;
    return mixed ? launch_pass_of<float>(s, p, g, kick, ef, kappa, els, deposit, dep, blocks,
                                         threads, line, bspline_phi)
                 : launch_pass_of<double>(s, p, g, kick, ef, kappa, els, deposit, dep, blocks,
                                          threads, line, bspline_phi);
}

hipError_t launch_pass_batched(hipStream_t s, const BatchLaunch &b, const ParticlePtrs &all,
                               const BatchStep *steps, bool kick, bool mixed, bool deposit,
                               const BatchPassForm &form, int blocks, int threads)
{
    if (blocks <= 0) return hipSuccess;
    return mixed ? launch_pass_batched_of<float>(s, b, all, steps, kick, deposit, form, blocks,
                                                 threads)
                 : launch_pass_batched_of<double>(s, b, all, steps, kick, deposit, form, blocks,
                                                  threads);
}

size_t pass_lds(bool six) { return six ? g_lds_limit6 : g_lds_limit; }

namespace {

constexpr int kMomentThreads = 256;

// Sums of the workgroups' partial moments, added in block order: the block
// brings them into LDS first, so that the chain of additions waits for nothing
// (read from memory one by one they took 34 us, now under 3).  Called by all
// threads; the result holds from the next barrier on.
__device__ __forceinline__ void sum_moments(const double *__restrict__ part, double *lds,
                                            double *sums)
{
    for (int t = threadIdx.x; t < kMomentBlocks * kMoments; t += kMomentThreads) lds[t] = part[t];
    __syncthreads();
    if (threadIdx.x < kMoments) {
        double s = 0.0;
#pragma unroll 16
        for (int b = 0; b < kMomentBlocks; ++b) s += lds[b * kMoments + threadIdx.x];
        sums[threadIdx.x] = s;
    }
}

// One pass of the beam moments over the alive particles (diagnostics).  PASS 1
// sums 1, x, px, y, py into part[block][k].  PASS 2 adds up pass 1's partials
// (every workgroup for itself; the first writes the sums to sums[0..5]) and
// sums the products of the deviations from the means into part2.  Each thread
// takes its particles in order, eight loaded at a time: with one in flight the
// 256 workgroups of four waves left memory idle (1e7 particles 210 us per pass
// for 330 MB).  Each workgroup reduces its threads in a fixed tree.
template <int PASS>
__global__ void __launch_bounds__(kMomentThreads)
    k_moments(ParticlePtrs P, double *__restrict__ part, double *__restrict__ part2,
              double *__restrict__ sums)
{
    __shared__ double red[kMoments][kMomentThreads];
    static_assert(kMomentBlocks == kMomentThreads, "red holds one value per workgroup and moment");
    double acc[kMoments] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    double mx = 0.0, mpx = 0.0, my = 0.0, mpy = 0.0;
    if (PASS == 2) {
        __shared__ double first[kMoments];
        sum_moments(part, &red[0][0], first);
        __syncthreads();
        if (blockIdx.x == 0 && threadIdx.x < kMoments) sums[threadIdx.x] = first[threadIdx.x];
        if (first[0] > 0.0) {
            mx = first[1] / first[0];
            mpx = first[2] / first[0];
            my = first[3] / first[0];
            mpy = first[4] / first[0];
        }
        __syncthreads();
    }
    constexpr int kAhead = 8;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p0 < P.n;
         p0 += kAhead * stride) {
        double x[kAhead], px[kAhead], y[kAhead], py[kAhead];
        bool alive[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t p = p0 + u * stride, q = p < P.n ? p : p0;
            x[u] = P.x[q];
            px[u] = P.px[q];
            y[u] = P.y[q];
            py[u] = P.py[q];
            alive[u] = p < P.n && !(P.lost && P.lost[q]);
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (!alive[u]) continue;
            if (PASS == 1) {
                acc[0] += 1.0;
                acc[1] += x[u];
                acc[2] += px[u];
                acc[3] += y[u];
                acc[4] += py[u];
            } else {
                const double dx = x[u] - mx, dpx = px[u] - mpx, dy = y[u] - my, dpy = py[u] - mpy;
                acc[0] += dx * dx;
                acc[1] += dpx * dpx;
                acc[2] += dx * dpx;
                acc[3] += dy * dy;
                acc[4] += dpy * dpy;
                acc[5] += dy * dpy;
            }
        }
    }
    const int t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < kMoments; ++k) red[k][t] = acc[k];
    __syncthreads();
    for (int h = kMomentThreads / 2; h > 0; h >>= 1) {
        if (t < h)
#pragma unroll
            for (int k = 0; k < kMoments; ++k) red[k][t] += red[k][t + h];
        __syncthreads();
    }
    double *out = PASS == 1 ? part : part2;
    if (t < kMoments) out[(size_t)blockIdx.x * kMoments + t] = red[t][0];
}

__global__ void __launch_bounds__(kMomentThreads)
    k_moments_sum(const double *__restrict__ part, double *__restrict__ out)
{
    __shared__ double lds[kMomentBlocks * kMoments];
    sum_moments(part, lds, out);
}

}  // namespace

hipError_t launch_moments(hipStream_t s, const ParticlePtrs &p, double *part, double *sums)
{
    double *part2 = part + kMomentBlocks * kMoments;
    hipLaunchKernelGGL(k_moments<1>, dim3(kMomentBlocks), dim3(kMomentThreads), 0, s, p, part,
                       (double *)nullptr, (double *)nullptr);
    hipLaunchKernelGGL(k_moments<2>, dim3(kMomentBlocks), dim3(kMomentThreads), 0, s, p, part,
                       part2, sums);
    hipLaunchKernelGGL(k_moments_sum, dim3(1), dim3(kMomentThreads), 0, s, (const double *)part2,
                       sums + kMoments);
    return hipGetLastError();
}

hipError_t launch_interleave(hipStream_t s, bool mixed, bool to_interleaved, void *ex, void *ey,
                             void *ef, int ncell)
{
    const dim3 grid((ncell + 255) / 256);
    if (mixed) {
        if (to_interleaved)
            hipLaunchKernelGGL((k_interleave<float, true>), grid, dim3(256), 0, s, (float *)ex,
                               (float *)ey, (float *)ef, ncell);
        else
            hipLaunchKernelGGL((k_interleave<float, false>), grid, dim3(256), 0, s, (float *)ex,
                               (float *)ey, (float *)ef, ncell);
    } else {
        if (to_interleaved)
            hipLaunchKernelGGL((k_interleave<double, true>), grid, dim3(256), 0, s, (double *)ex,
                               (double *)ey, (double *)ef, ncell);
        else
            hipLaunchKernelGGL((k_interleave<double, false>), grid, dim3(256), 0, s, (double *)ex,
                               (double *)ey, (double *)ef, ncell);
    }
    return hipGetLastError();
}

}  // namespace scpic

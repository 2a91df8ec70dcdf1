// gpd.hip — the particle hot path on gfx950: field gather from the Yee grid, the frame's
// Boris-like push, position update with the boundary conditions, leaky-box escape and the
// charge-conserving (Esirkepov) current deposit, fused in one kernel per tile.
//
// One workgroup owns one tile: it stages E and B of the tile plus the guard layers the gather
// reaches in LDS (one region per Yee component, sized for that component's lattice),
// accumulates the tile's current (plus the deposit halo) in LDS as 64-bit fixed point, and
// flushes it once to HBM with float atomics (only the halo overlaps a neighbour tile).  In boxes
// of few tiles several workgroups share one and the last of them flushes their sum.
// Particles are read through the sort permutation and written in sorted slot order, so the
// tile sort's scatter is fused into this pass.  A particle found outside its tile (only
// possible without a sort since the last push) takes the global-memory path.
#include "pic_internal.h"

namespace pic {

// ------------------------------------------------------------------ small vector helpers
struct f3 {
    float x, y, z;
};
__device__ inline f3 mk(float a, float b, float c) { return f3{a, b, c}; }
__device__ inline f3 operator+(f3 a, f3 b) { return mk(a.x + b.x, a.y + b.y, a.z + b.z); }
__device__ inline f3 operator*(float s, f3 a) { return mk(s * a.x, s * a.y, s * a.z); }
__device__ inline float dot(f3 a, f3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ inline f3 cross(f3 a, f3 b)
{
    return mk(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}

// Hardware reciprocal and square root (v_rcp_f32, v_sqrt_f32: about 1 ulp), used instead of
// the correctly rounded division and square-root sequences.
__device__ inline float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline float fsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
// v_rsq_f32 for arguments >= 1 (Lorentz factors): no denormal rescaling needed
__device__ inline float rsq1(float x) { return __builtin_amdgcn_rsqf(x); }

// Particle arrays are indexed with 32-bit byte offsets (capacity below 2^30 per species), so
// the loads and stores take a scalar base and one shared vector offset.
template <class T>
__device__ inline T ld_at(const T* __restrict__ base, uint32_t i)
{
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) +
                                       (size_t)(i * (uint32_t)sizeof(T)));
}
// Non-temporal: what a push writes is read by the next one at the earliest, and the caches are better kept for
// the reads, whose lines neighbouring tiles share (256^3 shear 5.84 -> 5.70 ms, 2048^2 leaky 4.27 -> 4.12 ms,
// 1024^2 leaky 0.675 -> 0.643 ms, a step of the 16 served boxes 704 -> 685 us; non-temporal loads made the push 20 % slower).
template <class T>
__device__ inline void st_at(T* __restrict__ base, uint32_t i, T v)
{
    __builtin_nontemporal_store(v, reinterpret_cast<T*>(reinterpret_cast<char*>(base) + (size_t)(i * (uint32_t)sizeof(T))));
}

// ------------------------------------------------------------------ interpolation
// Linear (CIC) interpolation of one component on its own staggered lattice (base index and
// weights per axis), from an array with element strides (1, sy, sz).
template <int DIM>
__device__ inline float interp(const float* __restrict__ F, int bx, int by, int bz, float wx,
                               float wy, float wz, int sy, int sz)
{
    const float* p = F + bx + sy * by + (DIM == 3 ? sz * bz : 0);
    float a = p[0] + wx * (p[1] - p[0]);
    float b = p[sy] + wx * (p[sy + 1] - p[sy]);
    float r = a + wy * (b - a);
    if (DIM == 3) {
        const float* q = p + sz;
        float c = q[0] + wx * (q[1] - q[0]);
        float d = q[sy] + wx * (q[sy + 1] - q[sy]);
        float r2 = c + wy * (d - c);
        r = r + wz * (r2 - r);
    }
    return r;
}

// Per axis: the integer lattice uses (cell, offset); the half-shifted lattice uses
// (cell-1, offset+1/2) below the cell centre and (cell, offset-1/2) above it.
struct AxisW {
    int b0, bh;
    float w0, wh;
};
__device__ inline AxisW axis_weights(int c, float o)
{
    AxisW a;
    const bool lo = o < 0.5f;
    a.b0 = c;
    a.w0 = o;
    a.bh = lo ? c - 1 : c;
    a.wh = lo ? o + 0.5f : o - 0.5f;
    return a;
}

// Gather the six Yee components at a particle.  Fields are arrays 0..2 = E, 3..5 = B.
template <int DIM, class FieldAt>
__device__ inline void gather(FieldAt fa, int sy, int sz, int cx, int cy, int cz, float ox,
                              float oy, float oz, f3& E, f3& B)
{
    const AxisW X = axis_weights(cx, ox), Y = axis_weights(cy, oy);
    AxisW Z = axis_weights(cz, oz);
    if (DIM == 2) Z = AxisW{0, 0, 0.f, 0.f};
    E.x = interp<DIM>(fa(0), X.bh, Y.b0, Z.b0, X.wh, Y.w0, Z.w0, sy, sz);
    E.y = interp<DIM>(fa(1), X.b0, Y.bh, Z.b0, X.w0, Y.wh, Z.w0, sy, sz);
    E.z = interp<DIM>(fa(2), X.b0, Y.b0, Z.bh, X.w0, Y.w0, Z.wh, sy, sz);
    B.x = interp<DIM>(fa(3), X.b0, Y.bh, Z.bh, X.w0, Y.wh, Z.wh, sy, sz);
    B.y = interp<DIM>(fa(4), X.bh, Y.b0, Z.bh, X.wh, Y.w0, Z.wh, sy, sz);
    B.z = interp<DIM>(fa(5), X.bh, Y.bh, Z.b0, X.wh, Y.wh, Z.w0, sy, sz);
}

// ------------------------------------------------------------------ pushers
// Standard Boris (the alpha = 0 and Lambda = 0 limits of the operators of Secs. 2.2, 3.2).
__device__ inline f3 push_boris(f3 u, f3 E, f3 B, float qm_hdt)
{
    const f3 eps = qm_hdt * E;
    const f3 um = u + eps;
    const float ig = rsq1(1.f + dot(um, um));
    const f3 t = (qm_hdt * ig) * B;
    const float d = 2.f * rcp(1.f + dot(t, t));
    const f3 c1 = cross(um, t);
    const f3 c2 = cross(c1, t);
    return um + d * (c1 + c2) + eps;
}

// Shearing-box push (Sec. 2.2, eq. OAu_disc): closed form
//   u+ = B(u-) + R(S u-) + R(S w)/(1-g),  w = B(u-) + R(S u-),  g = S_2 . R(e_y),
// with S u = e_y (s2 . u); R(e_y) written out.  gamma-bar from the printed first-order
// approximation refined by one fixed-point step of g^2 = 1 + A + K/g (the step contracts by
// about |K|/(2 g^3), so the approximation's error, at most ~4e-7, drops below FP32 rounding).
__device__ inline f3 push_shear(f3 u, f3 E, f3 B, float qm_hdt, float alpha1, float alpha2,
                                float om_dt)
{
    const f3 eps = qm_hdt * E;
    const f3 um = u + eps;
    const float uu = dot(um, um);
    const float ue = dot(um, eps);
    const float A = uu + 2.f * alpha1 * um.x * um.y;
    const float K = 2.f * alpha2 * ue * um.y;
    const float g0 = fsqrt(1.f + uu);
    float g = g0 + (alpha1 * um.x * um.y * g0 + alpha2 * ue * um.y) * rcp(1.f + uu);
    g = fsqrt(1.f + A + K * rcp(g));
    const float ig = rcp(g);
    f3 t = (qm_hdt * ig) * B;
    t.z += om_dt;
    const f3 et = ig * eps;
    const f3 s2 = mk(alpha1 + alpha2 * et.x, alpha2 * et.y, alpha2 * et.z);
    const float d = rcp(1.f + dot(t, t));
    const f3 c1 = cross(um, t);
    const f3 c2 = cross(c1, t);
    const f3 Bu = um + (2.f * d) * (c1 + c2);
    const f3 Rey = mk(d * (t.z + t.x * t.y), 1.f - d * (t.x * t.x + t.z * t.z), d * (t.y * t.z - t.x));
    const float gg = dot(s2, Rey);
    const f3 w = Bu + dot(s2, um) * Rey;
    const f3 up = w + (dot(s2, w) * rcp(1.f - gg)) * Rey;
    return up + eps;
}

// Expanding-box push (Sec. 3.2, eq. EBu_disc) with the printed modified Boris operator
//   B^(L)(v) = L~ v + ((1+L~) v x t~ + ((1+L~) v x t~) x t~)/(1 + t~^2),
// gamma-bar = sqrt(1 + ((1+Lambda) u-)^2), t~ = tau/(1-Lambda).
__device__ inline f3 push_expand(f3 u, f3 E, f3 B, float qm_hdt, const float lam1p[3],
                                 const float ltil[3], const float tfac[3])
{
    const f3 eps = qm_hdt * E;
    const f3 um = u + eps;
    const f3 lu = mk(lam1p[0] * um.x, lam1p[1] * um.y, lam1p[2] * um.z);
    const float ig = rsq1(1.f + dot(lu, lu));
    const float s = qm_hdt * ig;
    const f3 t = mk(s * tfac[0] * B.x, s * tfac[1] * B.y, s * tfac[2] * B.z);
    const f3 w = mk((1.f + ltil[0]) * um.x, (1.f + ltil[1]) * um.y, (1.f + ltil[2]) * um.z);
    const float d = rcp(1.f + dot(t, t));
    const f3 c1 = cross(w, t);
    const f3 c2 = cross(c1, t);
    const f3 up = mk(ltil[0] * um.x, ltil[1] * um.y, ltil[2] * um.z) + d * (c1 + c2);
    return up + eps;
}

// Combined shearing and expanding frame (the extension named in the conclusion, Sec. 5;
// reading): (1 - Lambda) u+ - u+ x tau~ - S u+ = (1 + Lambda) u- + u- x tau~ + S u-, i.e.
// eq. OAu_disc with the diagonal Lambda of eq. EBu_disc.  A u = (1 - Lambda) u - u x tau~ is
// inverted as the expanding push does, A^-1 r = R_t((1 - Lambda)^-1 r), t = (1 - Lambda)^-1
// tau~, so A^-1((1 + Lambda) v + v x tau~) is the printed B^(Lambda)(v); the rank-1 S is added
// by the Sherman-Morrison formula, as the shearing push adds it to R:
//   w = B^(Lambda)(u-) + (s2.u-) A^-1 e_y,  u+ = w + (s2.w) A^-1 e_y / (1 - s2.A^-1 e_y).
// gamma-bar solves g^2 = 1 + ((1+Lambda)u-)^2 + 2 alpha1 u-_x u-_y + 2 alpha2 (u-.eps) u-_y / g:
// the shearing push's first-order approximation (with (1+Lambda) u- in place of u-) and one
// fixed-point refinement.  Lambda = 0 is the shearing push, alpha = Omega0 = 0 the expanding.
__device__ inline f3 push_shear_expand(f3 u, f3 E, f3 B, float qm_hdt, float alpha1, float alpha2,
                                       float om_dt, const float lam1p[3], const float ltil[3],
                                       const float tfac[3])
{
    const f3 eps = qm_hdt * E;
    const f3 um = u + eps;
    const f3 lu = mk(lam1p[0] * um.x, lam1p[1] * um.y, lam1p[2] * um.z);
    const float ll = dot(lu, lu);
    const float ue = dot(um, eps);
    const float A = ll + 2.f * alpha1 * um.x * um.y;
    const float K = 2.f * alpha2 * ue * um.y;
    const float g0 = fsqrt(1.f + ll);
    float g = g0 + (alpha1 * um.x * um.y * g0 + alpha2 * ue * um.y) * rcp(1.f + ll);
    g = fsqrt(1.f + A + K * rcp(g));
    const float ig = rcp(g);
    f3 tt = (qm_hdt * ig) * B;
    tt.z += om_dt;
    const f3 t = mk(tfac[0] * tt.x, tfac[1] * tt.y, tfac[2] * tt.z);
    const f3 et = ig * eps;
    const f3 s2 = mk(alpha1 + alpha2 * et.x, alpha2 * et.y, alpha2 * et.z);
    const float d = rcp(1.f + dot(t, t));
    const f3 v = mk((1.f + ltil[0]) * um.x, (1.f + ltil[1]) * um.y, (1.f + ltil[2]) * um.z);
    const f3 c1 = cross(v, t);
    const f3 c2 = cross(c1, t);
    const f3 Bu = mk(ltil[0] * um.x, ltil[1] * um.y, ltil[2] * um.z) + d * (c1 + c2);
    // A^-1 e_y = R_t(e_y) / (1 - Lambda_y), R_t(e_y) written out
    const f3 Ae = tfac[1] * mk(d * (t.z + t.x * t.y), 1.f - d * (t.x * t.x + t.z * t.z), d * (t.y * t.z - t.x));
    const float gg = dot(s2, Ae);
    const f3 w = Bu + dot(s2, um) * Ae;
    const f3 up = w + (dot(s2, w) * rcp(1.f - gg)) * Ae;
    return up + eps;
}

// ------------------------------------------------------------------ positions
// In-cell offset renormalisation after s = off + delta (|delta| < 1), in FP32:
// s >= 1 -> (+1, s-1) exact; s < 0 -> t = s+1, (-1, t) if t < 1 else (0, 0).
__device__ inline float renorm(float s, int& dc)
{
    const float f = __builtin_amdgcn_fmed3f(floorf(s), -1.f, 1.f);
    const float r = __fsub_rn(s, f);
    // s + 1 rounded up to 1; or s is no number, for which f is -1: the particle stays in its cell, its offset NaN
    const bool full = !(r < 1.f) && f < 0.f;
    dc = (int)f + (full ? 1 : 0);
    return full ? __fsub_rn(r, 1.f) : r;
}

// ------------------------------------------------------------------ Esirkepov deposit
// CIC shape along one axis: L and U are the nodes around the old position (offset o from L, then o + D); a
// particle that leaves [0, 1] also reaches the node beyond, X (below L or above U).  Positions are taken
// from the nearer node, where they round least; c is that node, s the other.
struct Shape {
    float l, u;        // weights on L and U before the move
    float dl, du, dx;  // their changes and X's
    float e, x;        // what flows through the edge L-U, and through the one to X (towards +)
};
__device__ inline float flip(float v, uint32_t sign) { return __uint_as_float(__float_as_uint(v) ^ sign); }
__device__ inline Shape shape(float o, float D)
{
    Shape A;
    A.l = 1.f - o;
    A.u = o;
    const bool up = o >= 0.5f;  // s lies below c; 1 - o is exact then
    // by the magnitudes, so that an offset of -0, or rounded a unit beyond 0 or 1, has s on the side of one within
    const float x0 = up ? -fabsf(A.l) : fabsf(o), x1 = x0 + D;
    const uint32_t sign = __float_as_uint(x0) & 0x80000000u;
    const float t = flip(x1, sign);  // the new position counted towards s
    const float s0 = fabsf(x0), c0 = 1.f - s0;
    const float dc = (1.f - fabsf(x1)) - c0, ds = fmaxf(0.f, t) - s0;
    A.dx = fmaxf(0.f, -t);
    A.dl = up ? ds : dc;
    A.du = up ? dc : ds;
    A.e = flip(ds, sign);
    A.x = flip(A.dx, sign ^ 0x80000000u);
    return A;
}
// transverse factors of an axis with the charge factor q/dt folded in: node weight w gives
// (w0 + dw/2) and (w0/2 + dw/3)
struct Factor {
    float l1, l2, u1, u2, x1, x2;
};
__device__ inline Factor factor(const Shape& A, float q, float qh, float qt)
{
    return Factor{q * A.l + qh * A.dl, qh * A.l + qt * A.dl, q * A.u + qh * A.du,
                  qh * A.u + qt * A.du, qh * A.dx, qt * A.dx};
}

// Esirkepov decomposition of the density change into currents (CIC):
//   J_x on an edge: q/dt times what flows through it times P of its node across,
//   P = S0_y (S0_z + DS_z/2) + DS_y (S0_z/2 + DS_z/3) (cyclic for y and z);
//   2D: P = S0_y + DS_y/2, and J_z = q dz/dt (S0_x (S0_y + DS_y/2) + DS_x (S0_y/2 + DS_y/3)).
// A particle that crosses a node on no axis (61 % of them at theta = 0.3, 80 % at 0.05) has the 12
// (3D) / 8 (2D) terms of the cell's own edges out of 54 / 21, all at fixed ways from one place.  The terms on
// X nodes and edges stand in a branch per combination of crossed axes (seven in 3D) for all components.
// With a mask for each term about the nearest node instead, a wave ran all 54 on a quarter of its lanes.
// Fixed ways from one place keep the dense terms at one address register: 256^3 shear 6.05 -> 5.96 ms,
// 128 x 128 x 512 expand 5.04 -> 4.96 ms, 2048^2 leaky 4.38 -> 4.33 ms.
//
// Acc: add<C, IX, IY, IZ>(way, v) adds to component C at the particle's cell + (IX, IY, IZ) + way;
// node<A>(x), edge<A>(x): the way from L (from the edge L-U) along axis A to X by the sign of x.
template <int DIM, class Acc>
__device__ inline void esirkepov(Acc& acc, const Shape& X, const Shape& Y, const Shape& Z, float q_dt, float dz)
{
    const bool crx = X.x != 0.f, cry = Y.x != 0.f, crz = DIM == 3 && Z.x != 0.f;
    if constexpr (DIM == 3) {
        const float qh = 0.5f * q_dt, qt = (1.f / 3.f) * q_dt;
        const Factor FZ = factor(Z, q_dt, qh, qt), FY = factor(Y, q_dt, qh, qt);
        // products over two axes: nodes L and U of the first, then of the second
        const float yz00 = Y.l * FZ.l1 + Y.dl * FZ.l2, yz01 = Y.l * FZ.u1 + Y.dl * FZ.u2;
        const float yz10 = Y.u * FZ.l1 + Y.du * FZ.l2, yz11 = Y.u * FZ.u1 + Y.du * FZ.u2;
        const float xz00 = X.l * FZ.l1 + X.dl * FZ.l2, xz01 = X.l * FZ.u1 + X.dl * FZ.u2;
        const float xz10 = X.u * FZ.l1 + X.du * FZ.l2, xz11 = X.u * FZ.u1 + X.du * FZ.u2;
        const float xy00 = X.l * FY.l1 + X.dl * FY.l2, xy01 = X.l * FY.u1 + X.dl * FY.u2;
        const float xy10 = X.u * FY.l1 + X.du * FY.l2, xy11 = X.u * FY.u1 + X.du * FY.u2;
        acc.template add<0, 0, 0, 0>(0, X.e * yz00);
        acc.template add<0, 0, 0, 1>(0, X.e * yz01);
        acc.template add<0, 0, 1, 0>(0, X.e * yz10);
        acc.template add<0, 0, 1, 1>(0, X.e * yz11);
        acc.template add<1, 0, 0, 0>(0, Y.e * xz00);
        acc.template add<1, 0, 0, 1>(0, Y.e * xz01);
        acc.template add<1, 1, 0, 0>(0, Y.e * xz10);
        acc.template add<1, 1, 0, 1>(0, Y.e * xz11);
        acc.template add<2, 0, 0, 0>(0, Z.e * xy00);
        acc.template add<2, 0, 1, 0>(0, Z.e * xy01);
        acc.template add<2, 1, 0, 0>(0, Z.e * xy10);
        acc.template add<2, 1, 1, 0>(0, Z.e * xy11);
        if (crx) {
            const int d = acc.template edge<0>(X.x), k = acc.template node<0>(X.x);
            acc.template add<0, 0, 0, 0>(d, X.x * yz00);
            acc.template add<0, 0, 0, 1>(d, X.x * yz01);
            acc.template add<0, 0, 1, 0>(d, X.x * yz10);
            acc.template add<0, 0, 1, 1>(d, X.x * yz11);
            acc.template add<1, 0, 0, 0>(k, Y.e * (X.dx * FZ.l2));
            acc.template add<1, 0, 0, 1>(k, Y.e * (X.dx * FZ.u2));
            acc.template add<2, 0, 0, 0>(k, Z.e * (X.dx * FY.l2));
            acc.template add<2, 0, 1, 0>(k, Z.e * (X.dx * FY.u2));
        }
        if (cry) {
            const int d = acc.template edge<1>(Y.x), k = acc.template node<1>(Y.x);
            acc.template add<1, 0, 0, 0>(d, Y.x * xz00);
            acc.template add<1, 0, 0, 1>(d, Y.x * xz01);
            acc.template add<1, 1, 0, 0>(d, Y.x * xz10);
            acc.template add<1, 1, 0, 1>(d, Y.x * xz11);
            acc.template add<0, 0, 0, 0>(k, X.e * (Y.dx * FZ.l2));
            acc.template add<0, 0, 0, 1>(k, X.e * (Y.dx * FZ.u2));
            acc.template add<2, 0, 0, 0>(k, Z.e * (X.l * FY.x1 + X.dl * FY.x2));
            acc.template add<2, 1, 0, 0>(k, Z.e * (X.u * FY.x1 + X.du * FY.x2));
        }
        if (crz) {
            const int d = acc.template edge<2>(Z.x), k = acc.template node<2>(Z.x);
            acc.template add<2, 0, 0, 0>(d, Z.x * xy00);
            acc.template add<2, 0, 1, 0>(d, Z.x * xy01);
            acc.template add<2, 1, 0, 0>(d, Z.x * xy10);
            acc.template add<2, 1, 1, 0>(d, Z.x * xy11);
            acc.template add<0, 0, 0, 0>(k, X.e * (Y.l * FZ.x1 + Y.dl * FZ.x2));
            acc.template add<0, 0, 1, 0>(k, X.e * (Y.u * FZ.x1 + Y.du * FZ.x2));
            acc.template add<1, 0, 0, 0>(k, Y.e * (X.l * FZ.x1 + X.dl * FZ.x2));
            acc.template add<1, 1, 0, 0>(k, Y.e * (X.u * FZ.x1 + X.du * FZ.x2));
        }
        if (crx && cry) {
            const int kx = acc.template node<0>(X.x), ky = acc.template node<1>(Y.x);
            const int ax = acc.template edge<0>(X.x) + ky, ay = kx + acc.template edge<1>(Y.x);
            acc.template add<0, 0, 0, 0>(ax, X.x * (Y.dx * FZ.l2));
            acc.template add<0, 0, 0, 1>(ax, X.x * (Y.dx * FZ.u2));
            acc.template add<1, 0, 0, 0>(ay, Y.x * (X.dx * FZ.l2));
            acc.template add<1, 0, 0, 1>(ay, Y.x * (X.dx * FZ.u2));
            acc.template add<2, 0, 0, 0>(kx + ky, Z.e * (X.dx * FY.x2));
        }
        if (crx && crz) {
            const int kx = acc.template node<0>(X.x), kz = acc.template node<2>(Z.x);
            const int ax = acc.template edge<0>(X.x) + kz, az = kx + acc.template edge<2>(Z.x);
            acc.template add<0, 0, 0, 0>(ax, X.x * (Y.l * FZ.x1 + Y.dl * FZ.x2));
            acc.template add<0, 0, 1, 0>(ax, X.x * (Y.u * FZ.x1 + Y.du * FZ.x2));
            acc.template add<2, 0, 0, 0>(az, Z.x * (X.dx * FY.l2));
            acc.template add<2, 0, 1, 0>(az, Z.x * (X.dx * FY.u2));
            acc.template add<1, 0, 0, 0>(kx + kz, Y.e * (X.dx * FZ.x2));
        }
        if (cry && crz) {
            const int ky = acc.template node<1>(Y.x), kz = acc.template node<2>(Z.x);
            const int ay = acc.template edge<1>(Y.x) + kz, az = ky + acc.template edge<2>(Z.x);
            acc.template add<1, 0, 0, 0>(ay, Y.x * (X.l * FZ.x1 + X.dl * FZ.x2));
            acc.template add<1, 1, 0, 0>(ay, Y.x * (X.u * FZ.x1 + X.du * FZ.x2));
            acc.template add<2, 0, 0, 0>(az, Z.x * (X.l * FY.x1 + X.dl * FY.x2));
            acc.template add<2, 1, 0, 0>(az, Z.x * (X.u * FY.x1 + X.du * FY.x2));
            acc.template add<0, 0, 0, 0>(ky + kz, X.e * (Y.dx * FZ.x2));
            if (crx) {
                const int kx = acc.template node<0>(X.x);
                acc.template add<0, 0, 0, 0>(acc.template edge<0>(X.x) + ky + kz, X.x * (Y.dx * FZ.x2));
                acc.template add<1, 0, 0, 0>(kx + ay, Y.x * (X.dx * FZ.x2));
                acc.template add<2, 0, 0, 0>(kx + az, Z.x * (X.dx * FY.x2));
            }
        }
    } else {
        const float ex = q_dt * X.e, ey = q_dt * Y.e, jz = q_dt * dz;
        const float xl = X.l + 0.5f * X.dl, xu = X.u + 0.5f * X.du;
        const float yl = Y.l + 0.5f * Y.dl, yu = Y.u + 0.5f * Y.du;
        const float yl2 = 0.5f * Y.l + (1.f / 3.f) * Y.dl, yu2 = 0.5f * Y.u + (1.f / 3.f) * Y.du;
        acc.template add<0, 0, 0, 0>(0, ex * yl);
        acc.template add<0, 0, 1, 0>(0, ex * yu);
        acc.template add<1, 0, 0, 0>(0, ey * xl);
        acc.template add<1, 1, 0, 0>(0, ey * xu);
        acc.template add<2, 0, 0, 0>(0, jz * (X.l * yl + X.dl * yl2));
        acc.template add<2, 0, 1, 0>(0, jz * (X.l * yu + X.dl * yu2));
        acc.template add<2, 1, 0, 0>(0, jz * (X.u * yl + X.du * yl2));
        acc.template add<2, 1, 1, 0>(0, jz * (X.u * yu + X.du * yu2));
        if (crx) {
            const int d = acc.template edge<0>(X.x), k = acc.template node<0>(X.x);
            const float fx = q_dt * X.x;
            acc.template add<0, 0, 0, 0>(d, fx * yl);
            acc.template add<0, 0, 1, 0>(d, fx * yu);
            acc.template add<1, 0, 0, 0>(k, ey * (0.5f * X.dx));
            acc.template add<2, 0, 0, 0>(k, jz * (X.dx * yl2));
            acc.template add<2, 0, 1, 0>(k, jz * (X.dx * yu2));
        }
        if (cry) {
            const int d = acc.template edge<1>(Y.x), k = acc.template node<1>(Y.x);
            const float fy = q_dt * Y.x, x1 = 0.5f * Y.dx, x2 = (1.f / 3.f) * Y.dx;
            acc.template add<1, 0, 0, 0>(d, fy * xl);
            acc.template add<1, 1, 0, 0>(d, fy * xu);
            acc.template add<0, 0, 0, 0>(k, ex * x1);
            acc.template add<2, 0, 0, 0>(k, jz * (X.l * x1 + X.dl * x2));
            acc.template add<2, 1, 0, 0>(k, jz * (X.u * x1 + X.du * x2));
            if (crx) {
                const int kx = acc.template node<0>(X.x);
                acc.template add<0, 0, 0, 0>(acc.template edge<0>(X.x) + k, (q_dt * X.x) * x1);
                acc.template add<1, 0, 0, 0>(kx + d, fy * (0.5f * X.dx));
                acc.template add<2, 0, 0, 0>(kx + k, jz * (X.dx * x2));
            }
        }
    }
}

// ------------------------------------------------------------------ tile regions in LDS
// Field component f (0..2 = Ex, Ey, Ez; 3..5 = Bx, By, Bz) lies on the half-shifted lattice
// along the axes of its Yee offset: Ex x, Ey y, Ez z, Bx y and z, By x and z, Bz x and y.
__host__ __device__ constexpr bool yee_half(int f, int a) { return f < 3 ? f == a : f - 3 != a; }

template <int DIM, int TX, int TY, int TZ>
struct Geo {
    static constexpr int T(int a) { return a == 0 ? TX : (a == 1 ? TY : TZ); }
    // Staged field component f: per lower corner along x the value there and the step to the next one
    // (8 bytes): along a half-lattice axis the values at global indices t0-1 .. t0+T, along an integer
    // axis t0 .. t0+T, what CIC needs for a particle in the tile.  All components have the pitches of
    // the half lattices, so that one place and the three half-cell choices give every address.
    static constexpr int FX = TX + 1, FY = TY + 2, FXY = FX * FY;
    static constexpr int fdim(int f, int a)
    {
        return (DIM == 2 && a == 2) ? 1 : T(a) + (yee_half(f, a) ? 2 : 1);
    }
    static constexpr int fsize(int f) { return FXY * (fdim(f, 2) - 1) + FX * fdim(f, 1); }
    static constexpr int foff(int f) { return f == 0 ? 0 : foff(f - 1) + fsize(f - 1); }
    // Current component c, origin at global index t0-1 on every axis: along its own axis the
    // edges t0-1 .. t0+T (T+2), across it the nodes t0-1 .. t0+T+1 (T+3); the deposit of a
    // particle of the tile stays inside.  2D: J_z has nodes along x and y.  Pitches of the nodes.
    static constexpr int JX = TX + 3, JY = TY + 3;
    static constexpr int jdim(int c, int a)
    {
        return (DIM == 2 && a == 2) ? 1 : T(a) + (a == c ? 2 : 3);
    }
    static constexpr int jsize(int c) { return JX * (JY * (jdim(c, 2) - 1) + jdim(c, 1)); }
    static constexpr int joff(int c) { return c == 0 ? 0 : joff(c - 1) + jsize(c - 1); }
    static constexpr int JTOT = joff(2) + jsize(2);
    // words per tile of P.tsum: its sums, and in a line of its own the count of the parts that are done
    static constexpr int JSPLIT = (JTOT + 15) / 16 * 16 + 16;
    static constexpr int FTOT = foff(5) + fsize(5);
    static constexpr int FBYTES = (8 * FTOT + 15) & ~15;   // E, B first, then J (8-byte words)
    static constexpr int LDS_BYTES = FBYTES + 8 * JTOT;
};

// LDS accumulator: one region per current component (Geo::jdim).  The tile current is summed in
// 64-bit fixed point: a contribution arrives pre-scaled so that the largest possible single
// contribution is 2^30 units, is truncated to int32 and added with ds_add_u64 (integer LDS
// atomics cost a few cycles per wave instruction, while FP32 LDS atomics are serialised per
// lane).  Integer sums are exact and independent of the order.
template <class G, int DIM>
struct LdsAcc {
    char* J;
    int at;  // place in bytes of the particle's cell, counted from the tile's first
    static constexpr int pitch(int a) { return 8 * (a == 0 ? 1 : (a == 1 ? G::JX : G::JX * G::JY)); }
    template <int C, int IX, int IY, int IZ>
    __device__ inline void add(int way, float v)
    {
        constexpr int place = 8 * G::joff(C) + (1 + IX) * pitch(0) + (1 + IY) * pitch(1) + (DIM == 3 ? (1 + IZ) * pitch(2) : 0);
        // v_cvt_i32_f32: truncates, saturates
        atomicAdd(reinterpret_cast<unsigned long long*>(J + (at + way) + place), (unsigned long long)(long long)(int)v);
    }
    template <int A>
    __device__ inline int edge(float x) const { return x < 0.f ? -pitch(A) : pitch(A); }
    template <int A>
    __device__ inline int node(float x) const { return x < 0.f ? -pitch(A) : 2 * pitch(A); }
};
template <class G, int DIM>
__device__ inline LdsAcc<G, DIM> lds_acc(unsigned long long* Jl, int rx, int ry, int rz)
{
    using A = LdsAcc<G, DIM>;
    // 24-bit multiply-adds; region places are non-negative
    return A{reinterpret_cast<char*>(Jl), (int)(8u * (unsigned)rx + __umul24((unsigned)A::pitch(1), (unsigned)ry) +
                                                (DIM == 3 ? __umul24((unsigned)A::pitch(2), (unsigned)rz) : 0u))};
}

// Global accumulator on the guarded current arrays (slow path).
struct GlobalAcc {
    float* const* J;
    int at;  // the particle's cell; a guarded array holds less than 2^31 floats
    int sy, sz;
    template <int C, int IX, int IY, int IZ>
    __device__ inline void add(int way, float v)
    {
        if (v != 0.f) unsafeAtomicAdd(&J[C][at + IX + sy * IY + sz * IZ + way], v);
    }
    template <int A>
    __device__ inline int edge(float x) const { return (x < 0.f ? -1 : 1) * (A == 0 ? 1 : (A == 1 ? sy : sz)); }
    template <int A>
    __device__ inline int node(float x) const { return (x < 0.f ? -1 : 2) * (A == 0 ? 1 : (A == 1 ? sy : sz)); }
};
__device__ inline GlobalAcc global_acc(const StepDev& P, int x, int y, int z)
{
    return GlobalAcc{P.J, x + P.sy * y + P.sz * z, P.sy, P.sz};
}

// CIC interpolation of staged component F: ad is the place of the lower corner in bytes, (wa, wb, wc) the
// weights of the upper corner.  One 8-byte read per x row: for scattered lanes it costs the 6.3 cycles of a
// 4-byte one, two 4-byte values (ds_read2_b32) 12.5 and two rows in one instruction (ds_read2_b64) 22, which
// the atomic form of the load keeps the compiler from making.  LDS was active 81-86 % of a 3D push's cycles,
// now 64-70 %: 256^3 shear 6.35 -> 6.05 ms, 128 x 128 x 512 expand 5.30 -> 5.04 ms (2 x 134 M particles).
template <class G, int F>
__device__ inline float2 field_row(const char* Fl, unsigned ad, int row)
{
    const unsigned long long v = __hip_atomic_load(
        reinterpret_cast<const unsigned long long*>(Fl + ad + 8 * (G::foff(F) + row)), __ATOMIC_RELAXED,
        __HIP_MEMORY_SCOPE_SINGLETHREAD);
    return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}
template <class G, int DIM, int F>
__device__ inline float interp_lds(const char* Fl, unsigned ad, float wa, float wb, float wc)
{
    const float2 p = field_row<G, F>(Fl, ad, 0), q = field_row<G, F>(Fl, ad, G::FX);
    float2 s, t;
    if (DIM == 3) {
        s = field_row<G, F>(Fl, ad, G::FXY);
        t = field_row<G, F>(Fl, ad, G::FXY + G::FX);
    }
    const float a = p.x + wa * p.y, b = q.x + wa * q.y;
    float r = a + wb * (b - a);
    if (DIM == 3) {
        const float c = s.x + wa * s.y, d = t.x + wa * t.y;
        const float r2 = c + wb * (d - c);
        r = r + wc * (r2 - r);
    }
    return r;
}

// Gather from the staged tile: (rx, ry, rz) = cell - tile origin.  On a half-shifted axis the
// lower node is the one at cell - 1/2 below the cell centre and cell + 1/2 above it.
template <class G, int DIM>
__device__ inline void gather_lds(const char* Fl, int rx, int ry, int rz, float ox, float oy, float oz, f3& E,
                                  f3& B)
{
    const bool lx = ox < 0.5f, ly = oy < 0.5f, lz = oz < 0.5f;
    const float hx = ox + (lx ? 0.5f : -0.5f), hy = oy + (ly ? 0.5f : -0.5f);
    const float hz = oz + (lz ? 0.5f : -0.5f);
    // 24-bit multiply-adds (full rate); places are non-negative
    const unsigned ad = 8u * (unsigned)rx + __umul24((unsigned)ry, 8u * G::FX) +
                        (DIM == 3 ? __umul24((unsigned)rz, 8u * G::FXY) : 0u);
    const unsigned ax = lx ? 0u : 8u, ay = ly ? 0u : 8u * G::FX, az = DIM == 2 || lz ? 0u : 8u * G::FXY;
    E.x = interp_lds<G, DIM, 0>(Fl, ad + ax, hx, oy, oz);
    E.y = interp_lds<G, DIM, 1>(Fl, ad + ay, ox, hy, oz);
    E.z = interp_lds<G, DIM, 2>(Fl, ad + az, ox, oy, hz);
    B.x = interp_lds<G, DIM, 3>(Fl, ad + ay + az, ox, hy, hz);
    B.y = interp_lds<G, DIM, 4>(Fl, ad + ax + az, hx, oy, hz);
    B.z = interp_lds<G, DIM, 5>(Fl, ad + ax + ay, hx, hy, oz);
}

// Stage field component F (and the ones after it) of the tile into its LDS region.  All components'
// loads are in flight before the first store where a thread has few of them: a box of one round of
// workgroups waits for memory once instead of for each component.
template <class G, int DIM, int F, int NT>
__device__ inline void stage_fields(float2* __restrict__ Fl, const StepDev& P, const int t0[3],
                                    const int ext[3], int tid)
{
    constexpr int N = G::fsize(F), ROUNDS = (N + NT - 1) / NT;
    constexpr int hx = yee_half(F, 0), hy = yee_half(F, 1), hz = DIM == 3 && yee_half(F, 2);
    const float* src = F < 3 ? P.E[F] : P.B[F - 3];
    float a[ROUNDS], b[ROUNDS];
#pragma unroll
    for (int k = 0; k < ROUNDS; k++) {
        const int e = tid + k * NT;
        const int lx = e % G::FX, ly = (e / G::FX) % G::FY, lz = e / G::FXY;
        a[k] = b[k] = 0.f;
        if (lx < ext[0] + hx && ly < ext[1] + 1 + hy && lz < (DIM == 2 ? 1 : ext[2] + 1 + hz)) {
            const int64_t g = (int64_t)(t0[0] - hx + lx) + (int64_t)P.sy * (t0[1] - hy + ly) +
                              (DIM == 3 ? (int64_t)P.sz * (t0[2] - hz + lz) : 0);
            a[k] = src[g];
            b[k] = src[g + 1];
        }
    }
    if constexpr (F < 5 && ROUNDS <= 2) stage_fields<G, DIM, F + 1, NT>(Fl, P, t0, ext, tid);
#pragma unroll
    for (int k = 0; k < ROUNDS; k++) {
        const int e = tid + k * NT;
        if (e < N) Fl[G::foff(F) + e] = make_float2(a[k], b[k] - a[k]);
    }
    if constexpr (F < 5 && ROUNDS > 2) stage_fields<G, DIM, F + 1, NT>(Fl, P, t0, ext, tid);
}

// ------------------------------------------------------------------ the fused kernel
template <int DIM>
__device__ inline void tile_origin(const StepDev& P, int tile, int t0[3], int ext[3])
{
    const int tx = tile % P.tl.nt[0];
    const int r = tile / P.tl.nt[0];
    const int ty = r % P.tl.nt[1];
    const int tz = r / P.tl.nt[1];
    const int tc[3] = {tx, ty, tz};
#pragma unroll
    for (int d = 0; d < 3; d++) {
        t0[d] = tc[d] << P.tl.lt[d];
        const int e = P.n[d] - t0[d];
        ext[d] = e < (1 << P.tl.lt[d]) ? e : (1 << P.tl.lt[d]);
    }
    if (DIM == 2) {
        t0[2] = 0;
        ext[2] = 1;
    }
}

__device__ inline void latch(uint32_t* err, uint32_t bit) { atomicOr(err, bit); }

// int64 fixed-point tile sum -> FP32 current
__device__ inline float fixed_to_float(unsigned long long a, float unit)
{
    const long long v = (long long)a;
    const int hi = (int)(v >> 32);
    const unsigned lo = (unsigned)v;
    return (float)(((double)hi * 4294967296.0 + (double)lo) * (double)unit);
}

// Flush the tile current (interior + deposit halo) to the global arrays with float atomics.  The parts of a
// split tile add their integers to the tile's words of P.tsum first, and the one that comes last flushes
// the whole sum: exact and converted once, however the tile was split.  It leaves words and count at zero
// for the next launch; nobody waits.  The parts meet in device-scope atomics alone, so each needs only its
// own to be done before it counts itself; __threadfence() would write back and invalidate the L2 for every
// part (a step of the 64^2 box 115 us, an unfused one of the 384^2 box 333 us; 87 and 144 us this way), and
// counts of several tiles in one line made the parts queue for it (90 us).  Parts that rounded to FP32 each and
// met in the current's atomics took 83 and 140 us, but put the rounding of their gross sums and the order of the
// additions into every node.
// flag: a shared word that nothing else uses any more.
template <class G, int DIM, int NT>
__device__ inline void flush_current(unsigned long long* Jl, const StepDev& P, int tile,
                                     const int t0[3], const int ext[3], int tid, uint32_t* flag)
{
    if (P.lsplit) {
        unsigned long long* const sum = P.tsum + (size_t)tile * G::JSPLIT;
        uint32_t* const done = reinterpret_cast<uint32_t*>(sum + G::JSPLIT - 16);
        for (int e = tid; e < G::JTOT; e += NT)
            if (Jl[e]) __hip_atomic_fetch_add(&sum[e], Jl[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0)
            *flag = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == 1u << P.lsplit;
        __syncthreads();
        if (!*flag) return;
        constexpr int N = (G::JTOT + NT - 1) / NT;  // all loads on their way before the first is used
        unsigned long long v[N];
        int t = tid;
        asm volatile("" : "+v"(t));  // keeps the places out of the particle loop's registers
#pragma unroll
        for (int k = 0; k < N; k++)
            v[k] = t + k * NT < G::JTOT ? __hip_atomic_load(&sum[t + k * NT], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
#pragma unroll
        for (int k = 0; k < N; k++) {  // its own entries below: no barrier
            if (t + k * NT >= G::JTOT) break;
            Jl[t + k * NT] = v[k];
            __hip_atomic_store(&sum[t + k * NT], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (tid == 0) __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    for (int e = tid; e < G::JTOT; e += NT) {
        const unsigned long long a = Jl[e];
        if (a == 0ull) continue;
        const int c = (e >= G::joff(1)) + (e >= G::joff(2));
        const int r = e - (c == 0 ? 0 : (c == 1 ? G::joff(1) : G::joff(2)));
        const int lx = r % G::JX, ly = (r / G::JX) % G::JY, lz = r / (G::JX * G::JY);
        if (lx < ext[0] + (c == 0 ? 2 : 3) && ly < ext[1] + (c == 1 ? 2 : 3) &&
            (DIM == 2 || lz < ext[2] + (c == 2 ? 2 : 3))) {
            const int64_t g = (int64_t)(t0[0] - 1 + lx) + (int64_t)P.sy * (t0[1] - 1 + ly) +
                              (DIM == 3 ? (int64_t)P.sz * (t0[2] - 1 + lz) : 0);
            unsafeAtomicAdd(&P.J[c][g], fixed_to_float(a, P.junit));
        }
    }
}

// what a workgroup takes of a launch: its tile, of the species s0 .. s1 - 1 the rounds part, part + 2^lparts, ...
struct Share {
    int tile, part, lparts, s0, s1;
    __device__ inline Share(const StepDev& P, int unit)
    {
        tile = unit >> P.lsplit;
        part = (unit & ((1 << P.lsplit) - 1)) >> P.by_species;
        lparts = P.lsplit - P.by_species;
        s0 = P.by_species ? unit & 1 : 0;
        s1 = P.by_species ? s0 + 1 : P.nsp;
    }
};

// a particle as it is read through the sort permutation; in the leaky box with what its escape needs
template <int DIM, int FRAME>
struct Particle {
    int32_t cell;
    float o[DIM];
    f3 u;
    float dr[3];
    uint32_t id;
    __device__ inline void load(const StepDev& P, const SpeciesDev& S, uint32_t src)
    {
        cell = ld_at(S.cell_in, src);
#pragma unroll
        for (int d = 0; d < DIM; d++) o[d] = ld_at(S.off_in[d], src);
        u = mk(ld_at(S.u_in[0], src), ld_at(S.u_in[1], src), ld_at(S.u_in[2], src));
        if (FRAME == kLeaky) load_escape(P, S, src);
    }
    __device__ inline void load_escape(const StepDev& P, const SpeciesDev& S, uint32_t src)
    {
        id = ld_at(S.id_in, src);
        if (P.leaky_mode == 0) {
            dr[0] = ld_at(S.dr_in[0], src);
            dr[1] = ld_at(S.dr_in[1], src);
            if (P.use_3vec) dr[2] = ld_at(S.dr_in[2], src);
        }
    }
};

template <int DIM, int TX, int TY, int TZ, int FRAME, int NT>
__device__ __attribute__((always_inline)) inline void gpd_body(const StepDev& P, int blk, int nblk,
                                                                int fuse)
{
    using G = Geo<DIM, TX, TY, TZ>;
    __shared__ __attribute__((aligned(16))) unsigned char lds[G::LDS_BYTES];
    const char* const Fl = reinterpret_cast<const char*>(lds);                            // E, B
    unsigned long long* const Jl = reinterpret_cast<unsigned long long*>(lds + G::FBYTES);  // J

    const int unit = xcd_contiguous(blk, nblk);
    const Share share(P, unit);
    const int tile = share.tile;
    int t0[3], ext[3];
    tile_origin<DIM>(P, tile, t0, ext);
    const int tid = threadIdx.x;

    // migration counts of the next sort (per species, direction)
    __shared__ uint32_t mc[kMaxSpecies * kMigDirs];
    const int tsy = t0[1] >> P.tl.lt[1];  // y index of this tile
    const int mco = frame_sheared(FRAME) ? mig_center(P.mg, tsy, true) : tsy;
    const int mci = frame_sheared(FRAME) ? mig_center(P.mg, tsy, false) : tsy;

    stage_fields<G, DIM, 0, NT>(reinterpret_cast<float2*>(lds), P, t0, ext, tid);
    if (fuse)
        for (int e = tid; e < G::JTOT; e += NT) Jl[e] = 0ull;
    if (tid < kMaxSpecies * kMigDirs) mc[tid] = 0u;
    __syncthreads();

    const int nx = P.n[0], ny = P.n[1], nz = P.n[2];
    for (int s = share.s0; s < share.s1; s++) {
        const SpeciesDev& S = P.sp[s];
        bool far = false;   // a particle beyond the neighbouring tiles
        uint32_t nesc = 0;  // probabilistic escapes (one counter add per wave, at the end)
        uint32_t nsl = 0;   // shearing box: superluminal effective velocities (likewise)
        const uint32_t beg = (uint32_t)S.toff[tile], end = (uint32_t)S.toff[tile + 1];
        // The threads take the tile's slots from the first multiple of 32 on (the 128-byte lines of the
        // 4-byte particle arrays, so that a wave's stores fill whole lines) and those before it last.
        // A round's particle is read during the deposit of the round before, at an index read one round
        // earlier still; past the last round both stay on the last slot.  The kernel without gather, push
        // and deposit still takes 80-97 % of its time, so what counts is that every wave always has loads
        // on their way, and that it waits for its stores no earlier than after a deposit: 256^3 shear
        // 5.96 -> 5.84 ms, 128 x 128 x 512 expand 4.96 -> 4.80 ms, 1024^2 leaky 0.716 -> 0.675 ms.
        const uint32_t count = end - beg, head = min(-beg & 31u, count);
        auto slot_of = [&](uint32_t v) {
            const uint32_t r = min(v, count - 1) + head;
            return beg + (r < count ? r : r - count);
        };
        const uint32_t stride = (uint32_t)NT << share.lparts;
        uint32_t v = share.part * NT + tid, src = 0, src_next = 0;
        Particle<DIM, FRAME> p;
        if (v < count) {
            src = (uint32_t)ld_at(S.perm, slot_of(v));
            src_next = (uint32_t)ld_at(S.perm, slot_of(v + stride));
            p.load(P, S, src);
        }
        for (; v < count; v += stride) {
            uint32_t so = slot_of(v);
            asm("" : "+v"(so));  // keeps the 32-bit offset form (scalar base) for the stores
            int cx, cy, cz;
            P.cc.decode(p.cell, cx, cy, cz);
            const float ox = p.o[0], oy = p.o[1], oz = DIM == 3 ? p.o[2] : 0.f;
            f3 u = p.u;

            const int rx = cx - t0[0], ry = cy - t0[1], rz = DIM == 3 ? cz - t0[2] : 0;
            const bool in_tile = (unsigned)rx < (unsigned)ext[0] && (unsigned)ry < (unsigned)ext[1] &&
                                 (DIM == 2 || (unsigned)rz < (unsigned)ext[2]);
            f3 E, B;
            if (in_tile) {
                gather_lds<G, DIM>(Fl, rx, ry, rz, ox, oy, oz, E, B);
            } else {
                auto fa = [&](int c) -> const float* { return c < 3 ? P.E[c] : P.B[c - 3]; };
                gather<DIM>(fa, P.sy, P.sz, cx, cy, cz, ox, oy, oz, E, B);
                atomicAdd(&P.ctr[0], 1ull);
                latch(P.err, 4u);
            }

            // ---- push
            const float xr = __fadd_rn(__fsub_rn((float)cx, P.half_nx), ox);  // radial x (shearing box)
            if (FRAME == kShear)
                u = push_shear(u, E, B, S.qm_hdt, P.alpha1, P.sO * xr, P.om_dt);
            else if (FRAME == kShearExpand)
                u = push_shear_expand(u, E, B, S.qm_hdt, P.alpha1, P.sO * xr, P.om_dt, P.lam1p,
                                      P.ltil, P.tfac);
            else if (FRAME == kExpand)
                u = push_expand(u, E, B, S.qm_hdt, P.lam1p, P.ltil, P.tfac);
            else
                u = push_boris(u, E, B, S.qm_hdt);

            // ---- displacement of the deposit (comoving for the shearing box, primed for the
            // expanding box, both for the combined frame)
            const float ig = rsq1(1.f + dot(u, u));
            const float hs = P.dt * ig;
            f3 D = hs * u;
            if (frame_expanding(FRAME)) D = mk(D.x * P.linv[0], D.y * P.linv[1], D.z * P.linv[2]);
            // y increment of the position: the shearing box adds the shear move
            // y -= s Omega0 (x' + x^n)/2 dt (Sec. 2.2), x' + x^n = 2 x^n + D.x, each operation
            // rounded as written (the FP32 integer layer of the oracle repeats it bit for bit)
            float dyt = D.y, vs = 0.f;
            if (frame_sheared(FRAME)) {  // the combined frame: x and y scale together
                vs = __fmul_rn(-P.sO, __fmaf_rn(0.5f, D.x, xr));  // v_s at the midpoint x
                dyt = __fmaf_rn(P.dt, vs, D.y);
            }
            // one test catches both: a non-finite momentum makes D NaN, which fails every
            // comparison; a finite one fails it when a deposit displacement reaches half a cell
            // or the shear move takes the y increment to a whole cell (the offset
            // renormalisation needs |increment| < 1)
            if (!(fabsf(D.x) < 0.5f && fabsf(D.y) < 0.5f && (DIM == 2 || fabsf(D.z) < 0.5f) &&
                  fabsf(dyt) < 1.f))
                latch(P.err, (isfinite(u.x) && isfinite(u.y) && isfinite(u.z)) ? 1u : 2u);

            // ---- new position: x' = x^n + D, then (shearing box) the shear move
            // y -= s Omega0 (x' + x^n)/2 dt (Sec. 2.2)
            if (frame_sheared(FRAME)) {
                // the effective velocity u'/gamma' + v_s e_y (eq. OAx) can exceed c for
                // relativistic particles (Sec. 2.1): counted, not corrected.  With
                // |u'|^2/gamma'^2 = 1 - 1/gamma'^2, |v|^2 > 1 reads vs (2 u'_y/gamma' + vs) > 1/gamma'^2.
                if (P.count_sl) nsl += (vs * fmaf(2.f * u.y, ig, vs) > ig * ig) ? 1u : 0u;
            }
            int dcx, dcy, dcz = 0;
            const float nox = renorm(__fadd_rn(ox, D.x), dcx);
            float noy = renorm(__fadd_rn(oy, dyt), dcy);
            const float noz = DIM == 3 ? renorm(__fadd_rn(oz, D.z), dcz) : 0.f;
            int ncx = cx + dcx, ncy = cy + dcy, ncz = cz + dcz;
            const bool xwrap = ncx >= nx || ncx < 0;
            if (xwrap) {
                // shearing-periodic x (Sec. 2.1): leaving through x_o re-enters at x_i with
                // y + Delta y_s(t^{n+1}); leaving through x_i re-enters at x_o with y - Delta y_s
                const bool out = ncx >= nx;
                ncx += out ? -nx : nx;
                if (frame_sheared(FRAME)) {
                    int d2;
                    noy = renorm(__fadd_rn(noy, out ? P.dys_frac : -P.dys_frac), d2);
                    // ncy in [-1, ny], dys_int in [0, ny): the sum lies in (-ny-2, 2ny+1)
                    ncy += (out ? P.dys_int : -P.dys_int) + d2;
                    if (ncy >= ny) ncy -= ny;
                    if (ncy < 0) ncy += ny;
                }
            }
            if (ncy >= ny) ncy -= ny;
            if (ncy < 0) ncy += ny;
            if (DIM == 3) {
                if (ncz >= nz) ncz -= nz;
                if (ncz < 0) ncz += nz;
            }
            int32_t ncell = P.cc.encode(ncx, ncy, ncz);

            // ---- leaky box (Sec. 4.1); in the shearing and expanding frames on request, with the
            // displacement D of the deposit: comoving (relative to the shear flow), or primed
            if (FRAME == kLeaky || (FRAME != kPlain && P.escape)) {
                if (FRAME != kLeaky) p.load_escape(P, S, src);
                const uint32_t pid = p.id;
                if (P.leaky_mode == 0) {
                    // the z displacement is tracked only for the 3-vector test
                    float rx = p.dr[0] + D.x, ry = p.dr[1] + D.y;
                    float rz = 0.f;
                    float m = fmaxf(fabsf(rx), fabsf(ry));
                    if (P.use_3vec) {
                        rz = p.dr[2] + D.z;
                        m = fmaxf(m, fabsf(rz));
                    }
                    if (m >= P.l_esc) {
                        uint32_t w[4] = {pid, P.step_lo, 1u, P.box_id};
                        philox4x32_10(w, P.key0, P.key1);
                        // inverse CDF of |u| (bulk bins linear in p, top bin linear in -log2(1-p))
                        const uint32_t bin = w[0] >> 20, rr = w[0] & 0xFFFFFu;
                        float um;
                        if (bin < (uint32_t)(kMjBins - 1)) {
                            const float fr = (float)rr * (1.f / 1048576.f);
                            um = P.mj[bin] + fr * (P.mj[bin + 1] - P.mj[bin]);
                        } else {
                            const float sv = 20.f - log2f((float)(0x100000u - rr));
                            const float xk = sv * ((float)kMjTail / 20.f);
                            int k = (int)xk;
                            k = k > kMjTail - 1 ? kMjTail - 1 : k;
                            const float fr = xk - (float)k;
                            const float* T = P.mj + kMjBins - 1;
                            um = T[k] + fr * (T[k + 1] - T[k]);
                        }
                        const float mu = 2.f * ((float)(w[1] >> 8) * (1.f / 16777216.f)) - 1.f;
                        const float phi = 6.283185307179586f * ((float)(w[2] >> 8) * (1.f / 16777216.f));
                        float sp, cp;
                        sincosf(phi, &sp, &cp);
                        const float st = sqrtf(fmaxf(0.f, 1.f - mu * mu));
                        u = mk(um * st * cp, um * st * sp, um * mu);
                        rx = ry = rz = 0.f;
                    }
                    st_at(S.dr_out[0], so, rx);
                    st_at(S.dr_out[1], so, ry);
                    if (P.use_3vec) st_at(S.dr_out[2], so, rz);
                } else {
                    const double g2m1 = ((double)u.x * (double)u.x + (double)u.y * (double)u.y) +
                                        (double)u.z * (double)u.z;
                    if (g2m1 > P.g2thr) {
                        uint32_t w[4] = {pid, P.step_lo, 0u, P.box_id};
                        philox4x32_10(w, P.key0, P.key1);
                        if (w[0] < P.esc_thr) {
                            ncell = -1;
                            nesc++;
                        }
                    }
                }
            }

            if (P.count_mig) {
                // direction of the new tile from this one.  Whole tiles: the cell step r + dc in
                // [-1, edge] shifted right by log2(edge) is -1, 0 or +1, periodic wraps included;
                // one tile on an axis means 0.  A shearing-box x-face crossing moves in y by the
                // push's Delta y_s: its y step is taken from the face's centre.
                int d;
                if (P.mg.general) {
                    d = mig_dir(P.mg, t0[0] >> P.tl.lt[0], tsy, t0[2] >> P.tl.lt[2], mco, mci, ncx, ncy, ncz);
                } else {
                    const int dx = ((rx + dcx) >> P.tl.lt[0]) & P.mg.many[0];
                    int dy = ((ry + dcy) >> P.tl.lt[1]) & P.mg.many[1];
                    const int dz = DIM == 2 ? 0 : ((rz + dcz) >> P.tl.lt[2]) & P.mg.many[2];
                    if (frame_sheared(FRAME) && xwrap && P.mg.nt[1] > 1)
                        dy = ring_step((ncy >> P.tl.lt[1]) - (dx > 0 ? mco : mci), P.mg.nt[1]);
                    d = dy == 2 ? -1 : (dx + 1) + 3 * (dy + 1) + 9 * (dz + 1);
                    // the caller moved the particle since the sort: any number of tiles away
                    if (!in_tile && ((unsigned)(dx + 1) > 2u || (unsigned)(dy + 1) > 2u || (unsigned)(dz + 1) > 2u)) d = -1;
                }
                if (ncell < 0) d = kMigDead;
                // the particles that stay in the tile (the common direction) are not counted: the
                // sort takes them as the tile's particles less all the others
                if (d != kMigStay) {
                    if (d >= 0)
                        atomicAdd(&mc[s * kMigDirs + d], 1u);
                    else
                        far = true;
                }
            }
            st_at(S.cell_out, so, ncell);
            st_at(S.off_out[0], so, nox);
            st_at(S.off_out[1], so, noy);
            if (DIM == 3) st_at(S.off_out[2], so, noz);
            st_at(S.u_out[0], so, u.x);
            st_at(S.u_out[1], so, u.y);
            st_at(S.u_out[2], so, u.z);
            if (P.track_ids) st_at(S.id_out, so, FRAME == kLeaky ? p.id : ld_at(S.id_in, src));

            src = src_next;
            p.load(P, S, src);
            src_next = (uint32_t)ld_at(S.perm, slot_of(v + 2 * stride));

            // ---- deposit xn -> xn + D
            if (fuse) {
                const Shape SX = shape(ox, D.x), SY = shape(oy, D.y), SZ = shape(oz, D.z);
                if (in_tile) {
                    LdsAcc<G, DIM> acc = lds_acc<G, DIM>(Jl, rx, ry, rz);
                    esirkepov<DIM>(acc, SX, SY, SZ, S.q_dt * P.jscale, D.z);
                } else {
                    GlobalAcc acc = global_acc(P, cx, cy, DIM == 3 ? cz : 0);
                    esirkepov<DIM>(acc, SX, SY, SZ, S.q_dt, D.z);
                }
            } else {
                st_at(S.ws_cell, so, P.cc.encode(cx, cy, cz));
                st_at(S.ws_off[0], so, ox);
                st_at(S.ws_off[1], so, oy);
                if (DIM == 3) st_at(S.ws_off[2], so, oz);
                st_at(S.ws_disp[0], so, D.x);
                st_at(S.ws_disp[1], so, D.y);
                st_at(S.ws_disp[2], so, D.z);
            }
        }
        if (FRAME == kLeaky || (FRAME != kPlain && P.escape)) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) nesc += __shfl_xor(nesc, o, 64);
            if ((tid & 63) == 0 && nesc) atomicAdd(&P.ctr[1], (unsigned long long)nesc);
        }
        if (frame_sheared(FRAME) && P.count_sl) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) nsl += __shfl_xor(nsl, o, 64);
            if ((tid & 63) == 0 && nsl) atomicAdd(&P.ctr[3], (unsigned long long)nsl);
        }
        if (P.count_mig) {
            if (far) {
                *P.mfb[s] = 1;
                if (P.mig_latch) latch(P.err, kErrSort);
            }
        }
    }

    if (!fuse && !P.count_mig) return;
    __syncthreads();
    if (P.count_mig && tid < P.nsp * kMigDirs) {
        const int s = tid / kMigDirs, d = tid - s * kMigDirs;
        uint32_t* const cnt = &P.mcnt[s][(size_t)tile * kMigDirs + d];
        if (P.lsplit == 0)
            *cnt = mc[tid];
        else if (mc[tid])
            atomicAdd(cnt, mc[tid]);
    }
    if (fuse) flush_current<G, DIM, NT>(Jl, P, tile, t0, ext, tid, mc);
}

// Register budgets: 3D for the 6 waves per SIMD of two 12-wave workgroups a CU; 2D tiles of 8x8 (7 KB of
// LDS) fit eight waves per SIMD in 64 VGPRs, tiles of 16x16 (23 KB) seven in 72.
template <int DIM, int TX, int TY, int TZ, int FRAME, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(DIM == 3 ? 6 : (TX == 8 ? 8 : 7))))
void gpd_kernel(StepDev P, int fuse)
{
    gpd_body<DIM, TX, TY, TZ, FRAME, NT>(P, (int)blockIdx.x, (int)gridDim.x, fuse);
}

// Many boxes in one launch: the blocks of unit u (one box's tiles) take its descriptor.
template <int DIM, int TX, int TY, int TZ, int FRAME, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(DIM == 3 ? 6 : (TX == 8 ? 8 : 7))))
void gpd_batch(const StepDev* __restrict__ t, UnitMap m)
{
    const int u = unit_of(m, (int)blockIdx.x);
    gpd_body<DIM, TX, TY, TZ, FRAME, NT>(t[u], (int)blockIdx.x - (int)m.prefix[u],
                                         (int)(m.prefix[u + 1] - m.prefix[u]), 1);
}

// Unfused deposit: the same Esirkepov tile accumulation from the positions and deposit
// displacements saved by an unfused push (in sorted slot order).
template <int DIM, int TX, int TY, int TZ, int NT>
__global__ __launch_bounds__(NT) void deposit_kernel(StepDev P)
{
    using G = Geo<DIM, TX, TY, TZ>;
    __shared__ unsigned long long Jl[G::JTOT];
    __shared__ uint32_t flag;
    const int unit = xcd_contiguous(blockIdx.x, gridDim.x);
    const Share share(P, unit);
    const int tile = share.tile;
    int t0[3], ext[3];
    tile_origin<DIM>(P, tile, t0, ext);
    const int tid = threadIdx.x;
    for (int e = tid; e < G::JTOT; e += NT) Jl[e] = 0ull;
    __syncthreads();
    for (int s = share.s0; s < share.s1; s++) {
        const SpeciesDev& S = P.sp[s];
        const uint32_t beg = (uint32_t)S.toff[tile], end = (uint32_t)S.toff[tile + 1];
        for (uint32_t slot = beg + share.part * NT + tid; slot < end; slot += (uint32_t)NT << share.lparts) {
            int cx, cy, cz;
            P.cc.decode(ld_at(S.ws_cell, slot), cx, cy, cz);
            const float ox = ld_at(S.ws_off[0], slot), oy = ld_at(S.ws_off[1], slot);
            const float oz = DIM == 3 ? ld_at(S.ws_off[2], slot) : 0.f;
            const f3 D = mk(ld_at(S.ws_disp[0], slot), ld_at(S.ws_disp[1], slot),
                            ld_at(S.ws_disp[2], slot));
            const int rx = cx - t0[0], ry = cy - t0[1], rz = DIM == 3 ? cz - t0[2] : 0;
            const bool in_tile = (unsigned)rx < (unsigned)ext[0] && (unsigned)ry < (unsigned)ext[1] &&
                                 (DIM == 2 || (unsigned)rz < (unsigned)ext[2]);
            const Shape SX = shape(ox, D.x), SY = shape(oy, D.y), SZ = shape(oz, D.z);
            if (in_tile) {
                LdsAcc<G, DIM> acc = lds_acc<G, DIM>(Jl, rx, ry, rz);
                esirkepov<DIM>(acc, SX, SY, SZ, S.q_dt * P.jscale, D.z);
            } else {
                GlobalAcc acc = global_acc(P, cx, cy, DIM == 3 ? cz : 0);
                esirkepov<DIM>(acc, SX, SY, SZ, S.q_dt, D.z);
            }
        }
    }
    __syncthreads();
    flush_current<G, DIM, NT>(Jl, P, tile, t0, ext, tid, &flag);
}

// ------------------------------------------------------------------ launchers
// Threads per workgroup: the paired field regions leave LDS for two workgroups a CU at 8^3 tiles (72 KB each;
// three of 48 KB before), and twelve waves in each keep the CU's 24; the larger 2D tiles have as many more
// threads as cells.  Ten waves did not pair up on the four SIMDs (push at 256^3 7.8 ms against 6.1), eight
// with more registers were slower too (6.3).
constexpr int threads_for(int dim, int cells)
{
    return dim == 3 ? (cells == 512 ? 768 : 512) : (cells <= 256 ? 256 : cells);
}

// A tile's workgroup walks its particles a round of NT slots after another, each round waiting for
// its loads (3 to 5 us), so a box of few tiles is bound by that chain on an idle chip.  Its tiles are
// split as long as the launch has fewer workgroups than split_below, a part more than a round of a species (four
// from a workgroup a CU on: 320^2 with 4 particles a cell and species takes 31.5 us so and 35.0 in parts of one), and
// the workgroups are all resident at once (ragged tiles counted by their cells: a step of 17 x 199 x 14 cells, 150
// tiles, takes 210 us in 600 workgroups and 232 in 300); beyond that only parts of more than sixteen rounds.  Where the
// parts still leave the chip idle, one of two species each halves the chain again.  The push with its clears,
// us, whole / split: 64^2 with 16 particles a cell and species 66 / 21 (tiles of 8 x 8 29 / 19), 20 x 12 x 16 with 4
// 35 / 25, 24^3 with 8 52 / 29, 384^2 with 32 166 / 142; not resident at once: 48^3 with 8 60 / 86 (432 workgroups
// 65), 512^2 with 32 in tiles of 32 x 32 210 / 259, but 56^3 with 32 291 / 257; the species apart: 20 x 12 x 16 31 -> 25.
static int64_t split_below(int dim, const int t[3])  // 2 (3D, 32 x 16), 4 (to 16 x 16) or 1 (32 x 32) workgroups a CU
{
    const int cells = t[0] * t[1] * t[2];
    return dim == 3 ? 512 : (cells <= 256 ? 1024 : 256 * (1024 / cells));
}
void split_tiles(StepDev& P, const int t[3], int64_t n_tiles, int64_t whole_tiles, int64_t slots_per_tile)
{
    const int cells = t[0] * t[1] * t[2];
    const int64_t want = split_below(P.dim, t), nt = threads_for(P.dim, cells);
    const int64_t resident = P.dim == 2 && cells <= 256 ? 7 * 256 : want;
    P.lsplit = 0;
    auto more = [&] {
        return (n_tiles << P.lsplit) < want &&
               ((whole_tiles << (P.lsplit + 1)) <= resident || (slots_per_tile >> P.lsplit) > 16 * nt);
    };
    auto rounds = [&] { return (n_tiles << P.lsplit) < 256 ? 1 : 4; };
    while (P.lsplit < 6 && (slots_per_tile >> P.lsplit) > rounds() * nt && more()) P.lsplit++;
    P.by_species = P.nsp == 2 && more() ? 1 : 0;
    P.lsplit += P.by_species;
}

// words of P.tsum: a launch has at least the box's tiles, so a box of more is never split
int64_t split_words(int dim, const int t[3], int64_t n_tiles)
{
    if (n_tiles >= split_below(dim, t)) return 0;
    if (dim == 3) return n_tiles * (t[0] == 8 ? Geo<3, 8, 8, 8>::JSPLIT : Geo<3, 4, 4, 4>::JSPLIT);
    if (t[0] == 16) return n_tiles * Geo<2, 16, 16, 1>::JSPLIT;
    if (t[0] == 8) return n_tiles * Geo<2, 8, 8, 1>::JSPLIT;
    return n_tiles * (t[1] == 16 ? Geo<2, 32, 16, 1>::JSPLIT : Geo<2, 32, 32, 1>::JSPLIT);
}

template <int DIM, int TX, int TY, int TZ>
static hipError_t launch_shape(const StepDev& P, int fuse, hipStream_t st)
{
    constexpr int NT = threads_for(DIM, TX * TY * TZ);
    const dim3 grid((unsigned)P.tl.n_tiles << P.lsplit), block(NT);
    switch (P.frame) {
    case kShear:
        gpd_kernel<DIM, TX, TY, TZ, kShear, NT><<<grid, block, 0, st>>>(P, fuse);
        break;
    case kExpand:
        gpd_kernel<DIM, TX, TY, TZ, kExpand, NT><<<grid, block, 0, st>>>(P, fuse);
        break;
    case kLeaky:
        gpd_kernel<DIM, TX, TY, TZ, kLeaky, NT><<<grid, block, 0, st>>>(P, fuse);
        break;
    case kShearExpand:
        gpd_kernel<DIM, TX, TY, TZ, kShearExpand, NT><<<grid, block, 0, st>>>(P, fuse);
        break;
    default:
        gpd_kernel<DIM, TX, TY, TZ, kPlain, NT><<<grid, block, 0, st>>>(P, fuse);
        break;
    }
    return hipGetLastError();
}

template <int DIM, int TX, int TY, int TZ>
static hipError_t launch_dep_shape(const StepDev& P, hipStream_t st)
{
    constexpr int NT = threads_for(DIM, TX * TY * TZ);
    deposit_kernel<DIM, TX, TY, TZ, NT><<<dim3((unsigned)P.tl.n_tiles << P.lsplit), dim3(NT), 0, st>>>(P);
    return hipGetLastError();
}

// Tile shapes (edges in cells) with an instantiated fused kernel, and the subset the batched
// launch supports.  Returns the number of shapes written (at most max).
int tile_candidates(int dim, bool batched, int (*out)[3], int max)
{
    static const int k3[][3] = {{8, 8, 8}, {4, 4, 4}};
    static const int k2[][3] = {{16, 16, 1}, {8, 8, 1}, {32, 16, 1}, {32, 32, 1}};
    const int (*list)[3] = dim == 3 ? k3 : k2;
    const int n = dim == 3 ? (batched ? 1 : 2) : (batched ? 2 : 4);
    int w = 0;
    for (int i = 0; i < n && w < max; i++, w++)
        for (int k = 0; k < 3; k++) out[w][k] = list[i][k];
    return w;
}

static bool in_candidates(int dim, bool batched, const int t[3])
{
    int c[8][3];
    const int n = tile_candidates(dim, batched, c, 8);
    for (int i = 0; i < n; i++)
        if (c[i][0] == t[0] && c[i][1] == t[1] && c[i][2] == t[2]) return true;
    return false;
}

bool tile_shape_supported(int dim, const int t[3]) { return in_candidates(dim, false, t); }

template <int DIM, int TX, int TY, int TZ>
static hipError_t launch_batch_shape(const StepDev* table, UnitMap m, int blocks, int frame,
                                     hipStream_t st)
{
    constexpr int NT = threads_for(DIM, TX * TY * TZ);
    switch (frame) {
    case kShear: gpd_batch<DIM, TX, TY, TZ, kShear, NT><<<blocks, NT, 0, st>>>(table, m); break;
    case kExpand: gpd_batch<DIM, TX, TY, TZ, kExpand, NT><<<blocks, NT, 0, st>>>(table, m); break;
    case kShearExpand: gpd_batch<DIM, TX, TY, TZ, kShearExpand, NT><<<blocks, NT, 0, st>>>(table, m); break;
    case kLeaky: gpd_batch<DIM, TX, TY, TZ, kLeaky, NT><<<blocks, NT, 0, st>>>(table, m); break;
    default: gpd_batch<DIM, TX, TY, TZ, kPlain, NT><<<blocks, NT, 0, st>>>(table, m); break;
    }
    return hipGetLastError();
}

bool batch_tile_supported(int dim, const int t[3]) { return in_candidates(dim, true, t); }

hipError_t launch_gather_push_batch(const StepDev* table, UnitMap m, int blocks, int dim,
                                    const int t[3], int frame, hipStream_t st)
{
    if (blocks <= 0) return hipSuccess;
    if (dim == 3) return launch_batch_shape<3, 8, 8, 8>(table, m, blocks, frame, st);
    if (t[0] == 16) return launch_batch_shape<2, 16, 16, 1>(table, m, blocks, frame, st);
    return launch_batch_shape<2, 8, 8, 1>(table, m, blocks, frame, st);
}

hipError_t launch_gather_push(const StepDev& P, const int t[3], int fuse, hipStream_t st)
{
    if (P.dim == 3) {
        if (t[0] == 8) return launch_shape<3, 8, 8, 8>(P, fuse, st);
        return launch_shape<3, 4, 4, 4>(P, fuse, st);
    }
    if (t[0] == 16) return launch_shape<2, 16, 16, 1>(P, fuse, st);
    if (t[0] == 8) return launch_shape<2, 8, 8, 1>(P, fuse, st);
    if (t[1] == 16) return launch_shape<2, 32, 16, 1>(P, fuse, st);
    return launch_shape<2, 32, 32, 1>(P, fuse, st);
}

hipError_t launch_deposit(const StepDev& P, const int t[3], hipStream_t st)
{
    if (P.dim == 3) {
        if (t[0] == 8) return launch_dep_shape<3, 8, 8, 8>(P, st);
        return launch_dep_shape<3, 4, 4, 4>(P, st);
    }
    if (t[0] == 16) return launch_dep_shape<2, 16, 16, 1>(P, st);
    if (t[0] == 8) return launch_dep_shape<2, 8, 8, 1>(P, st);
    if (t[1] == 16) return launch_dep_shape<2, 32, 16, 1>(P, st);
    return launch_dep_shape<2, 32, 32, 1>(P, st);
}

}  // namespace pic

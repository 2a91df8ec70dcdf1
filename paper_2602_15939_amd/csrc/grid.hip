// grid.hip — grid kernels of the particle hot path (gfx950): guard fills with the
// shearing-periodic boundary (Sec. 2.1), the current fold with the J' transport along y
// (Sec. 2.2), the Maxwell steps of the three frames (Yee; Yee with the expanding-box scale
// factors of Sec. 3.2; implicit midpoint with upwinded advection solved by fixed-point
// iteration, Sec. 2.2) and the FP64 reductions.
//
// Every grid array carries kGuard guard cells on each side of each axis (z: none in 2D);
// pointers address the interior cell (0,0,0) and the x stride is 1.
#include "pic_internal.h"

namespace pic {

__device__ inline int64_t gidx(const GridDev& G, int x, int y, int z)
{
    return (int64_t)x + (int64_t)G.sy * y + (int64_t)G.sz * z;
}
// i mod n in [0, n); one add or subtract for i in [-n, 2n) (the indices here are within a
// period of the range), the remainder only beyond
__device__ inline int wrapn(int i, int n)
{
    if (i < 0) i += n;
    if (i >= n) i -= n;
    if ((unsigned)i >= (unsigned)n) {
        i %= n;
        if (i < 0) i += n;
    }
    return i;
}

// ------------------------------------------------------------------ guard fill
// Every guard cell takes its value from interior cells: y, z periodic; x periodic, or for the
// shearing box F(x_o + m, y) = F(x_i + m, y + dys) and F(x_i - m, y) = F(x_o - m, y - dys)
// with a fractional dys applied by linear interpolation along y.  No guard cell reads another one,
// so the slabs of the three axes are one launch.  The step fills guards once, at its end, for the
// push: the field kernels below read the periodic images themselves.

// the image of an x guard cell between the two interior values a (at y + js) and b (at
// y + js + 1), weight w on b; the guard fill and the 3D sweep's x halo share it
__device__ inline float shear_lerp(float a, float b, float w) { return fmaf(w, b, (1.f - w) * a); }

// y row offset js and weight w of the image of an x guard cell of the shearing box
// (hi: beyond x = nx - 1, lo: before x = 0): hi y + dys = y + dys_int + w,
// lo y - dys = y - dys_int - 1 + (1 - w)
__device__ inline void shear_image(bool hi, int dys_int, float dys_w, int& js, float& w)
{
    if (hi) {
        js = dys_int;
        w = dys_w;
    } else {
        js = -dys_int - (dys_w > 0.f ? 1 : 0);
        w = dys_w > 0.f ? 1.f - dys_w : 0.f;
    }
}

__device__ __attribute__((always_inline)) inline void fill_guards_body(const FillArgs& a, int blk, int, int c)
{
    const GridDev& G = a.G;
    const int shear = a.shear, dys_int = a.dys_int;
    const float dys_w = a.dys_w;
    float* F = a.A.p[c];
    // 32-bit index arithmetic: the x and y guard widths are kGuard, the other divisors are
    // invariant (precomputed multipliers)
    uint32_t t = (uint32_t)blk * kBlock + threadIdx.x;
    constexpr uint32_t g2 = 2 * kGuard;
    const int gz = G.g[2];
    const uint32_t NYg = (uint32_t)(G.n[1] + 2 * kGuard);
    int x, y, z;
    if (t < a.n[0]) {  // x guard slabs over the whole guarded y, z
        const uint32_t m = t % g2, r = t / g2;
        const uint32_t q = G.divyg.div(r);
        y = (int)(r - q * NYg) - kGuard;
        z = (int)q - gz;
        x = (int)m < kGuard ? (int)m - kGuard : G.n[0] + ((int)m - kGuard);
    } else if ((t -= a.n[0]) < a.n[1]) {  // y guard slabs over interior x, guarded z
        const uint32_t r = G.div0.div(t);
        x = (int)(t - r * (uint32_t)G.n[0]);
        const uint32_t m = r % g2;
        z = (int)(r / g2) - gz;
        y = (int)m < kGuard ? (int)m - kGuard : G.n[1] + ((int)m - kGuard);
    } else {  // z guard slabs over interior x, y
        if ((t -= a.n[1]) >= a.n[2]) return;
        const uint32_t r = G.div0.div(t);
        x = (int)(t - r * (uint32_t)G.n[0]);
        const uint32_t q = G.div1.div(r);
        y = (int)(r - q * (uint32_t)G.n[1]);
        const int m = (int)q;
        z = m < gz ? m - gz : G.n[2] + (m - gz);
    }
    const int sz_ = wrapn(z, G.n[2]);
    float v;
    if (x < 0 || x >= G.n[0]) {
        const bool hi = x >= G.n[0];
        const int sx = hi ? x - G.n[0] : x + G.n[0];
        if (shear) {
            int js;
            float w;
            shear_image(hi, dys_int, dys_w, js, w);
            const float a = F[gidx(G, sx, wrapn(y + js, G.n[1]), sz_)];
            const float b = F[gidx(G, sx, wrapn(y + js + 1, G.n[1]), sz_)];
            v = shear_lerp(a, b, w);
        } else {
            v = F[gidx(G, sx, wrapn(y, G.n[1]), sz_)];
        }
    } else {
        v = F[gidx(G, x, wrapn(y, G.n[1]), sz_)];
    }
    F[gidx(G, x, y, z)] = v;
}
PIC_BATCHED_KERNEL(fill_guards, FillArgs, kBlock)

// ------------------------------------------------------------------ current fold

// interior coordinates of linear interior index t = x + n0 (y + n1 z) (below 2^31)
__device__ inline void cell_of(const GridDev& G, int64_t t, int& x, int& y, int& z)
{
    const uint32_t u = (uint32_t)t;
    const uint32_t r = G.div0.div(u);
    x = (int)(u - r * (uint32_t)G.n[0]);
    const uint32_t zz = G.div1.div(r);
    y = (int)(r - zz * (uint32_t)G.n[1]);
    z = (int)zz;
}

// J' at guarded column xg moved along y by v_s(xg) dt/2 (Sec. 2.2), v_s taken at the
// component's staggered x: first-order upwind, i.e. linear interpolation between rows; N rows from y on
template <int N>
__device__ inline void shear_transport(const GridDev& G, const float* __restrict__ F, int c, int xg, int y, int z,
                                       float sO_hdt, float half_nx, float out[N])
{
    const float xc = (float)xg + (c == 0 ? 0.5f : 0.f) - half_nx;
    const float d = -sO_hdt * xc;
    const float fl = floorf(d);
    const int m = (int)fl;
    const float w = d - fl;
    float f[N + 1];
#pragma unroll
    for (int k = 0; k <= N; k++) f[k] = F[gidx(G, xg, wrapn(y + k - m - 1, G.n[1]), z)];
#pragma unroll
    for (int k = 0; k < N; k++) out[k] = fmaf(1.f - w, f[k + 1], w * f[k]);
}
// The transport and the shearing-periodic x fold in one pass (out-of-place): an interior cell
// takes its own transported value plus, on the first and last g columns, the transported
// guard column of the other face at the y shift of the shearing-periodic map (the exact
// transpose of the field guard fill's interpolation).  A thread takes kFoldRows cells along y, each row of
// which is read once for two of them, with all loads in flight together:
// 256^3 216 -> 114 us beside the sort, 150 x 90 x 84 cells 20.5 -> 11.2 us, 96^3 17.9 -> 9.4 us (a cell a thread before).
constexpr int kFoldRows = 4;
__device__ __attribute__((always_inline)) inline void shear_fold_cells(const ShearFoldArgs& a, int x, int y0, int z, int c)
{
    constexpr int N = kFoldRows;
    const GridDev& G = a.G;
    const int nx = G.n[0], ny = G.n[1], ga = G.g[0];
    const float* F = a.in.p[c];
    float v[N];
    shear_transport<N>(G, F, c, x, y0, z, a.sO_hdt, a.half_nx, v);
    if (x < ga) {  // guard column x + nx, the image of (x, y + dys)
        float t[N + 1];
        shear_transport<N + 1>(G, F, c, x + nx, y0 - a.dys_int - 1, z, a.sO_hdt, a.half_nx, t);
#pragma unroll
        for (int k = 0; k < N; k++) v[k] += fmaf(1.f - a.dys_w, t[k + 1], a.dys_w * t[k]);
    }
    if (x >= nx - ga) {  // guard column x - nx, the image of (x, y - dys)
        // shift -dys = js + w with js = -dys_int - 1, w = 1 - dys_w (dys_w > 0), else -dys_int
        int js = -a.dys_int;
        float w = 0.f;
        if (a.dys_w > 0.f) {
            js = -a.dys_int - 1;
            w = 1.f - a.dys_w;
        }
        float t[N + 1];
        shear_transport<N + 1>(G, F, c, x - nx, y0 - js - 1, z, a.sO_hdt, a.half_nx, t);
#pragma unroll
        for (int k = 0; k < N; k++) v[k] += fmaf(1.f - w, t[k + 1], w * t[k]);
    }
    float* out = a.out.p[c] + gidx(G, x, y0, z);
#pragma unroll
    for (int k = 0; k < N; k++)
        if (y0 + k < ny) out[(int64_t)G.sy * k] = v[k];
}
// grid-stride over the threads' cells (the batched launch gives each its own thread)
__device__ __attribute__((always_inline)) inline void shear_fold_body(const ShearFoldArgs& a, int blk, int nblk, int c)
{
    const uint32_t nx = (uint32_t)a.G.n[0], rows = (uint32_t)(a.G.n[1] + kFoldRows - 1) / kFoldRows;
    const int64_t n = (int64_t)nx * rows * a.G.n[2];
    for (int64_t t = (int64_t)blk * kBlock + threadIdx.x; t < n; t += (int64_t)nblk * kBlock) {
        const uint32_t u = (uint32_t)t, r = a.G.div0.div(u), z = r / rows;
        shear_fold_cells(a, (int)(u - r * nx), (int)(r - z * rows) * kFoldRows, (int)z, c);
    }
}
PIC_BATCHED_KERNEL(shear_fold, ShearFoldArgs, kBlock)

// Periodic fold in place: the cells of the first and last two layers of each axis take the guard
// cells that map onto them, in the order z, y, x.  A cell reads guards and itself and writes itself,
// so the axes are one launch (two and three before).  With the x fold the cells are the interior's;
// without it (the shearing box folds x with its transport) those of every guarded column.
// An axis has at most one image of a cell (it has four cells or more): all images are loaded at
// once, those that a cell has not at its own place, and the sums selected.
__device__ __attribute__((always_inline)) inline void fold_periodic_body(const FoldPArgs& a, int blk, int, int c)
{
    const GridDev& G = a.G;
    float* F = a.J.p[c];
    constexpr uint32_t g2 = 2 * kGuard;
    const int nx = G.n[0], ny = G.n[1], nz = G.n[2];
    uint32_t t = (uint32_t)blk * kBlock + threadIdx.x;
    auto layer = [](uint32_t m, int n) { return m < kGuard ? (int)m : n - (int)g2 + (int)m; };
    int x, y, z = 0;
    if (t < a.n[0]) {  // x layers: every y, z
        const uint32_t r = t / g2;
        x = layer(t % g2, nx);
        z = (int)G.div1.div(r);
        y = (int)(r - (uint32_t)z * (uint32_t)ny);
    } else {
        t -= a.n[0];
        const bool yl = t < a.n[1];
        if (!yl && (t -= a.n[1]) >= a.n[2]) return;
        const uint32_t r = t / a.wx;
        x = a.x0 + (int)(t - r * a.wx);
        if (yl) {
            y = layer(r % g2, ny);
            z = (int)(r / g2);
        } else {
            const uint32_t iny = (uint32_t)(ny - (int)g2), q = r / iny;
            y = kGuard + (int)(r - q * iny);
            z = layer(q, nz);
        }
    }
    auto image = [](int i, int n, int s) -> int64_t {
        return i < kGuard ? (int64_t)n * s : (i >= n - kGuard ? -(int64_t)n * s : 0);
    };
    const int64_t i = gidx(G, x, y, z), iy = image(y, ny, G.sy);
    const int64_t ix = a.n[0] ? image(x, nx, 1) : 0, iz = G.dim == 3 ? image(z, nz, G.sz) : 0;
    float v[2][2];
#pragma unroll
    for (int k = 0; k < 2; k++)
#pragma unroll
        for (int j = 0; j < 2; j++) {
            const float* p = F + i + (k ? ix : 0) + (j ? iy : 0);
            const float own = p[0], img = p[iz];
            v[k][j] = iz ? own + img : own;
        }
    const float v0 = iy ? v[0][0] + v[0][1] : v[0][0], v1 = iy ? v[1][0] + v[1][1] : v[1][0];
    F[i] = ix ? v0 + v1 : v0;
}
PIC_BATCHED_KERNEL(fold_periodic, FoldPArgs, kBlock)

// ------------------------------------------------------------------ Maxwell
// Yee curls (c = 1, dx = 1).  E_j and B_j enter multiplied by ge[j], gb[j] (the l_j of the
// expanding box, 1 otherwise).  Neighbours beyond a face are read at their periodic images, so the
// three updates of a step need no guard fill between them.

// element offsets from a cell to its periodic neighbour one up (or down) along an axis
__device__ inline int step_up(int i, int n, int s) { return i + 1 == n ? -(n - 1) * s : s; }
__device__ inline int step_down(int i, int n, int s) { return i == 0 ? (n - 1) * s : -s; }

// B_i <- fout_i (fin_i B_i - dt/2 curl(g E)_i)
__device__ __attribute__((always_inline)) inline void yee_b_cell(const MaxwellDev& M, int64_t t)
{
    const GridDev& G = M.G;
    int x, y, z;
    cell_of(G, t, x, y, z);
    const int64_t i = gidx(G, x, y, z);
    const bool d3 = G.dim == 3;
    const int sx = step_up(x, G.n[0], 1), sy = step_up(y, G.n[1], G.sy);
    const int sz = d3 ? step_up(z, G.n[2], G.sz) : 0;
    const float* Ex = M.E[0];
    const float* Ey = M.E[1];
    const float* Ez = M.E[2];
    const float g0 = M.gf[0], g1 = M.gf[1], g2 = M.gf[2];
    const float cx = g2 * (Ez[i + sy] - Ez[i]) - (d3 ? g1 * (Ey[i + sz] - Ey[i]) : 0.f);
    const float cy = (d3 ? g0 * (Ex[i + sz] - Ex[i]) : 0.f) - g2 * (Ez[i + sx] - Ez[i]);
    const float cz = g1 * (Ey[i + sx] - Ey[i]) - g0 * (Ex[i + sy] - Ex[i]);
    const float h = 0.5f * M.dt;
    M.B[0][i] = M.fout[0] * (M.fin[0] * M.B[0][i] - h * cx);
    M.B[1][i] = M.fout[1] * (M.fin[1] * M.B[1][i] - h * cy);
    M.B[2][i] = M.fout[2] * (M.fin[2] * M.B[2][i] - h * cz);
}
// grid-stride over the cells (the batched launch gives every cell its own thread)
__device__ __attribute__((always_inline)) inline void yee_b_body(const MaxwellDev& M, int blk, int nblk, int)
{
    const int64_t n = (int64_t)M.G.n[0] * M.G.n[1] * M.G.n[2];
    for (int64_t t = (int64_t)xcd_contiguous(blk, nblk) * kBlock + threadIdx.x; t < n; t += (int64_t)nblk * kBlock) yee_b_cell(M, t);
}
PIC_BATCHED_KERNEL(yee_b, MaxwellDev, kBlock)

// E_i <- fout_i (fin_i E_i + dt curl(g B)_i - 4 pi dt J_i)
__device__ __attribute__((always_inline)) inline void yee_e_cell(const MaxwellDev& M, int64_t t)
{
    const GridDev& G = M.G;
    int x, y, z;
    cell_of(G, t, x, y, z);
    const int64_t i = gidx(G, x, y, z);
    const bool d3 = G.dim == 3;
    const int sx = step_down(x, G.n[0], 1), sy = step_down(y, G.n[1], G.sy);
    const int sz = d3 ? step_down(z, G.n[2], G.sz) : 0;
    const float* Bx = M.B[0];
    const float* By = M.B[1];
    const float* Bz = M.B[2];
    const float g0 = M.gf[0], g1 = M.gf[1], g2 = M.gf[2];
    const float cx = g2 * (Bz[i] - Bz[i + sy]) - (d3 ? g1 * (By[i] - By[i + sz]) : 0.f);
    const float cy = (d3 ? g0 * (Bx[i] - Bx[i + sz]) : 0.f) - g2 * (Bz[i] - Bz[i + sx]);
    const float cz = g1 * (By[i] - By[i + sx]) - g0 * (Bx[i] - Bx[i + sy]);
    const float fp = 4.f * 3.14159265358979f * M.dt;
    M.E[0][i] = M.fout[0] * (M.fin[0] * M.E[0][i] + M.dt * cx - fp * M.J[0][i]);
    M.E[1][i] = M.fout[1] * (M.fin[1] * M.E[1][i] + M.dt * cy - fp * M.J[1][i]);
    M.E[2][i] = M.fout[2] * (M.fin[2] * M.E[2][i] + M.dt * cz - fp * M.J[2][i]);
}
// grid-stride over the cells (the batched launch gives every cell its own thread)
__device__ __attribute__((always_inline)) inline void yee_e_body(const MaxwellDev& M, int blk, int nblk, int)
{
    const int64_t n = (int64_t)M.G.n[0] * M.G.n[1] * M.G.n[2];
    for (int64_t t = (int64_t)xcd_contiguous(blk, nblk) * kBlock + threadIdx.x; t < n; t += (int64_t)nblk * kBlock) yee_e_cell(M, t);
}
PIC_BATCHED_KERNEL(yee_e, MaxwellDev, kBlock)

// FP contraction inside one expression only in the shearing-box sweeps: every kernel that
// computes an iterate (one sweep per launch, two per pass, the face columns of a pass) then
// rounds it the same way, so the paths agree bit for bit.
#pragma clang fp contract(on)

// Shearing box, fixed-point sweeps of the implicit midpoint rule (Sec. 2.2):
//   F^{k+1} = F^n + dt RHS((F^n + F^k)/2, J'),
// RHS of eq. OAB / eq. OAE with v = -s Omega0 x:
//   dB/dt  = -curl E' - v dB/dy (upwind) - s Omega0 <Bx> e_y
//   dE'/dt = curl B - 4 pi J' + (+v dEx/dy, -v dEy/dy, +v dEz/dy) (upwind)
//            - v (dEy/dx, dEx/dx + dEz/dz, dEy/dz) (central, averaged onto the component).
// The field part L of RHS is linear (the upwind side depends only on the sign of v at the
// component), so with C = F^n + dt/2 L(F^n) - 4 pi dt J' (fixed during the step) every sweep is
//   F^{k+1} = C + dt/2 L(F^k).
// The first sweep (F^0 = F^n) also writes C.
//
// The stencil is written once against an accessor V(c, dx, dy, dz) of the iterate.
enum { BX = 0, BY, BZ, EX, EY, EZ };

template <bool D3, class Acc>
__device__ inline void ksb_operator(const Acc& V, float v0, float vh, float sO, float L[6])
{
    // curl E' at the B locations, curl B at the E locations
    const float cEx = (V(EZ, 0, 1, 0) - V(EZ, 0, 0, 0)) - (D3 ? V(EY, 0, 0, 1) - V(EY, 0, 0, 0) : 0.f);
    const float cEy = (D3 ? V(EX, 0, 0, 1) - V(EX, 0, 0, 0) : 0.f) - (V(EZ, 1, 0, 0) - V(EZ, 0, 0, 0));
    const float cEz = (V(EY, 1, 0, 0) - V(EY, 0, 0, 0)) - (V(EX, 0, 1, 0) - V(EX, 0, 0, 0));
    const float cBx = (V(BZ, 0, 0, 0) - V(BZ, 0, -1, 0)) - (D3 ? V(BY, 0, 0, 0) - V(BY, 0, 0, -1) : 0.f);
    const float cBy = (D3 ? V(BX, 0, 0, 0) - V(BX, 0, 0, -1) : 0.f) - (V(BZ, 0, 0, 0) - V(BZ, -1, 0, 0));
    const float cBz = (V(BY, 0, 0, 0) - V(BY, -1, 0, 0)) - (V(BX, 0, 0, 0) - V(BX, 0, -1, 0));
    const float bxa = 0.25f * (V(BX, 0, 0, 0) + V(BX, 1, 0, 0) + V(BX, 0, -1, 0) + V(BX, 1, -1, 0));
    const float dEy_dx = 0.5f * ((V(EY, 1, 0, 0) - V(EY, 0, 0, 0)) + (V(EY, 1, -1, 0) - V(EY, 0, -1, 0)));
    const float dEx_dx = 0.5f * ((V(EX, 0, 0, 0) - V(EX, -1, 0, 0)) + (V(EX, 0, 1, 0) - V(EX, -1, 1, 0)));
    const float dEz_dz =
        D3 ? 0.5f * ((V(EZ, 0, 0, 0) - V(EZ, 0, 0, -1)) + (V(EZ, 0, 1, 0) - V(EZ, 0, 1, -1))) : 0.f;
    const float dEy_dz =
        D3 ? 0.5f * ((V(EY, 0, 0, 1) - V(EY, 0, 0, 0)) + (V(EY, 0, -1, 1) - V(EY, 0, -1, 0))) : 0.f;
    // upwind difference along y for transport velocity w
    auto updy = [&](int c, float w) {
        return w > 0.f ? V(c, 0, 0, 0) - V(c, 0, -1, 0) : V(c, 0, 1, 0) - V(c, 0, 0, 0);
    };
    L[BX] = -cEx - v0 * updy(BX, v0);
    L[BY] = -cEy - vh * updy(BY, vh) - sO * bxa;
    L[BZ] = -cEz - vh * updy(BZ, vh);
    L[EX] = cBx + vh * updy(EX, -vh) - vh * dEy_dx;
    L[EY] = cBy - v0 * updy(EY, v0) - v0 * (dEx_dx + dEz_dz);
    L[EZ] = cBz + v0 * updy(EZ, -v0) - v0 * dEy_dz;
}

// The operator of the combined shearing and expanding frame (reading: the step of Sec. 2.2 on
// the expanding-frame fields of Sec. 3.1): the curls act on (1/l) L^2 F, i.e. d[c] F_c, as in
// eqs. EBB/EBE; the transport and tidal terms keep their form in the expanding coordinates (x
// and y scale together) except v dE'y/dz in dE'z/dt, which takes kz = (l_y/l_z)^2.
template <bool D3, class Acc>
__device__ inline void ksb_operator_f(const Acc& V, float v0, float vh, float sO, const float d[3],
                                      float kz, float L[6])
{
    const float cEx = d[2] * (V(EZ, 0, 1, 0) - V(EZ, 0, 0, 0)) - (D3 ? d[1] * (V(EY, 0, 0, 1) - V(EY, 0, 0, 0)) : 0.f);
    const float cEy = (D3 ? d[0] * (V(EX, 0, 0, 1) - V(EX, 0, 0, 0)) : 0.f) - d[2] * (V(EZ, 1, 0, 0) - V(EZ, 0, 0, 0));
    const float cEz = d[1] * (V(EY, 1, 0, 0) - V(EY, 0, 0, 0)) - d[0] * (V(EX, 0, 1, 0) - V(EX, 0, 0, 0));
    const float cBx = d[2] * (V(BZ, 0, 0, 0) - V(BZ, 0, -1, 0)) - (D3 ? d[1] * (V(BY, 0, 0, 0) - V(BY, 0, 0, -1)) : 0.f);
    const float cBy = (D3 ? d[0] * (V(BX, 0, 0, 0) - V(BX, 0, 0, -1)) : 0.f) - d[2] * (V(BZ, 0, 0, 0) - V(BZ, -1, 0, 0));
    const float cBz = d[1] * (V(BY, 0, 0, 0) - V(BY, -1, 0, 0)) - d[0] * (V(BX, 0, 0, 0) - V(BX, 0, -1, 0));
    const float bxa = 0.25f * (V(BX, 0, 0, 0) + V(BX, 1, 0, 0) + V(BX, 0, -1, 0) + V(BX, 1, -1, 0));
    const float dEy_dx = 0.5f * ((V(EY, 1, 0, 0) - V(EY, 0, 0, 0)) + (V(EY, 1, -1, 0) - V(EY, 0, -1, 0)));
    const float dEx_dx = 0.5f * ((V(EX, 0, 0, 0) - V(EX, -1, 0, 0)) + (V(EX, 0, 1, 0) - V(EX, -1, 1, 0)));
    const float dEz_dz =
        D3 ? 0.5f * ((V(EZ, 0, 0, 0) - V(EZ, 0, 0, -1)) + (V(EZ, 0, 1, 0) - V(EZ, 0, 1, -1))) : 0.f;
    const float dEy_dz =
        D3 ? 0.5f * ((V(EY, 0, 0, 1) - V(EY, 0, 0, 0)) + (V(EY, 0, -1, 1) - V(EY, 0, -1, 0))) : 0.f;
    auto updy = [&](int c, float w) {
        return w > 0.f ? V(c, 0, 0, 0) - V(c, 0, -1, 0) : V(c, 0, 1, 0) - V(c, 0, 0, 0);
    };
    L[BX] = -cEx - v0 * updy(BX, v0);
    L[BY] = -cEy - vh * updy(BY, vh) - sO * bxa;
    L[BZ] = -cEz - vh * updy(BZ, vh);
    L[EX] = cBx + vh * updy(EX, -vh) - vh * dEy_dx;
    L[EY] = cBy - v0 * updy(EY, v0) - v0 * (dEx_dx + dEz_dz);
    L[EZ] = cBz + v0 * updy(EZ, -v0) - v0 * (kz * dEy_dz);
}

// ---- tolerance mode of the sweeps
// a sweep's (largest change, largest value) pair meets the tolerance (a finite change only)
__device__ inline bool ksb_met(const uint32_t* pair, float tol)
{
    const float d = __uint_as_float(pair[0]);
    return d <= tol * __uint_as_float(pair[1]) && d <= 3.4028235e38f;
}
// the sweep before this one met the tolerance: uniform over the grid, tested before any work, by each
// wave for itself
__device__ inline bool ksb_skip(const KsbDev& K)
{
    if (!K.conv || K.k == 0) return false;
    const uint32_t* p = K.conv + kConvSweep * (K.k - 1) + kConvStride * (threadIdx.x % kConvSlots);
    uint32_t pair[2] = {p[0], p[1]};
    for (int o = kConvSlots / 2; o > 0; o >>= 1)
        for (int j = 0; j < 2; j++) pair[j] = max(pair[j], (uint32_t)__shfl_xor(pair[j], o, 64));
    return ksb_met(pair, K.tol);
}
// running maxima of |F^{k+1} - F^k| (NaN -> +inf) and |F^{k+1}|
__device__ inline void ksb_track(float fo, float fk, float& dm, float& fm)
{
    const float d = fabsf(fo - fk);
    dm = d == d ? fmaxf(dm, d) : __int_as_float(0x7f800000);
    fm = fmaxf(fm, fabsf(fo));
}
// workgroup maxima (NT threads, whole waves), one atomic pair per workgroup
template <int NT>
__device__ inline void ksb_reduce(float dm, float fm, uint32_t* sweep)
{
    __shared__ float red[2][NT / 64];
    for (int o = 32; o > 0; o >>= 1) {
        dm = fmaxf(dm, __shfl_xor(dm, o, 64));
        fm = fmaxf(fm, __shfl_xor(fm, o, 64));
    }
    const int w = threadIdx.x / 64;
    if (threadIdx.x % 64 == 0) {
        red[0][w] = dm;
        red[1][w] = fm;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int j = 1; j < NT / 64; j++) {
            dm = fmaxf(dm, red[0][j]);
            fm = fmaxf(fm, red[1][j]);
        }
        uint32_t* const p = sweep + kConvStride * (blockIdx.x % kConvSlots);
        atomicMax(p, __float_as_uint(dm));
        atomicMax(p + 1, __float_as_uint(fm));
    }
}

// output of one cell: FIRST writes C and F^1 from F^n, later sweeps F^{k+1} from C; Fk is
// the iterate at the cell (F^n for the first sweep)
template <bool FIRST>
__device__ inline void ksb_store(const KsbDev& K, int64_t i, const float L[6], const float Fk[6],
                                 float& dm, float& fm)
{
    const float h = 0.5f * K.dt;
    const float fpdt = 4.f * 3.14159265358979f * K.dt;
#pragma unroll
    for (int c = 0; c < 6; c++) {
        float Cv;
        if (FIRST) {
            Cv = Fk[c] + h * L[c];
            if (c >= EX) Cv -= fpdt * K.J[c - EX][i];
            K.C[c][i] = Cv;
        } else {
            Cv = K.C[c][i];
        }
        const float v = Cv + h * L[c];
        K.Fo[c][i] = v;
        ksb_track(v, Fk[c], dm, fm);
    }
}

// The values the operator reads at one cell, all loaded before the first is used: the upwind sides
// and the faces then select between registers, and the loads of a cell wait once.
struct KsbCell {
    float v[6][3][3][3];  // [component][dx + 1][dy + 1][dz + 1], the places the operator reads
    __device__ inline float operator()(int c, int dx, int dy, int dz) const { return v[c][dx + 1][dy + 1][dz + 1]; }
};

// y, z periodic; x shearing-periodic: the column beyond a face is interpolated between the rows
// y + dy + js and the next one of the other face's column, as the guard fill does
template <bool D3>
__device__ inline void ksb_load(const KsbDev& K, int x, int y, int z, int64_t i, KsbCell& V)
{
    const GridDev& G = K.G;
    const float* const* F = K.Fk;
    const int nx = G.n[0], ny = G.n[1];
    const int yu = step_up(y, ny, G.sy), yd = step_down(y, ny, G.sy);
    const int zu = D3 ? step_up(z, G.n[2], G.sz) : 0, zd = D3 ? step_down(z, G.n[2], G.sz) : 0;
    const bool lo = x == 0, face = lo || x == nx - 1;
    // elements at dx = +1 (dy = 0, -1) and dx = -1 (dy = 0, +1); r1: the second row of an image
    int64_t u0 = i + 1, um = i + 1 + yd, d0 = i - 1, dp = i - 1 + yu;
    int64_t r1[2] = {0, 0};
    float w = 0.f;
    if (face) {
        int js;
        shear_image(!lo, K.ydys_int, K.ydys_w, js, w);
        const int64_t col = gidx(G, lo ? nx - 1 : 0, 0, z);
        const int t = wrapn(y + js, ny);  // rows t - 1 .. t + 2 of the other face
        const int64_t c0 = col + (int64_t)G.sy * t, cu = c0 + step_up(t, ny, G.sy);
        if (lo) {
            d0 = c0;
            dp = r1[0] = cu;
            r1[1] = col + (int64_t)G.sy * wrapn(t + 2, ny);
        } else {
            u0 = r1[1] = c0;
            um = c0 + step_down(t, ny, G.sy);
            r1[0] = cu;
        }
    }
#pragma unroll
    for (int c = 0; c < 6; c++) {
        V.v[c][1][1][1] = F[c][i];
        V.v[c][1][2][1] = F[c][i + yu];
        V.v[c][1][0][1] = F[c][i + yd];
    }
    const float ezu = F[EZ][u0], eyu = F[EY][u0], bxu = F[BX][u0], eyum = F[EY][um], bxum = F[BX][um];
    const float bzd = F[BZ][d0], byd = F[BY][d0], exd = F[EX][d0], exdp = F[EX][dp];
    if (D3) {
        V.v[EY][1][1][2] = F[EY][i + zu];
        V.v[EX][1][1][2] = F[EX][i + zu];
        V.v[EY][1][0][2] = F[EY][i + yd + zu];
        V.v[BY][1][1][0] = F[BY][i + zd];
        V.v[BX][1][1][0] = F[BX][i + zd];
        V.v[EZ][1][1][0] = F[EZ][i + zd];
        V.v[EZ][1][2][0] = F[EZ][i + yu + zd];
    }
    float s[5] = {0.f, 0.f, 0.f, 0.f, 0.f};  // the images' second row values, one face's at a time
    if (face) {
        s[0] = lo ? F[BZ][r1[0]] : F[EZ][r1[0]];
        s[1] = lo ? F[BY][r1[0]] : F[EY][r1[0]];
        s[2] = lo ? F[EX][r1[0]] : F[BX][r1[0]];
        s[3] = lo ? F[EX][r1[1]] : F[EY][r1[1]];
        s[4] = lo ? 0.f : F[BX][r1[1]];
    }
    const bool hi = face && !lo;
    V.v[EZ][2][1][1] = hi ? shear_lerp(ezu, s[0], w) : ezu;
    V.v[EY][2][1][1] = hi ? shear_lerp(eyu, s[1], w) : eyu;
    V.v[BX][2][1][1] = hi ? shear_lerp(bxu, s[2], w) : bxu;
    V.v[EY][2][0][1] = hi ? shear_lerp(eyum, s[3], w) : eyum;
    V.v[BX][2][0][1] = hi ? shear_lerp(bxum, s[4], w) : bxum;
    V.v[BZ][0][1][1] = lo ? shear_lerp(bzd, s[0], w) : bzd;
    V.v[BY][0][1][1] = lo ? shear_lerp(byd, s[1], w) : byd;
    V.v[EX][0][1][1] = lo ? shear_lerp(exd, s[2], w) : exd;
    V.v[EX][0][2][1] = lo ? shear_lerp(exdp, s[3], w) : exdp;
}

// 2D (and any size): one thread per cell, neighbours straight from memory, beyond a face at their
// images, so that no guard fill runs between sweeps.  On small grids a step is bound by its launches
// (the fills were two of three in 2D): the 64^2 box replayed as a graph 201 -> 176 us a step, a
// 20 x 12 x 16 box stepped call by call 223 -> 155 us.  A separate branch for the cells at the x faces was
// slower than the fills (213 us on 64^2: every wave of a row has such a lane and ran both branches).
// An XCD takes a contiguous range of the cells, so that its L2 serves the rows above and below (on
// 150 x 90 x 84 cells 25.5 -> 18.4 us a sweep, on 96^3 17.6 -> 13.7 us).
template <bool FIRST>
__device__ __attribute__((always_inline)) inline void ksb_sweep_body(const KsbDev& K, int blk, int nblk, int)
{
    if (ksb_skip(K)) return;
    const GridDev& G = K.G;
    const int64_t t = (int64_t)xcd_contiguous(blk, nblk) * kBlock + threadIdx.x;
    float dm = 0.f, fm = 0.f;
    if (t < (int64_t)G.n[0] * G.n[1] * G.n[2]) {
        int x, y, z;
        cell_of(G, t, x, y, z);
        const int64_t i = gidx(G, x, y, z);
        const float v0 = -K.sO * ((float)x - K.half_nx);         // at x = i
        const float vh = -K.sO * ((float)x + 0.5f - K.half_nx);  // at x = i + 1/2
        float L[6], Fk[6];
        KsbCell V;
        if (G.dim == 3) {
            ksb_load<true>(K, x, y, z, i, V);
            if (K.expand)
                ksb_operator_f<true>(V, v0, vh, K.sO, K.dfac, K.kz, L);
            else
                ksb_operator<true>(V, v0, vh, K.sO, L);
        } else {
            ksb_load<false>(K, x, y, z, i, V);
            if (K.expand)
                ksb_operator_f<false>(V, v0, vh, K.sO, K.dfac, K.kz, L);
            else
                ksb_operator<false>(V, v0, vh, K.sO, L);
        }
#pragma unroll
        for (int c = 0; c < 6; c++) Fk[c] = V(c, 0, 0, 0);
        ksb_store<FIRST>(K, i, L, Fk, dm, fm);
    }
    if (K.conv) ksb_reduce<kBlock>(dm, fm, K.conv + kConvSweep * K.k);
}
__device__ __attribute__((always_inline)) inline void ksb_first_body(const KsbDev& K, int blk, int n, int y) { ksb_sweep_body<true>(K, blk, n, y); }
__device__ __attribute__((always_inline)) inline void ksb_next_body(const KsbDev& K, int blk, int n, int y) { ksb_sweep_body<false>(K, blk, n, y); }
PIC_BATCHED_KERNEL(ksb_first, KsbDev, kBlock)
PIC_BATCHED_KERNEL(ksb_next, KsbDev, kBlock)

// Two sweeps in one launch on small grids, where a sweep's launch and its one chain of loads (4.5 us) cost
// more than its work: a thread per position of a tile and the cells around it computes F^{k+1} straight
// from memory into LDS (FIRST also C), a thread per cell of the tile F^{k+2} from there.  Beyond an x face
// F^{k+1} is interpolated between two rows of the other face, computed for the tile's rows and one more;
// so no position needs another workgroup's result, and every value is the single sweeps' bit for bit.
// A step of 8 sweeps: 64^2 38 -> 24 us, 512^2 71 -> 43 us, 20 x 12 x 16 42 -> 28 us.  2D tiles of 16 x 16 took
// 22 and 52 us on these grids, 3D tiles of 8 x 8 x 4 35 us, of 4^3 27 us but 39 us on 32^3 (8 x 4 x 4: 32).
template <bool D3>
struct PairTile {
    static constexpr int TX = D3 ? 8 : 32, TY = D3 ? 4 : 16, TZ = D3 ? 4 : 1;
    static constexpr int WX = TX + 2, WY = TY + 2, WZ = D3 ? TZ + 2 : 1;
    static constexpr int N = TX * TY * TZ, W = WX * WY * WZ, RING = 2 * WX + 2 * TY;
    static constexpr int XROWS = WY + 1, X = WZ * XROWS;  // rows of the other face, per component and side
    static constexpr int LDS = 6 * (W + 2 * X);
};
constexpr int kPairBlock = 640;
constexpr int kPairLds = PairTile<true>::LDS > PairTile<false>::LDS ? PairTile<true>::LDS : PairTile<false>::LDS;

template <bool D3, bool FIRST>
__device__ __attribute__((always_inline)) inline void ksb_pair_tile(const KsbDev& K, int blk, float* lds)
{
    using T = PairTile<D3>;
    static_assert(T::W + 2 * T::WZ <= kPairBlock, "a thread per position and per additional row");
    const GridDev& G = K.G;
    const int nx = G.n[0], ny = G.n[1], nz = G.n[2];
    const int ntx = (nx + T::TX - 1) / T::TX, nty = (ny + T::TY - 1) / T::TY;
    const int x0 = blk % ntx * T::TX, y0 = blk / ntx % nty * T::TY, z0 = blk / (ntx * nty) * T::TZ;
    const int ex = min(T::TX, nx - x0), ey = min(T::TY, ny - y0), ez = min(T::TZ, nz - z0);
    const int tid = threadIdx.x;
    float* const Bs = lds;                // F^{k+1}: [c][lz][ly][lx], position 1 the tile's first cell
    float* const XB = lds + 6 * T::W;     // F^{k+1} of the other face: [side][c][lz][row]
    int js[2];
    float w1[2];
    shear_image(false, K.y1_int, K.y1_w, js[0], w1[0]);
    shear_image(true, K.y1_int, K.y1_w, js[1], w1[1]);

    // the thread's position: the tile's cells, then those around it, then the additional rows
    int lx = 0, ly = 0, lz = 0, side = -1;
    bool need;
    if (tid < T::N) {
        lx = 1 + tid % T::TX;
        ly = 1 + tid / T::TX % T::TY;
        lz = D3 ? 1 + tid / (T::TX * T::TY) : 0;
    } else if (tid < T::W) {
        int h = tid - T::N;
        if (D3 && h < 2 * T::WX * T::WY) {
            lz = h < T::WX * T::WY ? 0 : T::WZ - 1;
            lx = h % T::WX;
            ly = h / T::WX % T::WY;
        } else {
            if (D3) h -= 2 * T::WX * T::WY;
            lz = D3 ? 1 + h / T::RING : 0;
            h %= T::RING;
            if (h < 2 * T::WX) {
                lx = h % T::WX;
                ly = h < T::WX ? 0 : T::WY - 1;
            } else {
                lx = (h & 1) ? T::WX - 1 : 0;
                ly = 1 + (h - 2 * T::WX) / 2;
            }
        }
    }
    const int gx = x0 - 1 + lx;
    if (tid < T::W) {
        need = lx <= ex + 1 && ly <= ey + 1 && (!D3 || lz <= ez + 1);
        if (gx < 0) side = 0;
        if (gx >= nx) side = 1;
    } else {
        const int e = tid - T::W;
        side = e / T::WZ;
        lz = e % T::WZ;
        ly = ey + 2;
        need = e < 2 * T::WZ && (side == 0 ? x0 == 0 : x0 + ex == nx) && (!D3 || lz <= ez + 1);
    }
    const int cx = side < 0 ? gx : (side == 0 ? nx - 1 : 0);
    float C[6] = {};
    const float h = 0.5f * K.dt;
    if (need) {
        const int cy = wrapn(y0 - 1 + ly + (side < 0 ? 0 : js[side]), ny), cz = D3 ? wrapn(z0 - 1 + lz, nz) : 0;
        const int64_t i = gidx(G, cx, cy, cz);
        const float fpdt = 4.f * 3.14159265358979f * K.dt;
        const float v0 = -K.sO * ((float)cx - K.half_nx);
        const float vh = -K.sO * ((float)cx + 0.5f - K.half_nx);
#pragma unroll
        for (int c = 0; c < 6; c++)
            if (!FIRST || c >= EX) C[c] = FIRST ? K.J[c - EX][i] : K.C[c][i];
        float L[6];
        KsbCell V;
        ksb_load<D3>(K, cx, cy, cz, i, V);
        if (K.expand)
            ksb_operator_f<D3>(V, v0, vh, K.sO, K.dfac, K.kz, L);
        else
            ksb_operator<D3>(V, v0, vh, K.sO, L);
        const bool cell = tid < T::N && lx <= ex && ly <= ey && lz <= ez;
        float* const to = side < 0 ? Bs + lx + T::WX * (ly + T::WY * lz) : XB + 6 * T::X * side + ly + T::XROWS * lz;
        const int step = side < 0 ? T::W : T::X;
#pragma unroll
        for (int c = 0; c < 6; c++) {
            if (FIRST) {
                float cv = V(c, 0, 0, 0) + h * L[c];
                if (c >= EX) cv -= fpdt * C[c];
                C[c] = cv;
                if (cell) K.C[c][i] = cv;
            }
            to[c * step] = C[c] + h * L[c];
        }
    }
    __syncthreads();
    if (need && side >= 0 && tid < T::W)
#pragma unroll
        for (int c = 0; c < 6; c++) {
            const float* const r = XB + 6 * T::X * side + T::X * c + ly + T::XROWS * lz;
            Bs[lx + T::WX * (ly + T::WY * lz) + T::W * c] = shear_lerp(r[0], r[1], w1[side]);
        }
    __syncthreads();
    if (tid < T::N && lx <= ex && ly <= ey && lz <= ez) {
        const float* const B = Bs + lx + T::WX * (ly + T::WY * lz);
        auto V = [&](int c, int dx, int dy, int dz) { return B[T::W * c + dx + T::WX * (dy + T::WY * dz)]; };
        const float v0 = -K.sO * ((float)gx - K.half_nx);
        const float vh = -K.sO * ((float)gx + 0.5f - K.half_nx);
        float L[6];
        if (K.expand)
            ksb_operator_f<D3>(V, v0, vh, K.sO, K.dfac, K.kz, L);
        else
            ksb_operator<D3>(V, v0, vh, K.sO, L);
        const int64_t i = gidx(G, gx, y0 - 1 + ly, D3 ? z0 - 1 + lz : 0);
#pragma unroll
        for (int c = 0; c < 6; c++) K.Fo[c][i] = C[c] + h * L[c];
    }
}
template <bool FIRST>
__device__ __attribute__((always_inline)) inline void ksb_pair_body(const KsbDev& K, int blk)
{
    __shared__ float lds[kPairLds];
    if (K.G.dim == 3)
        ksb_pair_tile<true, FIRST>(K, blk, lds);
    else
        ksb_pair_tile<false, FIRST>(K, blk, lds);
}
__device__ __attribute__((always_inline)) inline void ksb_pair_first_body(const KsbDev& K, int blk, int, int) { ksb_pair_body<true>(K, blk); }
__device__ __attribute__((always_inline)) inline void ksb_pair_next_body(const KsbDev& K, int blk, int, int) { ksb_pair_body<false>(K, blk); }
PIC_BATCHED_KERNEL(ksb_pair_first, KsbDev, kPairBlock)
PIC_BATCHED_KERNEL(ksb_pair_next, KsbDev, kPairBlock)

// 3D: a workgroup owns a KX x KY column tile and marches over a chunk of at most KZ planes; three
// consecutive planes of the iterate (tile plus a one-cell halo) sit in LDS.  Halo positions
// outside the interior are read through the boundary maps of the guard fill (y, z periodic;
// x shearing-periodic with the fractional shift interpolated along y, the same arithmetic), so
// the iterates need no guard fill between sweeps (only the last one's guards are filled, for
// the push).  128 x 4 columns and chunks of 64 planes, which 256^3 cells still take (512 threads, 56 KB of LDS, two workgroups
// per CU) measured fastest at 256^3 among 32..128 x 2..16 x 16..128 (8 % below 32 x 8 x 32).  The iterate written and C read once per sweep use
// nontemporal (streaming) stores and loads: a sweep moves far more than the caches hold, and
// the halo reads of the iterate, which neighbouring workgroups share, keep the normal policy
// (another 9 %).
constexpr int KX = 128, KY = 4, KZ = 64;
constexpr int KXH = KX + 2, KYH = KY + 2;

template <bool FIRST>
__global__ __launch_bounds__(KX * KY) void ksb_sweep3_kernel(KsbDev K)
{
    constexpr int NT = KX * KY;
    // staged plane positions: the KX tile columns of the KYH rows, then the 2 * KYH x halo
    // positions, two per thread: j = 0 covers the first NT column positions, j = 1 the rest
    // and the x halo (the grid's x size is a multiple of KX, so only these can be x halo)
    constexpr int NCOL = KX * KYH, NPOS = NCOL + 2 * KYH;
    static_assert(NCOL >= NT && NPOS <= 2 * NT, "two staged positions per thread");
    __shared__ float P[3][6][KYH * KXH];
    if (ksb_skip(K)) return;
    const GridDev& G = K.G;
    const int tid = threadIdx.x, tx = tid % KX, ty = tid / KX;
    // tiles x fastest, then y, then z chunk; each XCD takes a contiguous range so that the
    // halos of neighbouring tiles are shared in its L2
    const int nx = G.n[0], ny = G.n[1], nz = G.n[2];
    const int ntx = nx / KX, nty = (ny + KY - 1) / KY;
    const int tile = xcd_contiguous(blockIdx.x, gridDim.x);
    const int x0 = (tile % ntx) * KX, y0 = ((tile / ntx) % nty) * KY, z0 = (tile / (ntx * nty)) * K.zc;
    const int z1 = min(z0 + K.zc, nz);
    const int x = x0 + tx, y = y0 + ty;
    const bool inside = y < ny;
    const float* const* F = K.Fk;
    // staged position j: LDS slot and in-plane offset of its source.  y and z halo positions
    // are read at their periodic images; the x halo positions (x = -1, x = nx) at their
    // shearing-periodic images: two interior values of the opposite x face, y rows js and
    // js + 1 from the position's y, interpolated as the guard fill does, so that no guard fill
    // is needed between sweeps.  Rows beyond the first one outside the grid (ragged y tiles)
    // are never read by a valid cell.
    int slot[2], off[2];
    bool ok[2];
    bool xh = false;  // position j = 1 is an x halo image
    int off2 = 0;
    float wx = 0.f;
#pragma unroll
    for (int j = 0; j < 2; j++) {
        const int q = tid + j * NT;
        int lx, ly;
        if (q < NCOL) {
            lx = 1 + q % KX;
            ly = q / KX;
        } else {
            const int r = q - NCOL;
            lx = (r & 1) ? KXH - 1 : 0;
            ly = r >> 1;
        }
        const int gx = x0 - 1 + lx, gy = y0 - 1 + ly;
        ok[j] = q < NPOS && gy <= ny;
        slot[j] = ly * KXH + lx;
        int js = 0;
        float w = 0.f;
        const bool img = j == 1 && ok[j] && (gx < 0 || gx >= nx);
        if (img) shear_image(gx >= nx, K.ydys_int, K.ydys_w, js, w);
        const int sx = gx < 0 ? gx + nx : (gx >= nx ? gx - nx : gx);
        const int ya = wrapn(gy + js, ny);
        off[j] = ok[j] ? sx + G.sy * ya : 0;
        if (j == 1) {
            xh = img;
            off2 = img ? sx + G.sy * wrapn(ya + 1, ny) : 0;
            wx = w;
        }
    }
    // register stage of one plane (loads in flight while the previous plane is computed; the
    // x images are interpolated when the plane is stashed)
    float R[2][6], R2[6];
    auto fetch = [&](int z) {
        const int64_t pz = (int64_t)G.sz * (z < 0 ? z + nz : (z >= nz ? z - nz : z));
#pragma unroll
        for (int c = 0; c < 6; c++) {
            R[0][c] = ok[0] ? F[c][off[0] + pz] : 0.f;
            R[1][c] = ok[1] ? F[c][off[1] + pz] : 0.f;
            R2[c] = xh ? F[c][off2 + pz] : 0.f;
        }
    };
    auto stash = [&](int s) {
#pragma unroll
        for (int c = 0; c < 6; c++) {
            if (ok[0]) P[s][c][slot[0]] = R[0][c];
            if (ok[1]) P[s][c][slot[1]] = xh ? shear_lerp(R[1][c], R2[c], wx) : R[1][c];
        }
    };
    const float v0 = -K.sO * ((float)x - K.half_nx);
    const float vh = -K.sO * ((float)x + 0.5f - K.half_nx);
    fetch(z0 - 1);
    stash(0);
    fetch(z0);
    stash(1);
    fetch(z0 + 1);
    int sm = 0, sc = 1, sp = 2;
    const int c0 = (ty + 1) * KXH + (tx + 1);
    const int64_t i0 = gidx(G, x, y, 0);
    float dm = 0.f, fm = 0.f;
    for (int z = z0; z < z1; z++) {
        stash(sp);                   // plane z+1
        if (z + 2 <= z1) fetch(z + 2);  // in flight during this plane
        float Cv[6];
        const int64_t i = i0 + (int64_t)G.sz * z;
        if (!FIRST && inside)
#pragma unroll
            for (int c = 0; c < 6; c++) Cv[c] = __builtin_nontemporal_load(&K.C[c][i]);
        __syncthreads();
        auto V = [&](int c, int dx, int dy, int dz) {
            const int slot = dz < 0 ? sm : (dz > 0 ? sp : sc);
            return P[slot][c][c0 + dx + KXH * dy];
        };
        if (inside) {
            float L[6];
            ksb_operator<true>(V, v0, vh, K.sO, L);
            const float h = 0.5f * K.dt;
            if (FIRST) {
                const float fpdt = 4.f * 3.14159265358979f * K.dt;
#pragma unroll
                for (int c = 0; c < 6; c++) {
                    float cv = P[sc][c][c0] + h * L[c];
                    if (c >= EX) cv -= fpdt * K.J[c - EX][i];
                    __builtin_nontemporal_store(cv, &K.C[c][i]);
                    const float v = cv + h * L[c];
                    __builtin_nontemporal_store(v, &K.Fo[c][i]);
                    if (K.conv) ksb_track(v, P[sc][c][c0], dm, fm);
                }
            } else {
#pragma unroll
                for (int c = 0; c < 6; c++) {
                    const float v = Cv[c] + h * L[c];
                    __builtin_nontemporal_store(v, &K.Fo[c][i]);
                    if (K.conv) ksb_track(v, P[sc][c][c0], dm, fm);
                }
            }
        }
        __syncthreads();
        const int t = sm;
        sm = sc;
        sc = sp;
        sp = t;
    }
    if (K.conv) ksb_reduce<NT>(dm, fm, K.conv + kConvSweep * K.k);
}

// ---- two sweeps per pass (3D, fixed sweep count)
// A pass takes F^k to F^{k+2} = C + dt/2 L(F^{k+1}) with F^{k+1} = C + dt/2 L(F^k) kept in LDS:
// the workgroup computes F^{k+1} on its PX x PY tile plus a one-cell halo, from F^k on the tile
// plus a two-cell halo, then F^{k+2} on the tile, marching over z with three planes of each
// iterate in LDS.  Memory sees one read of F^k and C and one write of F^{k+2} for two sweeps
// (the first pass reads F^n and J and writes C and F^2).
// The x halo of F^{k+1} beyond a shearing-periodic face is an image of the opposite face's
// F^{k+1} at another y, which another workgroup owns: a face tile recomputes those values
// itself, from F^k on the opposite face's three columns (one of them an image again) over the
// rows the image interpolates between, one plane ahead of its own F^{k+1}.
// Every value is the same expression as in the one-sweep kernels (contraction inside one
// expression only), so a pass gives the two sweeps' iterate bit for bit.
// Pipeline per plane: the stores of the previous plane's results, then the loads for the
// next plane (F^k and C in two alternating register sets), which nothing reads before the
// next plane, so the loads of a whole plane overlap the computation.
// Roles: every thread stages one F^k column position (the PY + 4 window rows over the PX tile
// columns); the threads of the first PY + 2 rows compute F^{k+1} on the window rows, those of
// rows 1..PY also F^{k+2} on the tile; wave WXA stages the x-halo columns of F^k, WXB computes
// the x-halo columns of F^{k+1}, WO0 and WO1 stage the opposite-face columns of F^k (one side
// each), WAUX computes the opposite-face values of F^{k+1}.
template <int X>
struct PassTile {
    static constexpr int PX = X, PY = 4, PZ = 64;
    static constexpr int W0X = PX + 4, W0Y = PY + 4;  // F^k window: tile + 2 (x from x0 - 2, y from y0 - 2)
    static constexpr int W1X = PX + 2, W1Y = PY + 2;  // F^{k+1} window: tile + 1
    static constexpr int XR1 = W1Y + 1, XR0 = XR1 + 2;  // opposite-face rows of F^{k+1} and of F^k
    static constexpr int PN = W0Y * PX;                 // one staged F^k position per thread
    // the extra roles go to the waves past the window rows where there are some (a 1024-thread
    // tile), else to the two last waves, which also compute (a 512-thread tile)
    static constexpr int WXA = 0, WXB = W1Y * PX / 64;
    static constexpr int WO0 = PN == 1024 ? 13 : WXB, WO1 = PN == 1024 ? 15 : WXB + 1;
    static constexpr int WAUX = PN == 1024 ? 14 : WXB + 1;
};
// 64 x 4 tiles: 512 threads and 72 KB of LDS, two workgroups per CU.  At 256^3 a pass takes
// 0.44 ms, the same as the 128 x 4 tile (1024 threads, 137 KB, one workgroup per CU), against
// 0.49 ms for two single sweeps.  Neither the stencil (the pass without it takes as long) nor
// HBM bandwidth bounds it: the loads of one plane, one plane ahead, are its memory parallelism,
// and a second register set for two planes ahead spills (measured slower).
constexpr int kPassX = 64;

// element of an array at a 32-bit byte offset from its base (the array pointer itself, in
// scalar registers): plane and in-plane offsets are summed in 32 bits, so the compiler keeps
// one offset register per position instead of a 64-bit address per array (the arrays of a
// box that takes the pass span less than 4 GiB)
__device__ inline float ld_off(const float* base, uint32_t ob)
{
    return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + ob);
}
__device__ inline float* st_off(float* base, uint32_t ob)
{
    return reinterpret_cast<float*>(reinterpret_cast<char*>(base) + ob);
}

template <int TX, bool FIRST>
__global__ __launch_bounds__(PassTile<TX>::PN) __attribute__((amdgpu_waves_per_eu(4)))
void ksb_pass3_kernel(KsbDev K)
{
    using T = PassTile<TX>;
    constexpr int PX = T::PX, PY = T::PY, PN = T::PN;
    constexpr int W0X = T::W0X, W0Y = T::W0Y, W1X = T::W1X, W1Y = T::W1Y, XR0 = T::XR0, XR1 = T::XR1;
    static_assert(PX % 64 == 0 && W1Y * PX == 64 * T::WXB && T::WAUX < PN / 64 && T::WO1 < PN / 64,
                  "thread roles");
    static_assert(2 * W1Y <= 64 && PX + PY * PX <= 64 * T::WXB, "F^{k+2} on window-row waves");
    static_assert(3 * XR0 <= 32 && XR1 <= 32, "opposite-face roles fit half a wave per side");
    __shared__ float A[3][6][W0Y * W0X];  // planes of F^k
    __shared__ float Bs[3][6][W1Y * W1X];  // planes of F^{k+1}
    __shared__ float XA[3][2][6][3 * XR0];  // opposite-face F^k: [plane][side][c][row * 3 + col]
    __shared__ float XB[2][2][6][XR1];      // opposite-face F^{k+1}: [plane][side][c][row]
    const GridDev& G = K.G;
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
    const int nx = G.n[0], ny = G.n[1], nz = G.n[2];
    const int ntx = nx / PX, nty = (ny + PY - 1) / PY;
    const int tile = xcd_contiguous(blockIdx.x, gridDim.x);
    const int x0 = (tile % ntx) * PX, y0 = ((tile / ntx) % nty) * PY, z0 = (tile / (ntx * nty)) * K.zc;
    const int z1 = min(z0 + K.zc, nz);
    const float* const* F = K.Fk;
    const float h = 0.5f * K.dt;
    const float fpdt = 4.f * 3.14159265358979f * K.dt;
    // side 0: the face at x = 0 (x halo x = -1, an image of column nx - 1); side 1: x = nx - 1
    const bool face[2] = {x0 == 0, x0 + PX == nx};
    int js1[2];
    float w1[2];
    shear_image(false, K.y1_int, K.y1_w, js1[0], w1[0]);
    shear_image(true, K.y1_int, K.y1_w, js1[1], w1[1]);

    // ---- staged F^k position of every thread: window row tid / PX, tile column tid % PX
    const uint32_t aoff = 4u * (uint32_t)(x0 + tid % PX + G.sy * wrapn(y0 - 2 + tid / PX, ny));
    const int aslot = tid + (W0X - PX) * (tid / PX) + 2;
    // extra F^k position, lanes 0..31 of wave 0 (x-halo columns lx = 0, 1, W0X-2, W0X-1 of
    // F^k) and of waves WO0 and WO1 (column col, row r of the XR0 opposite-face rows of side 0 and
    // side 1).  An image position interpolates two values (shift ydys of F^k): lane l + 32
    // loads the second one for lane l.
    uint32_t xoff = 0;
    int xslot = 0;
    bool xa = false, ximg = false;
    float xw = 0.f;
    const int xs = wv == T::WO1 ? 1 : 0;
    const bool owave = wv == T::WO0 || wv == T::WO1;
    {
        const int l = lane & 31;
        int gx = 0, gy = 0;
        bool pos = false;
        if (wv == T::WXA && l < 4 * W0Y) {
            const int ly = l >> 2, e = l & 3;
            const int lx = e < 2 ? e : W0X - 4 + e;
            gx = x0 - 2 + lx;
            gy = y0 - 2 + ly;
            pos = gx >= -1 && gx <= nx;  // x = -2, nx + 1 beyond a face are never read
            xslot = ly * W0X + lx;
        } else if (owave && l < 3 * XR0) {
            const int col = l % 3, r = l / 3;
            gx = (xs == 0 ? nx - 2 : -1) + col;
            gy = y0 - 2 + js1[xs] + r;
            pos = face[xs];
            xslot = r * 3 + col;
        }
        int js = 0;
        ximg = pos && (gx < 0 || gx >= nx);
        if (ximg) shear_image(gx >= nx, K.ydys_int, K.ydys_w, js, xw);
        const int sx = gx < 0 ? gx + nx : (gx >= nx ? gx - nx : gx);
        const int ya = wrapn(gy + js, ny);
        const bool second = lane >= 32;
        xa = pos && (!second || ximg);  // this lane loads a value
        xoff = xa ? 4u * (uint32_t)(sx + G.sy * (second ? wrapn(ya + 1, ny) : ya)) : 0u;
        if (second) xa = xa && ximg;
        if (second) ximg = false;
        if (second) pos = false;
        xslot = pos ? xslot : -1;  // the lanes that store (lanes < 32 with a position)
    }

    // ---- F^{k+1} position: threads < W1Y * PX on the window rows over the tile columns
    const bool bmain = tid < W1Y * PX;
    const int blx = 1 + tid % PX, bly = bmain ? tid / PX : 0;
    const int bslot = bly * W1X + blx;
    const int bgx = x0 + tid % PX;
    const uint32_t boff = 4u * (uint32_t)(bgx + G.sy * wrapn(y0 - 1 + bly, ny));
    // extra F^{k+1} position (wave WXB: the x-halo columns lx = 0, W1X - 1, rows r >> 1 --
    // interior, or beyond a face an image of the opposite face's values; wave WAUX: row r of the
    // opposite face of side cs, one plane ahead)
    int cslot = 0, cs = 0, crow = 0, cgx = 0;
    bool cop = false, cimg = false, caux = false;
    uint32_t coff = 0;
    if (wv == T::WXB && lane < 2 * W1Y) {
        const int ly = lane >> 1, lx = (lane & 1) ? W1X - 1 : 0;
        cgx = x0 - 1 + lx;
        const int gy = y0 - 1 + ly;
        cslot = ly * W1X + lx;
        crow = ly;
        cimg = cgx < 0 || cgx >= nx;
        cop = !cimg;
        cs = cgx < 0 ? 0 : 1;
        coff = cop ? 4u * (uint32_t)(cgx + G.sy * wrapn(gy, ny)) : 0u;
    }
    if (wv == T::WAUX && (lane & 31) < XR1) {
        cs = lane >> 5;
        crow = lane & 31;
        caux = face[cs];
        cgx = cs == 0 ? nx - 1 : 0;
        coff = caux ? 4u * (uint32_t)(cgx + G.sy * wrapn(y0 - 1 + js1[cs] + crow, ny)) : 0u;
    }
    const bool cload = cop || caux;

    // ---- F^{k+2}: the tile cell of threads PX .. PX + PY * PX - 1 (their F^{k+1} position)
    const bool tmain = tid >= PX && tid < PX + PY * PX;
    const int ty = tid / PX - 1;
    const bool inside = tmain && y0 + ty < ny;
    const uint32_t i0 = 4u * (uint32_t)(bgx + G.sy * min(y0 + max(ty, 0), ny - 1));

    // C of the F^{k+1} positions in two register sets used on alternate planes: the loads
    // for plane q + 1 are issued at the top of plane q, beside the F^k loads
    float R[6], X[6], Ca[6], Cb[6], Cn[6], Ct[6], Ores[6];
#pragma unroll
    for (int c = 0; c < 6; c++) X[c] = Ca[c] = Cb[c] = Cn[c] = Ct[c] = Ores[c] = 0.f;
    auto plane_of = [&](int z) { return 4u * (uint32_t)G.sz * (uint32_t)wrapn(z, nz); };
    auto fetch_main = [&](int z) {
        const uint32_t pz = plane_of(z);
#pragma unroll
        for (int c = 0; c < 6; c++) R[c] = ld_off(F[c], pz + aoff);
        if (wv == T::WXA && xa)
#pragma unroll
            for (int c = 0; c < 6; c++) X[c] = ld_off(F[c], pz + xoff);
    };
    auto fetch_aux = [&](int z) {
        const uint32_t pz = plane_of(z);
        if (owave && xa)
#pragma unroll
            for (int c = 0; c < 6; c++) X[c] = ld_off(F[c], pz + xoff);
    };
    // the extra value of a lane, interpolated with lane + 32's for an image (whole wave)
    auto extra = [&](int c) {
        const float v2 = __shfl(X[c], (lane & 31) + 32, 64);
        return ximg ? shear_lerp(X[c], v2, xw) : X[c];
    };
    auto stash_main = [&](int s) {
#pragma unroll
        for (int c = 0; c < 6; c++) A[s][c][aslot] = R[c];
        if (wv == T::WXA)
#pragma unroll
            for (int c = 0; c < 6; c++) {
                const float v = extra(c);
                if (xslot >= 0) A[s][c][xslot] = v;
            }
    };
    auto stash_aux = [&](int s) {
        if (owave)
#pragma unroll
            for (int c = 0; c < 6; c++) {
                const float v = extra(c);
                if (xslot >= 0) XA[s][xs][c][xslot] = v;
            }
    };
    // C (first pass: J) of the F^{k+1} positions into Cd: main ones and wave WXB's at plane zm,
    // wave WAUX's at za
    auto load_c = [&](float* Cd, int zm, int za) {
        const uint32_t pm = plane_of(zm);
        const uint32_t o = bmain ? boff : coff;
        const uint32_t pc = caux ? plane_of(za) : pm;
        if (bmain || cload)
#pragma unroll
            for (int c = 0; c < 6; c++)
                if (!FIRST || c >= EX)
                    Cd[c] = FIRST ? ld_off(K.J[c - EX], pc + o) : ld_off(K.C[c], pc + o);
    };
    // F^{k+1} = C + dt/2 L(F^k) at one position, the operator read through V; the first pass
    // also gives C there (cout)
    auto next_iterate = [&](auto&& V, int gx, const float* cw, float* out, float* cout) {
        const float v0 = -K.sO * ((float)gx - K.half_nx);
        const float vh = -K.sO * ((float)gx + 0.5f - K.half_nx);
        float L[6];
        ksb_operator<true>(V, v0, vh, K.sO, L);
#pragma unroll
        for (int c = 0; c < 6; c++) {
            if (FIRST) {
                float cv = V(c, 0, 0, 0) + h * L[c];
                if (c >= EX) cv -= fpdt * cw[c];
                cout[c] = cv;
                out[c] = cv + h * L[c];
            } else {
                out[c] = cw[c] + h * L[c];
            }
        }
    };
    // opposite-face F^{k+1} at plane z from the opposite-face F^k planes (m, c, p)
    auto aux_iterate = [&](const float* cw, int m, int c0, int p, int xb) {
        if (!caux) return;
        auto V = [&](int c, int dx, int dy, int dz) {
            const int s = dz < 0 ? m : (dz > 0 ? p : c0);
            return XA[s][cs][c][(crow + 1 + dy) * 3 + 1 + dx];
        };
        float out[6], cv[6];
        next_iterate(V, cgx, cw, out, cv);
#pragma unroll
        for (int c = 0; c < 6; c++) XB[xb][cs][c][crow] = out[c];
    };

    // ---- prologue: F^k planes z0 - 2, z0 - 1 (opposite face: z0 - 2 .. z0), the opposite
    // face's F^{k+1} at z0 - 1, then the loads for the first plane
    fetch_main(z0 - 2);
    fetch_aux(z0 - 2);
    stash_main(0);
    stash_aux(0);
    fetch_main(z0 - 1);
    fetch_aux(z0 - 1);
    stash_main(1);
    stash_aux(1);
    fetch_aux(z0);
    load_c(Cb, z0 - 1, z0 - 1);
    stash_aux(2);
    __syncthreads();
    aux_iterate(Cb, 0, 1, 2, 0);
    __syncthreads();  // slot 0 of the opposite-face F^k is staged again at the first plane
    fetch_main(z0);
    fetch_aux(z0 + 1);
    load_c(Ca, z0 - 1, z0);
    int am = 0, ac = 1, ap = 2;  // F^k planes q - 1, q, q + 1
    int bm = 0, bc = 1, bp = 2;  // F^{k+1} planes q - 2, q - 1, q
    int xm = 1, xc = 2, xp = 0;  // opposite-face F^k planes q, q + 1, q + 2
    int xbq = 0;                 // opposite-face F^{k+1} plane q (the other slot: q + 1)
    // one plane: F^{k+1} at q with the C set Cu (loaded a plane earlier), the loads of the
    // next plane's C into Cl
    auto plane = [&](int q, float* Cu, float* Cl) {
        stash_main(ap);  // F^k plane q + 1
        stash_aux(xp);   // opposite-face F^k plane q + 2
        if (inside) {
            if (q - 2 >= z0) {
                const uint32_t pz = plane_of(q - 2);
#pragma unroll
                for (int c = 0; c < 6; c++) __builtin_nontemporal_store(Ores[c], st_off(K.Fo[c], pz + i0));
            }
            if (FIRST && q - 1 >= z0 && q - 1 < z1) {
                const uint32_t pz = plane_of(q - 1);
#pragma unroll
                for (int c = 0; c < 6; c++) __builtin_nontemporal_store(Ct[c], st_off(K.C[c], pz + i0));
            }
        }
        if (q + 2 <= z1 + 1) fetch_main(q + 2);
        if (q + 3 <= z1 + 1) fetch_aux(q + 3);
        if (q + 1 <= z1) load_c(Cl, q + 1, q + 2);
        __syncthreads();
        // F^{k+1} at plane q
        if (bmain) {
            const int base = bslot + 2 * bly + W0X + 1;  // the same cell in the F^k window
            auto V = [&](int c, int dx, int dy, int dz) {
                const int s = dz < 0 ? am : (dz > 0 ? ap : ac);
                return A[s][c][base + dx + W0X * dy];
            };
            float out[6];
            next_iterate(V, bgx, Cu, out, Cn);
#pragma unroll
            for (int c = 0; c < 6; c++) Bs[bp][c][bslot] = out[c];
        }
        if (cop) {
            const int base = cslot + 2 * crow + W0X + 1;
            auto V = [&](int c, int dx, int dy, int dz) {
                const int s = dz < 0 ? am : (dz > 0 ? ap : ac);
                return A[s][c][base + dx + W0X * dy];
            };
            float out[6], cv[6];
            next_iterate(V, cgx, Cu, out, cv);
#pragma unroll
            for (int c = 0; c < 6; c++) Bs[bp][c][cslot] = out[c];
        } else if (cimg && face[cs]) {
#pragma unroll
            for (int c = 0; c < 6; c++)
                Bs[bp][c][cslot] = shear_lerp(XB[xbq][cs][c][crow], XB[xbq][cs][c][crow + 1], w1[cs]);
        }
        if (q + 1 <= z1) aux_iterate(Cu, xm, xc, xp, xbq ^ 1);  // opposite face, plane q + 1
        __syncthreads();
        // F^{k+2} at plane q - 1
        if (tmain && q - 1 >= z0) {
            const int base = bslot;
            auto V = [&](int c, int dx, int dy, int dz) {
                const int s = dz < 0 ? bm : (dz > 0 ? bp : bc);
                return Bs[s][c][base + dx + W1X * dy];
            };
            const float v0 = -K.sO * ((float)bgx - K.half_nx);
            const float vh = -K.sO * ((float)bgx + 0.5f - K.half_nx);
            float L[6];
            ksb_operator<true>(V, v0, vh, K.sO, L);
#pragma unroll
            for (int c = 0; c < 6; c++) Ores[c] = Ct[c] + h * L[c];
        }
#pragma unroll
        for (int c = 0; c < 6; c++) Ct[c] = FIRST ? Cn[c] : Cu[c];  // C at the tile cell, plane q
        int t = am;
        am = ac;
        ac = ap;
        ap = t;
        t = bm;
        bm = bc;
        bc = bp;
        bp = t;
        t = xm;
        xm = xc;
        xc = xp;
        xp = t;
        xbq ^= 1;
    };
    int q = z0 - 1;
    for (; q + 1 <= z1; q += 2) {
        plane(q, Ca, Cb);
        plane(q + 1, Cb, Ca);
    }
    if (q <= z1) plane(q, Ca, Cb);
    if (inside && z1 - 1 >= z0) {
        const uint32_t pz = plane_of(z1 - 1);
#pragma unroll
        for (int c = 0; c < 6; c++) __builtin_nontemporal_store(Ores[c], st_off(K.Fo[c], pz + i0));
    }
}

// End of a tolerance-mode step (one record per box): find the first sweep that met the
// tolerance, report the sweep count, latch kErrNoConverge if none did, and move that sweep's
// iterate into the set the step hands on when it sits in the other one.
__device__ __attribute__((always_inline)) inline void ksb_final_body(const KsbFin& F, int blk, int nblk, int)
{
    __shared__ int kstar;
    if (threadIdx.x == 0) kstar = F.K;
    __syncthreads();
    for (int j = threadIdx.x; j < F.K; j += kBlock) {
        uint32_t pair[2] = {0u, 0u};
#pragma unroll
        for (int k = 0; k < kConvSlots; k++)
            for (int i = 0; i < 2; i++) pair[i] = max(pair[i], F.conv[kConvSweep * j + kConvStride * k + i]);
        if (ksb_met(pair, F.tol)) atomicMin(&kstar, j);
    }
    __syncthreads();
    const bool met = kstar < F.K;
    const int last = met ? kstar : F.K - 1;  // the sweep whose iterate the step hands on
    if (blk == 0 && threadIdx.x == 0) {
        *F.sweeps = last + 1;
        if (!met) atomicOr(F.err, kErrNoConverge);
    }
    if (((F.K - 1 - last) & 1) == 0) return;
    const GridDev& G = F.G;
    const int64_t n = (int64_t)G.n[0] * G.n[1] * G.n[2];
    for (int64_t t = (int64_t)blk * kBlock + threadIdx.x; t < n; t += (int64_t)nblk * kBlock) {
        int x, y, z;
        cell_of(G, t, x, y, z);
        const int64_t i = gidx(G, x, y, z);
#pragma unroll
        for (int c = 0; c < 6; c++) F.dst[c][i] = F.src[c][i];
    }
}
PIC_BATCHED_KERNEL(ksb_final, KsbFin, kBlock)
#pragma clang fp contract(fast)

// ------------------------------------------------------------------ utilities
// interior of six components (B then E) times f[c % 3] (the expanding-frame conversion of the
// combined frame's field step)
// grid-stride over the cells (the batched launch gives every cell its own thread)
__device__ __attribute__((always_inline)) inline void scale_fields_body(const ScaleArgs& a, int blk, int nblk, int)
{
    const GridDev& G = a.G;
    const int64_t n = (int64_t)G.n[0] * G.n[1] * G.n[2];
    for (int64_t t = (int64_t)blk * kBlock + threadIdx.x; t < n; t += (int64_t)nblk * kBlock) {
        int x, y, z;
        cell_of(G, t, x, y, z);
        const int64_t i = gidx(G, x, y, z);
#pragma unroll
        for (int c = 0; c < 6; c++) a.F[c][i] *= a.f[c % 3];
    }
}
PIC_BATCHED_KERNEL(scale_fields, ScaleArgs, kBlock)

// grid-stride, 16-byte stores where the array is 16-byte aligned (the batched launch gives
// every word its own thread, so most of its threads find nothing to do)
__device__ inline void zero_words(const ZeroArgs& a, int blk, int nblk)
{
    const int64_t stride = (int64_t)nblk * kBlock, i = (int64_t)blk * kBlock + threadIdx.x;
    int64_t head = 0;
    if ((reinterpret_cast<uintptr_t>(a.p) & 15) == 0) {
        uint4* q = reinterpret_cast<uint4*>(a.p);
        const int64_t n4 = a.n >> 2;
        for (int64_t j = i; j < n4; j += stride) q[j] = make_uint4(0u, 0u, 0u, 0u);
        head = n4 << 2;
    }
    for (int64_t j = head + i; j < a.n; j += stride) a.p[j] = 0u;
}
__device__ __attribute__((always_inline)) inline void zero_body(const ZeroArgs& a, int blk, int nblk, int)
{
    zero_words(a, blk, nblk);
}
PIC_BATCHED_KERNEL(zero, ZeroArgs, kBlock)

// one launch (five before): y = 0 .. 2 the current arrays, beyond them the counts of a species
__global__ __launch_bounds__(kBlock) void clear_kernel(ClearArgs a)
{
    const int y = (int)blockIdx.y, s = y - 3;
    if (y < 3)
        zero_words(ZeroArgs{reinterpret_cast<uint32_t*>(a.J[y]), a.n}, (int)blockIdx.x, (int)gridDim.x);
    else
        zero_words(ZeroArgs{a.mcnt[s], a.nm}, (int)blockIdx.x, (int)gridDim.x);
    if (y == 0 && blockIdx.x == 0 && threadIdx.x < kMaxSpecies && a.flag[threadIdx.x]) *a.flag[threadIdx.x] = 0;
}

// interior <-> dense copies of gridDim.y arrays: dense index x + n0*(y + n1*z)
typedef float Quad __attribute__((ext_vector_type(4), aligned(4)));  // a row may start at any element
// A thread moves up to four consecutive elements of a row (quads divides by the quads of a row).  E or B of
// 256^3 138 -> 112 us, of 128 x 64 x 64 8.1 -> 4.9 us against an element a thread.
__global__ __launch_bounds__(kBlock) void interior_copy_kernel(GridDev G, Comp6 guarded, Comp6 dense, int to_dense, FastDiv quads)
{
    const int c = (int)blockIdx.y, nx = G.n[0];
    const uint32_t per_row = (uint32_t)(nx + 3) / 4;
    const int64_t n = (int64_t)per_row * G.n[1] * G.n[2];
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < n; t += (int64_t)gridDim.x * kBlock) {
        const uint32_t r = quads.div((uint32_t)t), z = G.div1.div(r);
        const int x = 4 * (int)((uint32_t)t - r * per_row);
        float* const g = guarded.p[c] + gidx(G, x, (int)(r - z * (uint32_t)G.n[1]), (int)z);
        float* const d = dense.p[c] + (int64_t)r * nx + x;
        const float* const from = to_dense ? g : d;
        float* const to = to_dense ? d : g;
        if (x + 4 <= nx)
            *reinterpret_cast<Quad*>(to) = *reinterpret_cast<const Quad*>(from);
        else
            for (int k = 0; k < nx - x; k++) to[k] = from[k];
    }
}

// FP64 sum of a workgroup's values in a fixed order, on thread 0
__device__ inline double block_sum(double v, double* sh)
{
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int s = kBlock / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

// FP64 block partial sums of squares of 6 interior component arrays
__global__ __launch_bounds__(kBlock) void field_energy_kernel(GridDev G, Comp6 A, double* part)
{
    __shared__ double sh[kBlock];
    const int c = blockIdx.y;
    double acc = 0.0;
    const int64_t ncell = (int64_t)G.n[0] * G.n[1] * G.n[2];
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < ncell;
         t += (int64_t)gridDim.x * kBlock) {
        int x, y, z;
        cell_of(G, t, x, y, z);
        const double v = A.p[c][gidx(G, x, y, z)];
        acc += v * v;
    }
    const double r = block_sum(acc, sh);
    if (threadIdx.x == 0) part[c * gridDim.x + blockIdx.x] = r;
}

// FP64 block partial sums of (gamma-1), u and the kinetic stress diagonal u_c^2/gamma over the particles
// that have not escaped (an escape marks the cell -1 until the next sort drops the particle; cell null:
// a box without escapes), one species per blockIdx.y
__global__ __launch_bounds__(kBlock) void particle_sums_kernel(SumArgs P, double* part)
{
    __shared__ double sh[kBlock];
    const SumArgs::Species& S = P.s[blockIdx.y];
    double a[kPartSums] = {};
    const int n = *S.n_live;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock) {
        if (S.cell && S.cell[i] < 0) continue;
        const double x = S.u[0][i], y = S.u[1][i], z = S.u[2][i];
        const double uu = x * x + y * y + z * z;
        const double g = sqrt(1.0 + uu), rg = 1.0 / g;
        a[0] += uu / (g + 1.0);  // gamma - 1 without cancellation
        a[1] += x;
        a[2] += y;
        a[3] += z;
        a[4] += x * x * rg;
        a[5] += y * y * rg;
        a[6] += z * z * rg;
    }
    for (int k = 0; k < kPartSums; k++) {
        const double r = block_sum(a[k], sh);
        if (threadIdx.x == 0) part[(blockIdx.y * kPartSums + k) * gridDim.x + blockIdx.x] = r;
    }
}

// Energy distribution (Sec. 4.2) of the particles that have not escaped: slot = number of
// edges <= gamma - 1 (0: below the first edge, nbins + 1: at or above the last; non-finite
// energies go to the last slot).  Edges and the workgroup's counts sit in LDS, sized by the bins, so
// that a histogram of 200 bins leaves a CU full (three workgroups with the space for the most bins);
// each workgroup adds its non-zero counts once.  The chip is filled by two workgroups of sixteen waves
// a CU: the counts of 1024 smaller ones meet at the same few words of memory.  A thread searches for two
// particles at a time.
// 9.6M particles, 200 bins: 127 us with the fixed space and 1024 small workgroups, 50 us (2.3 TB/s).  (Several count words a slot, and a
// search by FP32 energies with the FP64 one where an edge is near, did not change that.)
constexpr int kHistBlock = 1024, kHistBlocks = 512;
__global__ __launch_bounds__(kHistBlock) void energy_hist_kernel(const int32_t* cell, const float* ux,
                                                             const float* uy, const float* uz,
                                                             const int32_t* n_live,
                                                             const double* edges, int nbins,
                                                             unsigned long long* counts)
{
    extern __shared__ double e[];
    uint32_t* const h = reinterpret_cast<uint32_t*>(e + nbins + 1);
    for (int b = threadIdx.x; b < nbins + 2; b += kHistBlock) h[b] = 0u;
    for (int b = threadIdx.x; b <= nbins; b += kHistBlock) e[b] = edges[b];
    __syncthreads();
    const int n = *n_live;
    int steps = 1;  // halvings that bring nbins + 1 edges down to none
    while ((nbins + 1) >> steps) steps++;
    const int64_t stride = (int64_t)gridDim.x * kHistBlock;
    for (int64_t i = (int64_t)blockIdx.x * kHistBlock + threadIdx.x; i < n; i += 2 * stride) {
        double k[2];
        int lo[2] = {0, 0}, len[2];
        bool on[2];
#pragma unroll
        for (int j = 0; j < 2; j++) {
            const int64_t p = i + j * stride, q = p < n ? p : i;
            on[j] = p < n && !(cell && cell[q] < 0);
            const double x = ux[q], y = uy[q], z = uz[q];
            const double uu = x * x + y * y + z * z;  // FP32 inputs: the products are exact
            k[j] = uu / (sqrt(1.0 + uu) + 1.0);
            len[j] = nbins + 1;  // edges[0 .. lo) <= k, edges[lo + len ..] > k
        }
        for (int s = 0; s < steps; s++)
#pragma unroll
            for (int j = 0; j < 2; j++) {
                const int half = len[j] >> 1, mid = lo[j] + half;
                const bool below = len[j] > 0 && e[mid < nbins ? mid : nbins] <= k[j];
                lo[j] = below ? mid + 1 : lo[j];
                len[j] = below ? len[j] - half - 1 : half;
            }
#pragma unroll
        for (int j = 0; j < 2; j++)
            if (on[j]) atomicAdd(&h[k[j] == k[j] ? lo[j] : nbins + 1], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nbins + 2; b += kHistBlock)
        if (h[b]) atomicAdd(&counts[b], (unsigned long long)h[b]);
}

// The record of a box: workgroup r < rows sums the row r of ncol partials in a fixed order, the one
// beyond them collects the counters.  (One thread per row took 82 us.)
__global__ __launch_bounds__(kBlock) void box_record_kernel(SumArgs P, const double* part, int rows, int ncol, BoxRecord* out)
{
    __shared__ double sh[kBlock];
    const int r = (int)blockIdx.x;
    if (r == rows) {
        if (threadIdx.x == 0) {
            for (int s = 0; s < P.nsp; s++) out->live[s] = *P.s[s].n_live;
            for (int k = 0; k < 4; k++) out->ctr[k] = P.ctr[k];
            out->err = *P.err;
            out->sweeps = P.sweeps ? *P.sweeps : 0;
        }
        return;
    }
    double v = 0.0;
    for (int k = threadIdx.x; k < ncol; k += kBlock) v += part[r * ncol + k];
    v = block_sum(v, sh);
    if (threadIdx.x == 0) out->row[r] = v;
}

// ------------------------------------------------------------------ host launchers
static inline unsigned nblocks(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }
// grid of the grid-stride cell kernels (the shear fold, the Yee updates, field copies): 16 blocks per CU, each
// thread taking a few cells.  It was faster for a fold of one cell a thread; now, a thread per cell (fold: per
// four rows) is as fast on 128 x 128 x 257 cells (fold 27.2 us, Yee step 98 us both ways) and slightly faster on
// 256^3 (fold 95 against 100 us, Yee step 512 against 549 us).
constexpr unsigned kStrideBlocks = 4096;

FillArgs fill_args(const GridDev& G, float* const* comps, int ncomp, int shear, double dys)
{
    FillArgs a{};
    a.G = G;
    for (int c = 0; c < ncomp; c++) a.A.p[c] = comps[c];
    const double fl = floor(dys);
    a.shear = shear;
    a.dys_int = (int)fl;
    a.dys_w = (float)(dys - fl);
    // a guarded array holds less than 2^31 floats: the slabs together stay below 2^32 threads
    const uint32_t NYg = (uint32_t)(G.n[1] + 2 * G.g[1]), NZg = (uint32_t)(G.n[2] + 2 * G.g[2]);
    a.n[0] = 2u * G.g[0] * NYg * NZg;
    a.n[1] = (uint32_t)G.n[0] * 2u * G.g[1] * NZg;
    a.n[2] = (uint32_t)G.n[0] * (uint32_t)G.n[1] * 2u * G.g[2];
    return a;
}
unsigned fill_blocks(const FillArgs& a) { return nblocks((int64_t)a.n[0] + a.n[1] + a.n[2]); }

hipError_t fill_guards(const GridDev& G, float* const* comps, int ncomp, int shear, double dys,
                       hipStream_t st)
{
    const FillArgs a = fill_args(G, comps, ncomp, shear, dys);
    fill_guards_kernel<<<dim3(fill_blocks(a), ncomp), kBlock, 0, st>>>(a);
    return hipGetLastError();
}

FoldPArgs fold_args(const GridDev& G, float* const* J, int shear)
{
    FoldPArgs a{};
    a.G = G;
    for (int c = 0; c < 3; c++) a.J.p[c] = J[c];
    const uint32_t g2 = 2 * kGuard, nx = G.n[0], ny = G.n[1], nz = G.n[2];
    a.x0 = shear ? -kGuard : kGuard;
    a.wx = shear ? nx + g2 : nx - g2;
    a.n[0] = shear ? 0 : g2 * ny * nz;
    a.n[1] = a.wx * g2 * nz;
    a.n[2] = G.dim == 3 ? a.wx * (ny - g2) * g2 : 0;
    return a;
}
unsigned fold_blocks(const FoldPArgs& a) { return nblocks((int64_t)a.n[0] + a.n[1] + a.n[2]); }

unsigned shear_fold_blocks(const GridDev& G)
{
    return nblocks((int64_t)G.n[0] * ((G.n[1] + kFoldRows - 1) / kFoldRows) * G.n[2]);
}
// Fold the deposited current: in place, or for the shearing box into `out`, every interior cell.
hipError_t fold_current(const GridDev& G, float* const* J, float* const* out, int shear,
                        double sO, double dt, double dys_half, hipStream_t st)
{
    const Comp3 Jc{{J[0], J[1], J[2]}};
    const FoldPArgs a = fold_args(G, J, shear);
    fold_periodic_kernel<<<dim3(fold_blocks(a), 3), kBlock, 0, st>>>(a);
    if (shear) {
        const double fl = floor(dys_half);
        const Comp3 Oc{{out[0], out[1], out[2]}};
        const unsigned nb = std::min(shear_fold_blocks(G), kStrideBlocks);
        shear_fold_kernel<<<dim3(nb, 3), kBlock, 0, st>>>(
            ShearFoldArgs{G, Jc, Oc, (float)(sO * dt / 2.0), 0.5f * G.n[0], (int)fl, (float)(dys_half - fl)});
    }
    return hipGetLastError();
}

hipError_t yee_b(const MaxwellDev& M, hipStream_t st)
{
    yee_b_kernel<<<std::min(nblocks((int64_t)M.G.n[0] * M.G.n[1] * M.G.n[2]), kStrideBlocks), kBlock, 0, st>>>(M);
    return hipGetLastError();
}
hipError_t yee_e(const MaxwellDev& M, hipStream_t st)
{
    yee_e_kernel<<<std::min(nblocks((int64_t)M.G.n[0] * M.G.n[1] * M.G.n[2]), kStrideBlocks), kBlock, 0, st>>>(M);
    return hipGetLastError();
}
// Where the staged sweep and the pass over z, which march over planes that each wait for the one before,
// win: on grids that the last-level cache does not hold.  us a step of 8 sweeps, passes / staged sweeps /
// one thread a cell: 64^3 74 / 54 / 56, 128 x 64 x 64 99 / 146 / 74, 128^3 265 / 336 / 221,
// 256 x 128 x 128 454 / 577 / 674, 256^3 1849 / 2117 / 2611; the line lies between 128^3 and 256 x 128 x 128.
constexpr int64_t kStagedCells = 3ll << 20;
bool ksb_staged(const GridDev& G)
{
    return G.dim == 3 && G.n[0] % KX == 0 && (int64_t)G.n[0] * G.n[1] * G.n[2] > kStagedCells;
}
bool ksb_pass_fits(const GridDev& G)
{
    return G.dim == 3 && G.n[0] % kPassX == 0 && (int64_t)G.n[0] * G.n[1] * G.n[2] > kStagedCells && 4 * (int64_t)G.sz * G.n[2] < (int64_t(1) << 32);
}

// Planes per workgroup of the staged kernels and the workgroups of a launch over `columns` column
// tiles: `most` planes on grids that fill the chip with them (two workgroups a CU), fewer on smaller
// ones (a chunk reads two planes, a pass four, beyond its own); on the grids of more than kStagedCells a
// staged sweep is down to 8 planes, a pass to 16.  A step of 8 sweeps, us, so / in chunks of 64: 128 x 255 x 97
// passes 465 / 630, single sweeps 616 / 1110; 256 x 128 x 128 464 / 605 and 606 / 1187; 256 x 256 x 128 871 / 872 and 1100 / 1351.
static unsigned z_chunks(int columns, int nz, int most, int& zc)
{
    zc = most;
    while (zc > 8 && (int64_t)columns * ((nz + zc - 1) / zc) < 2 * 256) zc /= 2;
    return (unsigned)(columns * ((nz + zc - 1) / zc));
}

hipError_t ksb_sweep_staged(const KsbDev& K, bool first, hipStream_t st)
{
    if (!ksb_staged(K.G) || K.expand) return hipErrorInvalidValue;
    KsbDev Z = K;
    const unsigned grid = z_chunks((K.G.n[0] / KX) * ((K.G.n[1] + KY - 1) / KY), K.G.n[2], KZ, Z.zc);
    if (first)
        ksb_sweep3_kernel<true><<<grid, KX * KY, 0, st>>>(Z);
    else
        ksb_sweep3_kernel<false><<<grid, KX * KY, 0, st>>>(Z);
    return hipGetLastError();
}
hipError_t ksb_sweep(const KsbDev& K, bool first, hipStream_t st)
{
    const unsigned nb = nblocks((int64_t)K.G.n[0] * K.G.n[1] * K.G.n[2]);
    if (first)
        ksb_first_kernel<<<nb, kBlock, 0, st>>>(K);
    else
        ksb_next_kernel<<<nb, kBlock, 0, st>>>(K);
    return hipGetLastError();
}
// Where two sweeps per launch win.  us a step of 8 sweeps, pairs / singles: 64^2 24 / 37, 512^2 43 / 71,
// 1024^2 130 / 142 (there its memory bounds it); 20 x 12 x 16 28 / 42, 32^3 32 / 41, 48^3 80 / 50 (a 3D
// tile computes 2.8 positions a cell, and many tiles share a CU).
bool ksb_pairs(const GridDev& G)
{
    return (int64_t)G.n[0] * G.n[1] * G.n[2] <= (G.dim == 2 ? 1ll << 20 : 1ll << 15);
}
unsigned ksb_pair_blocks(const GridDev& G)
{
    using T3 = PairTile<true>;
    using T2 = PairTile<false>;
    auto tiles = [](int n, int t) { return (unsigned)((n + t - 1) / t); };
    return G.dim == 3 ? tiles(G.n[0], T3::TX) * tiles(G.n[1], T3::TY) * tiles(G.n[2], T3::TZ)
                      : tiles(G.n[0], T2::TX) * tiles(G.n[1], T2::TY);
}
hipError_t ksb_pair(const KsbDev& K, bool first, hipStream_t st)
{
    if (!ksb_pairs(K.G) || K.conv) return hipErrorInvalidValue;
    if (first)
        ksb_pair_first_kernel<<<ksb_pair_blocks(K.G), kPairBlock, 0, st>>>(K);
    else
        ksb_pair_next_kernel<<<ksb_pair_blocks(K.G), kPairBlock, 0, st>>>(K);
    return hipGetLastError();
}
hipError_t ksb_pass(const KsbDev& K, bool first, hipStream_t st)
{
    if (!ksb_pass_fits(K.G) || K.conv) return hipErrorInvalidValue;
    using T = PassTile<kPassX>;
    KsbDev Z = K;
    const unsigned grid = z_chunks((K.G.n[0] / T::PX) * ((K.G.n[1] + T::PY - 1) / T::PY), K.G.n[2], T::PZ, Z.zc);
    if (first)
        ksb_pass3_kernel<kPassX, true><<<grid, T::PN, 0, st>>>(Z);
    else
        ksb_pass3_kernel<kPassX, false><<<grid, T::PN, 0, st>>>(Z);
    return hipGetLastError();
}
hipError_t scale_fields(const GridDev& G, float* const* F, const float f[3], hipStream_t st)
{
    ScaleArgs a{};
    a.G = G;
    for (int c = 0; c < 6; c++) a.F[c] = F[c];
    for (int c = 0; c < 3; c++) a.f[c] = f[c];
    scale_fields_kernel<<<std::min(nblocks((int64_t)G.n[0] * G.n[1] * G.n[2]), kStrideBlocks), kBlock, 0, st>>>(a);
    return hipGetLastError();
}
hipError_t ksb_finalize(const KsbFin& F, hipStream_t st)
{
    ksb_final_kernel<<<kKsbFinBlocks, kBlock, 0, st>>>(F);
    return hipGetLastError();
}
hipError_t grid_batch(GridBatchKind k, const void* table, UnitMap m, int blocks, int ydim,
                      hipStream_t st)
{
    if (blocks <= 0) return hipSuccess;
    const dim3 grid((unsigned)blocks, (unsigned)ydim);
    switch (k) {
    case kBatchZero: zero_batch<<<grid, kBlock, 0, st>>>(static_cast<const ZeroArgs*>(table), m); break;
    case kBatchFill:
        fill_guards_batch<<<grid, kBlock, 0, st>>>(static_cast<const FillArgs*>(table), m);
        break;
    case kBatchFoldP:
        fold_periodic_batch<<<grid, kBlock, 0, st>>>(static_cast<const FoldPArgs*>(table), m);
        break;
    case kBatchShearFold:
        shear_fold_batch<<<grid, kBlock, 0, st>>>(static_cast<const ShearFoldArgs*>(table), m);
        break;
    case kBatchYeeB: yee_b_batch<<<grid, kBlock, 0, st>>>(static_cast<const MaxwellDev*>(table), m); break;
    case kBatchYeeE: yee_e_batch<<<grid, kBlock, 0, st>>>(static_cast<const MaxwellDev*>(table), m); break;
    case kBatchKsbFirst:
        ksb_first_batch<<<grid, kBlock, 0, st>>>(static_cast<const KsbDev*>(table), m);
        break;
    case kBatchKsbNext: ksb_next_batch<<<grid, kBlock, 0, st>>>(static_cast<const KsbDev*>(table), m); break;
    case kBatchKsbPairFirst:
        ksb_pair_first_batch<<<grid, kPairBlock, 0, st>>>(static_cast<const KsbDev*>(table), m);
        break;
    case kBatchKsbPairNext:
        ksb_pair_next_batch<<<grid, kPairBlock, 0, st>>>(static_cast<const KsbDev*>(table), m);
        break;
    case kBatchKsbFinal: ksb_final_batch<<<grid, kBlock, 0, st>>>(static_cast<const KsbFin*>(table), m); break;
    case kBatchScale: scale_fields_batch<<<grid, kBlock, 0, st>>>(static_cast<const ScaleArgs*>(table), m); break;
    }
    return hipGetLastError();
}

unsigned grid_blocks(int64_t items) { return nblocks(items); }

hipError_t zero_floats(float* p, int64_t n, hipStream_t st)
{
    if (n > 0)
        zero_kernel<<<std::min(nblocks((n + 3) / 4), kStrideBlocks), kBlock, 0, st>>>(
            ZeroArgs{reinterpret_cast<uint32_t*>(p), n});
    return hipGetLastError();
}
hipError_t clear_for_push(const ClearArgs& a, hipStream_t st)
{
    const int ns = a.nm == 0 ? 0 : (a.mcnt[1] ? 2 : 1);
    const unsigned nb = std::min(nblocks((std::max(a.n, a.nm) + 3) / 4), kStrideBlocks / 4);
    clear_kernel<<<dim3(std::max(nb, 1u), 3 + ns), kBlock, 0, st>>>(a);
    return hipGetLastError();
}
hipError_t interior_copy(const GridDev& G, float* const* guarded, float* const* dense, int ncomp, int to_dense,
                         hipStream_t st)
{
    if (ncomp == 0) return hipSuccess;
    Comp6 A{}, D{};
    for (int c = 0; c < ncomp; c++) {
        A.p[c] = guarded[c];
        D.p[c] = dense[c];
    }
    const int64_t per_row = (G.n[0] + 3) / 4;
    const unsigned nb = std::min(nblocks(per_row * G.n[1] * G.n[2]), kStrideBlocks);
    interior_copy_kernel<<<dim3(nb, (unsigned)ncomp), kBlock, 0, st>>>(G, A, D, to_dense, FastDiv::make((uint32_t)per_row));
    return hipGetLastError();
}
hipError_t box_record(const GridDev& G, float* const* comps, const SumArgs& P, double* part, int nblk, BoxRecord* out,
                      hipStream_t st)
{
    Comp6 A{};
    for (int c = 0; c < 6; c++) A.p[c] = comps[c];
    const int rows = 6 + kPartSums * P.nsp;
    field_energy_kernel<<<dim3(nblk, 6), kBlock, 0, st>>>(G, A, part);
    particle_sums_kernel<<<dim3(nblk, (unsigned)P.nsp), kBlock, 0, st>>>(P, part + 6 * nblk);
    box_record_kernel<<<rows + 1, kBlock, 0, st>>>(P, part, rows, nblk, out);
    return hipGetLastError();
}
hipError_t energy_histogram(const int32_t* cell, const float* ux, const float* uy, const float* uz,
                            const int32_t* n_live, const double* edges, int nbins,
                            unsigned long long* counts, hipStream_t st)
{
    zero_kernel<<<nblocks(2 * (nbins + 2)), kBlock, 0, st>>>(
        ZeroArgs{reinterpret_cast<uint32_t*>(counts), (int64_t)2 * (nbins + 2)});
    const size_t lds = (size_t)(nbins + 1) * sizeof(double) + (size_t)(nbins + 2) * sizeof(uint32_t);
    energy_hist_kernel<<<kHistBlocks, kHistBlock, lds, st>>>(cell, ux, uy, uz, n_live, edges, nbins, counts);
    return hipGetLastError();
}

}  // namespace pic

// moments.hip -- moment-space storage of the D3Q27 recursive-regularized
// step (arXiv 2408.15115, App. A): the collided populations are
// C = f0(rho, u) + (1 - 1/tau) f1(P1, u), a function of rho, u and the
// off-equilibrium stress P1 alone, so a cell's post-collision state is fully
// given by ten numbers.  Stored per cell (FP32, SoA [10][nz][ny][nx]):
//   m0 = rho - 1,  m1..3 = rho u,  m4..9 = (1 - 1/tau) P1 as xx, yy, zz, xy, xz, yz.
// The step reads 40 bytes and writes 40 bytes per cell instead of 27 + 27
// populations.  Periodic in x and y; z periodic or bounded by the walls of the
// lattice kernel (free-slip, no-slip at rest or moving in x, constant
// pressure).  Cells forced in the last step carry their equilibrium shift in
// the forcing box of their case (moments.hpp); the expansion applies it.
//
// The step never forms the 27 populations of a cell.  With
//   phi_c(u) = w_c (1 + 3 c u + (9 c^2 - 3) u^2 / 2)     (one dimension)
// the regularized state is
//   C_i = rho phi_x phi_y phi_z + half the second derivatives of phi_x phi_y
//         phi_z along u contracted with (1 - 1/tau) P1,
// a sum of products of one-dimensional factors, and what a cell needs of the
// populations it pulls are ten raw moments.  So the streaming is done one
// dimension at a time, each taking the sums over its own velocity component
// as soon as it has moved the data:
//   x  a cell forms its state as T_c[m_y, m_z], c = -1, 0, 1 populations in x
//      and Hermite coefficients in y and z; T_1 and T_-1 move one cell along
//      x; the sums over c with c^p, p = 0, 1, 2, are taken;
//   y  each goes to populations in y, moves one row and is summed with c^q,
//      p + q <= 2;
//   z  the six remaining sums go to populations in z and are added to the
//      planes z - 1, z and z + 1.
// That is about 350 vector instructions per cell (counted, halo included)
// instead of the 650 of expanding a halo of cells into populations and
// gathering 27 of them.  256 x 256 x 768 takes 0.90 ms alone (1.14 with the
// expansion), of which the arithmetic alone would take 0.55: the step is bound
// by memory.  It reads 1.4 times its 40 bytes per cell (halo rows and side
// columns that have left the L2), and a plain copy that marches like it reaches
// 5.0 TB/s where one in address order reaches 5.8.  With the loads one plane
// ahead instead of two it took 6 % longer.
#include <algorithm>
#include <cmath>

#include "internal.hpp"
#include "lattice.hpp"
#include "moments.hpp"

namespace turret {

namespace mom {
// A workgroup owns a column of at most MX x MY cells and marches through a
// chunk of z planes.  Wave r + 1 holds row y0 + r of a plane, r = -1 .. the
// tile's row count, a cell per lane: the x exchange is a lane shift.  In tiles
// of at most MX - 2 columns lanes hold the columns x0 - 1 and x0 + width too;
// else one more wavefront (the side wave) forms what the columns x0 - 1 and
// x0 + MX pass into the tile, a plane ahead.
constexpr int MX = 64;
constexpr int kRowsLarge = 11, kRowsSmall = 5;   // MY of the two kernels (see moment_plan)

__device__ __forceinline__ int wrap1(int v, int n)
{
    return v < 0 ? v + n : (v >= n ? v - n : v);
}

// Lane i takes lane i - 1's (i + 1's) value; lane 0 (63) takes edge.
__device__ __forceinline__ float from_left(float v, float edge)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float from_right(float v, float edge)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x130, 0xf, 0xf, false));
}

constexpr int kRegular = 0, kNonTemporal = 2;   // cache policies of the buffer stores

// The workgroup's LDS is all that a barrier of the step orders: global loads
// in flight (the next plane's moments) stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// What all three T_c of a cell share.  Coefficients of order one or two in y
// (z) are kept times 3 and everything times 6 per dimension, which turns
// every one-dimensional transform into additions (see to_populations).
struct CellTerms {
    float r1, rho, j, u[3];
    float V, W, V2;                        // 3 u_y, 3 u_z, 3 u_y^2
    float q;                               // rho u_x^2 + P_xx
    float Pyy3, Pzz3, Pxy3, Pxz3, Pyz6;    // multiples of the stored stress
};

__device__ __forceinline__ CellTerms cell_terms(const float m[10])
{
    CellTerms k;
    k.r1 = m[0];
    k.rho = 1.0f + m[0];
    k.j = m[1];
    const float inv = inverse(k.rho);
    k.u[0] = m[1] * inv;
    k.u[1] = m[2] * inv;
    k.u[2] = m[3] * inv;
    k.V = 3.0f * k.u[1];
    k.W = 3.0f * k.u[2];
    k.V2 = k.V * k.u[1];
    k.q = fmaf(m[1], k.u[0], m[4]);
    k.Pyy3 = 3.0f * m[5];
    k.Pzz3 = 3.0f * m[6];
    k.Pxy3 = 3.0f * m[7];
    k.Pxz3 = 3.0f * m[8];
    k.Pyz6 = 6.0f * m[9];
    return k;
}

// T_c[m_y + 3 m_z] of one x velocity: phi, dphi = 6 phi_c(u_x) and its
// derivative, d = 6 times the coefficient of order zero (deviation form), w6
// = 6 w_c.
__device__ __forceinline__ void slab(const CellTerms &k, float phi, float dphi, float d, float w6, float t[9])
{
    const float a = d + w6;
    const float b3 = dphi * k.Pxy3, c3 = dphi * k.Pxz3;
    const float yy3 = phi * k.Pyy3, zz3 = phi * k.Pzz3, yz6 = phi * k.Pyz6;
    t[0] = d;
    t[1] = fmaf(a, k.V, b3);
    t[3] = fmaf(a, k.W, c3);
    t[2] = fmaf(k.u[1], t[1] + b3, yy3);
    t[4] = fmaf(k.W, t[1], fmaf(c3, k.V, 1.5f * yz6));
    t[6] = fmaf(k.u[2], t[3] + c3, zz3);
    const float n = k.V * fmaf(c3, k.u[1], yz6);
    t[5] = fmaf(k.W, t[2], n);
    t[7] = fmaf(k.V, t[6], k.W * fmaf(b3, k.u[2], yz6));
    t[8] = fmaf(k.u[2], t[5] + n, k.V2 * zz3);
}

// The same for velocity c = +1 or -1 (a float, so that it may differ between
// lanes) and for c = 0.
__device__ __forceinline__ void slab_side(const CellTerms &k, float c, float t[9])
{
    const float u = k.u[0];
    slab(k, fmaf(3.0f * u, u + c, 1.0f), fmaf(6.0f, u, 3.0f * c), fmaf(3.0f, fmaf(c, k.j, k.q), k.r1), 1.0f, t);
}
__device__ __forceinline__ void slab_rest(const CellTerms &k, float t[9])
{
    const float u = k.u[0];
    slab(k, fmaf(-6.0f * u, u, 4.0f), -12.0f * u, fmaf(4.0f, k.r1, -6.0f * k.q), 4.0f, t);
}

// A cell forced in the last step (shift sh = (Delta, lambda)): the change of
// its equilibrium part from u to u + Delta, and the first-order term's factor
// lambda; c as above, 0 for the rest velocity.
__device__ __forceinline__ void slab_shift(const CellTerms &k, const float sh[4], float c, float t[9])
{
    const float w6 = c == 0.0f ? 4.0f : 1.0f, e2 = c == 0.0f ? -1.5f : 3.0f;
    const float u = k.u[0], ue = u + sh[0];
    const float phi = k.rho * w6 * fmaf(u, fmaf(e2, u, 3.0f * c), 1.0f);
    const float phe = k.rho * w6 * fmaf(ue, fmaf(e2, ue, 3.0f * c), 1.0f);
    const float y[3] = {1.0f, k.V, k.V * k.u[1]}, z[3] = {1.0f, k.W, k.W * k.u[2]};
    const float vy = k.u[1] + sh[1], vz = k.u[2] + sh[2];
    const float ye[3] = {1.0f, 3.0f * vy, 3.0f * vy * vy}, ze[3] = {1.0f, 3.0f * vz, 3.0f * vz * vz};
    t[0] += k.rho * w6 * sh[0] * fmaf(e2, u + ue, 3.0f * c);
#pragma unroll
    for (int n = 1; n < 9; n++) t[n] += phe * ye[n % 3] * ze[n / 3] - phi * y[n % 3] * z[n / 3];
    const float g = k.rho * (1.0f - sh[3]) * w6;
    t[0] -= 3.0f * c * g * sh[0];
    t[1] -= 3.0f * g * sh[1];
    t[3] -= 3.0f * g * sh[2];
}

// Coefficients (a0, 3 a1, 3 a2) -> 6 x populations at +1 and -1 and 3 x at 0.
__device__ __forceinline__ void to_populations(float a0, float a1, float a2, float &up, float &down, float &rest)
{
    const float s = a0 + a2;
    up = s + a1;
    down = s - a1;
    rest = fmaf(2.0f, a0, -a2);
}
}  // namespace mom

namespace mom {
template <int MY, int POLICY>
struct Exchange {
    static constexpr int kRows = MY, kPolicy = POLICY;   // (the form of the march goes with its LDS)
    float edge[2][2][MY + 2][12];      // the side wave's T into the tile: [plane parity][side][row][9 of 12]
    float up[2][9][MY + 1][MX];    // row r - 1's +1 populations for row r: [plane parity][value][r][x]
    float down[2][9][MY + 1][MX];  // row r + 1's -1 populations for row r: [plane parity][value][r + 1][x]
};

// What the waves of a workgroup share: the tile, the case and its walls.
struct Tiling {
    int nx, ny, nz, z0, sponge, bc_lo, bc_hi;
    int x0, y0, zs, ze, width, rows, lane0;   // lane0: the lane of column x0 (1: the lanes hold the side columns)
    float uw_lo, uw_hi, tau0;
    long long plane;
    const float *s;
    float *d;
    ShiftBox sb;   // forcing shifts of the last correction
    // z walls: planes -1 and nz exist only when z is periodic; physical
    // plane z is stored in ring slot (z + z0) mod nz
    __device__ __forceinline__ bool wlo() const { return bc_lo != BC_PERIODIC; }
    __device__ __forceinline__ bool whi() const { return bc_hi != BC_PERIODIC; }
    __device__ __forceinline__ bool exists(int z) const { return (z >= 0 || !wlo()) && (z < nz || !whi()); }
    __device__ __forceinline__ int slot(int z) const { return wrap1(wrap1(z, nz) + z0, nz); }
    // A chunk without a wall row or a cell of the forcing box (side columns,
    // halo rows and neighbour planes included): its march needs neither test.
    __device__ __forceinline__ bool plain() const
    {
        if ((zs == 0 && wlo()) || (ze == nz && whi())) return false;
        if (!sb.valid) return true;
        // `count` coordinates from `first` on, modulo n, against the box's L from o on
        auto clear = [&](int first, int count, int o, int n) {
            const int rel = wrap1(first - o, n);
            return rel >= sb.L && rel + count <= n;
        };
        return clear(wrap1(x0 - 1, nx), width + 2, sb.o[0], nx) || clear(wrap1(y0 - 1, ny), rows + 2, sb.o[1], ny) ||
               clear(slot(zs - 1), ze - zs + 2, sb.o[2], nz);
    }
};

// Steps through the planes of a chunk: the base of the plane at hand in the
// ring, advanced a plane at a time.
struct PlaneCursor {
    const float *at;
    int slot, nz;
    long long slab;
    __device__ __forceinline__ PlaneCursor(const Tiling &t, const float *base, int z)
        : slot(t.slot(z)), nz(t.nz), slab((long long)t.ny * t.nx)
    {
        at = base + slot * slab;
    }
    __device__ __forceinline__ void advance()
    {
        const bool wrap = ++slot == nz;
        at += wrap ? slab - nz * slab : slab;
        slot = wrap ? 0 : slot;
    }
};

// The moments of the plane's cell at byte offset hoff.
__device__ __forceinline__ void load_plane(const PlaneCursor &c, long long plane, unsigned int hoff, float m[10])
{
    const char *at = (const char *)c.at;
#pragma unroll
    for (int k = 0; k < 10; k++) m[k] = *(const float *)(at + k * 4 * plane + hoff);
}

// Loads run two planes ahead (the memory latency under load is more than the
// work on one plane).  Every iteration issues the same ones: past the chunk's
// last plane, and for a plane that does not exist, an existing one is loaded
// and not used.
struct LoadAhead {
    PlaneCursor c;
    int z, last;   // plane at c; last existing plane of the chunk
    __device__ __forceinline__ LoadAhead(const Tiling &t)
        : c(t, t.s, t.exists(t.zs - 1) ? t.zs - 1 : 0), z(t.exists(t.zs - 1) ? t.zs - 1 : 0),
          last(t.exists(t.ze) ? t.ze : t.ze - 1)
    {
    }
    // on to plane zn, if it is the next one
    __device__ __forceinline__ void to(int zn)
    {
        if (zn > z && z < last) {
            c.advance();
            z++;
        }
    }
};

// The side wave: lane = 32 side + row.  It forms what the columns x0 - 1 and
// x0 + MX pass into the tile, of plane z + 1 while the rows work on plane z.
template <class Lds>
__device__ __forceinline__ void side_march(const Tiling &t, Lds &lds, int lane)
{
    static_assert(Lds::kRows + 2 <= 32, "the side wave holds the rows of one side in 32 lanes");
    if (t.lane0) {   // the lanes of the rows hold these columns
        for (int z = t.zs - 1; z <= t.ze + 1; z++) lds_barrier();
        return;
    }
    const int row = min(lane & 31, t.rows + 1);
    const int gx = lane < 32 ? (t.x0 == 0 ? t.nx - 1 : t.x0 - 1) : (t.x0 + MX) % t.nx;
    const int gy = (t.y0 - 1 + row + t.ny) % t.ny;
    const unsigned int hoff = 4u * (unsigned int)(gy * t.nx + gx);
    const float c = lane < 32 ? 1.0f : -1.0f;
    float m[2][10];
    LoadAhead ahead(t);
    load_plane(ahead.c, t.plane, hoff, m[0]);
    ahead.to(t.zs);
    load_plane(ahead.c, t.plane, hoff, m[1]);
    auto step = [&](int z, float *mz) {
        if (z <= t.ze && t.exists(z)) {
            const CellTerms k = cell_terms(mz);
            float v[9], sh[4];
            slab_side(k, c, v);
            if (shift_at(t.sb, t.nx, t.ny, t.nz, gx, gy, t.slot(z), sh)) slab_shift(k, sh, c, v);
            float *e = lds.edge[z & 1][lane >> 5][row];   // lanes past the rows repeat the last one's values
#pragma unroll
            for (int n = 0; n < 9; n++) e[n] = v[n];
        }
        ahead.to(z + 2);
        load_plane(ahead.c, t.plane, hoff, mz);
        lds_barrier();
    };
    int z = t.zs - 1;
    for (; z <= t.ze; z += 2) {
        step(z, m[0]);
        step(z + 1, m[1]);
    }
    if (z == t.ze + 1) step(z, m[0]);
}

// One row of the tile: the cells y0 + r, r = 0 .. rows - 1, or one of the two
// halo rows r = -1 and rows, which only pass values on.
enum { ROW_BELOW, ROW_INNER, ROW_ABOVE };
template <int KIND, bool PLAIN, class Lds>
__device__ __forceinline__ void row_march(const Tiling &t, Lds &lds, BodyDev &body, int r, int lane)
{
    constexpr bool INNER = KIND == ROW_INNER;
    const int nz = t.nz, wave = r + 1;
    // lanes past the column right of the tile repeat it
    const int col = min(lane - t.lane0, t.width);
    const int gx = (t.x0 + col + t.nx) % t.nx, gy = (t.y0 + r + t.ny) % t.ny;
    const unsigned int hoff = 4u * (unsigned int)(gy * t.nx + gx);
    // byte offset of the lane's cell in an output plane; lanes outside the
    // tile's cells store past the plane's end, which the buffer bounds drop:
    // no branch around the stores, so that the wait for the loads in flight
    // (issued before them) need not include them
    const bool out = lane >= t.lane0 && col < t.width;
    const unsigned int slab_bytes = 4u * (unsigned int)(t.ny * t.nx);
    const unsigned int ooff = out ? hoff : slab_bytes;
    const int shb = PLAIN ? 0 : wrap1(gy - t.sb.o[1], t.ny);   // the row's place in the forcing box
    const float om0 = 1.0f - 1.0f / t.tau0;
    // per unfinished output plane, in the order (p, q) = 00 10 01 20 11 02:
    // next = the +1 populations' sums for plane z + 1; cur = for plane z those
    // of 00, 10 and 01 (they also enter the odd sums in z), the rest of 00,
    // and the totals so far of the others
    float next[6], cur[9], m[2][10];
#pragma unroll
    for (int c = 0; c < 6; c++) next[c] = 0.0f;
#pragma unroll
    for (int c = 0; c < 9; c++) cur[c] = 0.0f;
    PlaneCursor oc(t, t.d, t.zs);   // the plane that the next store goes to
    auto store = [&](const float *mo, unsigned int off) {
#pragma unroll
        for (int c = 0; c < 10; c++)
            __builtin_amdgcn_raw_buffer_store_b32(
                __float_as_uint(mo[c]),
                __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(oc.at) + c * t.plane, 0, (int)slab_bytes, 0x00027000),
                (int)off, 0, Lds::kPolicy);
    };
    LoadAhead ahead(t);
    // (the dropped stores: the loop is then entered, as it is repeated, with
    // the loads of each plane followed by as many stores)
    const float none[10] = {};
    load_plane(ahead.c, t.plane, hoff, m[0]);
    if (INNER) store(none, slab_bytes);
    ahead.to(t.zs);
    load_plane(ahead.c, t.plane, hoff, m[1]);
    if (INNER) store(none, slab_bytes);
    lds_barrier();
    auto step = [&](int z, float *mz) __attribute__((always_inline)) {
        const int par = z & 1;
        const bool have = PLAIN || t.exists(z);   // the same for the whole workgroup
        const bool wall_lo = !PLAIN && z == 0 && t.wlo(), wall_hi = !PLAIN && z == nz - 1 && t.whi();
        float wl[6];      // bounce-back walls: what the wall passes in, unmoved
        float rest[9];    // the row's own y populations at 0, [p + 3 m_z]
        float tp[9], t0[9], tm[9];
        if (have) {
            const CellTerms k = cell_terms(mz);
            slab_side(k, 1.0f, tp);
            slab_rest(k, t0);
            slab_side(k, -1.0f, tm);
            if (!PLAIN && t.sb.valid && shb < t.sb.L && wrap1(t.slot(z) - t.sb.o[2], nz) < t.sb.L) {
                float sh[4];
                if (shift_at(t.sb, t.nx, t.ny, nz, gx, gy, t.slot(z), sh)) {
                    slab_shift(k, sh, 1.0f, tp);
                    slab_shift(k, sh, 0.0f, t0);
                    slab_shift(k, sh, -1.0f, tm);
                }
            }
        }
        ahead.to(z + 2);
        load_plane(ahead.c, t.plane, hoff, mz);
        if (have) {
            if (INNER && ((wall_lo && t.bc_lo != BC_FREESLIP) || (wall_hi && t.bc_hi != BC_FREESLIP))) {
                const int bc = wall_lo ? t.bc_lo : t.bc_hi;
                const float zdir = wall_lo ? -1.0f : 1.0f, sign = bc == BC_PRESSURE ? -1.0f : 1.0f;
                float G[6][3];
#pragma unroll
                for (int n = 0; n < 3; n++) {
                    const float a0 = tp[3 * n] + t0[3 * n] + tm[3 * n], a1 = tp[3 * n + 1] + t0[3 * n + 1] + tm[3 * n + 1],
                                a2 = tp[3 * n + 2] + tm[3 * n + 2];
                    G[0][n] = 6.0f * a0;
                    G[1][n] = -6.0f * (tp[3 * n] - tm[3 * n]);
                    G[2][n] = -2.0f * a1;
                    G[3][n] = 6.0f * (tp[3 * n] + tm[3 * n]);
                    G[4][n] = 2.0f * (tp[3 * n + 1] - tm[3 * n + 1]);
                    G[5][n] = 2.0f * (a0 + a2 + t0[3 * n + 2]);
                }
#pragma unroll
                for (int c = 0; c < 6; c++) wl[c] = sign * (G[c][0] + G[c][2] + zdir * G[c][1]);
                if (bc == BC_NOSLIP) wl[1] += 72.0f * (wall_lo ? t.uw_lo : t.uw_hi);   // 216 times u_w / 3
            }
            // x: move, sum over the x velocity, and on to y populations
            const float *el = lds.edge[par][0][wave], *er = lds.edge[par][1][wave];
#pragma unroll
            for (int n = 0; n < 3; n++) {
                float X[3][3];   // [p][m_y]
#pragma unroll
                for (int y = 0; y < 3; y++) {
                    const float L = from_left(tp[3 * n + y], el[3 * n + y]), R = from_right(tm[3 * n + y], er[3 * n + y]);
                    X[2][y] = L + R;
                    X[1][y] = L - R;
                    X[0][y] = X[2][y] + t0[3 * n + y];
                }
#pragma unroll
                for (int q = 0; q < 3; q++) {
                    float up, down;
                    to_populations(X[q][0], X[q][1], X[q][2], up, down, rest[q + 3 * n]);
                    if (KIND != ROW_ABOVE) lds.up[par][q + 3 * n][r + 1][lane] = up;
                    if (KIND != ROW_BELOW) lds.down[par][q + 3 * n][r][lane] = down;
                }
            }
        }
        lds_barrier();
        if constexpr (INNER) {
            float up[6], down[6], mid[6];
            if (have) {
                // y: sums over the y velocity, and on to z populations
                float G[6][3];
#pragma unroll
                for (int n = 0; n < 3; n++) {
                    float B[3], A[3];
#pragma unroll
                    for (int q = 0; q < 3; q++) {
                        B[q] = lds.up[par][q + 3 * n][r][lane];
                        A[q] = lds.down[par][q + 3 * n][r + 1][lane];
                    }
                    G[5][n] = B[0] + A[0];
                    G[2][n] = B[0] - A[0];
                    G[0][n] = fmaf(2.0f, rest[3 * n], G[5][n]);
                    G[4][n] = B[1] - A[1];
                    G[1][n] = fmaf(2.0f, rest[3 * n + 1], B[1] + A[1]);
                    G[3][n] = fmaf(2.0f, rest[3 * n + 2], B[2] + A[2]);
                }
#pragma unroll
                for (int c = 0; c < 6; c++) to_populations(G[c][0], G[c][1], G[c][2], up[c], down[c], mid[c]);
            } else {
                // beyond the top wall: what the wall passes into plane z - 1
#pragma unroll
                for (int c = 0; c < 6; c++) {
                    down[c] = next[c];
                    up[c] = mid[c] = 0.0f;
                }
            }
            // plane z - 1 is complete (from the chunk's third plane on)
            const bool stored = z > t.zs;
            constexpr float F = 1.0f / 216.0f;
            Moments rm;
            const float zz = cur[0] + down[0];
            rm.r1 = F * fmaf(2.0f, cur[3], zz);
            rm.j[0] = F * (cur[4] + down[1]);
            rm.j[1] = F * (cur[5] + down[2]);
            rm.j[2] = F * (cur[0] - down[0]);
            rm.pxx = F * (cur[6] + down[3]);
            rm.pyy = F * (cur[8] + down[5]);
            rm.pzz = F * zz;
            rm.pxy = F * (cur[7] + down[4]);
            rm.pxz = F * (cur[1] - down[1]);
            rm.pyz = F * (cur[2] - down[2]);
            float om = om0;
            if (t.sponge >= 2 && z - 1 >= nz - t.sponge) om = 1.0f - 1.0f / tau_at(t.tau0, nz, t.sponge, z - 1);
            float mo[10];
            bool bad;
            collide_to_moments(rm, om, mo, bad);
            const unsigned long long bm = __ballot(bad && stored && out);
            if (bm != 0ull && lane == __ffsll((unsigned long long)bm) - 1) atomicOr(&body.err, 4);
            store(mo, stored ? ooff : slab_bytes);
            if (stored) oc.advance();
            if (wall_lo)
#pragma unroll
                for (int c = 0; c < 6; c++) next[c] = t.bc_lo == BC_FREESLIP ? down[c] : wl[c];
#pragma unroll
            for (int c = 0; c < 3; c++) cur[c] = next[c];
            cur[3] = mid[0];
#pragma unroll
            for (int c = 1; c < 6; c++) cur[3 + c] = fmaf(2.0f, mid[c], next[c]);
#pragma unroll
            for (int c = 0; c < 6; c++) next[c] = wall_hi && t.bc_hi != BC_FREESLIP ? wl[c] : up[c];
        }
    };
    int z = t.zs - 1;
    for (; z < t.ze; z += 2) {
        step(z, m[0]);
        step(z + 1, m[1]);
    }
    if (z == t.ze) step(z, m[0]);
}

template <bool PLAIN, class Lds>
__device__ __forceinline__ void march(const Tiling &t, Lds &lds, BodyDev &body)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int r = wave - 1;
    if (wave == Lds::kRows + 2) side_march(t, lds, lane);
    else if (r < 0) row_march<ROW_BELOW, PLAIN>(t, lds, body, r, lane);
    else if (r < t.rows) row_march<ROW_INNER, PLAIN>(t, lds, body, r, lane);
    else if (r == t.rows) row_march<ROW_ABOVE, PLAIN>(t, lds, body, r, lane);
    else
        for (int z = t.zs - 1; z <= t.ze + 1; z++) lds_barrier();   // a tile of fewer rows
}
}  // namespace mom

// Tile t of a case: x fastest, then y, then the z chunk.  Workgroups are
// spread over the 8 XCDs round-robin; block b takes table entry
// (b mod 8) * ceil(n / 8) + b / 8, so that each XCD's L2 serves a contiguous
// run of neighbouring tiles and their shared halo rows.
//
// Output plane o takes population i from plane o - xi_z, so plane z feeds
// z - 1 (complete then), z and z + 1; what is known of the two unfinished
// planes stays in registers.  At a z wall the populations from outside are
// formed when the plane of the boundary row is there: free-slip, the plane's
// own opposite z direction, already moved along x and y; no-slip and constant
// pressure, the cell's own opposite direction, unmoved (no-slip plus the
// moving wall's momentum, constant pressure with the sign reversed).
template <int MY, int POLICY>
__global__ void __launch_bounds__(64 * (MY + 3)) k_moment_step(const float *__restrict__ src, float *__restrict__ dst,
                                                               DevPtrs p, int ntiles)
{
    using namespace mom;
    __shared__ Exchange<MY, POLICY> lds;
    const int b = blockIdx.x;
    const int ti = (b & 7) * ((ntiles + 7) >> 3) + (b >> 3);
    if (ti >= ntiles) return;
    const Tile tl = p.tiles[ti];
    const CaseDev &cd = p.cases[tl.c];
    BodyDev &body = p.body[tl.c];
    if (body.err != 0) return;
    Tiling t;
    t.nx = cd.nx;
    t.ny = cd.ny;
    t.nz = cd.nz;
    t.z0 = body.z0;
    const MomentTiles &mt = cd.mom;
    t.x0 = (tl.first % mt.ntx) * mt.width;
    t.y0 = ((tl.first / mt.ntx) % mt.nty) * mt.rows;
    t.zs = (tl.first / (mt.ntx * mt.nty)) * mt.planes;
    t.ze = min(t.zs + mt.planes, t.nz);
    t.width = min(mt.width, t.nx - t.x0);
    t.rows = min(mt.rows, t.ny - t.y0);
    t.lane0 = mt.width <= MX - 2 ? 1 : 0;
    t.sponge = cd.sponge;
    t.bc_lo = cd.bc_lo;
    t.bc_hi = cd.bc_hi;
    t.uw_lo = cd.uw_lo;
    t.uw_hi = cd.uw_hi;
    t.tau0 = cd.tau0;
    t.plane = cd.plane;
    t.s = src + cd.pop_off;
    t.d = dst + cd.pop_off;
    t.sb = shift_box(p, cd, body);
    if (t.plain()) march<true>(t, lds, body);
    else march<false>(t, lds, body);
}

// Moments (and forcing shifts) -> population deviations of case c, layout
// [27][plane] in the ring order of the storage.
__global__ void __launch_bounds__(256) k_moments_expand(const float *__restrict__ src, float *__restrict__ dst,
                                                        DevPtrs p, int c)
{
    const CaseDev cd = p.cases[c];
    const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (i >= cd.cells) return;
    const long long plane = cd.plane;
    const int x = (int)(i % cd.nx), y = (int)((i / cd.nx) % cd.ny), zs = (int)(i / ((long long)cd.nx * cd.ny));
    const mom::ShiftBox sb = mom::shift_box(p, cd, p.body[c]);
    float m[10], sh[4], out[Q];
#pragma unroll
    for (int k = 0; k < 10; k++) m[k] = src[k * plane + i];
    (void)mom::shift_at(sb, cd.nx, cd.ny, cd.nz, x, y, zs, sh);
    mom::expand(m, sh, out);
#pragma unroll
    for (int k = 0; k < Q; k++) dst[k * plane + i] = out[k];
}

// Population deviations of post-collision states -> stored moments: rho - 1,
// rho u and the off-equilibrium stress about f0(rho, u).  Exact for
// regularized states; any other state is replaced by its regularized part.
__global__ void __launch_bounds__(256) k_moments_project(const float *__restrict__ src, float *__restrict__ dst,
                                                         long long plane, long long cells)
{
    const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (i >= cells) return;
    float g[Q], m[10];
#pragma unroll
    for (int k = 0; k < Q; k++) g[k] = src[k * plane + i];
    bool bad;
    mom::collide_to_moments(raw_moments(g), 1.0f, m, bad);
#pragma unroll
    for (int k = 0; k < 10; k++) dst[k * plane + i] = m[k];
}

// The column tiles of a case for a row capacity: the least number of tiles
// that covers it, of even widths and heights.  Where even widths leave two
// lanes of a wave free those hold the side columns (150 columns: three tiles
// of 50 instead of 64 + 64 + 22).
static MomentTiles moment_tiling(int nx, int ny, int nz, int cap, int planes)
{
    auto up = [](int a, int b) { return (a + b - 1) / b; };
    MomentTiles m;
    m.cap = cap;
    m.ntx = up(nx, mom::MX);
    m.width = up(nx, mom::MX - 2) == m.ntx ? up(nx, m.ntx) : mom::MX;
    m.ntx = up(nx, m.width);
    m.rows = up(ny, up(ny, cap));
    m.nty = up(ny, m.rows);
    m.planes = up(nz, up(nz, planes));
    m.ntz = up(nz, m.planes);
    return m;
}

// Row capacity (11 rows: one workgroup of 14 waves per CU; 5 rows: two of 8)
// and planes per chunk, for all cases of a context together: the least
// estimate of a step's time.  A workgroup takes planes + 3 turns; a turn of
// rows + 2 row waves takes about 2.1 us x (rows + 2) / 15 on a CU to itself
// and 1.15 us x (rows + 2) / 7 per workgroup of the small kind (measured on
// boxes that fill few CUs).  The memory's time is that of each plane written
// once and read once with its halo, at 5 TB/s.  Long chunks and 11 rows read
// least: 256 x 256 x 768 takes 0.90 ms with 11 rows, 0.94 with 5; short chunks
// and 5 rows fill the chip: 64^3 takes 13 us with 5 rows and 6 planes, 65 with
// 11 rows and 32.  (13 rows, a full register file, are 3 % faster alone but
// leave the coupling no room beside them.)  With bodies the coupling's kernels
// run beside the step: a step of one workgroup per CU then leaves an eighth
// of the CUs (150 x 131 x 211: 159 us with 216 workgroups, 183 with 324).
void moment_plan(CaseDev *cd, int n, bool bodies)
{
    const double cus = bodies ? 224.0 : 256.0;
    double best = 0.0;
    int cap = 0, planes = 0;
    for (int r : {mom::kRowsLarge, mom::kRowsSmall})
        for (int lz : {4, 6, 8, 10, 12, 16, 20, 24, 32, 36, 40, 48, 64, 96}) {
            double wgs = 0.0, turns = 0.0, bytes = 0.0;
            for (int c = 0; c < n; c++) {
                const MomentTiles m = moment_tiling(cd[c].nx, cd[c].ny, cd[c].nz, r, lz);
                const double w = (double)m.ntx * m.nty * m.ntz;
                wgs += w;
                turns += w * (m.planes + 3) * (m.rows + 2);
                bytes += 40.0 * cd[c].cells * (1.0 + (m.rows + 2.0) / m.rows * (m.planes + 2.0) / m.planes);
            }
            const double turn = r == mom::kRowsLarge ? 2.1 / 15 : 1.15 / 7;
            const double compute = std::ceil(wgs / cus) * (turns / wgs) * turn, memory = bytes / 5e6;   // us
            const double t = std::max(compute, memory) + 0.25 * std::min(compute, memory);
            if (cap == 0 || t < best) {
                best = t;
                cap = r;
                planes = lz;
            }
        }
    for (int c = 0; c < n; c++) cd[c].mom = moment_tiling(cd[c].nx, cd[c].ny, cd[c].nz, cap, planes);
}

hipError_t launch_moment_step(const void *src, void *dst, const DevPtrs &p, int ntiles, int cap, int keep, hipStream_t s)
{
    const dim3 grid((ntiles + 7) / 8 * 8);
    const float *a = (const float *)src;
    float *b = (float *)dst;
    auto launch = [&](auto rows, auto policy) {
        constexpr int MY = decltype(rows)::value, POLICY = decltype(policy)::value;
        hipLaunchKernelGGL((k_moment_step<MY, POLICY>), grid, dim3(64 * (MY + 3)), 0, s, a, b, p, ntiles);
    };
    const std::integral_constant<int, mom::kRowsLarge> large;
    const std::integral_constant<int, mom::kRowsSmall> small;
    const std::integral_constant<int, mom::kRegular> regular;
    const std::integral_constant<int, mom::kNonTemporal> streamed;
    if (cap == mom::kRowsLarge) keep ? launch(large, regular) : launch(large, streamed);
    else keep ? launch(small, regular) : launch(small, streamed);
    return hipGetLastError();
}

hipError_t launch_moments_expand(const float *src, float *dst, const DevPtrs &p, int c, hipStream_t s)
{
    CaseDev cd;
    hipError_t e = hipMemcpy(&cd, p.cases + c, sizeof cd, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return e;
    const long long grid = (cd.cells + 255) / 256;
    hipLaunchKernelGGL(k_moments_expand, dim3((unsigned)grid), dim3(256), 0, s, src, dst, p, c);
    return hipGetLastError();
}

hipError_t launch_moments_expand_n(const float *src, float *dst, const DevPtrs &p, int c, long long cells,
                                   hipStream_t s)
{
    const long long grid = (cells + 255) / 256;
    hipLaunchKernelGGL(k_moments_expand, dim3((unsigned)grid), dim3(256), 0, s, src, dst, p, c);
    return hipGetLastError();
}

hipError_t launch_moments_project(const float *src, float *dst, long long plane, long long cells, hipStream_t s)
{
    const long long grid = (cells + 255) / 256;
    hipLaunchKernelGGL(k_moments_project, dim3((unsigned)grid), dim3(256), 0, s, src, dst, plane, cells);
    return hipGetLastError();
}

}  // namespace turret

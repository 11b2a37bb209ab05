// kernels.hip -- gfx950 kernels of the settling-particle time step
// (arXiv 2408.15115, Sec. 2) other than the lattice kernel (stream_collide.hip),
// and their stream launchers.
//
//   k_body_advance        Sec. 2.3: leapfrog / predictor-corrector, FP64
//   k_markers             Sec. 2.3: marker position, normal and rigid velocity;
//                         tile boxes and the marks of the cells they cover
//   k_region_gather       Sec. 2.1 stress and Sec. 2.2 u* on the particle region
//   k_interp_force_tiles  Sec. 2.2: l = 0 interpolation and the stress integral
//                         (+ the first spread); the last tile of a case forms
//                         its FP64 force / torque totals in a fixed order
//   k_spread_tiles        Sec. 2.2 spreading (deterministic fixed-point atomics)
//   k_interp_update_tiles Sec. 2.2 interpolation of u* + H and the residual
//                         (+ the next cycle's spread)
//   k_correct             Sec. 2.2 forced rule: add f0(u + tau h) - f0(u)
//   k_window_*            Sec. 2.5 re-injection as a ring-origin shift
//
// IBM kernels give one 64-lane wavefront to each marker: lane l is the
// stencil node (l & 3, (l >> 2) & 3, l >> 4) of the 4 x 4 x 4 weight support;
// a workgroup takes one tile of nearby markers and stages their common box of
// region cells in LDS.
#include <algorithm>

#include "internal.hpp"
#include "lattice.hpp"
#include "fine.hpp"
#include "pull.hpp"
#include "mlp.hpp"
#include "moments.hpp"
#include "worklist.hpp"
#include <type_traits>

// Register budget of the coupling's kernels (the reason stands at the tile kernels).
#define EIGHT_WAVES __attribute__((amdgpu_waves_per_eu(8, 8)))

namespace turret {


// ---------------------------------------------------------------- body
__device__ inline void cross3(const double a[3], const double b[3], double c[3])
{
    c[0] = a[1] * b[2] - a[2] * b[1];
    c[1] = a[2] * b[0] - a[0] * b[2];
    c[2] = a[0] * b[1] - a[1] * b[0];
}

__device__ inline void inverse3(const double A[9], double B[9])
{
    const double c00 = A[4] * A[8] - A[5] * A[7];
    const double c01 = A[5] * A[6] - A[3] * A[8];
    const double c02 = A[3] * A[7] - A[4] * A[6];
    const double inv = 1.0 / (A[0] * c00 + A[1] * c01 + A[2] * c02);
    B[0] = c00 * inv;
    B[1] = (A[2] * A[7] - A[1] * A[8]) * inv;
    B[2] = (A[1] * A[5] - A[2] * A[4]) * inv;
    B[3] = c01 * inv;
    B[4] = (A[0] * A[8] - A[2] * A[6]) * inv;
    B[5] = (A[2] * A[3] - A[0] * A[5]) * inv;
    B[6] = c02 * inv;
    B[7] = (A[1] * A[6] - A[0] * A[7]) * inv;
    B[8] = (A[0] * A[4] - A[1] * A[3]) * inv;
}

__device__ inline void mv3(const double A[9], const double x[3], double y[3])
{
#pragma unroll
    for (int a = 0; a < 3; a++) y[a] = A[3 * a] * x[0] + A[3 * a + 1] * x[1] + A[3 * a + 2] * x[2];
}

// Sec. 2.3 leapfrog with F(t), T(t): a = g + F/(kappa V), v(t+1/2), r(t+1);
// w(t+1/2) through M^-1 (J/m)^-1 M with the fluid torque plus the body's
// constant external torque; orientation predictor-corrector.  Then the IBM
// region origin for the new position.
__device__ inline void body_advance_case(const DevPtrs &p, int c)
{
    const CaseDev &cd = p.cases[c];
    BodyDev &B = p.body[c];
    // every field first, in one round of loads (no short-circuit between the
    // two tests, so both loads issue together), then the arithmetic, then the
    // stores
    const int M = cd.M, err = B.err;
    if ((M == 0) | (err != 0)) return;
    const double kappa = B.kappa, vol = B.vol, grav = B.gravity, Rb = B.Rb;
    double F[3], T[3], Te[3], v[3], r[3], w[3], d[9], J[9];
#pragma unroll
    for (int k = 0; k < 3; k++) {
        F[k] = B.F[k];
        T[k] = B.T[k];
        Te[k] = B.Text[k];
        v[k] = B.v[k];
        r[k] = B.r[k];
        w[k] = B.w[k];
    }
#pragma unroll
    for (int k = 0; k < 9; k++) {
        d[k] = B.d[k];
        J[k] = B.Jm_inv[k];
    }
    const int steps = B.steps;
    const double kv = kappa * vol;
    const double a[3] = {F[0] / kv, F[1] / kv, F[2] / kv - grav};
#pragma unroll
    for (int k = 0; k < 3; k++) {
        v[k] += a[k];
        r[k] += v[k];
    }
    double Minv[9], t1[3], t2[3], t3[3];
    inverse3(d, Minv);
    const double Ttot[3] = {T[0] + Te[0], T[1] + Te[1], T[2] + Te[2]};
    mv3(d, Ttot, t1);
    mv3(J, t1, t2);
    mv3(Minv, t2, t3);
#pragma unroll
    for (int k = 0; k < 3; k++) w[k] += t3[k] / kv;
#pragma unroll
    for (int i = 0; i < 3; i++) {
        double di[3] = {d[3 * i], d[3 * i + 1], d[3 * i + 2]}, wd[3], mid[3], wm[3];
        cross3(w, di, wd);
#pragma unroll
        for (int k = 0; k < 3; k++) mid[k] = 0.5 * (di[k] + (di[k] + wd[k]));
        cross3(w, mid, wm);
#pragma unroll
        for (int k = 0; k < 3; k++) d[3 * i + k] = di[k] + wm[k];
    }
#pragma unroll
    for (int k = 0; k < 3; k++) {
        B.v[k] = v[k];
        B.r[k] = r[k];
        B.w[k] = w[k];
        B.org[k] = (int)floor(r[k] - Rb) - 2;
    }
#pragma unroll
    for (int k = 0; k < 9; k++) B.d[k] = d[k];
    B.steps = steps + 1;
}

__global__ void k_body_advance(DevPtrs p, int n_cases)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < n_cases) body_advance_case(p, c);
}

// X_k = r + sum_j xb_kj d_j, n_k = sum_j nb_kj d_j, U_k = v + w x (X_k - r).
// The body fields the region and marker kernels read, copied into registers
// at a kernel's start: after the kernel's first global store the compiler
// must assume the body record may have changed and would reload each field
// with a vector load and a wait of its own.
struct BodyView {
    int err, active;
    int org[3];
    int z0;
    double r[3];
};

__device__ inline BodyView body_view(const BodyDev &B)
{
    BodyView v;
    v.err = B.err;
    v.active = B.active;
    v.z0 = B.z0;
#pragma unroll
    for (int d = 0; d < 3; d++) {
        v.org[d] = B.org[d];
        v.r[d] = B.r[d];
    }
    return v;
}

// The window test of Sec. 2.5 at the body's height rz.
__device__ inline bool window_shifts(const CaseDev &cd, double rz)
{
    return cd.M > 0 && cd.dz > 0 && cd.h_end > 0.0 && rz < cd.h_end;
}

// Moment storage: the tag that selects the moment forms of the region gather,
// the correction and the window reset.
struct CodecMom {
    using T = float;
};

// Moment storage, first pass of the region gather: the collided populations
// (forcing shifts included) of the cells that the gather pulls from (marked by
// k_markers in the region with a one-cell rim, edge E = L + 2), into rpop.  Rim
// planes beyond a z wall are never pulled and are left alone.
__global__ void __launch_bounds__(256) EIGHT_WAVES k_region_expand_mom(const float *__restrict__ src, DevPtrs p)
{
    __shared__ ScanList list;
    const int c = blockIdx.y;
    const CaseDev cd = p.cases[c];
    const BodyView B = body_view(p.body[c]);
    const int E = cd.L + 2, E3 = E * E * E, first = blockIdx.x * 256;
    if (cd.M == 0 || first >= E3) return;
    unsigned char *mk = p.xmark + cd.xreg_off;
    const int q = scan_cells(list, first, E3, B.err, [&](int i) { return mk[i]; });
    if (q < 0) return;
    mk[q] = 0;
    const int a = q % E, b = (q / E) % E, cc = q / (E * E);
    int z = B.org[2] - 1 + cc;
    if (z < 0 || z >= cd.nz) {
        if (cd.bc_lo != BC_PERIODIC) return;
        z = wrapi(z, cd.nz);
    }
    const int x = wrapi(B.org[0] - 1 + a, cd.nx), y = wrapi(B.org[1] - 1 + b, cd.ny);
    int slot = z + B.z0;
    if (slot >= cd.nz) slot -= cd.nz;
    const float *sp = src + cd.pop_off + ((long long)slot * cd.ny + y) * cd.nx + x;
    float m[10], sh[4], out[Q];
#pragma unroll
    for (int i = 0; i < 10; i++) m[i] = sp[i * cd.plane];
    (void)mom::shift_at(mom::shift_box(p, cd, p.body[c]), cd.nx, cd.ny, cd.nz, x, y, slot, sh);
    mom::expand(m, sh, out);
    float *dst = p.rpop + cd.xreg_off + q;
#pragma unroll
    for (int i = 0; i < Q; i++) dst[i * p.xstride] = out[i];
}

// Second pass: the pull of pull() from the expanded region, for region cell
// (a, b, cc) at physical height z, with the same z wall rules.
__device__ inline void pull_region(const DevPtrs &p, const CaseDev &cd, int a, int b, int cc, int z, float g[Q])
{
    const int E = cd.L + 2;
    const float *R = p.rpop + cd.xreg_off;
    const int cell = ((cc + 1) * E + b + 1) * E + a + 1;
    Unroll<0, Q>::run([&](auto I) {
        constexpr int i = decltype(I)::value;
        g[i] = R[i * p.xstride + (cell - (cz(i) * E + cy(i)) * E - cx(i))];
    });
    // cells at a wall: the populations that come from beyond it again
    const bool wlo = z == 0 && cd.bc_lo != BC_PERIODIC, whi = z == cd.nz - 1 && cd.bc_hi != BC_PERIODIC;
    if (!wlo && !whi) return;
    Unroll<0, Q>::run([&](auto I) {
        constexpr int i = decltype(I)::value;
        if constexpr (cz(i) != 0) {
            if (!(cz(i) == 1 ? wlo : whi)) return;
            const int bc = cz(i) == 1 ? cd.bc_lo : cd.bc_hi;
            if (bc == BC_FREESLIP) {
                g[i] = R[mirror_z(i) * p.xstride + (cell - cy(i) * E - cx(i))];
                return;
            }
            const float v = R[opposite(i) * p.xstride + cell];
            if (bc == BC_PRESSURE) g[i] = -v;
            else if constexpr (cx(i) != 0) g[i] = v + wall_momentum<i>(cz(i) == 1 ? cd.uw_lo : cd.uw_hi);
            else g[i] = v;
        }
    });
}

// ------------------------------------------------------------ region fields
// For every marked cell of the particle region (inside some tile's stencil box;
// the others are read by no interpolation and carry no force): pull f(t+1) from
// the buffer the lattice kernel read, then rho - 1, u* = sum xi f / sum f and
// the stress sigma = -p I + (1/(2 tau) - 1) P1 with p = cs^2 (rho - 1)
// (Sec. 2.1).  Also clears the cells' fixed-point immersed-force accumulators
// and the marks of the force-surface points (the correction clears the others).
// One region cell; fetch(cd, x, y, z, g) gives the populations pulled by the
// cell at (x, y, z).
template <class Fetch>
__device__ __forceinline__ void gather_cell(const DevPtrs &p, const CaseDev &cd, const int org[3], int q, Fetch &&fetch)
{
    const int L = cd.L, L3 = L * L * L;
    float *R = p.reg + cd.reg_off * kRegFields;
    long long *H = p.H + cd.reg_off * 3;
    p.mark2[cd.reg_off + q] = 0;
#pragma unroll
    for (int j = 0; j < kHBufs; j++) {
        H[j * p.hstride + q] = 0;
        H[j * p.hstride + L3 + q] = 0;
        H[j * p.hstride + 2 * L3 + q] = 0;
    }
    const int a = q % L, b = (q / L) % L, cc = q / (L * L);
    const int gz = org[2] + cc;
    if (gz < 0 || gz >= cd.nz) {
#pragma unroll
        for (int f = 0; f < kRegFields; f++) R[f * L3 + q] = 0.0f;
        return;
    }
    float g[Q];
    fetch(a, b, cc, gz, g);
    const Macro M = macro(raw_moments(g));
    const float tau = tau_at(cd.tau0, cd.nz, cd.sponge, gz);
    const float fac = 0.5f / tau - 1.0f;
    const float pr = CS2 * M.r1;
    R[0 * L3 + q] = M.r1;
    R[1 * L3 + q] = M.u[0];
    R[2 * L3 + q] = M.u[1];
    R[3 * L3 + q] = M.u[2];
    R[4 * L3 + q] = -pr + fac * M.P[0][0];
    R[5 * L3 + q] = -pr + fac * M.P[1][1];
    R[6 * L3 + q] = -pr + fac * M.P[2][2];
    R[7 * L3 + q] = fac * M.P[0][1];
    R[8 * L3 + q] = fac * M.P[0][2];
    R[9 * L3 + q] = fac * M.P[1][2];
}

// src: the buffer the lattice kernel read (moment storage: unused, the cells
// pull from the expanded region).
template <class CD>
__global__ void __launch_bounds__(256) EIGHT_WAVES k_region_gather(const typename CD::T *__restrict__ src, DevPtrs p, int sid)
{
    __shared__ ScanList list;
    const int c = blockIdx.y;
    const CaseDev cd = p.cases[c];
    const BodyView B = body_view(p.body[c]);
    const int L3 = cd.L * cd.L * cd.L, first = blockIdx.x * 256;
    if (cd.M == 0 || first >= L3) return;
    const int q = scan_cells(list, first, L3, B.err, [&](int i) { return p.mark[cd.reg_off + i] | p.mark2[cd.reg_off + i]; });
    if (q < 0) return;
    gather_cell(p, cd, B.org, q, [&](int a, int b, int cc, int gz, float g[Q]) {
        if constexpr (std::is_same<CD, CodecMom>::value) {
            pull_region(p, cd, a, b, cc, gz, g);
        } else {
            const int gx = wrapi(B.org[0] + a, cd.nx), gy = wrapi(B.org[1] + b, cd.ny);
            if constexpr (!std::is_same<CD, CodecF32>::value) {
                if (cd.LB[0] > 0) {
                    // reduced-precision store with a full-precision box around the body
                    const BodyDev &Bd = p.body[c];
                    const int fo[3] = {Bd.fo[sid][0], Bd.fo[sid][1], Bd.fo[sid][2]};
                    pull_fine<CD>(src + cd.pop_off, Bd.fvalid[sid] ? p.fine[sid] + cd.fine_off : nullptr, cd, B.z0, fo, gx,
                                  gy, gz, g);
                    return;
                }
            }
            pull<CD, true>(src + cd.pop_off, cd.plane, cd.nx, cd.ny, cd.nz, B.z0, cd.bc_lo, cd.bc_hi, cd.uw_lo, cd.uw_hi, gx, gy,
                     gz, g);
        }
    });
}

// --------------------------------------------------------- marker stencils
// One-dimensional four-point weight function of Sec. 2.2 (two branches).
// Written without branches (one square root per call): the lanes of a
// stencil fall on both branches.
__device__ inline double phi4(double r)
{
    const double a = fabs(r);
    const bool inner = a <= 1.0;
    const double arg = inner ? 1.0 + 4.0 * a - 4.0 * a * a : -7.0 + 12.0 * a - 4.0 * a * a;
    const double sq = sqrt(fmax(arg, 0.0));   // arg >= 1 wherever the value is used
    const double v = inner ? 0.125 * (3.0 - 2.0 * a + sq) : 0.125 * (5.0 - 2.0 * a - sq);
    return a <= 2.0 ? v : 0.0;
}

struct Node {
    int q;        // region cell index, -1 if outside the region
    double W;     // tensor-product weight
};

__device__ inline Node stencil_node(const double X[3], int lane, const CaseDev &cd, const int org[3])
{
    const int off[3] = {lane & 3, (lane >> 2) & 3, lane >> 4};
    const int n[3] = {cd.nx, cd.ny, cd.nz};
    const int L = cd.L;
    Node nd;
    nd.W = 1.0;
    int r[3];
    bool ok = true;
#pragma unroll
    for (int d = 0; d < 3; d++) {
        const int node = (int)floor(X[d]) - 1 + off[d];
        nd.W *= phi4((double)node - X[d]);
        int rel = node - org[d];
        if (d < 2) rel = wrapi(rel, n[d]);
        ok = ok && rel >= 0 && rel < L;
        r[d] = rel;
    }
    nd.q = ok ? r[0] + L * (r[1] + L * r[2]) : -1;
    return nd;
}

// v + the value of the lane that the DPP pattern CTRL pairs with this one
// (both 32-bit halves moved by DPP; no LDS traffic).
template <int CTRL>
__device__ inline double dpp_pair_add(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, false);
    return v + __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ inline double lane_value(double v, int l)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sum over a row of 16 lanes (all active), the same bits in every lane of
// the row: pairs (lane ^ 1), quads (lane ^ 2), half rows (mirror of 8) and
// rows (mirror of 16); each step adds the same two operands in both lanes of
// a pair, so the row ends uniform.
__device__ inline double row_sum(double v)
{
    v = dpp_pair_add<0xB1>(v);    // quad_perm [1, 0, 3, 2]
    v = dpp_pair_add<0x4E>(v);    // quad_perm [2, 3, 0, 1]
    v = dpp_pair_add<0x141>(v);   // row_half_mirror
    v = dpp_pair_add<0x140>(v);   // row_mirror
    return v;
}

// Sum over the 64 lanes of a wavefront (all active), the same bits in every
// lane: row sums, then the four row totals in a fixed order.
__device__ inline double wave_sum(double v)
{
    v = row_sum(v);
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// ------------------------------------------------------------ marker tiles
// One workgroup per marker tile (markers close together on the body): the
// tile's stencils share a box of region cells.  Interpolations stage the
// box's fields in LDS once and read every stencil node from there; spreading
// accumulates into an LDS copy of the box (int64 fixed point) and adds each
// touched cell to HBM once.  A box larger than kBoxCells (not expected for
// the tile span) falls back to per-node HBM access.
// Tile handled by workgroup b: the dispatcher deals workgroups round-robin
// over the 8 XCDs, so consecutive blocks are spread and each XCD is given a
// contiguous (Morton-ordered, hence spatially compact) run of tiles whose
// boxes overlap inside one L2.  The grid is padded to a multiple of 8.
__device__ inline int tile_of_block(int b, int n)
{
    const int per = (n + 7) >> 3;
    return (b & 7) * per + (b >> 3);
}

// Box-local index of a lane's stencil node and its weight W = (w_x w_y) w_z
// from the marker's one-dimensional weights w[4 d + o] (k_markers evaluates
// them once per step).
__device__ inline int box_node_w(const double X[3], const double *w, int lane, const TileBox &b, double &W)
{
    const int off[3] = {lane & 3, (lane >> 2) & 3, lane >> 4};
    int r[3];
    W = 1.0;
#pragma unroll
    for (int d = 0; d < 3; d++) {
        const int node = (int)floor(X[d]) - 1 + off[d];
        W *= w[4 * d + off[d]];
        r[d] = node - b.lo[d];
    }
    return r[0] + b.e[0] * (r[1] + b.e[1] * r[2]);
}

// Lane layout of the interpolation passes: thread t takes marker t / 16 of
// the tile and the stencil column (t & 3, (t >> 2) & 3); its nodes are the
// four z levels of that column.  A row of 16 lanes is one marker, so the
// stencil sums are row sums and the tile's markers run side by side.
static_assert(kTileMarkers * 16 == 256, "one workgroup row of 16 lanes per tile marker");
struct Column {
    int i[4];       // box cells of the four nodes (box path)
    int q[4];       // region cells of the four nodes (per-node path; -1 outside)
    double W[4];    // node weights
};

// The column's nodes: in a box that fits from the column's one-dimensional
// weights w(x, y, z level) = wx, wy, wz[4] (W = (w_x w_y) w_z, the product order
// of box_node_w), else from stencil_node.
__device__ inline Column column_nodes(const DevPtrs &p, const double X[3], double wx, double wy, const double wz[4], int col,
                                      const TileBox &tb)
{
    Column cn;
    const int cx = col & 3, cy = col >> 2;
    if (tb.fits) {
        const double wxy = wx * wy;
        const int b0 = ((int)floor(X[0]) - 1 + cx - tb.lo[0]) +
                       tb.e[0] * (((int)floor(X[1]) - 1 + cy - tb.lo[1]) + tb.e[1] * ((int)floor(X[2]) - 1 - tb.lo[2]));
#pragma unroll
        for (int z = 0; z < 4; z++) {
            cn.W[z] = wxy * wz[z];
            cn.i[z] = b0 + z * tb.e[0] * tb.e[1];
            cn.q[z] = -1;
        }
    } else {
#pragma unroll
        for (int z = 0; z < 4; z++) {
            const Node nd = stencil_node(X, col + 16 * z, p.cases[tb.c], p.body[tb.c].org);
            cn.W[z] = nd.W;
            cn.q[z] = nd.q;
            cn.i[z] = 0;
        }
    }
    return cn;
}

// Region cell index of cell i of a box that fits (quotients by the
// multiplication that wave_box's caller prepared: exact for i < 2^16 / e).
__device__ inline int box_region_cell(int i, const TileBox &b)
{
    const int t = (i * b.inv[0]) >> 16, bx = i - t * b.e[0], bz = (t * b.inv[1]) >> 16, by = t - bz * b.e[1];
    return b.base + bx + b.L * (by + b.L * bz);
}

// Marks stencil node `lane` of the point X as used in this step (region
// cells outside every stencil are neither gathered nor corrected).
__device__ inline void mark_node(unsigned char *mk, unsigned char *xmk, const CaseDev &cd, const BodyView &B, const double X[3], int lane)
{
    const int off[3] = {lane & 3, (lane >> 2) & 3, lane >> 4};
    const int n[3] = {cd.nx, cd.ny, cd.nz};
    const int L = cd.L;
    int r[3];
    bool ok = true;
#pragma unroll
    for (int d = 0; d < 3; d++) {
        int rel = (int)floor(X[d]) - 1 + off[d] - B.org[d];
        if (d < 2) rel = wrapi(rel, n[d]);
        ok = ok && rel >= 0 && rel < L;
        r[d] = rel;
    }
    if (!ok) return;
    mk[r[0] + L * (r[1] + L * r[2])] = 1;
    if (xmk)
        for (int n = 0; n < 27; n++)
            xmk[r[0] + n % 3 + (L + 2) * (r[1] + n / 3 % 3 + (L + 2) * (r[2] + n / 9))] = 1;
}

// Box of the stencil nodes of the points P held by the lanes with `on` set
// (at least one): first node lo = min floor(P) - 1 and extent
// max floor(P) - min floor(P) + 4 per axis, by butterfly min / max.
__device__ inline void wave_box(const double P[3], bool on, int lo[3], int e[3])
{
#pragma unroll
    for (int d = 0; d < 3; d++) {
        const int f = (int)floor(P[d]);
        int mn = on ? f : (1 << 30), mx = on ? f : -(1 << 30);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            mn = min(mn, __shfl_xor(mn, o));
            mx = max(mx, __shfl_xor(mx, o));
        }
        lo[d] = mn - 1;
        e[d] = mx - mn + 4;
    }
}

// Marks in mk the stencil cells of the tile's points P (lane j < count holds
// point j): the whole box when it lies inside the region, else node by node;
// and in xmk (moment storage) those and their neighbours.
// The box goes to the tile's entry of the tile table.
__device__ inline void mark_points(unsigned char *mk, unsigned char *xmk, const CaseDev &cd, const BodyView &B,
                                   const double P[3], int count, int lane, TileBox &out)
{
    int lo[3], e[3], o[3];
    wave_box(P, lane < count, lo, e);
    const int L = cd.L;
    bool in = true;
#pragma unroll
    for (int d = 0; d < 3; d++) {
        o[d] = lo[d] - B.org[d];
        in = in && o[d] >= 0 && o[d] + e[d] <= L;
    }
    const int base = o[0] + L * (o[1] + L * o[2]);
    if (in) {
        for (int r = lane; r < e[0] * e[1]; r += 64) {
            const int by = r / e[0], at = base + (r - by * e[0]) + L * by;
            for (int bz = 0; bz < e[2]; bz++) mk[at + L * L * bz] = 1;
        }
        if (xmk) {   // the same box with a one-cell rim, in the region with its rim
            const int E = L + 2, e0 = e[0] + 2, n = e0 * (e[1] + 2);
            for (int r = lane; r < n; r += 64) {
                const int by = r / e0, at = o[0] + (r - by * e0) + E * (o[1] + by + E * o[2]);
                for (int bz = 0; bz < e[2] + 2; bz++) xmk[at + E * E * bz] = 1;
            }
        }
    } else {
        for (int j = 0; j < count; j++) {
            const double Pj[3] = {__shfl(P[0], j), __shfl(P[1], j), __shfl(P[2], j)};
            mark_node(mk, xmk, cd, B, Pj, lane);
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int d = 0; d < 3; d++) {
            out.lo[d] = lo[d];
            out.e[d] = e[d];
        }
        out.inv[0] = (65535 + e[0]) / e[0];
        out.inv[1] = (65535 + e[1]) / e[1];
        out.base = base;
        out.fits = in && e[0] * e[1] * e[2] <= kBoxCells;
    }
}

// One wavefront per marker tile (Sec. 2.3 kinematics): lane j < count forms
// the position, normal and rigid velocity of marker first + j and checks the
// z range; the tile's stencil box goes to the tile table, and the cells of
// that box (and of the force-surface points' box) are marked for this step.
__global__ void __launch_bounds__(64) EIGHT_WAVES k_markers(DevPtrs p, int n_mtiles)
{
    const int tix = tile_of_block((int)blockIdx.x, n_mtiles);
    if (tix >= n_mtiles) return;
    const MarkerTile mt = p.mtiles[tix];
    const CaseDev cd = p.cases[mt.c];
    const BodyDev &Bd = p.body[mt.c];
    const BodyView B = body_view(Bd);
    if (B.err != 0) return;
    const int lane = threadIdx.x;
    if (tix == cd.tile_off && lane == 0) {   // the step's geometry, for the correction
        StepGeometry &G = p.geo[mt.c];
        G.z0 = Bd.z0;
        G.shift = window_shifts(cd, B.r[2]);
#pragma unroll
        for (int a = 0; a < 3; a++) {
            G.org[a] = B.org[a];
            G.fo[0][a] = Bd.fo[0][a];
            G.fo[1][a] = Bd.fo[1][a];
        }
        G.fvalid[0] = Bd.fvalid[0];
        G.fvalid[1] = Bd.fvalid[1];
    }
    const bool on = lane < mt.count;
    const int k = mt.first + (on ? lane : 0);
    const double xb[3] = {p.xb[3 * k], p.xb[3 * k + 1], p.xb[3 * k + 2]};
    const double nb[3] = {p.nb[3 * k], p.nb[3 * k + 1], p.nb[3 * k + 2]};
    double X[3], N[3], rel[3], wr[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        X[a] = B.r[a] + xb[0] * Bd.d[a] + xb[1] * Bd.d[3 + a] + xb[2] * Bd.d[6 + a];
        N[a] = nb[0] * Bd.d[a] + nb[1] * Bd.d[3 + a] + nb[2] * Bd.d[6 + a];
        rel[a] = X[a] - B.r[a];
    }
    const double w[3] = {Bd.w[0], Bd.w[1], Bd.w[2]}, vb[3] = {Bd.v[0], Bd.v[1], Bd.v[2]};
    const double dl = cd.force_offset;
    if (on) {
        cross3(w, rel, wr);
#pragma unroll
        for (int a = 0; a < 3; a++) {
            p.X[3 * k + a] = X[a];
            p.N[3 * k + a] = N[a];
            p.U[3 * k + a] = vb[a] + wr[a];
        }
        // the marker's one-dimensional stencil weights for this step
#pragma unroll
        for (int d = 0; d < 3; d++) {
            const int n0 = (int)floor(X[d]) - 1;
#pragma unroll
            for (int o = 0; o < 4; o++) p.wt[12 * k + 4 * d + o] = phi4((double)(n0 + o) - X[d]);
        }
        const int fz = (int)floor(X[2]);
        if (fz - 1 < 0 || fz + 2 > cd.nz - 1) atomicOr(&p.body[mt.c].err, 1);
        if (dl > 0.0) {
            const int gz = (int)floor(X[2] + dl * N[2]);
            if (gz - 1 < 0 || gz + 2 > cd.nz - 1) atomicOr(&p.body[mt.c].err, 1);
        }
    }
    unsigned char *xmk = p.xmark ? p.xmark + cd.xreg_off : nullptr;
    mark_points(p.mark + cd.reg_off, xmk, cd, B, X, mt.count, lane, p.tbox[tix]);
    if (dl > 0.0) {   // the force-surface points
        const double Y[3] = {X[0] + dl * N[0], X[1] + dl * N[1], X[2] + dl * N[2]};
        mark_points(p.mark2 + cd.reg_off, xmk, cd, B, Y, mt.count, lane, p.tbox[n_mtiles + tix]);
    }
}

// Epilogue of the l = 0 interpolation: plain start, warm-start features and the
// stress-integral parts, by one wavefront, four lanes per marker: lane a < 3 of
// a marker's quad takes component a (lane 3 repeats component 0 and stores
// nothing).  Its operands load with the tile's other data; one thread per
// marker, which held all components at once, spilled 24 registers.
struct Epilogue {
    int j, a, k;          // marker of the tile, component, marker
    bool on;
    double hp, hq, h0q;   // the final h of the previous step and of the one before, the previous plain start
    double n;             // the normal
    __device__ inline void load(const DevPtrs &p, const TileBox &tb)
    {
        j = (threadIdx.x & 63) >> 2;
        a = threadIdx.x & 3;
        on = threadIdx.x < 64 && j < tb.count && a < 3;
        a = a < 3 ? a : 0;
        k = tb.first + (j < tb.count ? j : 0);
        hp = hq = h0q = n = 0.0;
        if (threadIdx.x < 64) {
            hp = p.hk[3 * k + a];
            hq = p.hk2[3 * k + a];
            h0q = p.h0[3 * k + a];
            n = p.N[3 * k + a];
        }
    }
};

// Value of lane a of this lane's quad.
template <int A>
__device__ inline double quad_lane(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, A * 0x55, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), A * 0x55, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ inline double quad_at(double v, int a)
{
    const double v0 = quad_lane<0>(v), v1 = quad_lane<1>(v), v2 = quad_lane<2>(v);
    return a == 0 ? v0 : (a == 1 ? v1 : v2);
}
__device__ inline double quad_norm(double v)
{
    const double v0 = quad_lane<0>(v), v1 = quad_lane<1>(v), v2 = quad_lane<2>(v);
    return sqrt(v0 * v0 + v1 * v1 + v2 * v2);
}

// One wavefront: ev = a marker's interpolated rho - 1, u*, sigma (rewritten as
// its parts), rec = its record, r = the body's centre.  h_k becomes h0 when the
// first spread has been done (spread set), else 0.
template <int W>
__device__ inline void force_epilogue(const DevPtrs &p, const Epilogue &E, const double r[3], double (*ev)[kRegFields],
                                      const double (*rec)[W], int spread)
{
    const int a = E.a, b = a == 2 ? 0 : a + 1, c = b == 2 ? 0 : b + 1, j = E.on ? E.j : 0, k = E.k;
    const double *v = ev[j], *rc = rec[j];
    const double h0 = rc[3 + a] - v[1 + a], dS = rc[6], pr = (double)CS2 * v[0];
    // sigma's row a; fields 4..9 = xx yy zz xy xz yz
    const double sx = v[a == 0 ? 4 : (a == 1 ? 7 : 8)], sy = v[a == 0 ? 7 : (a == 1 ? 5 : 9)], sz = v[a == 0 ? 8 : (a == 1 ? 9 : 6)];
    const double s = sx * quad_lane<0>(E.n) + sy * quad_lane<1>(E.n) + sz * quad_lane<2>(E.n);
    const double rel_b = rc[b] - r[b], rel_c = rc[c] - r[c];
    const double ts = rel_b * quad_at(s, c) - rel_c * quad_at(s, b);
    // warm-start features: the plain start U - I[u*] (an invertible linear
    // map of I[u*] and U that keeps their small difference out of
    // cancellation), h(t-1), and the changes h(t-1) - h(t-2) and
    // h0(t) - h0(t-1), over the marker's scale |h0| + |h(t-1)|; the normal
    // and the area
    const double sc = fmax(quad_norm(h0) + quad_norm(E.hp), 1e-14);
    if (!E.on) return;
    float *ft = p.feat + (long long)kMlpIn * k;
    ft[kFeatH0 + a] = (float)(h0 / sc);
    ft[kFeatHPrev + a] = (float)(E.hp / sc);
    ft[kFeatDH + a] = (float)((E.hp - E.hq) / sc);
    ft[kFeatDH0 + a] = (float)((h0 - E.h0q) / sc);
    ft[kFeatNormal + a] = (float)E.n;
    if (a == 0) {
        ft[kFeatArea] = (float)dS;
        p.hs[k] = sc;
    }
    // h_k holds what has been spread so far; dh is the next increment
    p.hk2[3 * k + a] = E.hp;
    p.h0[3 * k + a] = h0;
    p.hk[3 * k + a] = spread ? 0.0 + h0 : 0.0;
    p.dh[3 * k + a] = h0;
    double *o = ev[E.j];   // (every lane of the wavefront has read its fields)
    o[a] = dS * s;
    o[3 + a] = dS * ts;
    o[6 + a] = dS * (-pr) * E.n;
}

// Tile sums of the per-marker parts (the first kPart entries of each row of
// tp, a row per marker), in marker order (deterministic).
template <int W>
__device__ inline void tile_part_sum(const DevPtrs &p, int tix, int count, const double (*tp)[W])
{
    __syncthreads();
    if (count > 0 && (int)threadIdx.x < kPart) {
        double acc = 0.0;
        for (int j = 0; j < count; j++) acc += tp[j][threadIdx.x];
        p.part[(long long)kPart * tix + threadIdx.x] = acc;
    }
}

// Case totals of the per-tile force, torque and pressure-force parts, in a
// fixed order: strided per-thread sums over the case's tiles, a fixed
// butterfly inside each wavefront, then the wavefronts in order.
__device__ inline void case_force_total(const DevPtrs &p, const CaseDev &cd, BodyDev &B)
{
    __shared__ double sh[4][kPart];
    double acc[kPart];
#pragma unroll
    for (int j = 0; j < kPart; j++) acc[j] = 0.0;
    for (int t = threadIdx.x; t < cd.n_tiles; t += blockDim.x) {
        const double *o = p.part + (long long)kPart * (cd.tile_off + t);
#pragma unroll
        for (int j = 0; j < kPart; j++) acc[j] += o[j];
    }
#pragma unroll
    for (int j = 0; j < kPart; j++) acc[j] = wave_sum(acc[j]);
    const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int j = 0; j < kPart; j++) sh[wave][j] = acc[j];
    __syncthreads();
    if (threadIdx.x < kPart) {
        double v = 0.0;
        for (int w = 0; w < nw; w++) v += sh[w][threadIdx.x];
        double *dst = threadIdx.x < 3 ? &B.F[threadIdx.x] : (threadIdx.x < 6 ? &B.T[threadIdx.x - 3] : &B.Fp[threadIdx.x - 6]);
        *dst = v;
    }
}

__device__ inline double wave_max(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}

// Case maximum of the per-tile residuals into resid and resid_hist[slot].
__device__ inline void case_resid_total(const DevPtrs &p, const CaseDev &cd, BodyDev &B, int slot)
{
    __shared__ double sh[4];
    double m = 0.0;
    for (int t = threadIdx.x; t < cd.n_tiles; t += blockDim.x) m = fmax(m, p.res[cd.tile_off + t]);
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        double v = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); w++) v = fmax(v, sh[w]);
        B.resid = v;
        if (slot >= 0 && slot < 16) B.resid_hist[slot] = v;
    }
}

// Spread of one marker's increment d (held by every lane) through the lane's
// stencil node with weight W dS_k: fixed point, into the tile's LDS
// accumulator (box cell i) or, when the box does not fit, straight into the
// region accumulator Hc (region cell q, -1 outside).
__device__ inline void spread_node(const DevPtrs &p, int c, const TileBox &tb, int i, int q, double wS,
                                   const double d[3], unsigned long long (*acc)[kBoxCells], long long *Hc, int L3)
{
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const double v = d[a] * wS;
        long long fx = 0;
        if (fabs(v) < 1.0e6) fx = __double2ll_rn(v * kFixScale);
        else atomicOr(&p.body[c].err, 2);
        if (tb.fits) atomicAdd(&acc[a][i], (unsigned long long)fx);
        else if (q >= 0) atomicAdd((unsigned long long *)&Hc[a * L3 + q], (unsigned long long)fx);
    }
}

// The tile's LDS accumulator into the region accumulator: one global atomic
// per touched cell and component (after a barrier).
__device__ inline void spread_flush(const TileBox &tb, int ncell, int L3, const unsigned long long (*acc)[kBoxCells],
                                    long long *Hc)
{
    for (int i = threadIdx.x; i < ncell; i += blockDim.x) {
        const int q = box_region_cell(i, tb);
#pragma unroll
        for (int a = 0; a < 3; a++)
            if (acc[a][i] != 0ull) atomicAdd((unsigned long long *)&Hc[a * L3 + q], acc[a][i]);
    }
}

// Entry f of marker k's record: X (0..2), U (3..5), dS (6), the stencil
// weights (7..18), h_k (19..21).  The force kernel keeps entries 0..18.
constexpr int kRecW = 7, kRecH = 19, kRecForce = 19, kRecUpdate = 22;

// The kernels of the coupling run beside the lattice kernel, whose waves each
// hold 64 VGPRs and 96 SGPRs and fill every wave slot of a SIMD (the moment
// step: 14 waves of 128 VGPRs).  A coupling wave starts only in a slot that is
// free, so they are compiled for 8 waves per SIMD, the lattice kernel's own
// budget: at 256 x 256 x 768 the coupling then runs during the lattice kernel
// instead of after it, 50 us less per step in FP32, 60 in BF16.  The LDS of the
// tile kernels is taken at launch (dynamic), so that the compiler's occupancy
// target is set by the register budget and not by the LDS size; the layouts
// are carved below, 8-byte arrays first.

struct LdsCarve {
    unsigned char *at;
    template <class A>
    __device__ A &take()
    {
        A &r = *reinterpret_cast<A *>(at);
        at += sizeof(A);
        return r;
    }
};

constexpr size_t kLdsForce = sizeof(unsigned long long[3][kBoxCells]) + sizeof(double[kTileMarkers][kRegFields]) +
                             sizeof(double[kTileMarkers][kRecForce]) + sizeof(double[kTileMarkers][3]) +
                             sizeof(float[kRegFields][kBoxCells]);
constexpr size_t kLdsSurface = sizeof(double[kTileMarkers][7]) + sizeof(double[kTileMarkers][kPart]) + sizeof(float[7][kBoxCells]);
constexpr size_t kLdsUpdate = sizeof(double[3][kBoxCells]) + sizeof(unsigned long long[3][kBoxCells]) +
                              sizeof(double[kTileMarkers][kRecUpdate]) + sizeof(double[kTileMarkers][3]) +
                              sizeof(double[kTileMarkers]);
static_assert(kLdsForce <= 65536 && kLdsUpdate <= 65536 && kLdsSurface <= kLdsUpdate, "tile kernel LDS");
__device__ inline double marker_record(const DevPtrs &p, int k, int f)
{
    if (f < 3) return p.X[3 * k + f];
    if (f < 6) return p.U[3 * k + f - 3];
    if (f == 6) return p.dS[k];
    if (f < kRecH) return p.wt[12 * k + f - kRecW];
    return p.hk[3 * k + f - kRecH];
}

// A tile's marker records into LDS (row j = marker first + j), in two loads
// per thread issued together; the caller stores them after its other loads
// and before its barrier.
template <int NREC>
struct RecordLoad {
    static_assert(kTileMarkers * NREC <= 512, "two loads per thread of a 256-thread workgroup");
    double v[2];
    __device__ inline void load(const DevPtrs &p, const TileBox &mt)
    {
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const int t = (int)threadIdx.x + 256 * u;
            v[u] = t < mt.count * NREC ? marker_record(p, mt.first + t / NREC, t % NREC) : 0.0;
        }
    }
    __device__ inline void store(const TileBox &mt, double (*rec)[NREC]) const
    {
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const int t = (int)threadIdx.x + 256 * u;
            if (t < mt.count * NREC) rec[t / NREC][t % NREC] = v[u];
        }
    }
};

// Spread of the tile's per-marker increments d[j] (LDS rows) after a
// barrier: wavefront w takes markers w, w+4, ...; lane l is stencil node l,
// so the 64 LDS atomics of one instruction go to 64 different cells.
__device__ inline void spread_tile(const DevPtrs &p, const TileBox &tb, const double *rbase, int nrec,
                                   const double (*d)[3], unsigned long long (*acc)[kBoxCells], long long *Hc, int L3)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int j = wave; j < tb.count; j += blockDim.x >> 6) {
        const double *rc = rbase + j * nrec;
        const double X[3] = {rc[0], rc[1], rc[2]};
        double W;
        int i = 0, q = -1;
        if (tb.fits) {
            i = box_node_w(X, rc + kRecW, lane, tb, W);
        } else {
            const Node nd = stencil_node(X, lane, p.cases[tb.c], p.body[tb.c].org);
            W = nd.W;
            q = nd.q;
        }
        spread_node(p, tb.c, tb, i, q, W * rc[6], d[j], acc, Hc, L3);
    }
}

// l = 0 and the stress integral over a tile (a row of 16 lanes per marker).
// With spread set, also the first forcing cycle's spread of the plain start
// h0 into accumulator 0 (h_k = h0).  The tile's force, torque and pressure
// force go to its parts unless the case has a force surface.
__device__ inline void force_tile(const DevPtrs &p, const TileBox &tb, int tix, int spread, unsigned char *lds)
{
    LdsCarve lc{lds};
    auto &acc = lc.take<unsigned long long[3][kBoxCells]>();
    auto &ep = lc.take<double[kTileMarkers][kRegFields]>();    // interpolated fields, then the marker's parts
    auto &mrec = lc.take<double[kTileMarkers][kRecForce]>();   // the tile's marker records
    auto &dinc = lc.take<double[kTileMarkers][3]>();           // the markers' increments (h0) to spread
    auto &box = lc.take<float[kRegFields][kBoxCells]>();
    const int L3 = tb.L * tb.L * tb.L;
    const float *R = p.reg + tb.reg_off * kRegFields;
    long long *H0 = p.H + tb.reg_off * 3;
    const int ncell = tb.e[0] * tb.e[1] * tb.e[2];
    // the markers' records, the epilogue's operands and the body load in the
    // same round as the box
    RecordLoad<kRecForce> rl;
    rl.load(p, tb);
    Epilogue ep_in;
    ep_in.load(p, tb);
    const BodyDev &B = p.body[tb.c];
    const int err = B.err;
    if (tb.fits) {
        for (int i = threadIdx.x; i < ncell; i += blockDim.x) {
            const int q = box_region_cell(i, tb);
#pragma unroll
            for (int f = 0; f < kRegFields; f++) box[f][i] = R[f * L3 + q];
            acc[0][i] = acc[1][i] = acc[2][i] = 0ull;
        }
    }
    if (err != 0) return;
    rl.store(tb, mrec);
    __syncthreads();
    // rows past the tile's markers repeat marker 0 and store nothing
    const int j = threadIdx.x >> 4, col = threadIdx.x & 15;
    const bool on = j < tb.count;
    const double *rc = mrec[on ? j : 0];
    const double X[3] = {rc[0], rc[1], rc[2]};
    const double *wr = rc + kRecW;   // 4 weights per axis
    const Column cn = column_nodes(p, X, wr[col & 3], wr[4 + (col >> 2)], wr + 8, col, tb);
    double v[kRegFields];
#pragma unroll
    for (int f = 0; f < kRegFields; f++) v[f] = 0.0;
#pragma unroll
    for (int z = 0; z < 4; z++) {
        if (tb.fits) {
#pragma unroll
            for (int f = 0; f < kRegFields; f++) v[f] += cn.W[z] * (double)box[f][cn.i[z]];
        } else if (cn.q[z] >= 0) {
#pragma unroll
            for (int f = 0; f < kRegFields; f++) v[f] += cn.W[z] * (double)R[f * L3 + cn.q[z]];
        }
    }
#pragma unroll
    for (int f = 0; f < kRegFields; f++) v[f] = row_sum(v[f]);
    if (on && col == 0) {
#pragma unroll
        for (int f = 0; f < kRegFields; f++) ep[j][f] = v[f];
#pragma unroll
        for (int a = 0; a < 3; a++) dinc[j][a] = rc[3 + a] - v[1 + a];
    }
    __syncthreads();
    if (spread) spread_tile(p, tb, &mrec[0][0], kRecForce, dinc, acc, H0, L3);
    if (threadIdx.x < 64) {
        const double r[3] = {B.r[0], B.r[1], B.r[2]};
        force_epilogue(p, ep_in, r, ep, mrec, spread);
    }
    tile_part_sum(p, tix, tb.surface ? 0 : tb.count, ep);
    if (spread && tb.fits) spread_flush(tb, ncell, L3, acc, H0);
}

// The stress integral on the parallel surface at distance force_offset outside
// the markers (points Y_k = X_k + delta n_k, same normals, areas dSo): the box
// of the tile's surface-point stencils (from k_markers) is staged in LDS with
// rho - 1 and sigma, a row of 16 lanes per marker sums its stencil, one thread
// per marker forms its parts.
__device__ inline void surface_force_tile(const DevPtrs &p, const TileBox &tb, int tix, unsigned char *lds)
{
    LdsCarve lc{lds};
    auto &ev = lc.take<double[kTileMarkers][7]>();
    auto &tp = lc.take<double[kTileMarkers][kPart]>();
    auto &box = lc.take<float[7][kBoxCells]>();
    const int L3 = tb.L * tb.L * tb.L;
    const float *R = p.reg + tb.reg_off * kRegFields;
    const int ncell = tb.e[0] * tb.e[1] * tb.e[2];
    const BodyDev &B = p.body[tb.c];
    const int err = B.err;
    const double r[3] = {B.r[0], B.r[1], B.r[2]};
    const int j = threadIdx.x >> 4, col = threadIdx.x & 15;
    const bool on = j < tb.count;
    const int k = tb.first + (on ? j : 0);
    const double dl = p.cases[tb.c].force_offset;
    double Y[3], w[6];   // this column's weights: x, y and the four z levels
#pragma unroll
    for (int a = 0; a < 3; a++) Y[a] = p.X[3 * k + a] + dl * p.N[3 * k + a];
    // fields 0 (rho - 1) and 4..9 (sigma xx yy zz xy xz yz)
    if (tb.fits) {
        for (int i = threadIdx.x; i < ncell; i += blockDim.x) {
            const int q = box_region_cell(i, tb);
            box[0][i] = R[q];
#pragma unroll
            for (int f = 1; f < 7; f++) box[f][i] = R[(f + 3) * L3 + q];
        }
    }
    if (err != 0) return;
    __syncthreads();
    w[0] = phi4((double)((int)floor(Y[0]) - 1 + (col & 3)) - Y[0]);
    w[1] = phi4((double)((int)floor(Y[1]) - 1 + (col >> 2)) - Y[1]);
#pragma unroll
    for (int z = 0; z < 4; z++) w[2 + z] = phi4((double)((int)floor(Y[2]) - 1 + z) - Y[2]);
    const Column cn = column_nodes(p, Y, w[0], w[1], w + 2, col, tb);
    double v[7];
#pragma unroll
    for (int f = 0; f < 7; f++) v[f] = 0.0;
#pragma unroll
    for (int z = 0; z < 4; z++) {
        if (tb.fits) {
#pragma unroll
            for (int f = 0; f < 7; f++) v[f] += cn.W[z] * (double)box[f][cn.i[z]];
        } else if (cn.q[z] >= 0) {
#pragma unroll
            for (int f = 0; f < 7; f++) v[f] += cn.W[z] * (double)R[(f == 0 ? 0 : f + 3) * L3 + cn.q[z]];
        }
    }
#pragma unroll
    for (int f = 0; f < 7; f++) v[f] = row_sum(v[f]);
    if (on && col == 0)
#pragma unroll
        for (int f = 0; f < 7; f++) ev[j][f] = v[f];
    __syncthreads();
    if ((int)threadIdx.x < tb.count) {
        const int m = tb.first + threadIdx.x;
        const double *e = ev[threadIdx.x];
        const double nk[3] = {p.N[3 * m], p.N[3 * m + 1], p.N[3 * m + 2]};
        const double pr = (double)CS2 * e[0];
        const double sg[3][3] = {{e[1], e[4], e[5]}, {e[4], e[2], e[6]}, {e[5], e[6], e[3]}};
        double s[3], rel[3], ts[3];
#pragma unroll
        for (int a = 0; a < 3; a++) {
            s[a] = sg[a][0] * nk[0] + sg[a][1] * nk[1] + sg[a][2] * nk[2];
            rel[a] = p.X[3 * m + a] + dl * nk[a] - r[a];
        }
        cross3(rel, s, ts);
        const double dA = p.dSo[m];
#pragma unroll
        for (int a = 0; a < 3; a++) {
            tp[threadIdx.x][a] = dA * s[a];
            tp[threadIdx.x][3 + a] = dA * ts[a];
            tp[threadIdx.x][6 + a] = dA * (-pr) * nk[a];
        }
    }
    tile_part_sum(p, tix, tb.count, tp);
}

__global__ void __launch_bounds__(256) EIGHT_WAVES k_interp_force_tiles(DevPtrs p, int n_mtiles, int spread)
{
    extern __shared__ __align__(16) unsigned char lds_dyn[];
    const int tix = tile_of_block((int)blockIdx.x, n_mtiles);
    if (tix >= n_mtiles) return;
    const TileBox tb = p.tbox[tix];
    force_tile(p, tb, tix, spread, lds_dyn);
}

__global__ void __launch_bounds__(256) EIGHT_WAVES k_surface_force_tiles(DevPtrs p, int n_mtiles)
{
    extern __shared__ __align__(16) unsigned char lds_dyn[];
    const int tix = tile_of_block((int)blockIdx.x, n_mtiles);
    if (tix >= n_mtiles) return;
    const TileBox tb = p.tbox[n_mtiles + tix];
    if (tb.surface) surface_force_tile(p, tb, tix, lds_dyn);
}

// Spreading of the increments dh over a tile into accumulator 0 (H += S[dh],
// h_k += dh): LDS accumulation, then one HBM atomic per touched cell.  With
// masked set, cases whose sequence has ended are skipped.
__global__ void __launch_bounds__(256) EIGHT_WAVES k_spread_tiles(DevPtrs p, int n_mtiles, int masked)
{
    __shared__ unsigned long long acc[3][kBoxCells];
    __shared__ double mrec[kTileMarkers][kRecForce];   // the tile's marker records
    __shared__ double dinc[kTileMarkers][3];           // the increments dh to spread
    const int tix = tile_of_block((int)blockIdx.x, n_mtiles);
    if (tix >= n_mtiles) return;
    const TileBox tb = p.tbox[tix];
    const int err = p.body[tb.c].err, active = p.body[tb.c].active;
    const int L3 = tb.L * tb.L * tb.L;
    long long *H = p.H + tb.reg_off * 3;
    const int ncell = tb.e[0] * tb.e[1] * tb.e[2];
    RecordLoad<kRecForce> rl;
    rl.load(p, tb);
    // thread j < count: marker j's increment, and h_k += dh
    const int t = threadIdx.x;
    double dh[3] = {0.0, 0.0, 0.0}, hk[3] = {0.0, 0.0, 0.0};
    if (t < tb.count)
#pragma unroll
        for (int a = 0; a < 3; a++) {
            dh[a] = p.dh[3 * (tb.first + t) + a];
            hk[a] = p.hk[3 * (tb.first + t) + a];
        }
    if (err != 0 || (masked && !active)) return;
    if (tb.fits)
        for (int i = threadIdx.x; i < ncell; i += blockDim.x) acc[0][i] = acc[1][i] = acc[2][i] = 0ull;
    rl.store(tb, mrec);
    if (t < tb.count)
#pragma unroll
        for (int a = 0; a < 3; a++) {
            dinc[t][a] = dh[a];
            p.hk[3 * (tb.first + t) + a] = hk[a] + dh[a];
        }
    __syncthreads();
    spread_tile(p, tb, &mrec[0][0], kRecForce, dinc, acc, H, L3);
    __syncthreads();
    if (tb.fits) spread_flush(tb, ncell, L3, acc, H);
}

// Interpolation of u* + H over a tile (staged in LDS, FP64; H the sum of
// accumulators 0 .. NB-1), the residual U_k - I[u* + H](X_k), the next
// increment dh = that residual, and the tile's largest residual component.
// With spread_to >= 0 the same pass spreads dh (the next cycle's spread,
// h_k += dh) into accumulator spread_to, which no interpolation of this
// pass reads.
template <int NB>
__global__ void __launch_bounds__(256) EIGHT_WAVES k_interp_update_tiles(DevPtrs p, int n_mtiles, int masked, int spread_to, int ft_total)
{
    extern __shared__ __align__(16) unsigned char lds_dyn[];
    LdsCarve lc{lds_dyn};
    auto &box = lc.take<double[3][kBoxCells]>();
    auto &acc = lc.take<unsigned long long[3][kBoxCells]>();
    auto &mrec = lc.take<double[kTileMarkers][kRecUpdate]>();   // the tile's marker records
    auto &dinc = lc.take<double[kTileMarkers][3]>();            // the markers' increments e to spread
    auto &rmax = lc.take<double[kTileMarkers]>();
    const int tix = tile_of_block((int)blockIdx.x, n_mtiles);
    if (tix >= n_mtiles) return;
    if (NB == 1 && blockIdx.y == 1) {
        const TileBox ts = p.tbox[n_mtiles + tix];
        if (ts.surface) surface_force_tile(p, ts, tix, lds_dyn);
        return;
    }
    const TileBox tb = p.tbox[tix];
    const int err = p.body[tb.c].err, active = p.body[tb.c].active;
    const int L3 = tb.L * tb.L * tb.L;
    const float *R = p.reg + tb.reg_off * kRegFields;
    const long long *H = p.H + tb.reg_off * 3;
    long long *Hs = p.H + (spread_to > 0 ? spread_to : 0) * p.hstride + tb.reg_off * 3;
    const int ncell = tb.e[0] * tb.e[1] * tb.e[2];
    // H at region cell q and component a: the exact integer sum of the accumulators
    const long long hstride = p.hstride;
    auto h_at = [&](int a, int q) {
        long long h = H[a * L3 + q];
#pragma unroll
        for (int b = 1; b < NB; b++) h += H[b * hstride + a * L3 + q];
        return h;
    };
    // the markers' records load in the same round as the box
    RecordLoad<kRecUpdate> rl;
    rl.load(p, tb);
    if (tb.fits) {
        for (int i = threadIdx.x; i < ncell; i += blockDim.x) {
            const int q = box_region_cell(i, tb);
#pragma unroll
            for (int a = 0; a < 3; a++) {
                box[a][i] = (double)R[(1 + a) * L3 + q] + (double)h_at(a, q) * kFixInv;
                acc[a][i] = 0ull;
            }
        }
    }
    if (err != 0 || (masked && !active)) return;
    rl.store(tb, mrec);
    __syncthreads();
    // rows past the tile's markers repeat marker 0 and store nothing
    const int j = threadIdx.x >> 4, col = threadIdx.x & 15;
    const bool on = j < tb.count;
    const double *rc = mrec[on ? j : 0];
    const double X[3] = {rc[0], rc[1], rc[2]};
    const double *wr = rc + kRecW;   // 4 weights per axis
    const Column cn = column_nodes(p, X, wr[col & 3], wr[4 + (col >> 2)], wr + 8, col, tb);
    double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int z = 0; z < 4; z++) {
        if (tb.fits) {
#pragma unroll
            for (int a = 0; a < 3; a++) v[a] += cn.W[z] * box[a][cn.i[z]];
        } else if (cn.q[z] >= 0) {
            const int q = cn.q[z];
#pragma unroll
            for (int a = 0; a < 3; a++)
                v[a] += cn.W[z] * ((double)R[(1 + a) * L3 + q] + (double)h_at(a, q) * kFixInv);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; a++) v[a] = row_sum(v[a]);
    const double e[3] = {rc[3] - v[0], rc[4] - v[1], rc[5] - v[2]};
    if (on && col == 0) {
        const int k = tb.first + j;
        double res = 0.0;
#pragma unroll
        for (int a = 0; a < 3; a++) {
            res = fmax(res, fabs(e[a]));
            p.dh[3 * k + a] = e[a];
            if (spread_to >= 0) p.hk[3 * k + a] = rc[kRecH + a] + e[a];
            dinc[j][a] = e[a];
        }
        rmax[j] = res;
    }
    __syncthreads();
    if (spread_to >= 0) spread_tile(p, tb, &mrec[0][0], kRecUpdate, dinc, acc, Hs, L3);
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = 0.0;
        for (int t = 0; t < tb.count; t++) m = fmax(m, rmax[t]);
        p.res[tix] = m;
    }
    if (spread_to >= 0 && tb.fits) spread_flush(tb, ncell, L3, acc, Hs);
    // the case's force totals from the force kernels' tile parts (complete at
    // this kernel's start), formed by the workgroup of its first tile
    if (ft_total && tix == tb.tile_off) case_force_total(p, p.cases[tb.c], p.body[tb.c]);
}

// FP64 force, torque and pressure-force totals of each case from its tile
// parts (one 256-thread workgroup per case, fixed order).
__global__ void __launch_bounds__(256) k_reduce_ft(DevPtrs p)
{
    const int c = blockIdx.x;
    const CaseDev &cd = p.cases[c];
    if (cd.M == 0 || p.body[c].err != 0) return;
    case_force_total(p, cd, p.body[c]);
}

// Max residual over the tiles of a case: into resid and resid_hist[slot].
// With masked set only cases still active are reduced; with gate_cycle > 0
// (a learned-start cycle) a case whose residual is at or below its gate is
// accepted and leaves the sequence.
__global__ void __launch_bounds__(256) k_reduce_resid(DevPtrs p, int slot, int masked, int gate_cycle)
{
    const int c = blockIdx.x;
    const CaseDev &cd = p.cases[c];
    BodyDev &B = p.body[c];
    if (cd.M == 0 || B.err != 0 || (masked && !B.active)) return;
    case_resid_total(p, cd, B, slot);
    if (threadIdx.x == 0 && gate_cycle > 0 && B.resid <= B.gate) {
        B.active = 0;
        B.accepts += 1;
        B.warm_cyc_sum += gate_cycle;
    }
}

// Start of a learned-start sequence: every live case runs cycles.
__global__ void k_gate_begin(DevPtrs p, int n_cases)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n_cases) return;
    BodyDev &B = p.body[c];
    B.active = 1;
    B.fallback = 0;
}

// End of the learned-start cycles: a case not accepted within them falls
// back to the plain start and stays active for the plain cycles.
__global__ void k_gate(DevPtrs p, int n_cases)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n_cases) return;
    BodyDev &B = p.body[c];
    if (p.cases[c].M == 0 || B.err != 0) return;
    B.fallback = B.active;
    if (B.fallback) B.rejects += 1;
}

// Warm start without a network: the previous step's final h_k (kept in the
// features over the marker's scale).
__global__ void k_warm_previous(DevPtrs p, int Mtot)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= Mtot || p.body[p.mcase[k]].err != 0) return;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const double h = (double)p.feat[(long long)kMlpIn * k + kFeatHPrev + a] * p.hs[k];
        p.hk[3 * k + a] = 0.0;
        p.dh[3 * k + a] = h;
    }
}

// Fallback preparation: plain start h_k = U_k - I[u*](X_k) ...
__global__ void k_fallback_markers(DevPtrs p, int Mtot)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= Mtot) return;
    const BodyDev &B = p.body[p.mcase[k]];
    if (B.err != 0 || !B.fallback) return;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        p.hk[3 * k + a] = 0.0;
        p.dh[3 * k + a] = p.h0[3 * k + a];
    }
}

// ... and an empty immersed-force accumulator.
__global__ void k_fallback_zero(DevPtrs p)
{
    const int c = blockIdx.y;
    const CaseDev &cd = p.cases[c];
    const BodyDev &B = p.body[c];
    if (cd.M == 0 || B.err != 0 || !B.fallback) return;
    const int L3 = cd.L * cd.L * cd.L;
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= L3 || !p.mark[cd.reg_off + q]) return;
    long long *H = p.H + cd.reg_off * 3;
#pragma unroll
    for (int j = 0; j < kHBufs; j++) {
        H[j * p.hstride + q] = 0;
        H[j * p.hstride + L3 + q] = 0;
        H[j * p.hstride + 2 * L3 + q] = 0;
    }
}

// Training targets: the final h_k minus the previous step's h, over the
// marker's feature scale: h_k / s_k - feature 9..11.
__global__ void k_targets(DevPtrs p, int Mtot, float *out)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= Mtot) return;
    const float *ft = p.feat + (long long)kMlpIn * k;
#pragma unroll
    for (int a = 0; a < 3; a++) out[3 * k + a] = (float)(p.hk[3 * k + a] / p.hs[k] - (double)ft[kFeatHPrev + a]);
}

// ----------------------------------------------------------------- window
// Sec. 2.5: below h_end the content and the body move up by dz rows.  With
// the ring layout the move is the origin change z0 -> z0 - dz; the dz rows
// that now form the bottom (the former top rows) restart at rest.
// The step's record for the case's log ring, taken after the window test.
struct StepRecord {
    double v[kLogFields];
};

__device__ inline StepRecord window_trigger_case(const DevPtrs &p, int c)
{
    const CaseDev &cd = p.cases[c];
    BodyDev &B = p.body[c];
    const int dz = cd.dz, nz = cd.nz;
    const double rz = B.r[2];
    const bool shift = B.err == 0 && window_shifts(cd, rz);
    B.shift_now = 0;
    if (shift) {
        B.r[2] = rz + (double)dz;
        B.z0 = wrapi(B.z0 - dz, nz);
        B.fo[0][2] += dz;   // the full-precision boxes move with the content
        B.fo[1][2] += dz;
        B.shift_now = 1;
        B.shifts += 1;
    }
    StepRecord rec;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        rec.v[a] = B.r[a];
        rec.v[12 + a] = B.v[a];
        rec.v[15 + a] = B.w[a];
        rec.v[18 + a] = B.F[a];
        rec.v[21 + a] = B.T[a];
        rec.v[24 + a] = B.Fp[a];
    }
#pragma unroll
    for (int a = 0; a < 9; a++) rec.v[3 + a] = B.d[a];
    rec.v[27] = B.resid;
    rec.v[28] = B.steps;
    rec.v[29] = B.shifts;
    rec.v[30] = B.z0;
    rec.v[31] = B.err;
    return rec;
}

// Appends a record to the case's log ring.  Written last in its kernel: the
// stores go through a plain double pointer, which the compiler must assume
// may alias the body state, so no body field is read after them.
__device__ inline void log_append(const DevPtrs &p, int c, const StepRecord &rec)
{
    BodyDev &B = p.body[c];
    const unsigned int n = B.logged;
    B.logged = n + 1;
    double *dst = p.log + ((long long)c * kLogCap + n % kLogCap) * kLogFields;
#pragma unroll
    for (int k = 0; k < kLogFields; k++) dst[k] = rec.v[k];
}

// The re-injected rows to rest, by thread t of nt: ring origin z0 and
// full-precision box origin fo after the shift.
template <class CD>
__device__ inline void reset_rows(typename CD::T *cur, const DevPtrs &p, const CaseDev &cd, int z0, const int fo[3],
                                  int fvalid, int cid, int t, int nt)
{
    const int slab = cd.nx * cd.ny;
    for (int idx = t; idx < cd.dz * slab; idx += nt) {
        const int zrow = idx / slab, rem = idx - zrow * slab;
        int zc = zrow + z0;
        if (zc >= cd.nz) zc -= cd.nz;
        typename CD::T *dst = cur + cd.pop_off + (long long)zc * slab + rem;
        if constexpr (std::is_same<CD, CodecMom>::value) {
#pragma unroll
            for (int k = 0; k < 10; k++) dst[(long long)k * cd.plane] = 0.0f;   // the rest state's moments
        } else {
            Unroll<0, Q>::run([&](auto I) {
                constexpr int i = decltype(I)::value;
                dst[(long long)i * cd.plane] = CD::template enc<i>(0.0f);
            });
            if (cd.LB[0] > 0 && fvalid) {
                const int slot = fine_slot(cd, fo, rem % cd.nx, rem / cd.nx, zrow);
                if (slot >= 0) {
                    float *F = p.fine[cid] + cd.fine_off;
                    const long long fplane = fine_plane(cd);
#pragma unroll
                    for (int i = 0; i < Q; i++) F[(long long)i * fplane + slot] = 0.0f;
                }
            }
        }
    }
}

// The end of a step, one workgroup per case, in the correction's launch: the
// forcing sequence's residual (its tile maxima are complete there) and, for
// steps that the library sequences itself (lbm_run, graph capture), the window
// test, the step's record and (TAIL_ADVANCE) the next step's body advance.  The
// correction's other workgroups, which take place at the same time, read the
// body's geometry from the copy that k_markers left (StepGeometry) and reset
// the re-injected rows.  The window test, the reset and the launches between
// them took 14 us at the end of every step; here they take none beside the
// correction.
enum { TAIL_NONE, TAIL_WINDOW, TAIL_ADVANCE };

__device__ inline void step_end(const DevPtrs &p, int c, bool live, int resid_slot, int tail)
{
    if (live && resid_slot >= 0) case_resid_total(p, p.cases[c], p.body[c], resid_slot);
    if (tail == TAIL_NONE || threadIdx.x != 0) return;
    const StepRecord rec = window_trigger_case(p, c);
    if (tail == TAIL_ADVANCE) body_advance_case(p, c);
    log_append(p, c, rec);
}

// Forced collision of Sec. 2.2: the lattice kernel wrote
// f0(rho, u) + (1 - 1/tau) f1; cells carrying an immersed force get
// f0(rho, u + tau h) - f0(rho, u) added (in the momentum-exact variant less
// the first-order term w_i xi_i . (tau - 1) rho h / cs^2).  Only cells
// marked this step can carry a force; their marks are cleared here.
template <class CD>
__global__ void __launch_bounds__(256) k_correct(typename CD::T *__restrict__ cur, DevPtrs p, int did, int resid_slot,
                                                 int tail)
{
    __shared__ ScanList list;
    const int c = blockIdx.y;
    const CaseDev &cd = p.cases[c];
    const bool live = cd.M > 0 && p.body[c].err == 0;
    if (blockIdx.x == 0) {
        step_end(p, c, live, resid_slot, tail);
        return;
    }
    if (!live) return;
    const StepGeometry &G = p.geo[c];
    const int L = cd.L, L3 = L * L * L, first = (blockIdx.x - 1) * 256;
    const bool shift = tail && G.shift;
    if (shift) {
        const int fo[3] = {G.fo[did][0], G.fo[did][1], G.fo[did][2] + cd.dz};
        reset_rows<CD>(cur, p, cd, wrapi(G.z0 - cd.dz, cd.nz), fo, G.fvalid[did], did, first + threadIdx.x,
                       (gridDim.x - 1) * 256);
    }
    if (first >= L3) return;
    unsigned char *mk = p.mark + cd.reg_off;
    const int q = scan_cells(list, first, L3, 0, [&](int i) { return mk[i]; });   // (err is settled: both streams have joined)
    if (q < 0) return;
    mk[q] = 0;
    const int a = q % L, b = (q / L) % L, cc = q / (L * L);
    const int gz = G.org[2] + cc;
    if (gz < 0 || gz >= (shift ? cd.nz - cd.dz : cd.nz)) return;   // (rows at rest from here on are left alone)
    const int gx = wrapi(G.org[0] + a, cd.nx), gy = wrapi(G.org[1] + b, cd.ny);
    int zc = gz + G.z0;
    if (zc >= cd.nz) zc -= cd.nz;
    const int off = (zc * cd.ny + gy) * cd.nx + gx;
    typename CD::T *dst = cur + cd.pop_off;
    // the accumulators, the fields and the populations in one round of loads
    const long long *H = p.H + cd.reg_off * 3;
    const float *R = p.reg + cd.reg_off * kRegFields;
    long long h0 = 0, h1 = 0, h2 = 0;
#pragma unroll
    for (int j = 0; j < kHBufs; j++) {
        h0 += H[j * p.hstride + q];
        h1 += H[j * p.hstride + L3 + q];
        h2 += H[j * p.hstride + 2 * L3 + q];
    }
    const float rho = 1.0f + R[q];
    const float u[3] = {R[L3 + q], R[2 * L3 + q], R[3 * L3 + q]};
    // a cell of the full-precision box is corrected there (FP32) and stored
    // rounded once; elsewhere the stored value is decoded and re-rounded
    int slot = -1;
    float *F = nullptr;
    long long fplane = 0;
    if (cd.LB[0] > 0 && G.fvalid[did]) {
        const int fo[3] = {G.fo[did][0], G.fo[did][1], G.fo[did][2]};
        slot = fine_slot(cd, fo, gx, gy, gz);
        F = p.fine[did] + cd.fine_off;
        fplane = fine_plane(cd);
    }
    float g[Q];
    if (slot >= 0) {
#pragma unroll
        for (int i = 0; i < Q; i++) g[i] = F[(long long)i * fplane + slot];
    } else {
        Unroll<0, Q>::run([&](auto I) {
            constexpr int i = decltype(I)::value;
            g[i] = CD::template dec<i>(dst[(long long)i * cd.plane + off]);
        });
    }
    if ((h0 | h1 | h2) == 0) return;
    const float tau = tau_at(cd.tau0, cd.nz, cd.sponge, gz);
    const float us[3] = {u[0] + tau * (float)((double)h0 * kFixInv), u[1] + tau * (float)((double)h1 * kFixInv),
                         u[2] + tau * (float)((double)h2 * kFixInv)};
    float A[Q], d[Q];
    shift_coeffs(rho, u, us, A);
    if (cd.forcing == 1) {
        // momentum-exact variant: the first-order coefficients (m = e_x, e_y,
        // e_z) become rho h instead of rho tau h
        const float k = (tau - 1.0f) * rho;
        A[1] -= k * (float)((double)h0 * kFixInv);
        A[3] -= k * (float)((double)h1 * kFixInv);
        A[9] -= k * (float)((double)h2 * kFixInv);
    }
    hermite_to_populations(A, d);
    Unroll<0, Q>::run([&](auto I) {
        constexpr int i = decltype(I)::value;
        const float v = g[i] + d[i];
        if constexpr (!std::is_same<CD, CodecF32>::value)
            if (slot >= 0) F[(long long)i * fplane + slot] = v;
        dst[(long long)i * cd.plane + off] = CD::template enc<i>(v);
    });
}

// The forced correction on moment storage: the stored moments stay the
// regularized state; the shift of every cell of the particle region goes to
// the case's forcing box, (tau h, lambda) on forced cells and zero elsewhere,
// with lambda = 1, or 1 / tau in the momentum-exact variant (the first-order
// term then carries rho h).  The box's origin is recorded in ring-slot
// coordinates, which a window shift leaves in place.  Marks are cleared.
__global__ void __launch_bounds__(256) k_correct_mom(float *__restrict__ cur, DevPtrs p, int did, int resid_slot, int tail)
{
    const int c = blockIdx.y;
    const CaseDev &cd = p.cases[c];
    const StepGeometry &G = p.geo[c];
    const bool live = cd.M > 0 && p.body[c].err == 0;
    if (blockIdx.x == 0) {
        if (live && threadIdx.x == 0) {
            BodyDev &B = p.body[c];
            B.dorg[0] = wrapi(G.org[0], cd.nx);
            B.dorg[1] = wrapi(G.org[1], cd.ny);
            B.dorg[2] = wrapi(G.org[2] + G.z0, cd.nz);
            B.dvalid = 1;
        }
        step_end(p, c, live, resid_slot, tail);
        return;
    }
    if (!live) return;
    const int L = cd.L, L3 = L * L * L, q = (blockIdx.x - 1) * 256 + threadIdx.x;
    if (tail && G.shift)
        reset_rows<CodecMom>(cur, p, cd, wrapi(G.z0 - cd.dz, cd.nz), nullptr, 0, did, q, (gridDim.x - 1) * 256);
    if (q >= L3) return;
    float *D = p.dsh + cd.reg_off * 4;
    float sh[4] = {0.0f, 0.0f, 0.0f, 1.0f};
    unsigned char &mk = p.mark[cd.reg_off + q];
    const int gz = G.org[2] + q / (L * L);
    if (mk && gz >= 0 && gz < cd.nz) {
        const long long *H = p.H + cd.reg_off * 3;
        long long h0 = 0, h1 = 0, h2 = 0;
#pragma unroll
        for (int j = 0; j < kHBufs; j++) {
            h0 += H[j * p.hstride + q];
            h1 += H[j * p.hstride + L3 + q];
            h2 += H[j * p.hstride + 2 * L3 + q];
        }
        const float tau = tau_at(cd.tau0, cd.nz, cd.sponge, gz);
        sh[0] = tau * (float)((double)h0 * kFixInv);
        sh[1] = tau * (float)((double)h1 * kFixInv);
        sh[2] = tau * (float)((double)h2 * kFixInv);
        if (cd.forcing == 1) sh[3] = 1.0f / tau;
    }
    if (mk) mk = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) D[k * (long long)L3 + q] = sh[k];
}

__global__ void k_window_trigger(DevPtrs p, int n_cases)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n_cases) return;
    const StepRecord rec = window_trigger_case(p, c);
    log_append(p, c, rec);
}

// The unread records of case c (cur of them read so far, at most room wanted) to
// pinned host memory, with the case's count.
__global__ void __launch_bounds__(256) k_log_fetch(DevPtrs p, int c, unsigned int cur, int room, LogStage *__restrict__ out)
{
    const unsigned int logged = p.body[c].logged;
    const int n = log_available(logged, cur, room);
    const unsigned int at = log_start(logged, cur);
    for (int i = threadIdx.x; i < min(n, kLogStage) * kLogFields; i += 256)
        out->rec[i] = p.log[((long long)c * kLogCap + (at + i / kLogFields) % kLogCap) * kLogFields + i % kLogFields];
    if (threadIdx.x == 0) out->logged = logged;
}

template <class CD>
__global__ void k_window_reset(typename CD::T *__restrict__ cur, DevPtrs p, int cid)
{
    const int c = blockIdx.y;
    const CaseDev &cd = p.cases[c];
    const BodyDev &B = p.body[c];
    if (!B.shift_now) return;
    // grid-strided: the launch stays small on the many steps without a shift
    reset_rows<CD>(cur, p, cd, B.z0, B.fo[cid], B.fvalid[cid], cid, blockIdx.x * blockDim.x + threadIdx.x,
                   gridDim.x * blockDim.x);
}

// --------------------------------------------------------------- launchers
hipError_t launch_body_advance(const DevPtrs &p, int n_cases, hipStream_t s)
{
    hipLaunchKernelGGL(k_body_advance, dim3((n_cases + 63) / 64), dim3(64), 0, s, p, n_cases);
    return hipGetLastError();
}

template <class CD>
static hipError_t ibm_impl(const void *prev, void *cur, const DevPtrs &p, int n_cases, int Mtot, int n_mtiles,
                           int maxL3, int cycles, int warm_mode, const _Float16 *th16, int warm_cycles, int diag,
                           int force_surface, int prev_id, hipStream_t s)
{
    using T = typename CD::T;
    const dim3 blk(256);
    const dim3 reg_grid((maxL3 + 255) / 256, n_cases);
    const dim3 tile_grid((n_mtiles + 7) / 8 * 8);
    const dim3 mark_grid((Mtot + 255) / 256);
    hipLaunchKernelGGL(k_markers, tile_grid, dim3(64), 0, s, p, n_mtiles);
    if constexpr (std::is_same<CD, CodecMom>::value) {
        int L = 1;
        while ((long long)L * L * L < maxL3) L++;
        const long long E3 = (long long)(L + 2) * (L + 2) * (L + 2);
        hipLaunchKernelGGL(k_region_expand_mom, dim3((unsigned)((E3 + 255) / 256), n_cases), blk, 0, s,
                           (const T *)prev, p);
    }
    hipLaunchKernelGGL(k_region_gather<CD>, reg_grid, blk, 0, s, (const T *)prev, p, prev_id);
    // plain start with at most kHBufs cycles: each cycle's spread rides on
    // the pass before it (force + spread 1, update c + spread c + 1)
    static_assert(kHBufs == 4, "the launch below instantiates 1..4 accumulators");
    const int fused = ibm_fused(warm_mode, cycles);
    hipLaunchKernelGGL(k_interp_force_tiles, tile_grid, blk, kLdsForce, s, p, n_mtiles, fused);
    // the fused sequence takes the force surface beside its first update pass
    // (both need the gathered region alone of what the force kernel leaves) and
    // forms the force totals in its second
    if (!fused || cycles < 2) {
        if (force_surface) hipLaunchKernelGGL(k_surface_force_tiles, tile_grid, blk, kLdsSurface, s, p, n_mtiles);
        hipLaunchKernelGGL(k_reduce_ft, dim3(n_cases), blk, 0, s, p);
    }
    // one sequence of multi-direct forcing cycles (Sec. 2.2, l = 1..4): spread
    // the increment, then interpolate and form the next increment; the
    // residual after the last spread is the sequence's residual
    auto sequence = [&](int ncyc, int slot0, int masked) {
        for (int cyc = 1; cyc <= ncyc; cyc++) {
            hipLaunchKernelGGL(k_spread_tiles, tile_grid, blk, 0, s, p, n_mtiles, masked);
            hipLaunchKernelGGL(k_interp_update_tiles<1>, tile_grid, blk, kLdsUpdate, s, p, n_mtiles, masked, -1, 0);
            if (diag || cyc == ncyc)
                hipLaunchKernelGGL(k_reduce_resid, dim3(n_cases), blk, 0, s, p, slot0 + cyc - 1, masked, 0);
        }
    };
    if (fused) {
        for (int cyc = 1; cyc <= cycles; cyc++) {
            const int to = cyc < cycles ? cyc : -1;
            // the second pass forms the force totals; the last pass's residual
            // is reduced by the forced correction (or, with diag, every
            // cycle's by its own kernel)
            const int ft = cyc == 2;
            const dim3 first(tile_grid.x, force_surface && cycles >= 2 ? 2 : 1);
            switch (cyc) {
            case 1: hipLaunchKernelGGL(k_interp_update_tiles<1>, first, blk, kLdsUpdate, s, p, n_mtiles, 0, to, ft); break;
            case 2: hipLaunchKernelGGL(k_interp_update_tiles<2>, tile_grid, blk, kLdsUpdate, s, p, n_mtiles, 0, to, ft); break;
            case 3: hipLaunchKernelGGL(k_interp_update_tiles<3>, tile_grid, blk, kLdsUpdate, s, p, n_mtiles, 0, to, ft); break;
            default: hipLaunchKernelGGL(k_interp_update_tiles<4>, tile_grid, blk, kLdsUpdate, s, p, n_mtiles, 0, to, ft); break;
            }
            if (diag)
                hipLaunchKernelGGL(k_reduce_resid, dim3(n_cases), blk, 0, s, p, cyc - 1, 0, 0);
        }
        (void)cur;
        return hipGetLastError();
    }
    if (warm_mode != 0) {
        // learned (or previous-h) start: cycles until the case's residual is
        // at or below its gate, at most warm_cycles; the rest restart plain
        if (warm_mode == 2) {
            hipError_t e = launch_mlp_warm_start(th16, p, Mtot, s);   // the network lives in mlp.hip
            if (e != hipSuccess) return e;
        } else {
            hipLaunchKernelGGL(k_warm_previous, mark_grid, blk, 0, s, p, Mtot);
        }
        const dim3 case_grid((n_cases + 63) / 64), case_blk(64);
        hipLaunchKernelGGL(k_gate_begin, case_grid, case_blk, 0, s, p, n_cases);
        for (int cyc = 1; cyc <= warm_cycles; cyc++) {
            hipLaunchKernelGGL(k_spread_tiles, tile_grid, blk, 0, s, p, n_mtiles, 1);
            hipLaunchKernelGGL(k_interp_update_tiles<1>, tile_grid, blk, kLdsUpdate, s, p, n_mtiles, 1, -1, 0);
            hipLaunchKernelGGL(k_reduce_resid, dim3(n_cases), blk, 0, s, p, cyc - 1, 1, cyc);
        }
        hipLaunchKernelGGL(k_gate, case_grid, case_blk, 0, s, p, n_cases);
        hipLaunchKernelGGL(k_fallback_markers, mark_grid, blk, 0, s, p, Mtot);
        hipLaunchKernelGGL(k_fallback_zero, reg_grid, blk, 0, s, p);
        sequence(cycles, 8, 1);
    } else {
        sequence(cycles, 0, 0);
    }
    (void)cur;
    return hipGetLastError();
}

template <class CD>
static hipError_t correct_impl(void *cur, const DevPtrs &p, int n_cases, int maxL3, int max_slab, int cur_id,
                               int resid_slot, int tail, hipStream_t s)
{
    // The first workgroup of a case ends its step; the others correct the region
    // and, on a step whose window moves, reset the rows.  A small body's region
    // has too few workgroups for the rows of a wide box (230 x 230 with a body of
    // 8 cells, 64 rows: 340 us more on such a step, 43 with one workgroup per CU,
    // no less with 1024; 160 x 160 with one of 16 in FP16: 75 and 16).
    const int reset = tail == TAIL_NONE ? 0 : std::min((max_slab + 255) / 256, std::max(8, 256 / n_cases));
    const dim3 grid(1 + std::max((maxL3 + 255) / 256, reset), n_cases);
    if constexpr (std::is_same<CD, CodecMom>::value)
        hipLaunchKernelGGL(k_correct_mom, grid, dim3(256), 0, s, (float *)cur, p, cur_id, resid_slot, tail);
    else
        hipLaunchKernelGGL(k_correct<CD>, grid, dim3(256), 0, s, (typename CD::T *)cur, p, cur_id, resid_slot, tail);
    return hipGetLastError();
}

hipError_t launch_correct(int storage, void *cur, const DevPtrs &p, int n_cases, int Mtot, int maxL3, int max_slab,
                          int cur_id, int resid_slot, int tail, hipStream_t s)
{
    if (Mtot == 0) return hipSuccess;
    switch (storage) {
    case ST_MOM: return correct_impl<CodecMom>(cur, p, n_cases, maxL3, max_slab, cur_id, resid_slot, tail, s);
    case ST_F16: return correct_impl<CodecF16>(cur, p, n_cases, maxL3, max_slab, cur_id, resid_slot, tail, s);
    case ST_BF16: return correct_impl<CodecBF16>(cur, p, n_cases, maxL3, max_slab, cur_id, resid_slot, tail, s);
    default: return correct_impl<CodecF32>(cur, p, n_cases, maxL3, max_slab, cur_id, resid_slot, tail, s);
    }
}

hipError_t launch_ibm(int storage, const void *prev, void *cur, const DevPtrs &p, int n_cases, int Mtot,
                      int n_mtiles, int maxL3, int cycles, int warm_mode, const _Float16 *th16, int warm_cycles,
                      int diag, int force_surface, int prev_id, hipStream_t s)
{
    if (Mtot == 0) return hipSuccess;
    switch (storage) {
    case ST_MOM:
        return ibm_impl<CodecMom>(prev, cur, p, n_cases, Mtot, n_mtiles, maxL3, cycles, warm_mode, th16, warm_cycles,
                                  diag, force_surface, prev_id, s);
    case ST_F16:
        return ibm_impl<CodecF16>(prev, cur, p, n_cases, Mtot, n_mtiles, maxL3, cycles, warm_mode, th16, warm_cycles,
                                  diag, force_surface, prev_id, s);
    case ST_BF16:
        return ibm_impl<CodecBF16>(prev, cur, p, n_cases, Mtot, n_mtiles, maxL3, cycles, warm_mode, th16,
                                   warm_cycles, diag, force_surface, prev_id, s);
    default:
        return ibm_impl<CodecF32>(prev, cur, p, n_cases, Mtot, n_mtiles, maxL3, cycles, warm_mode, th16, warm_cycles,
                                  diag, force_surface, prev_id, s);
    }
}

hipError_t launch_targets(const DevPtrs &p, int Mtot, float *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_targets, dim3((Mtot + 255) / 256), dim3(256), 0, s, p, Mtot, out);
    return hipGetLastError();
}

hipError_t launch_log_fetch(const DevPtrs &p, int c, unsigned int cur, int room, LogStage *out, hipStream_t s)
{
    // the launch's own status: a read does not answer for errors of earlier calls
    DevPtrs ptrs = p;
    void *args[] = {&ptrs, &c, &cur, &room, &out};
    return hipLaunchKernel((const void *)k_log_fetch, dim3(1), dim3(256), args, 0, s);
}

template <class CD>
static hipError_t window_impl(void *cur, const DevPtrs &p, int n_cases, int max_slab, int cur_id, hipStream_t s)
{
    hipLaunchKernelGGL(k_window_trigger, dim3((n_cases + 63) / 64), dim3(64), 0, s, p, n_cases);
    if (max_slab > 0) {
        // about 2048 workgroups in all, at least 8 per case
        const int per_case = std::max(8, std::min((max_slab + 255) / 256, 2048 / n_cases));
        hipLaunchKernelGGL(k_window_reset<CD>, dim3(per_case, n_cases), dim3(256), 0, s, (typename CD::T *)cur, p,
                           cur_id);
    }
    return hipGetLastError();
}

hipError_t launch_window(int storage, void *cur, const DevPtrs &p, int n_cases, int max_slab, int cur_id, hipStream_t s)
{
    switch (storage) {
    case ST_MOM: return window_impl<CodecMom>(cur, p, n_cases, max_slab, cur_id, s);
    case ST_F16: return window_impl<CodecF16>(cur, p, n_cases, max_slab, cur_id, s);
    case ST_BF16: return window_impl<CodecBF16>(cur, p, n_cases, max_slab, cur_id, s);
    default: return window_impl<CodecF32>(cur, p, n_cases, max_slab, cur_id, s);
    }
}

}  // namespace turret

// pull.hpp -- pull streaming with the boundary rules of the domain
// (arXiv 2408.15115, Sec. 2.1 and Sec. 2.5), shared by the lattice kernel and
// the particle-region gather.
#pragma once
#include "internal.hpp"
#include "lattice.hpp"

namespace turret {

// ------------------------------------------------------------------ pull
// The 27 populations arriving at cell (x, y, z): g_i = C_i(x - xi_i) from the
// previous post-collision buffer.  x, y periodic; at the z walls the missing
// population comes from specular reflection (free-slip: C_{mirror_z(i)} of the
// lateral neighbour in the same row), bounce-back (no-slip: C_{opposite(i)}
// of the cell itself) or anti-bounce-back at density 1 (constant pressure:
// f_i = -C_{opposite(i)} + 2 w_i, i.e. g_i = -g^C_{opposite(i)} in deviation
// form); periodic z wraps.  A no-slip wall may move in x at uw_lo / uw_hi:
// bounce-back then adds the wall's momentum, 6 w_i rho0 (xi_i . u_w) with
// rho0 = 1.  Physical row z sits in ring slot (z + z0) mod nz.
// WIDE: 64-bit cell offsets, which FP32 planes past 4 GiB need; also taken where
// they are the faster form (wide_planes), by the persistent FP32 schedules and by
// the region gather.
// The rest addresses each plane by its scalar base: with a direction per lane, as
// the rules of the walls need it, the addresses were half of the kernel's vector
// instructions.  Cells at a wall then load the populations that come from beyond
// it over the first ones, all of a side's in the same round and before anything
// waits for the first (one after the other they cost low boxes up to 14 %: 78 x 199
// x 13 in BF16 9.8 us a step against 8.4).
template <class CD, bool WIDE>
__device__ __forceinline__ void pull(const typename CD::T *__restrict__ src, long long plane, int nx, int ny, int nz,
                                     int z0, int bc_lo, int bc_hi, float uw_lo, float uw_hi, int x, int y, int z,
                                     float g[Q])
{
    using T = typename CD::T;
    const int xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1;
    const int ym = y == 0 ? ny - 1 : y - 1, yp = y == ny - 1 ? 0 : y + 1;
    int zc = z + z0;
    if (zc >= nz) zc -= nz;
    const int zlo = zc == 0 ? nz - 1 : zc - 1;
    const int zhi = zc == nz - 1 ? 0 : zc + 1;
    const bool wlo = (z == 0) && bc_lo != BC_PERIODIC;
    const bool whi = (z == nz - 1) && bc_hi != BC_PERIODIC;
    if constexpr (WIDE) {
        const int rowc = zc * ny, rowlo = zlo * ny, rowhi = zhi * ny;
        Unroll<0, Q>::run([&](auto I) {
            constexpr int i = decltype(I)::value;
            int sx = cx(i) == 1 ? xm : (cx(i) == -1 ? xp : x);
            int sy = cy(i) == 1 ? ym : (cy(i) == -1 ? yp : y);
            int srow = cz(i) == 1 ? rowlo : (cz(i) == -1 ? rowhi : rowc);
            int dir = i;
            bool neg = false;
            float add = 0.0f;
            if constexpr (cz(i) != 0) {
                const bool wall = cz(i) == 1 ? wlo : whi;
                const int bc = cz(i) == 1 ? bc_lo : bc_hi;
                if (wall) {
                    srow = rowc;
                    if (bc == BC_FREESLIP) {
                        dir = mirror_z(i);
                    } else {
                        dir = opposite(i);
                        sx = x;
                        sy = y;
                        neg = bc == BC_PRESSURE;
                        if constexpr (cx(i) != 0)
                            if (bc == BC_NOSLIP) add = wall_momentum<i>(cz(i) == 1 ? uw_lo : uw_hi);
                    }
                }
            }
            const float v = CD::template dec<i>(src[(long long)dir * plane + (long long)((srow + sy) * nx + sx)]);
            g[i] = (neg ? -v : v) + add;
        });
    } else {
        const unsigned int ex = sizeof(T), ey = (unsigned int)nx * ex, ez = (unsigned int)ny * ey;
        const unsigned int Z[3] = {zhi * ez, zc * ez, zlo * ez}, Y[3] = {yp * ey, y * ey, ym * ey},
                           X[3] = {xp * ex, x * ex, xm * ex};   // by component of xi, -1 .. 1
        T r[Q];
        Unroll<0, Q>::run([&](auto I) {
            constexpr int i = decltype(I)::value;
            r[i] = *plane_at(src + i * plane, Z[cz(i) + 1] + Y[cy(i) + 1] + X[cx(i) + 1]);
        });
        // side S = xi_z of the populations that come from beyond the wall
        auto from_wall = [&](auto S, int bc) {
            const bool slip = bc == BC_FREESLIP;
            Unroll<0, Q>::run([&](auto I) {
                constexpr int i = decltype(I)::value;
                if constexpr (cz(i) == decltype(S)::value)
                    r[i] = *plane_at(src + (slip ? mirror_z(i) : opposite(i)) * plane,
                                     Z[1] + (slip ? Y[cy(i) + 1] + X[cx(i) + 1] : Y[1] + X[1]));
            });
        };
        if (wlo) from_wall(std::integral_constant<int, 1>{}, bc_lo);
        if (whi) from_wall(std::integral_constant<int, -1>{}, bc_hi);
        Unroll<0, Q>::run([&](auto I) {
            constexpr int i = decltype(I)::value;
            g[i] = CD::template dec<i>(r[i]);
        });
        auto wall_rule = [&](auto S, int bc, float uw) {
            Unroll<0, Q>::run([&](auto I) {
                constexpr int i = decltype(I)::value;
                if constexpr (cz(i) == decltype(S)::value) {
                    if (bc == BC_PRESSURE) g[i] = -g[i];
                    else if constexpr (cx(i) != 0) g[i] += wall_momentum<i>(uw);
                }
            });
        };
        if (wlo && (bc_lo == BC_PRESSURE || (bc_lo == BC_NOSLIP && uw_lo != 0.0f)))
            wall_rule(std::integral_constant<int, 1>{}, bc_lo, uw_lo);
        if (whi && (bc_hi == BC_PRESSURE || (bc_hi == BC_NOSLIP && uw_hi != 0.0f)))
            wall_rule(std::integral_constant<int, -1>{}, bc_hi, uw_hi);
    }
}

}  // namespace turret

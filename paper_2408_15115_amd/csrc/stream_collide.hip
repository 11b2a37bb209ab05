// stream_collide.hip -- the fused pull-streaming + recursive-regularized
// collision kernel of the lattice Boltzmann step (arXiv 2408.15115, Sec. 2.1
// and App. A), one thread per cell over SoA storage, its launch schedules,
// and the plain streaming copy that calibrates HBM bandwidth and counters.
#include <type_traits>

#include "fine.hpp"
#include "internal.hpp"
#include "lattice.hpp"
#include "pull.hpp"

namespace turret {

// Every population is written once per step and not read again before the
// next step: the stores carry the non-temporal hint (measured faster; the
// same hint on the loads is not), unless the context's two FP32 buffers stay
// in the memory-side cache (KEEP).
template <class CD, bool KEEP, bool WIDE>
__device__ __forceinline__ void store_all(typename CD::T *__restrict__ dst, long long plane, int off, const float out[Q])
{
    Unroll<0, Q>::run([&](auto I) {
        constexpr int i = decltype(I)::value;
        typename CD::T *at = WIDE ? dst + i * plane + off
                                  : plane_at(dst + i * plane, (unsigned int)off * (unsigned int)sizeof(typename CD::T));
        if constexpr (KEEP) *at = CD::template enc<i>(out[i]);
        else __builtin_nontemporal_store(CD::template enc<i>(out[i]), at);
    });
}

// ------------------------------------------------------------ stream-collide
// One tile = blockDim.x consecutive cells of one case.  A case whose error
// bits are set is masked (frozen) so the rest of a batch goes on.  The guard
// flags non-finite density or |u| > 0.5 (bit 4) with one atomic per wave.
// COLL 0: recursive-regularized collision (App. A); COLL 1: BGK for
// comparison, f0 + (1 - 1/tau)(f - f0) with the raw off-equilibrium.
template <class CD, int COLL, bool KEEP, bool WIDE>
__device__ __forceinline__ void stream_collide_tile(const typename CD::T *__restrict__ src, typename CD::T *__restrict__ dst,
                                                    const CaseDev *__restrict__ cases, BodyDev *__restrict__ body, Tile tl,
                                                    int off)
{
    const CaseDev &cd = cases[tl.c];
    const int nx = cd.nx, ny = cd.ny, nz = cd.nz;
    const int cell = tl.first + off;   // off: this thread's cell in the tile
    if (body[tl.c].err != 0 || cell >= (int)cd.cells) return;
    const int z0 = body[tl.c].z0;
    const int x = cell % nx;
    const int t2 = cell / nx;
    const int y = t2 % ny;
    const int z = t2 / ny;
    // FP16 / BF16 with the full-precision box: the box step writes the box's
    // cells (it may run beside this kernel), so their stores are skipped
    // here (the cells are still collided for the stability guard).  The box
    // of this step starts one cell before the particle region, whose origin
    // the body advance has set.
    bool in_box = false;
    if constexpr (!std::is_same<CD, CodecF32>::value) {
        if (cd.LB[0] > 0) {
            const BodyDev &Bb = body[tl.c];
            int kx = x - wrap_mod(Bb.org[0] - 1, nx), ky = y - wrap_mod(Bb.org[1] - 1, ny);
            kx += kx < 0 ? nx : 0;
            ky += ky < 0 ? ny : 0;
            const int kz = z - (Bb.org[2] - 1);
            in_box = kx < cd.LB[0] && ky < cd.LB[1] && kz >= 0 && kz < cd.LB[2];
        }
    }
    float g[Q];
    pull<CD, WIDE>(src + cd.pop_off, cd.plane, nx, ny, nz, z0, cd.bc_lo, cd.bc_hi, cd.uw_lo, cd.uw_hi, x, y, z, g);
    const Macro M = macro(raw_moments(g));
    const float u2 = M.u[0] * M.u[0] + M.u[1] * M.u[1] + M.u[2] * M.u[2];
    const bool bad = !(fabsf(M.r1) < 1.0f) || !(u2 < 0.25f);
    const unsigned long long m = __ballot(bad);
    if (m != 0ull && (int)(threadIdx.x & 63) == __ffsll((unsigned long long)m) - 1) atomicOr(&body[tl.c].err, 4);
    const float tau = tau_at(cd.tau0, nz, cd.sponge, z);
    const float om = 1.0f - 1.0f / tau;
    float A[Q], out[Q];
    if constexpr (COLL == 1) {
        post_collision_coeffs(M, M.u, 0.0f, A);   // equilibrium coefficients only
        hermite_to_populations(A, out);
#pragma unroll
        for (int i = 0; i < Q; i++) out[i] += om * (g[i] - out[i]);
    } else {
        post_collision_coeffs(M, M.u, om, A);
        hermite_to_populations(A, out);
    }
    if (in_box) return;
    int zc = z + z0;
    if (zc >= nz) zc -= nz;
    store_all<CD, KEEP, WIDE>(dst + cd.pop_off, cd.plane, (zc * ny + y) * nx + x, out);
}

// SCHED 0: tile = workgroup; 1: XCD-grouped tiles (workgroups go
// round-robin over the 8 XCDs, so workgroup b handles tile
// (b mod 8) * (grid / 8) + b / 8 and neighbouring rows share one L2);
// 2: persistent workgroups striding over the table; 3: persistent work
// queue.  The queue is split in 8 contiguous segments with one counter each
// (a single device-wide counter serializes every grab across the XCDs);
// workgroup b starts on segment b mod 8, takes `chunk` tiles per grab and
// moves on to the other segments when its own is exhausted.  Counters only
// grow, so every workgroup leaves the loop.  4: the same 8 counters, but
// interleaved: counter g hands out chunks g, g + 8, g + 16, ... of the whole
// table, so the 8 XCDs advance through the table side by side and only the
// cases around one point of the table stream at a time (with contiguous
// segments each XCD streams a case of its own, 8 times the plane streams).
// (A queue of single wavefronts, without the barriers, was slower: four
// times the grabs on the same counters.)
// What bounds the queue is the counters: atomics of all XCDs on one address take
// their turns (some 12 ns each).  So a workgroup's first chunk is its own
// without a grab, the next grab is under way while a chunk is worked on, each
// counter has a line of its own, and a workgroup whose part is exhausted looks
// at all eight counters by loads before it grabs from another.  (With 1024
// workgroups trying all eight counters at the end, a step took 105 us at least:
// 97 x 46 x 101 in BF16, schedule 0: 15 us.)
// One instantiation per schedule keeps the register allocation of the plain
// schedules free of the loops.
constexpr int kQueueChunk = 4;

// First tile of the j-th chunk of a counter's part of the table, and the part's end.
template <int SCHED>
__device__ __forceinline__ int queue_tile(int grp, int j, int chunk, int ntiles)
{
    if constexpr (SCHED == 3) return grp * ((ntiles + 7) >> 3) + j * chunk;
    else return (8 * j + grp) * chunk;
}
template <int SCHED>
__device__ __forceinline__ int queue_end(int grp, int ntiles)
{
    if constexpr (SCHED == 3) return min(ntiles, (grp + 1) * ((ntiles + 7) >> 3));
    else return ntiles;
}

template <class CD, int SCHED, int COLL = 0, bool KEEP = false, bool WIDE = false>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(SCHED < 2 && COLL == 0 && !WIDE ? 8 : 4)))
k_stream_collide(const typename CD::T *__restrict__ src,
                                                        typename CD::T *__restrict__ dst,
                                                        const CaseDev *__restrict__ cases, BodyDev *__restrict__ body,
                                                        const Tile *__restrict__ tiles, int ntiles,
                                                        int *__restrict__ counter, int chunk)
{
    if constexpr (SCHED == 3 || SCHED == 4) {
        __shared__ int s_next[2];
        int grp = blockIdx.x & 7, j = blockIdx.x >> 3;
        for (;;) {
            const int t0 = queue_tile<SCHED>(grp, j, chunk, ntiles), end = queue_end<SCHED>(grp, ntiles);
            int next = 0;
            if (t0 < end) {
                if (threadIdx.x == 0) next = atomicAdd(&counter[kQueueStride * grp], 1);
                for (int t = t0; t < min(t0 + chunk, end); t++)
                    stream_collide_tile<CD, COLL, KEEP, WIDE>(src, dst, cases, body, tiles[t], (int)threadIdx.x);
            } else if (threadIdx.x < 64) {
                // the next part, in this workgroup's order, that has chunks left
                const int lane = threadIdx.x & 7, g = (blockIdx.x + lane) & 7;
                const int n = __hip_atomic_load(&counter[kQueueStride * g], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const bool left = queue_tile<SCHED>(g, ((int)gridDim.x - g + 7) / 8 + n, chunk, ntiles) <
                                  queue_end<SCHED>(g, ntiles);
                const int k = __ffsll((unsigned long long)(__ballot(left) & 0xff)) - 1;
                grp = k < 0 ? -1 : (blockIdx.x + k) & 7;
                if (k >= 0 && threadIdx.x == 0) next = atomicAdd(&counter[kQueueStride * grp], 1);
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                s_next[0] = grp;
                s_next[1] = next;
            }
            __syncthreads();
            grp = __builtin_amdgcn_readfirstlane(s_next[0]);
            if (grp < 0) break;
            j = ((int)gridDim.x - grp + 7) / 8 + __builtin_amdgcn_readfirstlane(s_next[1]);
        }
    } else if constexpr (SCHED == 2) {
        for (int t = blockIdx.x; t < ntiles; t += gridDim.x) stream_collide_tile<CD, COLL, KEEP, WIDE>(src, dst, cases, body, tiles[t], (int)threadIdx.x);
    } else {
        int t = blockIdx.x;
        if constexpr (SCHED == 1) t = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
        if (t < ntiles) stream_collide_tile<CD, COLL, KEEP, WIDE>(src, dst, cases, body, tiles[t], (int)threadIdx.x);
    }
}

__global__ void k_reset_counter(int *counter)
{
    if (threadIdx.x < 8) counter[kQueueStride * threadIdx.x] = 0;
}

// ------------------------------------------------------------ copy kernel
// Plain copy, one 16-byte element per lane and one element per thread (a
// flat grid reaches a higher HBM rate than a grid-strided loop).
__global__ void __launch_bounds__(256) k_copy(int4 *__restrict__ dst, const int4 *__restrict__ src, long long n)
{
    const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

hipError_t launch_copy(void *dst, const void *src, long long bytes, hipStream_t s)
{
    const long long n = bytes / 16;
    const long long grid = (n + 255) / 256;
    if (grid < 1 || grid > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_copy, dim3((unsigned)grid), dim3(256), 0, s, (int4 *)dst, (const int4 *)src, n);
    return hipGetLastError();
}

// --------------------------------------------------------------- launchers
template <class CD>
static hipError_t stream_collide_impl(const void *src, void *dst, const DevPtrs &p, int ntiles, int block,
                                      int schedule, int persist_wgs, int collision, int keep, hipStream_t s)
{
    using T = typename CD::T;
    int grid = ntiles;
    if (schedule == 1) grid = (ntiles + 7) / 8 * 8;
    if (schedule >= 2) grid = persist_wgs > 0 ? persist_wgs : 2048;
    // few tiles: smaller chunks, so that every workgroup still gets some
    const int chunk = std::max(1, std::min(kQueueChunk, ntiles / (4 * std::max(grid, 1))));
    const T *a = (const T *)src;
    T *b = (T *)dst;
    auto run = [&](auto sched, auto keep_form, auto wide) {
        hipLaunchKernelGGL((k_stream_collide<CD, decltype(sched)::value, 0, decltype(keep_form)::value, decltype(wide)::value>),
                           dim3(grid), dim3(block), 0, s, a, b, p.cases, p.body, p.tiles, ntiles, p.counter, chunk);
    };
    constexpr std::integral_constant<bool, std::is_same<CD, CodecF32>::value> f32;   // (only FP32 has the 64-bit form)
    if (collision == 1) {   // the comparison collision runs with the plain schedule only
        auto bgk = [&](auto wide) {
            hipLaunchKernelGGL((k_stream_collide<CD, 0, 1, false, decltype(wide)::value>), dim3(ntiles), dim3(block), 0, s, a,
                               b, p.cases, p.body, p.tiles, ntiles, p.counter, 1);
        };
        if (f32 && p.wide) bgk(f32);
        else bgk(std::false_type{});
        return hipGetLastError();
    }
    if (schedule == 3 || schedule == 4) hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(64), 0, s, p.counter);
    switch (schedule) {
    case 1:
        if (f32 && p.wide) run(std::integral_constant<int, 1>{}, std::false_type{}, f32);
        else run(std::integral_constant<int, 1>{}, std::false_type{}, std::false_type{});
        break;
    case 2: run(std::integral_constant<int, 2>{}, std::false_type{}, f32); break;
    case 3: run(std::integral_constant<int, 3>{}, std::false_type{}, f32); break;
    case 4: run(std::integral_constant<int, 4>{}, std::false_type{}, f32); break;
    default:
        if (f32 && p.wide) run(std::integral_constant<int, 0>{}, std::false_type{}, f32);
        else if (f32 && keep) run(std::integral_constant<int, 0>{}, f32, std::false_type{});
        else run(std::integral_constant<int, 0>{}, std::false_type{}, std::false_type{});
    }
    return hipGetLastError();
}

hipError_t launch_stream_collide(int storage, const void *src, void *dst, const DevPtrs &p, int ntiles,
                                 int block, int schedule, int persist_wgs, int collision, int keep, hipStream_t s)
{
    switch (storage) {
    case ST_F16:
        return stream_collide_impl<CodecF16>(src, dst, p, ntiles, block, schedule, persist_wgs, collision, keep, s);
    case ST_BF16:
        return stream_collide_impl<CodecBF16>(src, dst, p, ntiles, block, schedule, persist_wgs, collision, keep, s);
    default:
        return stream_collide_impl<CodecF32>(src, dst, p, ntiles, block, schedule, persist_wgs, collision, keep, s);
    }
}

}  // namespace turret

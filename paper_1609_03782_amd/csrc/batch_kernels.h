// Kernels of the batched filter's steps and what they share with the host
// side (batch.hip): instantiated per conductance by batch_inst.hip.
#pragma once
#include "internal.h"

namespace igk {

struct BatchCube {
    const float* in;
    float* out;
    float* scratch;
    BlockGeom g;
    int V;
    int npieces;       // pieces per pass (persistent launch)
    int nlast;         // items of the last pass
    int piece_off;     // first piece in the shared table
    int npass;         // passes
    int stage;         // 1: input copied to scratch first (in place, odd passes); 2: no passes, copy in -> out
    int niter;         // iterations (the resident kernel runs them all)
    long n;
};

struct BatchItem {
    int cube, pass, piece, depth;
};

constexpr int kCtrNext = 0;    // persistent launch: next item to take
constexpr int kCtrAbort = 1;   // persistent launch: set when a dependency wait ran out of time
constexpr int kCtrFin = 2;     // + cube: pieces done (rounds: of the last pass; persistent: of every pass)
// A dependency wait of the persistent launch gives up after 2 s of the
// 100 MHz constant clock (the whole 96-cube batch takes ~12 ms): every cube
// is then marked failed and every workgroup leaves, so a mistake ends in an
// error, never in a wait without end.
constexpr unsigned long long kWaitTicks = 200000000ULL;

constexpr int kResThreads = 1024;    // LDS-resident cubes: threads of the largest workgroup ...
constexpr int kResPerThread = 32;    // ... and voxels per thread

using ResidentKernel = void (*)(const BatchCube*, const int*, const DevParams*, unsigned long long*);
using BatchKernel = void (*)(const BatchCube*, const BatchItem*, const int*, const Piece*, const DevParams*, int*,
                             unsigned long long*);
using PersistKernel = void (*)(const BatchCube*, const BatchItem*, int, const Piece*, DevParams*, int, int*,
                               unsigned long long*);
// one conductance's kernels; rounds and persistent launches by pass depth 1..4
struct BatchKernels {
    ResidentKernel resident;
    BatchKernel round[4];
    PersistKernel persist[4];
};
const BatchKernels* batch_kernels(int cond);

// Batch cubes have nx <= 256: 4 voxels per lane with 1, 2 or 4 rows per
// wavefront, 3 where those still cover the row (passes of depth 1 and 2), or 1
// or 2 voxels per lane when nx < 4.
template <int COND, int T, int D>
__device__ __forceinline__ void run_piece_v(const BatchCube& cb, const float* src, float* dst, const Piece pc,
                                            const DevParams& P, float* lds) {
    const bool vec = cb.g.vec;
    if (cb.V == 1) {
        stream_piece<COND, float, 1, D, true, 1>(src, dst, cb.g, pc, P, lds);
        return;
    }
    if (cb.V == 2) {
        vec ? stream_piece<COND, float, 2, D, true, 1>(src, dst, cb.g, pc, P, lds)
            : stream_piece<COND, float, 2, D, false, 1>(src, dst, cb.g, pc, P, lds);
        return;
    }
    if constexpr (D <= 2) {
        if (cb.V == 3) {
            switch (cb.g.R) {
                case 4: vec ? stream_piece<COND, float, 3, D, true, 4>(src, dst, cb.g, pc, P, lds)
                            : stream_piece<COND, float, 3, D, false, 4>(src, dst, cb.g, pc, P, lds); break;
                case 2: vec ? stream_piece<COND, float, 3, D, true, 2>(src, dst, cb.g, pc, P, lds)
                            : stream_piece<COND, float, 3, D, false, 2>(src, dst, cb.g, pc, P, lds); break;
                default: vec ? stream_piece<COND, float, 3, D, true, 1>(src, dst, cb.g, pc, P, lds)
                             : stream_piece<COND, float, 3, D, false, 1>(src, dst, cb.g, pc, P, lds); break;
            }
            return;
        }
    }
    switch (cb.g.R) {
        case 4: vec ? stream_piece<COND, float, 4, D, true, 4>(src, dst, cb.g, pc, P, lds)
                    : stream_piece<COND, float, 4, D, false, 4>(src, dst, cb.g, pc, P, lds); break;
        case 2: vec ? stream_piece<COND, float, 4, D, true, 2>(src, dst, cb.g, pc, P, lds)
                    : stream_piece<COND, float, 4, D, false, 2>(src, dst, cb.g, pc, P, lds); break;
        default: vec ? stream_piece<COND, float, 4, D, true, 1>(src, dst, cb.g, pc, P, lds)
                     : stream_piece<COND, float, 4, D, false, 1>(src, dst, cb.g, pc, P, lds); break;
    }
}

// One round: workgroup b runs items [first[b], first[b + 1]) in turn (each one
// piece of one pass of one cube).  The loop bounds and everything the
// workgroup branches on around its barriers are the same for all its lanes; the
// completion count is one atomic of wavefront 0 to which the other lanes add 0.
template <int COND, int T>
__global__ void __launch_bounds__(1024)
k_batch_round(const BatchCube* __restrict__ cubes, const BatchItem* __restrict__ items, const int* __restrict__ first,
              const Piece* __restrict__ pieces, const DevParams* __restrict__ prm, int* __restrict__ ctr,
              unsigned long long* __restrict__ stamps) {
    extern __shared__ float lds[];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int one = threadIdx.x == 0 ? 1 : 0;
    const int it0 = __builtin_amdgcn_readfirstlane(first[blockIdx.x]);
    const int it1 = __builtin_amdgcn_readfirstlane(first[blockIdx.x + 1]);
    for (int it = it0; it < it1; ++it) {
        const BatchItem item = items[it];
        const BatchCube& cb = cubes[item.cube];
        const DevParams P = prm[item.cube];
        __syncthreads();   // the previous item is done with the LDS
        if (P.abort) continue;
        // pass k (1-based) writes out if (npass - k) is even, else scratch
        const int k = item.pass + 1;
        const float* src = item.pass == 0 ? (cb.stage ? cb.scratch : cb.in)
                                          : (((cb.npass - (k - 1)) % 2 == 0) ? cb.out : cb.scratch);
        float* dst = ((cb.npass - k) % 2 == 0) ? cb.out : cb.scratch;
        const Piece pc = pieces[cb.piece_off + item.piece];
        if constexpr (T >= 1) if (item.depth == 1) run_piece_v<COND, T, 1>(cb, src, dst, pc, P, lds);
        if constexpr (T >= 2) if (item.depth == 2) run_piece_v<COND, T, 2>(cb, src, dst, pc, P, lds);
        if constexpr (T >= 3) if (item.depth == 3) run_piece_v<COND, T, 3>(cb, src, dst, pc, P, lds);
        if constexpr (T >= 4) if (item.depth == 4) run_piece_v<COND, T, 4>(cb, src, dst, pc, P, lds);
        if (item.pass == cb.npass - 1) {   // completion stamp of the cube
            __syncthreads();
            if (w == 0) {
                const int prev = __builtin_amdgcn_readfirstlane(atomicAdd(&ctr[kCtrFin + item.cube], one));
                if (prev + 1 == cb.nlast) stamps[1 + item.cube] = wall_clock64();
            }
        }
    }
}

// The whole item list in one launch: each workgroup takes the next item from
// a counter, waits until every piece of the previous pass of its cube is
// done, runs the piece and counts it done.  Items are listed pass-major (all
// cubes' pass r before any cube's pass r + 1), so an item waits only on items
// taken earlier by running workgroups, which wait only on still earlier ones:
// every wait ends.  Cross-XCD visibility (each XCD has its own L2): the
// waiting wavefront polls with relaxed device-scope loads (no cache
// invalidation per poll), then takes one acquire fence (invalidate) before
// the workgroup reads the previous pass; after a piece, every wavefront
// drains its stores, the workgroup synchronises, and wavefront 0 takes one
// release fence (L2 write-back) before counting the piece.  Pieces of a cube
// whose input was non-finite run nothing but are still counted.
//
// All control flow around the barriers is wave-uniform: wavefront 0 as a
// whole takes, waits for and publishes items, every value it branches on is
// made uniform with readfirstlane, and each counter update is one atomic whose
// other lanes add 0.  (With a single-lane `if` around the dequeue, the
// compiler let the other lanes of the loop pass the start barrier without the
// dequeue, so they kept rerunning the previous item.)
template <int COND, int T>
__global__ void __launch_bounds__(1024)
k_batch_persist(const BatchCube* __restrict__ cubes, const BatchItem* __restrict__ items, int nitems,
                const Piece* __restrict__ pieces, DevParams* __restrict__ prm, int ncubes, int* __restrict__ ctr,
                unsigned long long* __restrict__ stamps) {
    extern __shared__ float lds[];
    __shared__ int s_item, s_go;
    const int lane = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const unsigned long long t_end = wall_clock64() + kWaitTicks;
    const int one = lane == 0 ? 1 : 0;
    for (;;) {
        if (w == 0) {
            const int it = __builtin_amdgcn_readfirstlane(atomicAdd(&ctr[kCtrNext], one));
            int go = it < nitems ? 1 : 0;
            if (go && __builtin_amdgcn_readfirstlane(
                          __hip_atomic_load(&ctr[kCtrAbort], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)))
                go = 0;
            if (go) {
                const int cube = __builtin_amdgcn_readfirstlane(items[it].cube);
                const int need = __builtin_amdgcn_readfirstlane(items[it].pass * cubes[cube].npieces);
                if (need > 0) {
                    for (;;) {
                        const int fin = __builtin_amdgcn_readfirstlane(
                            __hip_atomic_load(&ctr[kCtrFin + cube], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                        if (fin >= need) break;
                        if (__builtin_amdgcn_readfirstlane(
                                __hip_atomic_load(&ctr[kCtrAbort], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
                            go = 0;
                            break;
                        }
                        if (wall_clock64() > t_end) {
                            __hip_atomic_store(&ctr[kCtrAbort], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            for (int c = lane; c < ncubes; c += 64)
                                __hip_atomic_store(&prm[c].abort, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            go = 0;
                            break;
                        }
                        __builtin_amdgcn_s_sleep(8);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                    __builtin_amdgcn_s_waitcnt(0);
                }
            }
            s_item = it;   // every lane writes the same values
            s_go = go;
        }
        __syncthreads();
        const int go = __builtin_amdgcn_readfirstlane(s_go);
        if (!go) break;
        const int it = __builtin_amdgcn_readfirstlane(s_item);
        const BatchItem item = items[it];
        const BatchCube& cb = cubes[item.cube];
        const DevParams P = prm[item.cube];
        if (!P.abort) {
            const int k = item.pass + 1;
            const float* src = item.pass == 0 ? (cb.stage ? cb.scratch : cb.in)
                                              : (((cb.npass - (k - 1)) % 2 == 0) ? cb.out : cb.scratch);
            float* dst = ((cb.npass - k) % 2 == 0) ? cb.out : cb.scratch;
            const Piece pc = pieces[cb.piece_off + item.piece];
            if constexpr (T >= 1) if (item.depth == 1) run_piece_v<COND, T, 1>(cb, src, dst, pc, P, lds);
            if constexpr (T >= 2) if (item.depth == 2) run_piece_v<COND, T, 2>(cb, src, dst, pc, P, lds);
            if constexpr (T >= 3) if (item.depth == 3) run_piece_v<COND, T, 3>(cb, src, dst, pc, P, lds);
            if constexpr (T >= 4) if (item.depth == 4) run_piece_v<COND, T, 4>(cb, src, dst, pc, P, lds);
        }
        __builtin_amdgcn_s_waitcnt(0);   // this wavefront's stores have reached its L2
        __syncthreads();
        if (w == 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            __builtin_amdgcn_s_waitcnt(0);
            const int prev = __builtin_amdgcn_readfirstlane(
                __hip_atomic_fetch_add(&ctr[kCtrFin + item.cube], one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            if (prev + 1 == cb.npass * cb.npieces) stamps[1 + item.cube] = wall_clock64();
        }
    }
}

// LDS-resident cubes.  One workgroup holds the whole cube in LDS; with nth
// threads (64 to kResThreads, sized to the cube so that small cubes share a
// compute unit), voxel v = tid + nth k belongs to thread tid.  Each
// step, every thread evaluates its voxels from LDS into registers with the
// per-voxel formula of every other schedule (the edge terms and combine()
// in the same order), the workgroup synchronises, the new values go back to
// LDS, and it synchronises again.  A neighbour outside the cube is read as
// the voxel itself, so its difference is +0 and its edge term +0, bitwise
// what the closed coefficient gives.  HBM is read once and written once.
template <int COND>
__global__ void __launch_bounds__(kResThreads)
k_batch_resident(const BatchCube* __restrict__ cubes, const int* __restrict__ res, const DevParams* __restrict__ prm,
                 unsigned long long* __restrict__ stamps) {
    extern __shared__ float lds[];
    const int c = res[blockIdx.x];
    const BatchCube& cb = cubes[c];
    const DevParams P = prm[c];
    if (P.abort) return;
    const int nx = cb.g.nx, ny = cb.g.ny, nz = cb.g.nz;
    const int plane = nx * ny, N = plane * nz;
    const int tid = threadIdx.x, nth = blockDim.x;
    for (int v = tid; v < N; v += nth) lds[v] = cb.in[v];
    // which of the six neighbours of each of this thread's voxels exist: six
    // bits per voxel, four voxels per register
    // (coordinates stepped from voxel to voxel: v grows by nth)
    unsigned fm[kResPerThread / 4];
#pragma unroll
    for (int j = 0; j < kResPerThread / 4; ++j) fm[j] = 0u;
    {
        const int dx = nth % nx, dy = (nth / nx) % ny, dz = nth / plane;
        int x = tid % nx, y = (tid / nx) % ny, z = tid / plane;
#pragma unroll
        for (int k = 0; k < kResPerThread; ++k) {
            const unsigned b = (x > 0 ? 1u : 0u) | (x + 1 < nx ? 2u : 0u) | (y > 0 ? 4u : 0u) |
                               (y + 1 < ny ? 8u : 0u) | (z > 0 ? 16u : 0u) | (z + 1 < nz ? 32u : 0u);
            fm[k / 4] |= b << (8 * (k % 4));
            x += dx;
            if (x >= nx) { x -= nx; ++y; }
            y += dy;
            if (y >= ny) { y -= ny; ++z; }
            z += dz;
        }
    }
    __syncthreads();
    for (int s = 0; s < cb.niter; ++s) {
        // recompute the neighbour addresses every step rather than keep 6 per
        // voxel live across the loop (they would not fit in registers)
        int t0 = tid;
        asm volatile("" : "+v"(t0));
        unsigned fs[kResPerThread / 4];
#pragma unroll
        for (int j = 0; j < kResPerThread / 4; ++j) {
            fs[j] = fm[j];
            asm volatile("" : "+v"(fs[j]));
        }
        float nv[kResPerThread];
#pragma unroll
        for (int k = 0; k < kResPerThread; ++k) {
            const int v = t0 + nth * k;
            if (v < N) {
                const unsigned m = fs[k / 4] >> (8 * (k % 4));
                const float I = lds[v];
                const float xm = lds[(m & 1u) ? v - 1 : v], xp = lds[(m & 2u) ? v + 1 : v];
                const float ym = lds[(m & 4u) ? v - nx : v], yp = lds[(m & 8u) ? v + nx : v];
                const float zm = lds[(m & 16u) ? v - plane : v], zp = lds[(m & 32u) ? v + plane : v];
                const float exm = edge_term<COND>(I - xm, P.coef[0], P.kap);
                const float exp_ = edge_term<COND>(xp - I, P.coef[0], P.kap);
                const float eym = edge_term<COND>(I - ym, P.coef[1], P.kap);
                const float eyp = edge_term<COND>(yp - I, P.coef[1], P.kap);
                const float ezm = edge_term<COND>(I - zm, P.coef[2], P.kap);
                const float ezp = edge_term<COND>(zp - I, P.coef[2], P.kap);
                nv[k] = combine<COND>(I, exm, exp_, eym, eyp, ezm, ezp, P.kap, P.tau);
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kResPerThread; ++k) {
            const int v = t0 + nth * k;
            if (v < N) lds[v] = nv[k];
        }
        __syncthreads();
    }
    for (int v = tid; v < N; v += nth) cb.out[v] = lds[v];
    __syncthreads();
    if (tid == 0) stamps[1 + c] = wall_clock64();
}

}  // namespace igk

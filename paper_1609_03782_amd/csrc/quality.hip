// Filtering-quality diagnostics (Section 6): masked FP64 sums over a region
// of interest for a sweep of mask thresholds, then F, sigma_F, F_M, sigma_FM.
// See include/igquality.h.
//
// Partial sums live in 192 FP64 slots per partial: slot 3j + {0, 1, 2} holds
// (sum of original values, sum of model values, voxel count) under mask j,
// j < n_thr for the M_f thresholds and j = 63 for M_o (whose model slot is the
// unmasked model sum).  Two ways to produce the partials, both with a fixed
// work split and fixed-order sums, so results are bitwise reproducible run to
// run (no atomics):
//
//  * up to 8 thresholds (the sweep's case): voxel-parallel.  Each thread keeps
//    every mask's sums in registers and walks its voxels in a fixed order
//    (a contiguous range of ROI rows per workgroup, four loads in flight per
//    thread); a fixed shuffle tree and the wavefronts in order make one
//    partial per workgroup.  Bound by HBM.
//  * more thresholds: binned.  With the thresholds sorted, a voxel's filtered
//    value falls into one bin (the number of thresholds at or below it) and
//    mask j's sums are the sums of the bins from its rank up, so a voxel costs
//    one binary search and one addition per sum instead of one per threshold.
//    The bins live in LDS as FP64, one column per pair of lanes of a
//    wavefront, the lower lanes' voxels of a chunk added before the upper
//    lanes', so no two lanes ever meet on an address and the order of every sum
//    is fixed (the counts, whole numbers, have none).  One partial per
//    workgroup.
//
// k_quality_fold folds each slot over the partials (block b folds slot b:
// strided per-thread sums, then a fixed tree); k_quality_derive turns the 192
// sums into the diagnostics.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "igquality.h"
#include "internal.h"

namespace igk {

struct QGeom {
    long nx, ny;          // row and plane strides of the cube
    long x0, y0, z0;      // ROI origin
    long rx, ry;          // ROI extents in x and y
    long nroi;            // voxels in the ROI
    long nrows;           // ROI rows (ry * rz)
    int has_model;
    int pad;
    double thr[64];       // absolute threshold per mask (+inf: unused)
};

constexpr int kQWaves = 4;          // wavefronts per workgroup
constexpr int kQMaxBlocks = 1024;
constexpr int kQSlots = 192;        // 64 masks x (orig sum, model sum, count)
constexpr int kQSeg = 256;          // row-segment length of the voxel-parallel kernel

__device__ __forceinline__ double wsum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

template <int K>
__global__ void __launch_bounds__(256)
k_quality_vox(const float* __restrict__ orig, const float* __restrict__ filt, const float* __restrict__ model,
              QGeom g, double* __restrict__ part) {
    constexpr int NA = 3 * (K + 1);
    double acc[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[a] = 0.0;
    double thr[K];
#pragma unroll
    for (int k = 0; k < K; ++k) thr[k] = g.thr[k];
    const double thr_o = g.thr[63];
    // workgroup b takes a contiguous range of ROI rows (sequential memory),
    // (y, z) carried from row to row; within a row, thread t takes voxels
    // t, t + kQSeg, ... (kQUnroll loads of each cube in flight: every lane
    // loads, at x clamped into the row, and lanes past the row skip the sums;
    // loads under a branch made the compiler wait for each one in turn)
    constexpr int kQUnroll = 4;
    const float* mp = g.has_model ? model : orig;   // any readable cube when there is no model
    const long per = (g.nrows + gridDim.x - 1) / gridDim.x;
    const long r0 = (long)blockIdx.x * per, r1 = min(g.nrows, r0 + per);
    long y = r0 % g.ry, z = r0 / g.ry;
    for (long row = r0; row < r1; ++row) {
        const long base = g.x0 + g.nx * ((g.y0 + y) + g.ny * (g.z0 + z));
        for (long x0 = 0; x0 < g.rx; x0 += (long)kQSeg * kQUnroll) {
            float fo[kQUnroll], ff[kQUnroll], fm[kQUnroll];
            bool in[kQUnroll];
#pragma unroll
            for (int u = 0; u < kQUnroll; ++u) {
                const long x = x0 + u * kQSeg + threadIdx.x;
                const long xc = min(x, g.rx - 1);
                in[u] = x < g.rx;
                fo[u] = orig[base + xc];
                ff[u] = filt[base + xc];
                fm[u] = mp[base + xc];
            }
#pragma unroll
            for (int u = 0; u < kQUnroll; ++u) {
                if (!in[u]) continue;
                const double o = (double)fo[u], f = (double)ff[u], m = g.has_model ? (double)fm[u] : 0.0;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const bool p = f >= thr[k];
                    acc[3 * k] += p ? o : 0.0;
                    acc[3 * k + 1] += p ? m : 0.0;
                    acc[3 * k + 2] += p ? 1.0 : 0.0;
                }
                const bool po = o >= thr_o;
                acc[3 * K] += po ? o : 0.0;
                acc[3 * K + 1] += m;
                acc[3 * K + 2] += po ? 1.0 : 0.0;
            }
        }
        if (++y == g.ry) {
            y = 0;
            ++z;
        }
    }
    __shared__ double red[kQWaves][NA];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int a = 0; a < NA; ++a) {
        const double v = wsum(acc[a]);
        if (lane == 0) red[wid][a] = v;
    }
    __syncthreads();
    double* out = part + (long)blockIdx.x * kQSlots;
    for (int sl = threadIdx.x; sl < kQSlots; sl += 256) {
        const int j = sl / 3, c = sl % 3;
        const int a = j < K ? 3 * j + c : (j == 63 ? 3 * K + c : -1);
        double v = 0.0;
        if (a >= 0)
            for (int w = 0; w < kQWaves; ++w) v += red[w][a];
        out[sl] = v;
    }
}

// The M_f thresholds in ascending order as FP32 (the smallest value not below
// the FP64 threshold: the same test), NaN past the last; rank[j]: place of the
// caller's threshold j.
struct QSorted {
    float thr[64];
    unsigned char rank[64];
    int n;
    int pad;
};
constexpr int kQCols = 32;      // bin columns of a wavefront
constexpr int kQU = 16;         // voxels per lane and step, the next step's loads in flight
constexpr int kQChunk = 256 * kQU;

size_t bins_lds(int n, bool model) {
    return (size_t)kQWaves * n * kQCols * (model ? 20 : 12);
}

// STEPS: binary search steps (2^STEPS > n).  FLAT: the ROI is contiguous.  What
// bounds it: the search and the LDS additions, about 160 cycles of issue per 64
// voxels with one wavefront per SIMD (the bins fill the LDS).  46 thresholds, a
// model, 512^3: 438 us (3.7 TB/s), from 4085 us when every voxel was compared with
// every threshold (410 with the pairs' additions in one instruction, whose order
// nothing fixes); the whole call, two noise scans included, 4241 -> 738.
template <int STEPS, bool MODEL, bool FLAT>
__global__ void __launch_bounds__(256, 2)
k_quality_bins(const float* __restrict__ orig, const float* __restrict__ filt, const float* __restrict__ model,
               QGeom g, QSorted q, double* __restrict__ part) {
    extern __shared__ double qb[];
    __shared__ float T[64];
    __shared__ double tot[3][64];
    __shared__ double red[kQWaves][3];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int n = q.n, cells = n * kQCols;
    if (tid < 64) T[tid] = q.thr[tid];
    double* so = qb + w * cells;                               // bin b (1..n), column c at [(b - 1) kQCols + c]
    double* sm = qb + (kQWaves + w) * cells;
    unsigned* sc = reinterpret_cast<unsigned*>(qb + (MODEL ? 2 : 1) * kQWaves * cells) + w * cells;
    for (int k = lane; k < cells; k += 64) {
        so[k] = 0.0;
        if (MODEL) sm[k] = 0.0;
        sc[k] = 0;
    }
    __syncthreads();
    const int col = lane & (kQCols - 1);
    const bool second = lane >= kQCols;
    const double thr_o = g.thr[63];
    double a_oo = 0.0, a_m = 0.0, a_n = 0.0;
    typedef __attribute__((address_space(3))) double* ldp;

    const long chunks = (g.nroi + kQChunk - 1) / kQChunk;
    const bool big = g.rx >= (1L << 31) || g.ry >= (1L << 31);
    const long flat0 = g.x0 + g.nx * (g.y0 + g.ny * g.z0);     // FLAT: first voxel of the ROI
    auto load = [&](long ch, float (&fo)[kQU], float (&ff)[kQU], float (&fm)[kQU]) {
        const long e0 = min(ch, chunks - 1) * kQChunk;
        const int last = (int)min((long)kQChunk, g.nroi - e0) - 1;
        long rz = 0, ry = 0, rx = 0;                           // of element e0 (the same for the whole workgroup)
        if constexpr (!FLAT) {
            const long row = e0 / g.rx;
            rx = e0 - row * g.rx;
            rz = row / g.ry;
            ry = row - rz * g.ry;
        }
#pragma unroll
        for (int u = 0; u < kQU; ++u) {
            const int k = min(u * 256 + tid, last);
            long idx;
            if constexpr (FLAT) {
                idx = flat0 + e0 + k;
            } else if (big) {
                const long x = rx + k, dr = x / g.rx, y = ry + dr, dz = y / g.ry;
                idx = (g.x0 + (x - dr * g.rx)) + g.nx * ((g.y0 + (y - dz * g.ry)) + g.ny * (g.z0 + rz + dz));
            } else {   // 32-bit divisions: at most one row and kQChunk voxels past the chunk's start
                const unsigned x = (unsigned)rx + k, dr = x / (unsigned)g.rx;
                const unsigned y = (unsigned)ry + dr, dz = y / (unsigned)g.ry;
                idx = (g.x0 + (x - dr * (unsigned)g.rx)) +
                      g.nx * ((g.y0 + (y - dz * (unsigned)g.ry)) + g.ny * (g.z0 + rz + dz));
            }
            fo[u] = orig[idx];
            ff[u] = filt[idx];
            if constexpr (MODEL) fm[u] = model[idx];
        }
    };
    auto take = [&](long ch, const float (&fo)[kQU], const float (&ff)[kQU], const float (&fm)[kQU]) {
        const int count = (int)max(0L, min((long)kQChunk, g.nroi - ch * kQChunk));
        int bin[kQU], at[kQU];
        float vo[kQU], vm[kQU];
#pragma unroll
        for (int u = 0; u < kQU; ++u) {
            int b = 0;
#pragma unroll
            for (int st = 1 << (STEPS - 1); st > 0; st >>= 1) b += ff[u] >= T[b + st - 1] ? st : 0;
            bin[u] = b;
        }
#pragma unroll
        for (int u = 0; u < kQU; ++u) {
            const bool in = u * 256 + tid < count;
            const double o = fo[u];
            const bool po = in && o >= thr_o;
            a_oo += po ? o : 0.0;
            a_n += po ? 1.0 : 0.0;
            double m = 0.0;
            if constexpr (MODEL) {
                m = fm[u];
                a_m += in ? m : 0.0;
            }
            // a voxel below every threshold adds zeros to the first bin
            const bool on = in && bin[u] > 0;
            at[u] = max(bin[u] - 1, 0) * kQCols + col;
            vo[u] = on ? fo[u] : 0.0f;
            if constexpr (MODEL) vm[u] = on ? fm[u] : 0.0f;
            __hip_atomic_fetch_add(sc + at[u], on ? 1u : 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        // the pairs' lower lanes, then the upper: the statements between keep the
        // compiler from making one addition of the two, and the values FP32 meanwhile
        auto add = [&]() {
#pragma unroll
            for (int u = 0; u < kQU; ++u) {
                __builtin_amdgcn_ds_atomic_fadd_f64((ldp)(so + at[u]), (double)vo[u]);
                if constexpr (MODEL) __builtin_amdgcn_ds_atomic_fadd_f64((ldp)(sm + at[u]), (double)vm[u]);
            }
        };
        if (!second) add();
#pragma unroll
        for (int u = 0; u < kQU; ++u) {
            asm volatile("" : "+v"(vo[u]) : : "memory");
            if constexpr (MODEL) asm volatile("" : "+v"(vm[u]));
        }
        if (second) add();
    };
    float fo[2][kQU], ff[2][kQU], fm[2][kQU];
    load(blockIdx.x, fo[0], ff[0], fm[0]);
    for (long ch = blockIdx.x; ch < chunks; ch += 2L * gridDim.x) {
        load(ch + gridDim.x, fo[1], ff[1], fm[1]);             // past the last chunk: the last again, not taken
        take(ch, fo[0], ff[0], fm[0]);
        load(ch + 2L * gridDim.x, fo[0], ff[0], fm[0]);
        take(ch + gridDim.x, fo[1], ff[1], fm[1]);
    }
    const double r0 = wsum(a_oo), r1 = wsum(a_m), r2 = wsum(a_n);
    if (lane == 0) {
        red[w][0] = r0;
        red[w][1] = r1;
        red[w][2] = r2;
    }
    __syncthreads();
    // bin totals: a wavefront per bin, its 4 x 32 columns in a fixed tree
    for (int b = w; b < n; b += kQWaves) {
        double t[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < kQWaves / 2; ++k) {
            const int ww = 2 * k + (second ? 1 : 0), at = b * kQCols + col;
            t[0] += qb[ww * cells + at];
            if constexpr (MODEL) t[1] += qb[(kQWaves + ww) * cells + at];
            t[2] += (double)(reinterpret_cast<unsigned*>(qb + (MODEL ? 2 : 1) * kQWaves * cells)[ww * cells + at]);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double v = wsum(t[c]);
            if (lane == 0) tot[c][b] = v;
        }
    }
    __syncthreads();
    double* out = part + (long)blockIdx.x * kQSlots;
    for (int sl = tid; sl < kQSlots; sl += 256) {
        const int j = sl / 3, c = sl % 3;
        double v = 0.0;
        if (j < n)
            for (int b = q.rank[j]; b < n; ++b) v += tot[c][b];
        else if (j == 63)
            for (int ww = 0; ww < kQWaves; ++ww) v += red[ww][c];
        out[sl] = v;
    }
}

// Block b folds slot b over `count` partials: thread t sums partials t,
// t + 256, ... in order, then a fixed tree over the threads.
__global__ void __launch_bounds__(256)
k_quality_fold(const double* __restrict__ part, long count, double* __restrict__ sums) {
    const int sl = blockIdx.x;
    double v = 0.0;
    for (long i = threadIdx.x; i < count; i += 256) v += part[i * kQSlots + sl];
    v = wsum(v);
    __shared__ double sh[4];
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) sums[sl] = ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

// One wavefront: lane j derives the diagnostics of mask j.
__global__ void __launch_bounds__(64)
k_quality_derive(const double* __restrict__ sums, int nthr, int has_model, double rms_o, double rms_f, double indep,
                 long nroi, ig_quality_result* __restrict__ out) {
    const int j = threadIdx.x;
    const double s1 = sums[3 * j], s2 = sums[3 * j + 1];
    const long long n = (long long)sums[3 * j + 2];
    const double S_oo = sums[3 * 63], S_m = sums[3 * 63 + 1];
    const long long N_o = (long long)sums[3 * 63 + 2];
    const double nan = __builtin_nan("");
    if (j == 63) {
        out->rms_o = rms_o;
        out->rms_f = rms_f;
        out->S_oo = S_oo;
        out->S_m = has_model ? S_m : 0.0;
        out->N_o = N_o;
        out->n_roi = nroi;
    }
    if (j < IG_QUALITY_MAX_THR) {
        const bool on = j < nthr;
        const double sig_oo = sqrt((double)N_o / indep) * rms_o;
        const double sig_of = sqrt((double)n / indep) * rms_f;
        double F = nan, sF = nan, FM = nan, sFM = nan;
        if (on && S_oo != 0.0) {
            F = fabs(s1) / fabs(S_oo);
            sF = sqrt(sig_of * sig_of / (S_oo * S_oo) + s1 * s1 * sig_oo * sig_oo / (S_oo * S_oo * S_oo * S_oo));
        }
        if (on && has_model && S_m != 0.0) {
            FM = fabs(s2) / fabs(S_m);
            sFM = sig_of / fabs(S_m);
        }
        out->S_of[j] = on ? s1 : 0.0;
        out->S_mf[j] = on && has_model ? s2 : 0.0;
        out->N_f[j] = on ? n : 0;
        out->F[j] = F;
        out->sigma_F[j] = sF;
        out->F_M[j] = FM;
        out->sigma_FM[j] = sFM;
    }
}

}  // namespace igk

// ====================================================================== host
using namespace igk;
#define fail igk_fail
#define HIP_TRY(expr)                                                                              \
    do {                                                                                           \
        hipError_t e_ = (expr);                                                                    \
        if (e_ != hipSuccess)                                                                      \
            return fail(e_ == hipErrorOutOfMemory ? IG_ERR_OUT_OF_MEMORY : IG_ERR_DEVICE, "%s: %s", \
                        #expr, hipGetErrorString(e_));                                             \
    } while (0)

namespace {

struct QScratch {   // per-device partials, folded sums and result slot, kept for the process
    double* part = nullptr;
    double* sums = nullptr;
    ig_quality_result* res = nullptr;
};
std::mutex g_qmu;
QScratch g_qs[64];

ig_status noise_level(const float* d, long n, int device, void* stream, double given, double* rms) {
    if (given > 0.0) {
        *rms = given;
        return IG_OK;
    }
    double sum = 0.0, sumsq = 0.0;
    int64_t bad = 0;
    ig_status st = ig_reduce(d, IG_F32, n, device, stream, &sum, &sumsq, &bad);
    if (st != IG_OK) return st;
    if (bad) return fail(IG_ERR_NONFINITE, "a cube whose rms is to be estimated holds %lld non-finite voxels",
                         (long long)bad);
    *rms = n > 0 ? std::sqrt(sumsq / (double)n) : 0.0;
    return IG_OK;
}

}  // namespace

extern "C" ig_status ig_quality(const ig_quality_params* q, const float* d_orig, const float* d_filt,
                                const float* d_model, int64_t nx, int64_t ny, int64_t nz, int device,
                                void* hip_stream, ig_quality_result* out) {
    if (!q || !out || !d_orig || !d_filt) return fail(IG_ERR_INVALID_ARG, "NULL argument");
    if (q->struct_size != (int32_t)sizeof(ig_quality_params)) return fail(IG_ERR_INVALID_ARG, "struct_size");
    if (nx < 1 || ny < 1 || nz < 1) return fail(IG_ERR_INVALID_ARG, "bad cube size");
    if (q->n_thr < 1 || q->n_thr > IG_QUALITY_MAX_THR) return fail(IG_ERR_INVALID_ARG, "n_thr out of range");
    for (int j = 0; j < q->n_thr; ++j)
        if (!std::isfinite(q->thr_f[j])) return fail(IG_ERR_INVALID_ARG, "thr_f[%d] is not finite", j);
    if (!std::isfinite(q->thr_o)) return fail(IG_ERR_INVALID_ARG, "thr_o is not finite");
    if (!(q->indep > 0.0) || !std::isfinite(q->indep)) return fail(IG_ERR_INVALID_ARG, "indep must be > 0");
    if (!std::isfinite(q->rms_o) || !std::isfinite(q->rms_f)) return fail(IG_ERR_INVALID_ARG, "rms not finite");
    int64_t r[6] = {q->roi[0], q->roi[1], q->roi[2], q->roi[3], q->roi[4], q->roi[5]};
    if (!(r[0] | r[1] | r[2] | r[3] | r[4] | r[5])) {
        r[1] = nx; r[3] = ny; r[5] = nz;
    }
    if (r[0] < 0 || r[1] > nx || r[0] >= r[1] || r[2] < 0 || r[3] > ny || r[2] >= r[3] || r[4] < 0 || r[5] > nz ||
        r[4] >= r[5])
        return fail(IG_ERR_INVALID_ARG, "ROI empty or outside the cube");
    if (device < 0 || device >= 64) return fail(IG_ERR_INVALID_ARG, "bad device %d", device);
    {
        const size_t bytes = (size_t)(nx * ny * nz) * 4;
        ig_status cb = igk_check_buffer(d_orig, bytes, device, "d_orig");
        if (cb == IG_OK) cb = igk_check_buffer(d_filt, bytes, device, "d_filt");
        if (cb == IG_OK && d_model) cb = igk_check_buffer(d_model, bytes, device, "d_model");
        if (cb != IG_OK) return cb;
    }
    int prev = -1;
    (void)hipGetDevice(&prev);
    if (hipSetDevice(device) != hipSuccess) return fail(IG_ERR_DEVICE, "hipSetDevice(%d)", device);
    struct Restore { int d; ~Restore() { if (d >= 0) (void)hipSetDevice(d); } } restore{prev};
    hipStream_t s = (hipStream_t)hip_stream;

    const long n = (long)(nx * ny * nz);
    double rms_o = 0.0, rms_f = 0.0;
    ig_status st = noise_level(d_orig, n, device, hip_stream, q->rms_o, &rms_o);
    if (st != IG_OK) return st;
    st = noise_level(d_filt, n, device, hip_stream, q->rms_f, &rms_f);
    if (st != IG_OK) return st;

    QGeom g{};
    g.nx = nx; g.ny = ny;
    g.x0 = r[0]; g.y0 = r[2]; g.z0 = r[4];
    g.rx = r[1] - r[0]; g.ry = r[3] - r[2];
    g.nroi = g.rx * g.ry * (r[5] - r[4]);
    g.has_model = d_model != nullptr;
    for (int j = 0; j < 64; ++j) g.thr[j] = INFINITY;
    for (int j = 0; j < q->n_thr; ++j) g.thr[j] = q->thr_f[j] * rms_f;
    g.thr[63] = q->thr_o * rms_o;

    g.nrows = g.ry * (r[5] - r[4]);
    std::lock_guard<std::mutex> lk(g_qmu);
    QScratch& qs = g_qs[device];
    if (!qs.part) {   // all three or none: a failure leaves the cache empty
        QScratch fresh{};
        hipError_t e = igk_malloc((void**)&fresh.part, (size_t)kQMaxBlocks * kQWaves * kQSlots * sizeof(double));
        if (e == hipSuccess) e = igk_malloc((void**)&fresh.sums, (size_t)kQSlots * sizeof(double));
        if (e == hipSuccess) e = igk_malloc((void**)&fresh.res, sizeof(ig_quality_result));
        if (e != hipSuccess) {
            igk_free(fresh.part);
            igk_free(fresh.sums);
            igk_free(fresh.res);
            return fail(e == hipErrorOutOfMemory ? IG_ERR_OUT_OF_MEMORY : IG_ERR_DEVICE, "quality scratch: %s",
                        hipGetErrorString(e));
        }
        qs = fresh;
    }
    long count;
    if (q->n_thr <= 8) {
        const int K = q->n_thr <= 1 ? 1 : q->n_thr <= 2 ? 2 : q->n_thr <= 4 ? 4 : 8;
        const int blocks = (int)std::min<long>(kQMaxBlocks * 2, g.nrows);
        auto k = K == 1 ? k_quality_vox<1> : K == 2 ? k_quality_vox<2> : K == 4 ? k_quality_vox<4> : k_quality_vox<8>;
        hipLaunchKernelGGL(k, dim3(blocks), dim3(256), 0, s, d_orig, d_filt, d_model, g, qs.part);
        count = blocks;
    } else {
        QSorted qsrt{};
        int order[64];
        for (int j = 0; j < q->n_thr; ++j) order[j] = j;
        std::stable_sort(order, order + q->n_thr, [&](int a, int b) { return g.thr[a] < g.thr[b]; });
        for (int r = 0; r < 64; ++r) {
            qsrt.thr[r] = NAN;
            if (r >= q->n_thr) continue;
            const float f = (float)g.thr[order[r]];
            qsrt.thr[r] = (double)f < g.thr[order[r]] ? std::nextafterf(f, INFINITY) : f;
            qsrt.rank[order[r]] = (unsigned char)r;
        }
        qsrt.n = q->n_thr;
        const bool flat = g.rx == nx && (g.ry == ny || r[5] - r[4] == 1), mod = g.has_model != 0;
        using Kern = void (*)(const float*, const float*, const float*, QGeom, QSorted, double*);
        const Kern kerns[3][2][2] = {
            {{k_quality_bins<4, false, false>, k_quality_bins<4, false, true>},
             {k_quality_bins<4, true, false>, k_quality_bins<4, true, true>}},
            {{k_quality_bins<5, false, false>, k_quality_bins<5, false, true>},
             {k_quality_bins<5, true, false>, k_quality_bins<5, true, true>}},
            {{k_quality_bins<6, false, false>, k_quality_bins<6, false, true>},
             {k_quality_bins<6, true, false>, k_quality_bins<6, true, true>}}};
        const Kern k = kerns[q->n_thr < 16 ? 0 : q->n_thr < 32 ? 1 : 2][mod][flat];
        const size_t lds = bins_lds(q->n_thr, mod);
        if (lds > 65536)
            HIP_TRY(hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        // one round of workgroups: what the compute units hold with these bins
        const int per_cu = (int)std::max<size_t>(1, std::min<size_t>(4, (kMaxLds - 2048) / lds));
        int ncu = 256;
        (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device);
        const int blocks = (int)std::min<long>(std::min<long>((long)ncu * per_cu, kQMaxBlocks), (g.nroi + kQChunk - 1) / kQChunk);
        hipLaunchKernelGGL(k, dim3(blocks), dim3(256), lds, s, d_orig, d_filt, d_model, g, qsrt, qs.part);
        count = blocks;
    }
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_quality_fold, dim3(kQSlots), dim3(256), 0, s, qs.part, count, qs.sums);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_quality_derive, dim3(1), dim3(64), 0, s, qs.sums, q->n_thr, g.has_model, rms_o, rms_f,
                       q->indep, g.nroi, qs.res);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpyAsync(out, qs.res, sizeof(ig_quality_result), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    return IG_OK;
}

// Free the per-device quality scratch (the next ig_quality allocates it again).
void igk_quality_cache_release() {
    std::lock_guard<std::mutex> lk(g_qmu);
    int prev = -1;
    (void)hipGetDevice(&prev);
    for (int d = 0; d < 64; ++d) {
        QScratch& qs = g_qs[d];
        if (!qs.part && !qs.sums && !qs.res) continue;
        (void)hipSetDevice(d);
        igk_free(qs.part);
        igk_free(qs.sums);
        igk_free(qs.res);
        qs = QScratch{};
    }
    if (prev >= 0) (void)hipSetDevice(prev);
}

// Batched filter: many independent FP32 cubes of uneven sizes and parameters,
// captured once per batch signature into one HIP graph and replayed.  See
// ig_filter_batch in include/igfilter.h.
//
// Work items are (cube, pass, piece).  Round r of the graph is one launch of
// k_batch_round over pass r of every cube that has one, largest cubes first,
// dealt to the workgroups in equal shares of (cube, tile, plane) steps; the
// kernel boundary between rounds orders the passes, so no workgroup ever waits
// on another.  Cubes small enough to live in one compute
// unit's LDS (at most kResidentMax voxels, when enabled) skip the passes: one
// workgroup of k_batch_resident loads the cube, runs all n steps in LDS and
// writes the result.  The graph holds the counter reset (which also stamps
// the start on the GPU's constant-rate clock), the per-cube FP64 noise-level
// scan, the staging copies, the resident launch and the rounds; the
// descriptor tables are uploaded once when the plan is built.  The last piece
// of a cube's last pass (or its resident workgroup) stamps the clock, giving
// each cube's completion latency.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "batch_kernels.h"

using namespace igk;

namespace igk {

// ------------------------------------------------------------ rms pre-pass
struct SumChunk {
    int cube;
    int pad;
    long off, len;
};

__global__ void __launch_bounds__(256)
k_batch_sum(const BatchCube* __restrict__ cubes, const SumChunk* __restrict__ chunks, double* __restrict__ part,
            int from_out) {
    const SumChunk ch = chunks[blockIdx.x];
    const float* x = from_out ? cubes[ch.cube].out : cubes[ch.cube].in;
    double s1 = 0.0, s2 = 0.0, bad = 0.0;
    auto add = [&](float f) {
        if (!isfinite(f)) {
            bad += 1.0;
            return;
        }
        s1 += (double)f;
        s2 += (double)f * (double)f;
    };
    // groups of 8 loads in flight together, summed in the same order as one
    // at a time
    long i = threadIdx.x;
    for (; i + 7 * 256 < ch.len; i += 8 * 256) {
        float f[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) f[u] = x[ch.off + i + u * 256];
#pragma unroll
        for (int u = 0; u < 8; ++u) add(f[u]);
    }
    for (; i < ch.len; i += 256) add(x[ch.off + i]);
    __shared__ double sh[3][4];
    for (int o = 32; o > 0; o >>= 1) {
        s1 += __shfl_xor(s1, o, 64);
        s2 += __shfl_xor(s2, o, 64);
        bad += __shfl_xor(bad, o, 64);
    }
    const int wid = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { sh[0][wid] = s1; sh[1][wid] = s2; sh[2][wid] = bad; }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int k = 0; k < 3; ++k) part[3 * blockIdx.x + k] = ((sh[k][0] + sh[k][1]) + sh[k][2]) + sh[k][3];
}

// One workgroup per cube: fold its chunk partials in order, derive DevParams.
__global__ void __launch_bounds__(64)
k_batch_params(const ParamIn* __restrict__ pin, const int* __restrict__ chunk_first, const double* __restrict__ part,
               const long* __restrict__ nvox, DevParams* __restrict__ out, int sums_only) {
    const int c = blockIdx.x;
    if (threadIdx.x != 0) return;
    double s1 = 0.0, s2 = 0.0, bad = 0.0;
    for (int j = chunk_first[c]; j < chunk_first[c + 1]; ++j) {
        s1 += part[3 * j];
        s2 += part[3 * j + 1];
        bad += part[3 * j + 2];
    }
    if (sums_only) {   // output sums for the statistics: only the sum slot
        out[c].sum = s1;
        return;
    }
    const ParamIn in = pin[c];
    const long n = nvox[c];
    DevParams P;
    P.sum = s1;
    P.sumsq = s2;
    P.nonfinite = (long long)bad;
    P.abort = P.nonfinite > 0 ? 1 : 0;
    P.pad = 0;
    const double rho = in.rms > 0.0 ? in.rms : (n > 0 ? sqrt(s2 / (double)n) : 0.0);
    P.rho = rho;
    const double kr2 = ((double)in.K * rho) * ((double)in.K * rho);
    const double inv = kr2 > 0.0 ? 1.0 / kr2 : 0.0;
    double kap = in.cond == COND_PM_EXP ? -1.4426950408889634 * inv : inv;
    if (!(fabs(kap) <= 3.0e38)) kap = kap < 0 ? -3.0e38 : 3.0e38;
    P.kap = (float)kap;
    P.tau = in.tau;
    for (int a = 0; a < 3; ++a) {
        if (in.cond == COND_PM_EXP) P.coef[a] = (float)log2((double)in.tau * in.C[a]);
        else if (in.cond == COND_PM_RATIONAL) P.coef[a] = (float)((double)in.tau * in.C[a]);
        else P.coef[a] = in.C[a];
    }
    P.closed = in.cond == COND_PM_EXP ? -INFINITY : 0.0f;
    out[c] = P;
}

// Clear the counters and stamps (a kernel, so graph replays start clean) and
// stamp the start of the batch.
__global__ void k_batch_reset(int* __restrict__ ctr, int nctr, unsigned long long* __restrict__ stamps, int nst) {
    for (int i = threadIdx.x; i < nctr; i += blockDim.x) ctr[i] = 0;
    const unsigned long long t0 = wall_clock64();
    for (int i = threadIdx.x; i < nst; i += blockDim.x) stamps[i] = i == 0 ? t0 : 0ULL;
}

// Stage in-place inputs with an odd pass count through scratch (copy), so
// the last pass lands in the output buffer.
__global__ void __launch_bounds__(256)
k_batch_stage(const BatchCube* __restrict__ cubes, const SumChunk* __restrict__ chunks, const DevParams* __restrict__ prm) {
    const SumChunk ch = chunks[blockIdx.x];
    const BatchCube& cb = cubes[ch.cube];
    if (!cb.stage || prm[ch.cube].abort) return;
    float* to = cb.stage == 1 ? cb.scratch : cb.out;
    for (long i = threadIdx.x; i < ch.len; i += 256) to[ch.off + i] = cb.in[ch.off + i];
}

// A cube whose input held NaN or Inf ran no step: its output becomes NaN, so
// the failure is visible without the statistics.  A no-op for other cubes.
__global__ void __launch_bounds__(256)
k_batch_nan(const BatchCube* __restrict__ cubes, const SumChunk* __restrict__ chunks, const DevParams* __restrict__ prm) {
    const SumChunk ch = chunks[blockIdx.x];
    if (!prm[ch.cube].abort) return;
    float* out = cubes[ch.cube].out;
    const float q = __builtin_nanf("");
    for (long i = threadIdx.x; i < ch.len; i += 256) out[ch.off + i] = q;
}

const BatchKernels* batch_kernels_c0();
const BatchKernels* batch_kernels_c1();
const BatchKernels* batch_kernels_c2();
const BatchKernels* batch_kernels(int cond) {
    return cond == COND_INTENSITY ? batch_kernels_c0() : cond == COND_PM_EXP ? batch_kernels_c1() : batch_kernels_c2();
}

}  // namespace igk

// ====================================================================== host
#define fail igk_fail
#define HIP_TRY(expr)                                                                              \
    do {                                                                                           \
        hipError_t e_ = (expr);                                                                    \
        if (e_ != hipSuccess)                                                                      \
            return fail(e_ == hipErrorOutOfMemory ? IG_ERR_OUT_OF_MEMORY : IG_ERR_DEVICE, "%s: %s", \
                        #expr, hipGetErrorString(e_));                                             \
    } while (0)

namespace {

constexpr long kChunk = 1L << 16;   // voxels per rms partial (many workgroups even for small batches)

template <typename T>
struct DevBuf {
    T* p = nullptr;
    size_t n = 0;
    ~DevBuf() { igk_free(p); }
    hipError_t alloc(size_t count) {
        n = count;
        return igk_malloc((void**)&p, std::max<size_t>(1, count) * sizeof(T));
    }
};
struct BatchPlan {
    int device = 0;
    int cond = 0, T = 1, W = 16;
    int persist = 0;              // 1: one persistent launch instead of one launch per round
    int grid = 0;                 // persistent launch: workgroups
    int count = 0;
    std::vector<int> passes;
    DevBuf<float> scratch;
    DevBuf<BatchCube> d_cubes;
    DevBuf<BatchItem> d_items;
    DevBuf<Piece> d_pieces;
    DevBuf<SumChunk> d_chunks;
    DevBuf<int> d_chunk_first;
    DevBuf<double> d_part;
    DevBuf<ParamIn> d_pin;
    DevBuf<long> d_nvox;
    DevBuf<DevParams> d_params;
    DevBuf<DevParams> d_outsum;
    DevBuf<int> d_ctr;
    DevBuf<unsigned long long> d_stamps;
    DevBuf<int> d_res;             // cubes run LDS-resident, grouped by workgroup size
    int nres = 0;
    std::vector<int> res_off{0};  // class j (64 << j threads): d_res[res_off[j], res_off[j+1])
    std::vector<size_t> res_lds;  // per class: LDS bytes of its largest cube
    std::vector<int> resident;    // per cube: wavefronts of its resident workgroup (0: not resident)
    std::vector<int> niter;
    std::vector<int> round_off;   // round r: workgroups [round_off[r], round_off[r+1]), first items at d_first[round_off[r] + r]
    DevBuf<int> d_first;
    int nitems = 0, nchunks = 0;
    size_t lds = 0;
    hipStream_t cap = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    // the descriptor table as last uploaded (pinned, so the upload of a later
    // call's buffer addresses is a plain asynchronous copy) and its addresses
    BatchCube* h_cubes = nullptr;
    std::vector<std::pair<const void*, void*>> bufs;
    hipEvent_t done = nullptr;    // recorded after every launch of the graph
    uint64_t last_use = 0;        // for least-recently-used eviction
    ~BatchPlan() {
        if (done) {   // the graph may still run on the caller's stream
            (void)hipEventSynchronize(done);
            (void)hipEventDestroy(done);
        }
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
        if (cap) (void)hipStreamDestroy(cap);
        igk_host_free(h_cubes);
    }
};

std::mutex g_mu;
// Plans keyed by shapes, parameters and settings (not buffer addresses): a
// call with other tensors of the same shapes reuses the plan and rewrites its
// descriptor table.  At most kMaxPlans are kept; the least recently used one
// is dropped (after its last launch has finished) to make room.
constexpr size_t kMaxPlans = 8;
std::map<std::vector<uint64_t>, std::unique_ptr<BatchPlan>> g_cache;
uint64_t g_use = 0;
// The last call's items (validated) and plan: a call with byte-identical items
// and the same settings reuses it without validating or hashing again.
struct LastCall {
    std::vector<ig_batch_item> items;
    int device = -1, T = 0, W = 0, Z = 0, res = 0, persist = 0;
    BatchPlan* plan = nullptr;
};
LastCall g_last;
int g_batch_T = 0;    // 0: default choice
int g_batch_W = 16;
int g_batch_Z = 32;   // planes per z-chunk of a piece
int g_batch_persist = 0;   // 1: one persistent launch runs every pass
constexpr int kResidentMax = kResThreads * kResPerThread;   // 32768 voxels: 128 KiB of LDS
int g_batch_res = kResidentMax;   // cubes of at most this many voxels run LDS-resident (0: none)

std::vector<uint64_t> signature(const ig_batch_item* items, int count, int device) {
    std::vector<uint64_t> key;
    key.push_back((uint64_t)device);
    key.push_back((uint64_t)g_batch_T);
    key.push_back((uint64_t)g_batch_W);
    key.push_back((uint64_t)(g_batch_persist ? g_batch_Z : 0));   // the rounds deal shares, not chunks
    key.push_back((uint64_t)g_batch_res);
    key.push_back((uint64_t)g_batch_persist);
    for (int i = 0; i < count; ++i) {
        uint64_t w[(sizeof(ig_params) + 7) / 8] = {};
        std::memcpy(w, &items[i].p, sizeof(ig_params));
        for (uint64_t v : w) key.push_back(v);
        // what the plan depends on besides shapes: in place or not (staging)
        // and the buffers' alignment within 16 bytes (vector access)
        const uintptr_t a = (uintptr_t)items[i].d_in, b = (uintptr_t)items[i].d_out;
        key.push_back((uint64_t)((a % 16) << 8 | (b % 16) << 1 | (a == b ? 1 : 0)));
    }
    return key;
}

// Point the plan's descriptor table at this call's buffers (same shapes,
// alignment and in-place pattern as when it was built).  Enqueued on the
// caller's stream before the graph launch; the pinned table is rewritten only
// once the previous launch of the plan (and so its upload) has finished.
ig_status rebind(BatchPlan* bp, const ig_batch_item* items, int count, hipStream_t s) {
    bool same = (int)bp->bufs.size() == count;
    for (int c = 0; same && c < count; ++c)
        same = bp->bufs[c].first == items[c].d_in && bp->bufs[c].second == items[c].d_out;
    if (same) return IG_OK;
    HIP_TRY(hipEventSynchronize(bp->done));
    bp->bufs.resize(count);
    for (int c = 0; c < count; ++c) {
        bp->h_cubes[c].in = (const float*)items[c].d_in;
        bp->h_cubes[c].out = (float*)items[c].d_out;
        bp->bufs[c] = {items[c].d_in, items[c].d_out};
    }
    HIP_TRY(hipMemcpyAsync(bp->d_cubes.p, bp->h_cubes, count * sizeof(BatchCube), hipMemcpyHostToDevice, s));
    return IG_OK;
}

// The rounds: round r lays the tiles of pass r of every cube (largest cubes
// first) end to end as a sequence of plane steps and deals it to the workgroups
// in contiguous shares of equal cost, so that no round waits for a longest
// piece (fixed chunks of 32 planes left the 96-cube batch's first rounds six
// turns of the GPU for 5.7 turns' work, and paid the pipeline's fill on every
// chunk; 96 cubes of 32 .. 256 voxels a side: 9.11 -> 6.96 ms, the rows of 3
// voxels per lane included).  A share's items are its
// parts of the tiles it meets; each refills the pipeline (3 depths), which
// counts at the start of a tile.  A plane step's weight is the line of
// step_weight (idle rows of a tile that is taller than its cube cost little).
void deal_rounds(std::vector<BatchCube>& cubes, const std::vector<std::vector<int>>& depths,
                 const std::vector<int>& order, int maxpass, long slots, int W, std::vector<BatchItem>* its,
                 std::vector<Piece>* pieces, std::vector<int>* first, std::vector<int>* round_off) {
    struct Tile { int cube, tx, ty; double w, start; };   // start: its cost position
    for (int k = 0; k < maxpass; ++k) {
        std::vector<Tile> tiles;
        double tot = 0.0;
        long planes = 0;
        for (int c : order) {
            if (k >= cubes[c].npass) continue;
            const BlockGeom& g = cubes[c].g;
            const int busy = std::min(W, (std::min(g.ny, W * g.R) + g.R - 1) / g.R);
            const double w = step_weight(cubes[c].V, g.R, busy, g.vec == 0);
            for (int t = 0; t < g.ntx * g.nty; ++t) {
                tiles.push_back(Tile{c, t % g.ntx, t / g.ntx, w, tot});
                tot += w * (g.nz + 3 * depths[c][k]);
                planes += g.nz;
            }
            if (k + 1 == cubes[c].npass) cubes[c].nlast = 0;   // counted below
        }
        const long G = std::max(1L, std::min(slots, planes));
        size_t t = 0;
        int z = 0;                                   // next plane of tile t
        for (long b = 0; b < G; ++b) {
            first->push_back((int)its->size());
            const double end = b + 1 == G ? 1e300 : tot * (double)(b + 1) / (double)G;
            while (t < tiles.size()) {
                const Tile& tl = tiles[t];
                BatchCube& cb = cubes[tl.cube];
                const int fill = 3 * depths[tl.cube][k];
                // planes of this tile that start before the share's end
                const double upto = (end - tl.start) / tl.w - fill;
                const int z1 = upto >= cb.g.nz ? cb.g.nz : std::max(z, (int)upto);
                if (z1 > z) {
                    its->push_back(BatchItem{tl.cube, k, (int)pieces->size() - cb.piece_off, depths[tl.cube][k]});
                    pieces->push_back(Piece{tl.tx, tl.ty, z, z1});
                    if (k + 1 == cb.npass) ++cb.nlast;
                }
                z = z1;
                if (z < cb.g.nz) break;              // the share ends inside this tile
                ++t;
                z = 0;
            }
        }
        first->push_back((int)its->size());
        round_off->push_back(round_off->back() + (int)G);
    }
}

ig_status build_plan(const ig_batch_item* items, int count, int device, BatchPlan* bp) {
    bp->device = device;
    bp->count = count;
    bp->cond = items[0].p.cond;
    // LDS-resident: small cubes with at least one step
    bp->resident.assign(count, 0);
    bp->niter.assign(count, 0);
    int maxn = 0;
    long maxnx = 0;
    for (int i = 0; i < count; ++i) {
        const ig_params& p = items[i].p;
        bp->niter[i] = p.n_iter;
        bp->resident[i] = (g_batch_res > 0 && p.n_iter > 0 && p.nx * p.ny * p.nz <= g_batch_res) ? 1 : 0;
        if (bp->resident[i]) continue;
        maxn = std::max(maxn, p.n_iter);
        maxnx = std::max<long>(maxnx, p.nx);
    }
    bp->W = g_batch_W;
    bp->persist = g_batch_persist;
    bp->T = g_batch_T > 0 ? g_batch_T : std::max(1, std::min(2, maxn));
    const int T = bp->T, W = bp->W;
    if (maxnx > 256) return fail(IG_ERR_UNSUPPORTED, "batch items need nx <= 256 (unless LDS-resident)");
    int ncu = 256;
    (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device);

    // per-cube plans (persistent launch: pieces of ~32 planes), scratch offsets, chunk tables
    std::vector<BatchCube> cubes(count);
    std::vector<Piece> pieces;
    std::vector<SumChunk> chunks;
    std::vector<int> chunk_first(count + 1, 0);
    std::vector<ParamIn> pin(count);
    std::vector<long> nvox(count);
    std::vector<std::vector<int>> depths(count);
    size_t scratch_total = 0;
    std::vector<size_t> scratch_off(count);
    size_t lds = 0;
    constexpr int kResClasses = 5;   // 64, 128, 256, 512, 1024 threads
    std::vector<std::vector<int>> res(kResClasses);
    bp->res_lds.assign(kResClasses, 0);
    for (int c = 0; c < count; ++c) {
        const ig_params& p = items[c].p;
        const long n = (long)(p.nx * p.ny * p.nz);
        nvox[c] = n;
        scratch_off[c] = scratch_total;
        chunk_first[c] = (int)chunks.size();
        for (long off = 0; off < n; off += kChunk) chunks.push_back(SumChunk{c, 0, off, std::min(kChunk, n - off)});
        ParamIn& q = pin[c];
        q.K = p.K; q.tau = p.tau;
        for (int a = 0; a < 3; ++a) q.C[a] = p.C[a];
        q.cond = p.cond;
        q.abort_on_nonfinite = 1;
        q.rms = p.rms;
        BatchCube& cb = cubes[c];
        cb.in = (const float*)items[c].d_in;
        cb.out = (float*)items[c].d_out;
        cb.n = n;
        cb.niter = p.n_iter;
        if (bp->resident[c]) {   // no passes, no pieces, no scratch
            cb.g = BlockGeom{};
            cb.g.nx = (int)p.nx; cb.g.ny = (int)p.ny; cb.g.nz = (int)p.nz;
            cb.V = 1;
            cb.npieces = 0;
            cb.piece_off = (int)pieces.size();
            cb.npass = 0;
            cb.stage = 0;
            // the fewest threads (64 << j) that hold it at kResPerThread voxels each
            int j = 0;
            while (j + 1 < kResClasses && (64L << j) * kResPerThread < n) ++j;
            res[j].push_back(c);
            bp->resident[c] = 1 << j;
            bp->res_lds[j] = std::max(bp->res_lds[j], (size_t)n * sizeof(float));
            continue;
        }
        scratch_total += (size_t)((n + 63) / 64 * 64);
        ig_schedule s{};
        s.kind = IG_SCHED_BLOCKED;
        s.t_block = T;
        s.waves = W;
        s.zchunk = bp->persist ? g_batch_Z : (int)p.nz;
        // 3 voxels per lane cover rows of up to 48, 96 and 192 voxels with 4, 2
        // and 1 rows per wavefront: fewer idle lanes than 4 do
        int V, R;
        auto_vec_rows(p.nx, &V, &R);
        if (T <= 2 && V == 4 && (64 / R) * 3 >= p.nx) V = 3;
        s.vec = V;
        s.rows = R;
        PassPlan pp;
        const char* why = plan_pass(p, s, T, ncu, &pp, true);
        if (why) return fail(IG_ERR_INVALID_ARG, "batch item %d: %s", c, why);
        if (pp.g.grouped) return fail(IG_ERR_DEVICE, "batch item %d: unexpected grouped plan", c);
        if (pp.V > 4)
            return fail(IG_ERR_UNSUPPORTED, "batch item %d: layout with %d voxels per lane", c, pp.V);
        lds = std::max(lds, stream_lds_bytes(pp.V, T, W));
        cb.g = pp.g;
        const uintptr_t al = (uintptr_t)chunk_align(pp.V, 4);
        if (((uintptr_t)cb.in % al) || ((uintptr_t)cb.out % al)) cb.g.vec = 0;
        cb.V = pp.V;
        cb.npieces = bp->persist ? (int)pp.pieces.size() : 0;   // (deal_rounds makes the rounds' own)
        cb.piece_off = (int)pieces.size();
        pieces.insert(pieces.end(), pp.pieces.begin(), pp.pieces.begin() + cb.npieces);
        // pass depths (a remainder pass is shallower); in place with an odd count: stage
        std::vector<int>& d = depths[c];
        if (p.n_iter > 0) {
            d.assign(p.n_iter / T, T);
            if (p.n_iter % T) d.push_back(p.n_iter % T);
        }
        cb.npass = (int)d.size();
        cb.stage = (items[c].d_in == items[c].d_out && cb.npass % 2 == 1) ? 1
                   : (cb.npass == 0 && items[c].d_in != items[c].d_out) ? 2 : 0;
    }
    chunk_first[count] = (int)chunks.size();
    if (lds > kMaxLds) return fail(IG_ERR_UNSUPPORTED, "batch tile needs too much LDS");
    bp->lds = lds;
    bp->passes.resize(count);
    for (int c = 0; c < count; ++c) bp->passes[c] = bp->resident[c] ? 1 : cubes[c].npass;
    std::vector<int> res_all;
    bp->res_off.assign(1, 0);
    for (int j = 0; j < kResClasses; ++j) {
        res_all.insert(res_all.end(), res[j].begin(), res[j].end());
        bp->res_off.push_back((int)res_all.size());
        if (bp->res_lds[j] > kMaxLds) return fail(IG_ERR_UNSUPPORTED, "resident cube needs too much LDS");
    }
    bp->nres = (int)res_all.size();

    // rounds: round r holds pass r of every cube that has one, largest cubes first
    std::vector<int> order(count);
    for (int c = 0; c < count; ++c) order[c] = c;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return nvox[a] > nvox[b]; });
    int maxpass = 0;
    for (int c = 0; c < count; ++c) maxpass = std::max(maxpass, cubes[c].npass);
    std::vector<BatchItem> its;
    std::vector<int> first;
    bp->round_off.assign(1, 0);
    for (int c = 0; c < count; ++c) cubes[c].nlast = cubes[c].npieces;
    if (bp->persist) {
        for (int k = 0; k < maxpass; ++k)
            for (int c : order)
                if (k < cubes[c].npass)
                    for (int j = 0; j < cubes[c].npieces; ++j) its.push_back(BatchItem{c, k, j, depths[c][k]});
    } else {
        deal_rounds(cubes, depths, order, maxpass, (long)ncu * resident_per_cu(W, lds), W, &its, &pieces, &first,
                    &bp->round_off);
    }
    bp->nitems = (int)its.size();
    bp->nchunks = (int)chunks.size();

    HIP_TRY(bp->scratch.alloc(scratch_total));
    for (int c = 0; c < count; ++c) cubes[c].scratch = bp->scratch.p + scratch_off[c];
    HIP_TRY(bp->d_cubes.alloc(count));
    HIP_TRY(bp->d_items.alloc(its.size()));
    HIP_TRY(bp->d_pieces.alloc(pieces.size()));
    HIP_TRY(bp->d_first.alloc(first.size()));
    HIP_TRY(bp->d_chunks.alloc(chunks.size()));
    HIP_TRY(bp->d_chunk_first.alloc(count + 1));
    HIP_TRY(bp->d_part.alloc(3 * chunks.size()));
    HIP_TRY(bp->d_pin.alloc(count));
    HIP_TRY(bp->d_nvox.alloc(count));
    HIP_TRY(bp->d_params.alloc(count));
    HIP_TRY(bp->d_outsum.alloc(count));
    HIP_TRY(bp->d_ctr.alloc(kCtrFin + count));
    HIP_TRY(bp->d_stamps.alloc(1 + count));
    HIP_TRY(bp->d_res.alloc(res_all.size()));
    if (!res_all.empty())
        HIP_TRY(hipMemcpy(bp->d_res.p, res_all.data(), res_all.size() * sizeof(int), hipMemcpyHostToDevice));
    // descriptor tables: fixed for the plan's signature, uploaded once
    HIP_TRY(hipMemcpy(bp->d_cubes.p, cubes.data(), count * sizeof(BatchCube), hipMemcpyHostToDevice));
    HIP_TRY(igk_host_malloc((void**)&bp->h_cubes, count * sizeof(BatchCube)));
    std::memcpy(bp->h_cubes, cubes.data(), count * sizeof(BatchCube));
    bp->bufs.resize(count);
    for (int c = 0; c < count; ++c) bp->bufs[c] = {items[c].d_in, items[c].d_out};
    HIP_TRY(hipEventCreateWithFlags(&bp->done, hipEventDisableTiming));
    if (!its.empty())
        HIP_TRY(hipMemcpy(bp->d_items.p, its.data(), its.size() * sizeof(BatchItem), hipMemcpyHostToDevice));
    if (!pieces.empty())
        HIP_TRY(hipMemcpy(bp->d_pieces.p, pieces.data(), pieces.size() * sizeof(Piece), hipMemcpyHostToDevice));
    if (!first.empty())
        HIP_TRY(hipMemcpy(bp->d_first.p, first.data(), first.size() * sizeof(int), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(bp->d_chunks.p, chunks.data(), chunks.size() * sizeof(SumChunk), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(bp->d_chunk_first.p, chunk_first.data(), (count + 1) * sizeof(int), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(bp->d_pin.p, pin.data(), count * sizeof(ParamIn), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(bp->d_nvox.p, nvox.data(), count * sizeof(long), hipMemcpyHostToDevice));

    const BatchKernels* kernels = batch_kernels(bp->cond);
    BatchKernel kern = kernels->round[T - 1];
    PersistKernel pkern = kernels->persist[T - 1];
    if (lds > 65536) {
        HIP_TRY(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        HIP_TRY(hipFuncSetAttribute((const void*)pkern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    }
    // persistent launch: as many workgroups as the GPU holds at once (no more
    // than there are items; the kernel's own 8 bytes of LDS counted), so
    // every workgroup that takes an item is running
    bp->grid = (int)std::min<long>(bp->nitems, (long)ncu * resident_per_cu(W, lds + 16));
    ResidentKernel rkern = kernels->resident;
    const size_t res_lds_max = *std::max_element(bp->res_lds.begin(), bp->res_lds.end());
    if (res_lds_max > 65536)
        HIP_TRY(hipFuncSetAttribute((const void*)rkern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)res_lds_max));

    // capture: counter reset, noise-level pre-pass, staging, resident cubes, the rounds
    HIP_TRY(hipStreamCreateWithFlags(&bp->cap, hipStreamNonBlocking));
    HIP_TRY(hipStreamBeginCapture(bp->cap, hipStreamCaptureModeThreadLocal));
    hipStream_t s = bp->cap;
    hipError_t e = hipSuccess;
    auto chk = [&](hipError_t r) { if (e == hipSuccess) e = r; };
    hipLaunchKernelGGL(k_batch_reset, dim3(1), dim3(256), 0, s, bp->d_ctr.p, kCtrFin + count, bp->d_stamps.p,
                       1 + count);
    chk(hipGetLastError());
    if (bp->nchunks > 0) {
        hipLaunchKernelGGL(k_batch_sum, dim3(bp->nchunks), dim3(256), 0, s, bp->d_cubes.p, bp->d_chunks.p,
                           bp->d_part.p, 0);
        chk(hipGetLastError());
    }
    hipLaunchKernelGGL(k_batch_params, dim3(count), dim3(64), 0, s, bp->d_pin.p, bp->d_chunk_first.p,
                       bp->d_part.p, bp->d_nvox.p, bp->d_params.p, 0);
    chk(hipGetLastError());
    if (bp->nchunks > 0) {
        hipLaunchKernelGGL(k_batch_stage, dim3(bp->nchunks), dim3(256), 0, s, bp->d_cubes.p, bp->d_chunks.p,
                           bp->d_params.p);
        chk(hipGetLastError());
    }
    for (size_t j = 0; j + 1 < bp->res_off.size(); ++j) {
        const int n = bp->res_off[j + 1] - bp->res_off[j];
        if (n <= 0) continue;
        hipLaunchKernelGGL(rkern, dim3(n), dim3(64 << j), bp->res_lds[j], s, bp->d_cubes.p,
                           bp->d_res.p + bp->res_off[j], bp->d_params.p, bp->d_stamps.p);
        chk(hipGetLastError());
    }
    if (bp->persist) {
        if (bp->nitems > 0) {
            hipLaunchKernelGGL(pkern, dim3(bp->grid), dim3(64, W), lds, s, bp->d_cubes.p, bp->d_items.p, bp->nitems,
                               bp->d_pieces.p, bp->d_params.p, count, bp->d_ctr.p, bp->d_stamps.p);
            chk(hipGetLastError());
        }
    } else {
        for (size_t r = 0; r + 1 < bp->round_off.size(); ++r) {
            const int n = bp->round_off[r + 1] - bp->round_off[r];
            if (n <= 0) continue;
            hipLaunchKernelGGL(kern, dim3(n), dim3(64, W), lds, s, bp->d_cubes.p, bp->d_items.p,
                               bp->d_first.p + bp->round_off[r] + r, bp->d_pieces.p, bp->d_params.p, bp->d_ctr.p, bp->d_stamps.p);
            chk(hipGetLastError());
        }
    }
    if (bp->nchunks > 0) {
        hipLaunchKernelGGL(k_batch_nan, dim3(bp->nchunks), dim3(256), 0, s, bp->d_cubes.p, bp->d_chunks.p,
                           bp->d_params.p);
        chk(hipGetLastError());
    }
    hipGraph_t g = nullptr;
    hipError_t e2 = hipStreamEndCapture(s, &g);
    if (e != hipSuccess) { if (g) (void)hipGraphDestroy(g); return fail(IG_ERR_DEVICE, "capture: %s", hipGetErrorString(e)); }
    HIP_TRY(e2);
    bp->graph = g;
    HIP_TRY(hipGraphInstantiate(&bp->exec, g, nullptr, nullptr, 0));
    return IG_OK;
}

}  // namespace

static bool same_as_last(const ig_batch_item* items, int count, int device) {
    return g_last.plan && g_last.device == device && (int)g_last.items.size() == count && g_last.T == g_batch_T &&
           g_last.W == g_batch_W && (!g_batch_persist || g_last.Z == g_batch_Z) && g_last.res == g_batch_res &&
           g_last.persist == g_batch_persist && std::memcmp(g_last.items.data(), items, (size_t)count * sizeof(ig_batch_item)) == 0;
}

extern "C" ig_status ig_filter_batch(const ig_batch_item* items, int32_t count, int device, void* hip_stream,
                                     ig_stats* per_item, double* latency_ms) {
    if (!items || count < 1) return fail(IG_ERR_INVALID_ARG, "empty batch");
    if (per_item)
        for (int i = 0; i < count; ++i)
            if (per_item[i].struct_size != sizeof(ig_stats))
                return fail(IG_ERR_INVALID_ARG, "per_item[%d].struct_size", i);
    // held for the whole call: a plan stays alive while it is used
    std::lock_guard<std::mutex> lk(g_mu);
    BatchPlan* bp = same_as_last(items, count, device) ? g_last.plan : nullptr;
    if (!bp) {
    for (int i = 0; i < count; ++i) {
        ig_status st = igk_validate_params(&items[i].p);
        if (st != IG_OK) return st;
        if (items[i].p.dtype != IG_F32) return fail(IG_ERR_UNSUPPORTED, "batch item %d: only FP32 storage", i);
        if (items[i].p.cond != items[0].p.cond)
            return fail(IG_ERR_UNSUPPORTED, "batch items must share one conductance");
        if (!items[i].d_in || !items[i].d_out) return fail(IG_ERR_INVALID_ARG, "batch item %d: NULL buffer", i);
        const size_t bytes = (size_t)(items[i].p.nx * items[i].p.ny * items[i].p.nz) * 4;
        ig_status cb = igk_check_buffer(items[i].d_in, bytes, device, "batch item d_in");
        if (cb == IG_OK) cb = igk_check_buffer(items[i].d_out, bytes, device, "batch item d_out");
        if (cb != IG_OK) return fail(cb, "batch item %d: %s", i, std::string(ig_last_error()).c_str());
    }
    // buffers of distinct items must not overlap
    {
        std::vector<std::pair<uintptr_t, uintptr_t>> rng;
        for (int i = 0; i < count; ++i) {
            const size_t bytes = (size_t)(items[i].p.nx * items[i].p.ny * items[i].p.nz) * 4;
            const uintptr_t a = (uintptr_t)items[i].d_in, b = (uintptr_t)items[i].d_out;
            if (a != b && a < b + bytes && b < a + bytes)
                return fail(IG_ERR_INVALID_ARG, "batch item %d: input and output overlap partially", i);
            rng.push_back({a, a + bytes});
            if (b != a) rng.push_back({b, b + bytes});
        }
        std::sort(rng.begin(), rng.end());
        for (size_t k = 1; k < rng.size(); ++k)
            if (rng[k].first < rng[k - 1].second) return fail(IG_ERR_INVALID_ARG, "batch items share buffers");
    }
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev)
        return fail(IG_ERR_INVALID_ARG, "bad device %d", device);
    }
    int prev = -1;
    (void)hipGetDevice(&prev);
    if (hipSetDevice(device) != hipSuccess) return fail(IG_ERR_DEVICE, "hipSetDevice(%d)", device);
    struct Restore { int d; ~Restore() { if (d >= 0) (void)hipSetDevice(d); } } restore{prev};

    hipStream_t s = (hipStream_t)hip_stream;
    if (!bp) {
        auto key = signature(items, count, device);
        auto it = g_cache.find(key);
        if (it == g_cache.end()) {
            while (g_cache.size() >= kMaxPlans) {   // drop the least recently used plan
                auto lru = g_cache.begin();
                for (auto j = g_cache.begin(); j != g_cache.end(); ++j)
                    if (j->second->last_use < lru->second->last_use) lru = j;
                if (g_last.plan == lru->second.get()) g_last = LastCall{};
                g_cache.erase(lru);
            }
            auto plan = std::make_unique<BatchPlan>();
            ig_status st = build_plan(items, count, device, plan.get());
            if (st != IG_OK) return st;
            bp = plan.get();
            g_cache[key] = std::move(plan);
        } else {
            bp = it->second.get();
            ig_status st = rebind(bp, items, count, s);
            if (st != IG_OK) return st;
        }
        g_last.items.assign(items, items + count);
        g_last.device = device;
        g_last.T = g_batch_T; g_last.W = g_batch_W; g_last.Z = g_batch_Z; g_last.res = g_batch_res;
        g_last.persist = g_batch_persist;
        g_last.plan = bp;
    }
    bp->last_use = ++g_use;
    HIP_TRY(hipGraphLaunch(bp->exec, s));
    HIP_TRY(hipEventRecord(bp->done, s));
    if (!per_item && !latency_ms) return IG_OK;

    std::vector<unsigned long long> stamps(1 + count);
    HIP_TRY(hipMemcpyAsync(stamps.data(), bp->d_stamps.p, stamps.size() * 8, hipMemcpyDeviceToHost, s));
    std::vector<DevParams> prm(count);
    HIP_TRY(hipMemcpyAsync(prm.data(), bp->d_params.p, count * sizeof(DevParams), hipMemcpyDeviceToHost, s));
    if (per_item) {
        hipLaunchKernelGGL(k_batch_sum, dim3(bp->nchunks), dim3(256), 0, s, bp->d_cubes.p, bp->d_chunks.p,
                           bp->d_part.p, 1);
        hipLaunchKernelGGL(k_batch_params, dim3(count), dim3(64), 0, s, bp->d_pin.p, bp->d_chunk_first.p,
                           bp->d_part.p, bp->d_nvox.p, bp->d_outsum.p, 1);
        HIP_TRY(hipGetLastError());
    }
    std::vector<DevParams> osum(count);
    if (per_item)
        HIP_TRY(hipMemcpyAsync(osum.data(), bp->d_outsum.p, count * sizeof(DevParams), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    int khz = 0;
    (void)hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, device);
    bool bad = false, timed_out = false;
    for (int c = 0; c < count; ++c) {
        if (latency_ms)
            latency_ms[c] = (khz > 0 && stamps[1 + c] >= stamps[0]) ? (double)(stamps[1 + c] - stamps[0]) / khz : 0.0;
        if (per_item) {
            ig_stats& st = per_item[c];
            const ig_params& p = items[c].p;
            st.passes = bp->passes[c];
            st.rms_used = prm[c].rho;
            st.sum_in = prm[c].sum;
            st.sum_out = osum[c].sum;
            st.nonfinite = prm[c].nonfinite;
            st.monotone = (2.0 * (double)p.tau * ((double)p.C[0] + p.C[1] + p.C[2]) <= 1.0) ? 1 : 0;
            st.schedule = bp->resident[c] ? ig_schedule{IG_SCHED_BLOCKED, bp->niter[c], bp->resident[c], (int)p.nz, 1, 0, 0}
                                          : ig_schedule{IG_SCHED_BLOCKED, bp->T, bp->W, g_batch_Z, 4, 0, 0};
        }
        if (prm[c].abort == 2) timed_out = true;
        else if (prm[c].abort) bad = true;
    }
    if (timed_out)
        return fail(IG_ERR_DEVICE, "persistent batch: a dependency wait ran out of time (every output is set to NaN)");
    if (bad) return fail(IG_ERR_NONFINITE, "a batch item holds non-finite voxels (its output is set to NaN)");
    return IG_OK;
}

extern "C" void ig_batch_cache_clear(void) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_last = LastCall{};
    g_cache.clear();
}

extern "C" int32_t ig_batch_cache_size(void) {
    std::lock_guard<std::mutex> lk(g_mu);
    return (int32_t)g_cache.size();
}

extern "C" ig_status ig_batch_autotune(const ig_batch_item* items, int32_t count, int device, void* hip_stream,
                                       int32_t* best_t_block, int32_t* best_waves, int32_t* best_zchunk,
                                       double* best_ms) {
    if (!items || count < 1) return fail(IG_ERR_INVALID_ARG, "empty batch");
    for (int i = 0; i < count; ++i)
        if (items[i].d_in == items[i].d_out) return fail(IG_ERR_INVALID_ARG, "autotuning needs d_in != d_out");
    hipStream_t s = (hipStream_t)hip_stream;
    hipEvent_t e0, e1;
    HIP_TRY(hipEventCreate(&e0));
    HIP_TRY(hipEventCreate(&e1));
    int maxn = 0;
    for (int i = 0; i < count; ++i) maxn = std::max(maxn, items[i].p.n_iter);
    // drop the plan of a candidate that is not kept (each plan holds scratch
    // cubes for the whole batch)
    // small cubes: LDS-resident or streamed like the others (both are tried
    // when some cube qualifies)
    bool any_small = false;
    for (int i = 0; i < count; ++i)
        any_small |= items[i].p.n_iter > 0 && items[i].p.nx * items[i].p.ny * items[i].p.nz <= kResidentMax;
    std::vector<int> res_modes = any_small ? std::vector<int>{kResidentMax, 0} : std::vector<int>{g_batch_res};
    auto drop = [&](int T, int W, int Z, int R, int P) {
        std::lock_guard<std::mutex> lk(g_mu);
        const int t0 = g_batch_T, w0 = g_batch_W, z0 = g_batch_Z, r0 = g_batch_res, p0 = g_batch_persist;
        g_batch_T = T; g_batch_W = W; g_batch_Z = Z; g_batch_res = R; g_batch_persist = P;
        auto it = g_cache.find(signature(items, count, device));
        if (it != g_cache.end()) {
            if (g_last.plan == it->second.get()) g_last = LastCall{};
            g_cache.erase(it);
        }
        g_batch_T = t0; g_batch_W = w0; g_batch_Z = z0; g_batch_res = r0; g_batch_persist = p0;
    };
    double best = 1e300;
    int bT = 0, bW = 16, bZ = 32, bR = g_batch_res, bP = 0;
    for (int P : {0, 1})
        for (int R : res_modes)
            for (int T = 1; T <= std::max(1, std::min(4, maxn)); ++T)
                for (int W : {8, 12, 16})
                    for (int Z : {16, 32, 64}) {
                        if (W <= 2 * T) continue;
                        if (P == 0 && Z != 32) continue;   // the rounds deal shares, not chunks
                        if (ig_batch_set_schedule(T, W, Z) != IG_OK || ig_batch_set_resident(R) != IG_OK ||
                            ig_batch_set_launch(P) != IG_OK)
                            continue;
                        if (ig_filter_batch(items, count, device, hip_stream, nullptr, nullptr) != IG_OK) {   // build + warm
                            drop(T, W, Z, R, P);
                            continue;
                        }
                        float ms = 0.0f;
                        bool ok = hipEventRecord(e0, s) == hipSuccess;
                        for (int k = 0; k < 2 && ok; ++k)
                            ok = ig_filter_batch(items, count, device, hip_stream, nullptr, nullptr) == IG_OK;
                        ok = ok && hipEventRecord(e1, s) == hipSuccess && hipEventSynchronize(e1) == hipSuccess &&
                             hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
                        if (ok && ms / 2 < best) {
                            if (best < 1e300) drop(bT, bW, bZ, bR, bP);
                            best = ms / 2; bT = T; bW = W; bZ = Z; bR = R; bP = P;
                        } else {
                            drop(T, W, Z, R, P);
                        }
                    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (best >= 1e300) return fail(IG_ERR_UNSUPPORTED, "no batch schedule ran");
    ig_status st = ig_batch_set_schedule(bT, bW, bZ);
    if (st == IG_OK) st = ig_batch_set_resident(bR);
    if (st == IG_OK) st = ig_batch_set_launch(bP);
    if (st != IG_OK) return st;
    if (best_t_block) *best_t_block = bT;
    if (best_waves) *best_waves = bW;
    if (best_zchunk) *best_zchunk = bZ;
    if (best_ms) *best_ms = best;
    return IG_OK;
}

extern "C" ig_status ig_batch_set_schedule(int32_t t_block, int32_t waves, int32_t zchunk) {
    if (t_block < 0 || t_block > 4 || waves < 1 || waves > 16 || zchunk < 1 || zchunk > 4096)
        return fail(IG_ERR_INVALID_ARG, "bad batch schedule");
    std::lock_guard<std::mutex> lk(g_mu);
    g_batch_T = t_block;
    g_batch_W = waves;
    g_batch_Z = zchunk;
    return IG_OK;
}

extern "C" ig_status ig_batch_set_launch(int32_t persistent) {
    if (persistent != 0 && persistent != 1) return fail(IG_ERR_INVALID_ARG, "launch mode must be 0 or 1");
    std::lock_guard<std::mutex> lk(g_mu);
    g_batch_persist = persistent;
    return IG_OK;
}

extern "C" int32_t ig_batch_get_launch(void) {
    std::lock_guard<std::mutex> lk(g_mu);
    return g_batch_persist;
}

extern "C" ig_status ig_batch_set_resident(int32_t max_voxels) {
    if (max_voxels < 0 || max_voxels > kResidentMax)
        return fail(IG_ERR_INVALID_ARG, "resident limit must be in 0..%d voxels", kResidentMax);
    std::lock_guard<std::mutex> lk(g_mu);
    g_batch_res = max_voxels;
    return IG_OK;
}

extern "C" ig_status ig_batch_get_resident(int32_t* max_voxels) {
    if (!max_voxels) return fail(IG_ERR_INVALID_ARG, "max_voxels is NULL");
    std::lock_guard<std::mutex> lk(g_mu);
    *max_voxels = g_batch_res;
    return IG_OK;
}

// Kernels of the learned surrogate: a 3-D CNN of 3x3x3 convolutions that
// approximates n steps of the filter in one pass.
//
// Data layout.  Activations are bf16, channels-last: a[(z*ny + y)*nx + x][C].
// Convolutions are implicit GEMMs on the gfx950 matrix cores with
// v_mfma_f32_16x16x32_bf16 (D[16x16] += A[16x32] B[32x16], FP32 accumulate):
//   forward:  M = voxels (16 consecutive x), N = output channels,
//             K = 32 input channels of one tap (27 taps = 27 K-steps); for a
//             1-channel input K = the 27 taps themselves (padded to 32).
//   input gradient: the same kernel on the output gradient with the weights
//             mirrored in space and transposed in channels.
//   weight gradient: M = input channels (or taps), N = output channels,
//             K = voxels; per-workgroup partials, folded in a fixed order.
// Operand lane layout (wave64, checked on the device): A[i][k] sits in lane
// i + 16*(k/8), element k%8; B[k][n] in lane n + 16*(k/8), element k%8;
// D[m][n] in lane n + 16*(m/4), element m%4.
//
// Weights are kept packed in that B layout: Wp[t][nb][lane][8] holds
// B[k = 8*(lane/16) + e][n = 16*nb + lane%16] of tap t, so a lane's fragment
// is one 16-byte load.  For a 1-channel input the taps are the K index:
// Wp[nb][lane][8] with k = tap.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace igs {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16;

enum { EPI_RAW = 0, EPI_GELU = 1, EPI_BACK_GELU = 2, EPI_RESID = 3 };

__device__ __forceinline__ float bf2f(u16 h) { return __uint_as_float((unsigned)h << 16); }
__device__ __forceinline__ u16 f2bf(float f) {   // round to nearest, ties to even (finite inputs)
    unsigned u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (u16)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
    u += 0x7fffu + ((u >> 16) & 1u);
    return (u16)(u >> 16);
}

// f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>): a loop whose
// index is a constant in the body whatever the body's size
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(static_cast<F&&>(f), std::make_integer_sequence<int, N>{});
}

// ------------------------------------------------ conv, z-streaming, 32 in
// Error function by Abramowitz & Stegun, Handbook of Mathematical Functions,
// formula 7.1.26: erf(x) = 1 - (a1 t + ... + a5 t^5) e^{-x^2}, t = 1/(1 + p x)
// for x >= 0, |error| <= 1.5e-7 (far below the bf16 rounding of every value
// it feeds).
// gelu(z) = z/2 (1 + erf(z/sqrt2)); gelu'(z) = (1 + erf(z/sqrt2))/2 + z e^{-z^2/2}/sqrt(2 pi)
// GELU through the complementary function the same formula gives directly,
// erfc(x) = (a1 t + ... + a5 t^5) e^{-x^2} for x >= 0: with c = erfc(|z|/sqrt2),
// gelu(z) = max(z, 0) - |z|/2 c on both sides of 0 (11 VALU operations, a
// reciprocal and an exp2).
__device__ __forceinline__ float gelu_fast(float z) {
    const float az = fabsf(z);
    const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.3275911f * 0.70710678118654752f, az, 1.0f));
    const float ex = __builtin_amdgcn_exp2f((z * -0.72134752044448170f) * z);   // e^{-z^2/2}
    // the coefficients halved: c / 2 with the same roundings, one product fewer
    float pl = __builtin_fmaf(0.5f * 1.061405429f, t, 0.5f * -1.453152027f);
    pl = __builtin_fmaf(pl, t, 0.5f * 1.421413741f);
    pl = __builtin_fmaf(pl, t, 0.5f * -0.284496736f);
    pl = __builtin_fmaf(pl, t, 0.5f * 0.254829592f);
    const float c = (pl * t) * ex;
    return __builtin_fmaf(-az, c, fmaxf(z, 0.0f));
}
// With h = erfc(|x|)/2, x = z/sqrt2: (1 + erf(x))/2 = 1/2 + sign(z) (1/2 - h), the
// coefficients halved as above (every rounding is that of the formula as written).
__device__ __forceinline__ float gelu_grad_fast(float z) {
    const float x = z * 0.70710678118654752f;
    const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.3275911f, fabsf(x), 1.0f));
    const float ex = __builtin_amdgcn_exp2f((x * x) * -1.4426950408889634f);   // e^{-z^2/2}
    float pl = __builtin_fmaf(0.5f * 1.061405429f, t, 0.5f * -1.453152027f);
    pl = __builtin_fmaf(pl, t, 0.5f * 1.421413741f);
    pl = __builtin_fmaf(pl, t, 0.5f * -0.284496736f);
    pl = __builtin_fmaf(pl, t, 0.5f * 0.254829592f);
    const float u = 0.5f - (pl * t) * ex;
    const float su = __uint_as_float(__float_as_uint(u) ^ (__float_as_uint(z) & 0x80000000u));
    return (0.5f + su) + z * (0.39894228040143268f * ex);
}
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
// four FP32 values to four bf16 (round to nearest, ties to even; the gfx950
// conversion instruction packs two per operation)
__device__ __forceinline__ uint2 pack_bf16x4(float a, float b, float c, float d) {
    const bf16x4 v = {(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};
    return __builtin_bit_cast(uint2, v);
}

// The convolution of a 32-channel input as a z-stream: a workgroup of 8
// wavefronts owns an output tile of 32 voxels in x by 8 rows in y and a chunk of
// planes [z0, z1).  Wavefront (nb, xs, yg)
// computes 16 output channels (nb) of 16 voxels (xs) of 4 rows (yg), and holds
// the weights of its channels, all 27 taps, in registers (108) for the whole
// chunk, so the LDS only feeds activations.  A step takes one input plane and
// adds it to the sums of the three output planes it reaches: each fragment
// (row, x shift) is read once and multiplied with every weight it meets, up to 3
// rows by 3 planes: 18 reads of 1 KB for 108 products, where weights in LDS and
// one row per wavefront took 81, and two output planes at a time from four input
// planes 36.  The three sums of a row move on by name: a plane's first product
// takes the sum of the plane before as its addend.  The first two and the last
// two steps of a chunk leave out the tap planes that reach no output of it.
// Input planes (tile plus a one-voxel margin, zeros outside the cube) sit in a
// ring of three LDS slots: plane z is read (and z + 1 at the end, so no step
// starts by waiting for LDS) while z + 2 is staged, one barrier per plane.  The
// weights are the MFMA's A operand and the activations its B operand, so each
// lane ends with four consecutive output channels of one voxel and stores them
// with one 8-byte write.  Per output the taps are accumulated in the order
// 0..26, then the bias is added.  The step is one block of code whose issue order
// is laid out (below), the epilogue's VALU work behind the products.
// What bounds it now is power: 960 TFLOP/s of products executed on 360 x 360 x
// 150 (a library matrix product reaches 1127 on the same card), the matrix cores
// 53 % busy at 1.74 GHz; staging straight to LDS took 9 % of the cycles and none
// of the time (the clock fell with them).  A prediction on that cube (six such
// layers) went from 9.0 ms with weights in LDS to 7.7 with weights in registers
// and 7.4 with every fragment read once; a training step on four 96^3 cubes from
// 4.96 to 4.82 ms by the last.
constexpr int kZsRows = 8;    // tile rows
constexpr int kZsX = 32;      // tile columns
constexpr int kZsAhead = 2;   // activation fragments in flight ahead of their products (across steps)
constexpr int kZsSlots = 3;   // LDS ring
constexpr int kZsValu = 3;    // VALU operations issued behind a product
constexpr int kZsLX = kZsX + 2, kZsLY = kZsRows + 2;
constexpr int kZsPer = (kZsLX * kZsLY * 4 + 511) / 512;   // 16-byte chunks of a staged plane per thread
constexpr int kZsPl = kZsPer * 512 * 8;     // u16 of a slot: a plane and what the last threads write past it
constexpr size_t kZsLds = (size_t)kZsSlots * kZsPl * 2;

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
// A raw buffer over `bytes` from p: accesses at or past its end are dropped
// (loads give zeros), so a store that must not happen needs no branch around it
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_buffer(const void* p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}

// FP32 epilogues of the 1-channel z-stream kernel: lane (i + 16 kg) holds D[m = 4 kg +
// e][n = i] of each (s, nb), output channels 16 nb + 4 kg + e of voxel 16 s + i of row
// y, plane z; four consecutive channels go out in one 16-byte store.  Output channels
// are padded to 16 NB.  aux: the FP32 input cube for the residual (EPI_RESID, output
// channel 0 only).
template <int NB, int EPI, int MT>
__device__ __forceinline__ void zs_store(const f32x4 (&acc)[MT][NB], const float* __restrict__ bias,
                                         float* __restrict__ out, const float* __restrict__ aux, int x0, int y, int z,
                                         int nx, int ny, int i, int kg) {
    static_assert(EPI == EPI_RAW || EPI == EPI_RESID, "FP32 outputs");
#pragma unroll
    for (int s = 0; s < MT; ++s)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const f32x4& d = acc[s][nb];
            const int x = x0 + 16 * s + i, n0 = 16 * nb + 4 * kg;
            if (y >= ny || x >= nx) continue;
            const long v = (long)(z * ny + y) * nx + x;
            if constexpr (EPI == EPI_RAW) {
                float4 r;
                r.x = d[0] + (bias ? bias[n0] : 0.0f);
                r.y = d[1] + (bias ? bias[n0 + 1] : 0.0f);
                r.z = d[2] + (bias ? bias[n0 + 2] : 0.0f);
                r.w = d[3] + (bias ? bias[n0 + 3] : 0.0f);
                *reinterpret_cast<float4*>(out + v * 16 * NB + n0) = r;
            } else {
                if (n0 == 0) out[v] = aux[v] + (d[0] + bias[0]);
            }
        }
}

// How the tile planes (tiles of 32 x 8 voxels) of `cubes` cubes of one shape, laid
// one after another, are dealt to the workgroups: chunks of zch planes of one
// tile, or (zch = 0) equal contiguous shares of the sequence cube, tile, plane,
// which a workgroup takes as runs of planes of one tile.
struct ZsSplit {
    int ntx, nty, zch, cubes;
    __device__ __forceinline__ void share(int nz, int* u0, int* u1) const {
        const int tiles = ntx * nty;
        if (zch > 0) {
            const int nzc = (nz + zch - 1) / zch, t = blockIdx.x % tiles, q = blockIdx.x / tiles;
            const int z0 = q % nzc * zch;
            *u0 = (q / nzc * tiles + t) * nz + z0;
            *u1 = *u0 + min(zch, nz - z0);
        } else {
            const long total = (long)tiles * cubes * nz;
            *u0 = (int)(total * blockIdx.x / gridDim.x);
            *u1 = (int)(total * (blockIdx.x + 1) / gridDim.x);
        }
    }
    // the run that starts at u of a share that ends at u1; returns the cube
    __device__ __forceinline__ int run(int nz, int u, int u1, int* x0, int* y0, int* z0, int* z1) const {
        const int tiles = ntx * nty, t = u / nz, tile = t % tiles;
        *x0 = tile % ntx * kZsX;
        *y0 = tile / ntx * kZsRows;
        *z0 = u - t * nz;
        *z1 = min(nz, *z0 + (u1 - u));
        return t / tiles;
    }
};

// products per tap plane of fragment m of a step, and the epilogue values begun
// before it (16 over a step)
constexpr int zs_products(int m) {
    const int j = m / 3;
    return j == 0 || j == 5 ? 1 : j == 1 || j == 4 ? 2 : 3;
}
constexpr int zs_value(int m) {
    int n = 0;
    for (int k = 0; k < m; ++k) n += zs_products(k);
    return n * 16 / 36;
}

// NB = 1 (up to 16 output channels): the wavefronts nb = 1 compute nothing that
// is stored.  KEEP: the pre-activations go to aux (EPI_GELU).
template <int NB, int EPI, bool KEEP>
__global__ void __launch_bounds__(512)
k_conv_zs(const u16* __restrict__ in0, const bf16x8* __restrict__ wp, const float* __restrict__ bias,
          void* __restrict__ out0, const void* __restrict__ aux0, int nx, int ny, int nz, ZsSplit sp) {
    constexpr int NT = 512, PER = kZsPer;
    extern __shared__ uint4 zs_smem[];
    u16* ring = reinterpret_cast<u16*>(zs_smem);
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = w & 1, xs = (w >> 1) & 1, yg = w >> 2;
    const int i = lane & 15, kg = lane >> 4;
    const int n0 = 16 * nb + 4 * kg;
    const bool act = nb < NB;                      // this wavefront's channels exist

    bf16x8 wf[27];
#pragma unroll
    for (int t = 0; t < 27; ++t) wf[t] = wp[(t * NB + (act ? nb : 0)) * 64 + lane];
    f32x4 bv = {0.f, 0.f, 0.f, 0.f};
    if (EPI != EPI_BACK_GELU && bias && act)
#pragma unroll
        for (int e = 0; e < 4; ++e) bv[e] = bias[n0 + e];

    // runs of planes of one tile of one cube
    int u0, u1;
    sp.share(nz, &u0, &u1);
    for (int u = u0; u < u1;) {
        int x0, y0, z0, z1;
        const long cube = sp.run(nz, u, u1, &x0, &y0, &z0, &z1) * ((long)nx * ny * nz);
        u += z1 - z0;
        const u16* in = in0 + cube * 32;
        const void* aux = static_cast<const char*>(aux0) + cube * 64;   // (bf16, with 32 channels)
        void* out = static_cast<char*>(out0) + cube * (EPI == EPI_RAW ? 64 * NB : 64);

        // the chunks this thread stages: offset from the tile's first row of a
        // plane in units of 16 bytes (below 2^32: a piece has at most 2^28
        // voxels), clamped into the cube; mask: all ones if the chunk lies in it
        unsigned off[PER], mask[PER];
        const int yb = max(y0 - 1, 0);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int q = tid + NT * k, vox = q >> 2;
            const int x = x0 + vox % kZsLX - 1, y = y0 + vox / kZsLX - 1;
            mask[k] = x >= 0 && x < nx && y >= 0 && y < ny ? ~0u : 0u;
            off[k] = (unsigned)(((long)(min(max(y, 0), ny - 1) - yb) * nx + min(max(x, 0), nx - 1)) * 4 + (q & 3));
        }
        uint4 st[PER];
        auto fetch = [&](int z) {
            const uint4* base = reinterpret_cast<const uint4*>(in) + ((long)min(max(z, 0), nz - 1) * ny + yb) * nx * 4;
#pragma unroll
            for (int k = 0; k < PER; ++k) st[k] = base[off[k]];
        };
        auto put = [&](int z, int slot) {
            const bool zin = z >= 0 && z < nz;
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const unsigned m = zin ? mask[k] : 0u;
                reinterpret_cast<uint4*>(ring + slot * kZsPl)[tid + NT * k] =
                    make_uint4(st[k].x & m, st[k].y & m, st[k].z & m, st[k].w & m);
            }
        };
        // plane z0 - 1 + k sits in slot k mod 3
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            fetch(z0 - 1 + k);
            put(z0 - 1 + k, k);
        }
        fetch(z0 + 1);
        __syncthreads();

        const u16* lb = ring + ((4 * yg) * kZsLX + 16 * xs + i) * 32 + 8 * kg;
        // this wavefront's part of output row y + r, plane z: a buffer of bytes
        // `vb` per voxel from voxel x0, empty where nothing is to be stored
        const int y = y0 + 4 * yg;
        const int cols = min(nx - x0, kZsX);
        auto row = [&](const void* p, int z, int r, int vb) {   // no branch: it would split the pass's schedule
            const int on = -(int)(act & (z >= z0) & (z < z1) & (y + r < ny));
            return raw_buffer(static_cast<const char*>(p) +
                                  (((long)max(z, 0) * ny + min(y + r, ny - 1)) * nx + x0) * vb, on & (cols * vb));
        };
        const int lo = (16 * xs + i) * 64 + 2 * n0;    // this lane's four bf16 channels in such a row
        // a0, a1, a2: the sums that the current input plane reaches with the taps of
        // plane 0, 1 and 2.  prev: the finished output plane zp; its epilogue (GELU,
        // packing, stores) is spread over the next step's products, a value at a time
        // and with no branch, so that it runs beside the matrix cores
        constexpr int NV = 16;
        f32x4 a0[4], a1[4], a2[4], prev[4];
        uint2 pre[4];
        int zp = z0 - 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            prev[r] = f32x4{0.f, 0.f, 0.f, 0.f};
            pre[r] = make_uint2(0, 0);
        }
        auto store2 = [&](void* p, int z, int r, uint2 v) {
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{v.x, v.y}, row(p, z, r, 64), lo, 0, 0);
        };
        auto epi = [&](auto vc) {   // value e of row r
            constexpr int v = decltype(vc)::value, r = v / 4, e = v % 4;
            f32x4& d = prev[r];
            if constexpr (EPI == EPI_GELU) {
                if constexpr (e == 0) {
                    d += bv;
                    if constexpr (KEEP) store2(const_cast<void*>(aux), zp, r, pack_bf16x4(d[0], d[1], d[2], d[3]));
                }
                d[e] = gelu_fast(d[e]);
                if constexpr (e == 3) store2(out, zp, r, pack_bf16x4(d[0], d[1], d[2], d[3]));
            } else if constexpr (EPI == EPI_BACK_GELU) {
                const unsigned u = e < 2 ? pre[r].x : pre[r].y;
                d[e] *= gelu_grad_fast(__uint_as_float(e & 1 ? u & 0xffff0000u : u << 16));
                if constexpr (e == 3) store2(out, zp, r, pack_bf16x4(d[0], d[1], d[2], d[3]));
            } else if constexpr (e == 3) {
                typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
                const f32x4 o = d + bv;
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), row(out, zp, r, 64 * NB),
                                                       (16 * xs + i) * 64 * NB + 4 * n0, 0, 0);
            }
        };
        // fragment m: row 4 yg - 1 + j (j = m / 3) of the tile, shift dx = m % 3
        constexpr int FR = kZsAhead + 1;
        static_assert(18 % FR == 0, "the ring of fragments repeats with the steps");
        bf16x8 f[FR];
        int sl = 0;                                    // slot of the current plane
        const u16 *lq = lb, *lq1 = lb + kZsPl;         // the current plane and the next
        auto load = [&](auto mc) {                     // (18 and up: of the next plane, staged two steps ahead)
            constexpr int m = decltype(mc)::value, n = m % 18;
            f[m % FR] = *reinterpret_cast<const bf16x8*>((m < 18 ? lq : lq1) + ((n / 3) * kZsLX + n % 3) * 32);
        };
        static_for<kZsAhead>(load);
        // input plane z with the tap planes LO .. HI
        auto step = [&](auto loc, auto hic, int z) {
            constexpr int LO = decltype(loc)::value, HI = decltype(hic)::value;
            const int sw = sl == 0 ? 2 : sl - 1;       // slot of plane z + 2
            auto part = [&](auto hc) {
                constexpr int M0 = 9 * decltype(hc)::value;
                static_for<9>([&](auto mc) {
                    constexpr int m = M0 + decltype(mc)::value, j = m / 3, dx = m % 3;
                    load(std::integral_constant<int, m + kZsAhead>{});
                    // tap plane 2 first: a sum moves on by being the next plane's
                    // first addend, before its place is taken
#pragma unroll
                    for (int d = HI; d >= LO; --d)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (j - r >= 0 && j - r < 3) {
                                const bool first = j == r && dx == 0;
                                f32x4* o = d == 0 ? a0 : d == 1 ? a1 : a2;
                                const f32x4 c = !first ? o[r] : d == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : d == 1 ? a0[r] : a1[r];
                                o[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[9 * d + 3 * (j - r) + dx], f[m % FR], c,
                                                                               0, 0, 0);
                            }
                    if constexpr (HI == 2) {
                        constexpr int v0 = zs_value(m), v1 = zs_value(m + 1);
                        static_for<v1 - v0>([&](auto k) { epi(std::integral_constant<int, v0 + decltype(k)::value>{}); });
                    }
                });
                // the order to issue it in: each fragment's read kZsAhead fragments
                // ahead, and behind each product the two or three VALU operations that
                // fit under its 16 cycles
                static_for<9>([&](auto mc) {
                    constexpr int m = M0 + decltype(mc)::value;
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    static_for<zs_products(m) * (HI - LO + 1)>([&](auto) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, kZsValu, 0);
                    });
                });
                __builtin_amdgcn_sched_barrier(0);
            };
            __builtin_amdgcn_sched_barrier(0);
            part(std::integral_constant<int, 0>{});
            if constexpr (LO == 0) {                   // the last two steps stage nothing
                put(z + 2, sw);
                fetch(z + 3);
                __builtin_amdgcn_sched_barrier(0);
            }
            part(std::integral_constant<int, 1>{});
            if constexpr (HI == 2) {
                zp = z - 1;
#pragma unroll
                for (int r = 0; r < 4; ++r) prev[r] = a2[r];
                if constexpr (EPI == EPI_BACK_GELU)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(row(aux, zp, r, 64), lo, 0, 0);
                        pre[r] = make_uint2(v.x, v.y);
                    }
            }
            sl = sl == 2 ? 0 : sl + 1;
            lq = lq1;
            lq1 = lb + (sl == 2 ? 0 : sl + 1) * kZsPl;
            __syncthreads();
        };
        constexpr std::integral_constant<int, 0> D0{};
        constexpr std::integral_constant<int, 1> D1{};
        constexpr std::integral_constant<int, 2> D2{};
        step(D0, D0, z0 - 1);
        step(D0, D1, z0);
        for (int z = z0 + 1; z < z1 - 1; ++z) step(D0, D2, z);
        if (z1 - 1 > z0) step(D1, D2, z1 - 1);
        step(D2, D2, z1);
        static_for<NV>(epi);
    }
}

// The convolution of a 1-channel input as a z-stream (the network's first
// layer, and the input gradient of its 1-channel last layer): the tiles and z
// chunks of k_conv_zs, with K = the 27 taps of one voxel (padded to 32).  The
// three input planes z-1 .. z+1 of the tile and its margin (one bf16 value per
// voxel) sit in a small LDS ring, each lane gathers its 8 taps from it, and the
// weights, the MFMA's A operand, stay in registers, so each lane ends with
// four consecutive output channels of one voxel like k_conv_zs.  Per output
// the taps are summed inside the MFMA, then the bias is added.
template <int NB, int EPI, int MT>
__global__ void __launch_bounds__(512)
k_conv1_zs(const u16* __restrict__ in, const bf16x8* __restrict__ wp, const float* __restrict__ bias,
           void* __restrict__ out, const void* __restrict__ aux, int nx, int ny, int nz, int ntx, int nty, int zch) {
    // z chunks of one cube after another
    const int nzc = (nz + zch - 1) / zch;
    const long cube = (int)(blockIdx.x / (ntx * nty)) / nzc * ((long)nx * ny * nz);
    in += cube;
    if (aux) aux = static_cast<const char*>(aux) + cube * (EPI == EPI_RESID ? 4 : 32 * NB);
    out = static_cast<char*>(out) + cube * (EPI == EPI_RAW ? 64 * NB : EPI == EPI_RESID ? 4 : 32 * NB);
    constexpr int XW = 16 * MT, LX = XW + 2, LY = kZsRows + 2, NPL = LX * LY;
    static_assert(NPL <= 64 * kZsRows, "one staged voxel per thread");
    __shared__ u16 ring[3 * NPL + 16 * MT];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i = lane & 15, kg = lane >> 4;
    const int bt = blockIdx.x;
    const int tx = bt % ntx, ty = (bt / ntx) % nty, tz = bt / (ntx * nty) % nzc;
    const int x0 = tx * XW, y0 = ty * kZsRows;
    const int z0 = tz * zch, z1 = min(nz, z0 + zch);

    bf16x8 wf[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) wf[nb] = wp[nb * 64 + lane];

    // thread q stages voxel q of every plane (zero outside the cube); plane p
    // sits in slot (p - z0 + 1) mod 3, and zeros after the three slots stand
    // for the padding taps 27..31
    const int q = threadIdx.x;
    const int qx = x0 + q % LX - 1, qy = y0 + q / LX - 1;
    const bool qin = q < NPL && qx >= 0 && qx < nx && qy >= 0 && qy < ny;
    const long qoff = qin ? (long)qy * nx + qx : 0;
    const long plane = (long)nx * ny;
    auto fetch = [&](int z) -> u16 { return (qin && z >= 0 && z < nz) ? in[z * plane + qoff] : (u16)0; };
    auto put = [&](int z, u16 v) {
        if (q < NPL) ring[((z - z0 + 1) % 3) * NPL + q] = v;
    };
    if (threadIdx.x < 16 * MT) ring[3 * NPL + threadIdx.x] = 0;
    // this lane's 8 taps t = 8 kg + e of voxel i, for each of the three ring
    // rotations r = (z - z0) mod 3: the LDS index of the tap's input voxel
    int gidx[3][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int t = 8 * kg + e;
        const int dz = t / 9, dy = (t / 3) % 3, dx = t % 3;
        const int off = (w + dy) * LX + i + dx;
#pragma unroll
        for (int r = 0; r < 3; ++r) gidx[r][e] = t < 27 ? ((r + dz) % 3) * NPL + off : 3 * NPL;
    }
    put(z0 - 1, fetch(z0 - 1));
    put(z0, fetch(z0));
    u16 nxt = fetch(z0 + 1);

    const int y = y0 + w;
    // 32 bf16 output channels go out through a buffer over this wavefront's row of
    // the tile: no branch, and the addresses of a plane are scalar (360 x 360 x 150
    // 560 -> 452 us, the GELU of every value what is left)
    constexpr bool BUF = EPI == EPI_GELU || EPI == EPI_BACK_GELU;
    static_assert(!BUF || NB == 2, "the bf16 outputs have 32 channels");
    const int lo = i * 64 + 8 * kg;
    const int row_bytes = __builtin_amdgcn_readfirstlane(y < ny ? min(nx - x0, XW) * 64 : 0);
    const int yc = __builtin_amdgcn_readfirstlane(min(y, ny - 1));
    auto row = [&](const void* p, int z) {
        return raw_buffer(static_cast<const char*>(p) + (((long)z * ny + yc) * nx + x0) * 64, row_bytes);
    };
    f32x4 bv[NB];
    if constexpr (BUF && EPI == EPI_GELU)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int e = 0; e < 4; ++e) bv[nb][e] = bias[16 * nb + 4 * kg + e];
    // one plane; R = (z - z0) mod 3 known at compile time
    auto plane_step = [&](int z, auto R) {
        put(z + 1, nxt);
        u32x2 pre[MT][NB];
        if constexpr (BUF && EPI == EPI_BACK_GELU) {
            const auto ra = row(aux, z);
#pragma unroll
            for (int s = 0; s < MT; ++s)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    pre[s][nb] = __builtin_amdgcn_raw_buffer_load_b64(ra, lo + 1024 * s + 32 * nb, 0, 0);
        }
        __syncthreads();
        if (z + 1 < z1) nxt = fetch(z + 2);

        f32x4 acc[MT][NB];
#pragma unroll
        for (int s = 0; s < MT; ++s) {
            bf16x8 a;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                a[e] = __builtin_bit_cast(__bf16, ring[gidx[decltype(R)::value][e] + 16 * s]);
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                acc[s][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[nb], a, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        }
        if constexpr (BUF) {
            const auto ro = row(out, z);
            auto store = [&](const auto& rs, int s, int nb, uint2 v) {
                __builtin_amdgcn_raw_buffer_store_b64(u32x2{v.x, v.y}, rs, lo + 1024 * s + 32 * nb, 0, 0);
            };
#pragma unroll
            for (int s = 0; s < MT; ++s)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    f32x4 d = acc[s][nb];
                    if constexpr (EPI == EPI_GELU) {
                        d += bv[nb];
                        if (aux) store(row(aux, z), s, nb, pack_bf16x4(d[0], d[1], d[2], d[3]));
                        store(ro, s, nb, pack_bf16x4(gelu_fast(d[0]), gelu_fast(d[1]), gelu_fast(d[2]), gelu_fast(d[3])));
                    } else {
                        const unsigned px = pre[s][nb].x, py = pre[s][nb].y;
                        store(ro, s, nb,
                              pack_bf16x4(d[0] * gelu_grad_fast(__uint_as_float(px << 16)),
                                          d[1] * gelu_grad_fast(__uint_as_float(px & 0xffff0000u)),
                                          d[2] * gelu_grad_fast(__uint_as_float(py << 16)),
                                          d[3] * gelu_grad_fast(__uint_as_float(py & 0xffff0000u))));
                    }
                }
        } else {
            zs_store<NB, EPI, MT>(acc, bias, static_cast<float*>(out), static_cast<const float*>(aux), x0, y, z, nx, ny, i, kg);
        }
        __syncthreads();   // every wavefront is done with slot (z - 1) before it takes plane z + 2
    };
    for (int z = z0; z < z1; z += 3) {
        plane_step(z, std::integral_constant<int, 0>{});
        if (z + 1 < z1) plane_step(z + 1, std::integral_constant<int, 1>{});
        if (z + 2 < z1) plane_step(z + 2, std::integral_constant<int, 2>{});
    }
}

// A 32-channel input to one output channel (the network's last layer) as a
// z-stream.  For each plane u of the tile and its one-voxel margin the MFMA
// computes the 27 per-tap sums P_t(v) = sum_c X(v, c) W[t][c] of every voxel
// (weights as the A operand, M = taps, K = channels; activations as B, 16
// voxels per MFMA), into LDS.  Output (x, y, z) then adds P_t at its 27
// neighbours: the dz = 0 taps from plane z-1, the dz = 1 taps from plane z, the
// dz = 2 taps from plane z+1, so it sums its taps in the order 0..26 and then
// adds the bias (and, for the residual, adds that to the input).  Each
// activation is read from memory and multiplied once, instead of once per tap
// with 15 of 16 MFMA columns idle.  P is double-buffered, one barrier per plane.
constexpr int kO1X = 32;                                    // output tile: 32 x kZsRows
constexpr int kO1Vox = (kO1X + 2) * (kZsRows + 2);          // voxels of the tile and margin
constexpr int kO1Groups = (kO1Vox + 15) / 16;               // MFMA column groups of 16 voxels
constexpr int kO1Stride = kO1Groups * 16 + 4;               // floats per tap (4 taps apart: 16 banks apart)
constexpr size_t kO1Lds = (size_t)2 * 27 * kO1Stride * 4;

template <int EPI>
__global__ void __launch_bounds__(512)
k_conv_out1(const u16* __restrict__ in, const bf16x8* __restrict__ wp, const float* __restrict__ bias,
            float* __restrict__ out, const float* __restrict__ aux, int nx, int ny, int nz, int ntx, int nty,
            int zch) {
    static_assert(EPI == EPI_RAW || EPI == EPI_RESID, "raw or residual output");
    constexpr int LX = kO1X + 2;
    constexpr int GPW = (kO1Groups + kZsRows - 1) / kZsRows;   // column groups per wavefront
    extern __shared__ float o1_smem[];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i = lane & 15, kg = lane >> 4;
    const int bt = blockIdx.x;
    const int tx = bt % ntx, ty = (bt / ntx) % nty, tz = bt / (ntx * nty);
    const int x0 = tx * kO1X, y0 = ty * kZsRows;
    const int z0 = tz * zch, z1 = min(nz, z0 + zch);
    const long plane = (long)nx * ny;

    // A fragments: lane (i + 16 kg) holds W[tap 16 mb + i][channels 8 kg .. 8 kg + 7];
    // the packed B layout of tap t keeps exactly that in its lane 16 kg
    bf16x8 wa[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
        const int t = 16 * mb + i;
        wa[mb] = t < 27 ? wp[t * 64 + 16 * kg] : bf16x8{};
    }
    // this lane's B column: voxel 16 g + i of the tile and margin, channels 8 kg ..
    long voff[GPW];
    bool vin[GPW];
#pragma unroll
    for (int k = 0; k < GPW; ++k) {
        const int g = w + kZsRows * k, q = 16 * g + i;
        const int qx = x0 + q % LX - 1, qy = y0 + q / LX - 1;
        vin[k] = g < kO1Groups && q < kO1Vox && qx >= 0 && qx < nx && qy >= 0 && qy < ny;
        voff[k] = vin[k] ? ((long)qy * nx + qx) * 32 + 8 * kg : 0;
    }
    // a plane's fragments are loaded two steps ahead, the residual's input one (a
    // step is shorter than a load under way: 360 x 360 x 150 421 -> 322 us, 3.9 TB/s)
    uint4 b0[GPW], b1[GPW];
    auto fetch = [&](int u, uint4 (&b)[GPW]) {
#pragma unroll
        for (int k = 0; k < GPW; ++k)
            b[k] = (vin[k] && u >= 0 && u < nz) ? *reinterpret_cast<const uint4*>(in + u * plane * 32 + voff[k])
                                                : make_uint4(0, 0, 0, 0);
    };

    // output voxel of this thread (threads 256 .. 511 only compute P)
    const int ox = threadIdx.x % kO1X, oy = threadIdx.x / kO1X;
    const bool owner = threadIdx.x < kO1X * kZsRows;
    const int x = x0 + ox, y = y0 + oy;
    const bool store = owner && x < nx && y < ny;
    float a_prev = 0.f, a_cur = 0.f;   // sums of outputs z = u - 1 and z = u

    float ax = 0.f;
    auto step = [&](int u, uint4 (&b)[GPW]) {
        float* P = o1_smem + (u & 1) * 27 * kO1Stride;
#pragma unroll
        for (int k = 0; k < GPW; ++k) {
            const int g = w + kZsRows * k;
            if (g < kO1Groups) {
                const bf16x8 bv = __builtin_bit_cast(bf16x8, b[k]);
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) {
                    const f32x4 d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[mb], bv, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int t = 16 * mb + 4 * kg + e;
                        if (t < 27) P[t * kO1Stride + 16 * g + i] = d[e];
                    }
                }
            }
        }
        if (u + 1 < z1) fetch(u + 2, b);
        __syncthreads();
        if (owner) {
            const float res = ax;
            if (EPI == EPI_RESID && store && u < z1) ax = aux[(long)max(u, 0) * plane + (long)y * nx + x];
            const float* c = P + oy * LX + ox;
            float a_next = c[0];
#pragma unroll
            for (int t = 1; t < 9; ++t) a_next += c[t * kO1Stride + (t / 3) * LX + t % 3];
#pragma unroll
            for (int t = 9; t < 18; ++t) a_cur += c[t * kO1Stride + ((t / 3) % 3) * LX + t % 3];
#pragma unroll
            for (int t = 18; t < 27; ++t) a_prev += c[t * kO1Stride + ((t / 3) % 3) * LX + t % 3];
            const int zo = u - 1;   // a_prev is complete
            if (store && zo >= z0) {
                const long v = (long)zo * plane + (long)y * nx + x;
                if constexpr (EPI == EPI_RESID) {
                    out[v] = res + (a_prev + bias[0]);
                } else {
                    float4 r0, r1, r2, r3;
                    r0.x = a_prev + (bias ? bias[0] : 0.0f);
                    r0.y = bias ? bias[1] : 0.0f; r0.z = bias ? bias[2] : 0.0f; r0.w = bias ? bias[3] : 0.0f;
                    r1 = bias ? make_float4(bias[4], bias[5], bias[6], bias[7]) : make_float4(0.f, 0.f, 0.f, 0.f);
                    r2 = bias ? make_float4(bias[8], bias[9], bias[10], bias[11]) : make_float4(0.f, 0.f, 0.f, 0.f);
                    r3 = bias ? make_float4(bias[12], bias[13], bias[14], bias[15]) : make_float4(0.f, 0.f, 0.f, 0.f);
                    float4* o = reinterpret_cast<float4*>(out + v * 16);
                    o[0] = r0; o[1] = r1; o[2] = r2; o[3] = r3;
                }
            }
            a_prev = a_cur;
            a_cur = a_next;
        }
    };
    fetch(z0 - 1, b0);
    fetch(z0, b1);
    for (int u = z0 - 1; u <= z1; u += 2) {
        step(u, b0);
        if (u + 1 <= z1) step(u + 1, b1);
    }
}

// ---------------------------------------------------------- weight grad
// dW[t][c][n] = sum over voxels v of a[v + t][c] dz[v][n]: the matrix cores sum
// over K = 32 voxels of a row, so both operands are wanted voxel-minor while
// memory holds them channel-minor.  gfx950's transposing LDS read
// (ds_read_b64_tr_b16) does that: of each 16 lanes, lane l passes the address
// of voxel l / 4, channels 4 (l % 4) .., and receives channel l of the four
// voxels, so two reads make one operand fragment at the full LDS rate.
//
// The order of the FP32 sums is fixed by the cube's shape alone: a cube's units
// (32 x 4 voxels of one plane, u = (z nty + ty) ntx + tx) are cut into `groups`
// contiguous runs, the same for every call; a run's sums go through its units
// and their four rows in order, one product of 32 voxels per row, and its bias
// sums voxel by voxel; the runs of a cube are folded in quarters and the cubes of
// a batch added one after another (k_wgrad_fold).  So a gradient depends neither
// on how many cubes share a launch nor on the device's memory, and weights
// trained with it stay the same to the last bit from one version to the next.
typedef short s16x4 __attribute__((ext_vector_type(4)));
constexpr int kWgX = 32, kWgY = 4;                          // a unit
constexpr int kWgAhead = 2;                                 // activation fragments in flight ahead of their products
constexpr int kWgLX = kWgX + 2, kWgLY = kWgY + 2;           // with the margin
constexpr int kWgPlA = kWgLX * kWgLY * 32, kWgPlB = kWgX * kWgY * 32;   // u16 of a staged plane

typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
// the fragment [voxels 8 kg ..][channel l % 16]: lo = (voxel 8 kg + (l % 16) / 4,
// channels 4 (l % 4) ..) of rows of 32 channels, hi the same four voxels on
__device__ __forceinline__ bf16x8 tr_frag(const u16* lo, const u16* hi) {
    const s16x4 l = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(lo));
    const s16x4 h = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(hi));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(l, h, 0, 1, 2, 3, 4, 5, 6, 7));
}
// A staged voxel x of a row keeps its two halves of 16 channels in turn where bit 3
// of x is set, so that the 32 lanes of one LDS pass, which read 16 channels of
// voxels x and x + 8, meet no bank twice.
__device__ __forceinline__ int wg_half(int x, int half) { return x * 32 + ((half ^ (x >> 3)) & 1) * 16; }

// The gradient of a unit: NB = 2, 32 channels a voxel; NB = 1, one channel, a voxel per
// dword.  This lane's place in a row's fragment of channels 16 nb .., and that of row r
// at S = the gradient + the place
template <int NB>
__device__ __forceinline__ int wg_grad_lane(int lane, int nb) {
    const int i = lane & 15, kg = lane >> 4;
    return NB == 2 ? wg_half(8 * kg + i / 4, nb) + 4 * (i & 3) : 16 * kg;
}
template <int NB>
__device__ __forceinline__ bf16x8 wg_grad_frag(const u16* S, int r) {
    if constexpr (NB == 2) {
        return tr_frag(S + r * kWgX * 32, S + (r * kWgX + 4) * 32);
    } else {
        const uint4 p = *reinterpret_cast<const uint4*>(S + r * 2 * kWgX);
        const uint4 q = *reinterpret_cast<const uint4*>(S + r * 2 * kWgX + 8);
        return __builtin_bit_cast(bf16x8, make_uint4(p.x | p.y << 16, p.z | p.w << 16, q.x | q.y << 16, q.z | q.w << 16));
    }
}
constexpr int wg_grad(int NB) { return NB == 2 ? kWgPlB : 2 * kWgX * kWgY; }   // u16

// The runs of one workgroup and their units, one after another.  Workgroups are
// dispatched to the 8 XCDs in turn; each XCD takes an eighth of the runs and its
// workgroups neighbouring ones at a time, so that the planes they share meet in
// one L2.
struct WgUnits {
    int ntx, nty, groups, units;
    int run, end, by;       // run, the one past the last, and from run to run
    int cube, u1;           // of the run
    int u, tx, ty, z;       // the unit
    __device__ __forceinline__ WgUnits(int ntx_, int nty_, int nz, int groups_, int runs)
        : ntx(ntx_), nty(nty_), groups(groups_), units(ntx_ * nty_ * nz) {
        const int g = gridDim.x, b = blockIdx.x, parts = g % 8 == 0 ? 8 : 1, part = b % parts;
        by = g / parts;
        run = (int)((long)runs * part / parts) + b / parts;
        end = (int)((long)runs * (part + 1) / parts);
        if (more()) enter();
    }
    __device__ __forceinline__ bool more() const { return run < end; }
    __device__ __forceinline__ void enter() {
        cube = run / groups;
        const long r = run - cube * groups;
        u = (int)(r * units / groups);
        u1 = (int)((r + 1) * units / groups);
        tx = u % ntx;
        ty = u / ntx % nty;
        z = u / (ntx * nty);
    }
    __device__ __forceinline__ void next_run() {
        run += by;
        if (more()) enter();
    }
    // to the next unit; true where a run has ended
    __device__ __forceinline__ bool step() {
        if (++u < u1) {
            if (++tx == ntx) {
                tx = 0;
                if (++ty == nty) ty = 0, ++z;
            }
            return false;
        }
        return true;
    }
};

// The bias sums of a unit, voxel after voxel: lane (i + 16 g) adds channel 16 (g & 1) + i
// (NB = 1: every lane the same).  Half a row is read ahead of its additions.
template <int NB>
__device__ __forceinline__ void wg_bias(const u16* Bs, int lane, float* sum) {
    const int i = lane & 15;
    // voxels 16 h + 4 k .. + 3 of a row, as FP32 values
    auto read = [&](auto kc, const u16* row) {
        constexpr int v = 4 * decltype(kc)::value;
        f32x4 r;
        if constexpr (NB == 1) {
            const uint4 q = *reinterpret_cast<const uint4*>(row + 2 * v);   // a voxel per dword
            r = f32x4{__uint_as_float(q.x << 16), __uint_as_float(q.y << 16), __uint_as_float(q.z << 16), __uint_as_float(q.w << 16)};
        } else {
            const s16x4 q = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (lds_s16x4)(row + (i >> 2) * 32 + (((lane >> 4) ^ (v >> 3)) & 1) * 16 + 4 * (i & 3) + v * 32));
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = bf2f((u16)q[e]);
        }
        return r;
    };
    constexpr int ROW = NB == 2 ? kWgX * 32 : 2 * kWgX;     // u16
    float s = *sum;
    f32x4 r[2][4];
    static_for<4>([&](auto k) { r[0][decltype(k)::value] = read(k, Bs); });
    static_for<2 * kWgY>([&](auto hc) {
        constexpr int h = decltype(hc)::value;
        if constexpr (h + 1 < 2 * kWgY)
            static_for<4>([&](auto k) {
                constexpr int kk = 4 * ((h + 1) & 1) + decltype(k)::value;
                r[(h + 1) & 1][decltype(k)::value] = read(std::integral_constant<int, kk>{}, Bs + (h + 1) / 2 * ROW);
            });
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) s += r[h & 1][k][e];
        __builtin_amdgcn_sched_barrier(0);
    });
    *sum = s;
}

// 32 input channels and 32 output channels (NB = 2), or one (NB = 1, its gradient rows
// read as a column that all 16 lanes share, a voxel per dword).  Six wavefronts per
// 16 output channels multiply: (ms, p, nb) owns input channels 16 ms .., output
// channels 16 nb .. and the nine taps of plane p, with their sums in registers.  Each
// activation fragment is read once and multiplied with the gradient rows that it
// meets, which stay in registers: 22 fragment reads for 36 products.  Of four more
// wavefronts one adds the bias sums and three load the units straight into a ring of
// three in the LDS, two ahead, zeros outside the cube (loads past a buffer's end):
// one barrier a unit, without a wait for the loads under way.  The bias sums are a
// chain of 128 additions a unit, so that wavefront and the loading ones go first
// (s_setprio).  Four 96^3 cubes: 212 us a layer (4 x 263 with gathered LDS reads and
// one pair of fragments per product; 200 in a form that kept no order of the sums and
// streamed whole columns of planes); one output channel 132 us (4 x 185).  What
// bounds it: per unit and compute unit 1728 cycles of products, 2500 of the bias
// chain, and the wait for 47 KB of loads, in 3500.
constexpr int wg_threads(int NB) { return 64 * (6 * NB + 4); }
constexpr int wg_slot(int NB) { return 3 * kWgPlA + wg_grad(NB); }   // u16 of a staged unit
constexpr size_t wg_lds(int NB) { return (size_t)3 * wg_slot(NB) * 2; }
template <int NB>
__global__ void __launch_bounds__(wg_threads(NB), NB == 2 ? 4 : 3)
k_wgrad32(const u16* __restrict__ a0, const u16* __restrict__ dz0, float* __restrict__ part, int nx, int ny, int nz,
          int ntx, int nty, int groups, int runs) {
    constexpr int CO = NB == 2 ? 32 : 1, MW = 6 * NB, SLOT = wg_slot(NB), B0 = 3 * kWgPlA;
    constexpr long PART = 27L * 32 * CO + CO;
    extern __shared__ uint4 wg_smem[];
    u16* sm = reinterpret_cast<u16*>(wg_smem);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long n = (long)nx * ny * nz;
    WgUnits it(ntx, nty, nz, groups, runs);
    // a barrier that waits for no load: LDS accesses stay on their side of it
    auto barrier = [] {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    if (w > MW) {
        // Loading thread lt takes the 16-byte chunks lt + 192 k of the activations (KA)
        // and of the gradient (KB): a chunk's offset in bytes from the unit's first
        // voxel, and its column and row (bit of a mask) in the staged block.
        constexpr int QA = 3 * kWgLX * kWgLY * 4, KA = (QA + 191) / 192, QB = kWgX * kWgY * 4, KB = NB == 2 ? 3 : 1;
        const int lw = w - MW - 1, lt = 64 * lw + lane;
        unsigned rel[KA], col[KA], bit[KA], relb[KB], colb[KB], bitb[KB];
#pragma unroll
        for (int k = 0; k < KA; ++k) {
            const int q = lt + 192 * k, vox = q >> 2, x = vox % kWgLX, r = vox / kWgLX;
            const int c = (q & 3) ^ ((x >> 2) & 2);          // (wg_half)
            rel[k] = (unsigned)(((r / kWgLY - 1) * ny + r % kWgLY - 1) * nx + x - 1) * 64u + 16 * c;
            col[k] = x;
            bit[k] = 1u << r;
        }
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            const int q = lt + 192 * k, vox = NB == 2 ? q >> 2 : 64 * k + lane, x = vox % kWgX, r = vox / kWgX;
            relb[k] = (unsigned)(r * nx + x) * (NB == 2 ? 64u : 2u) + (NB == 2 ? 16 * ((q & 3) ^ ((x >> 2) & 2)) : 0);
            colb[k] = x;
            bitb[k] = 1u << r;
        }
        const unsigned bytes = (unsigned)(n * 64), bytesb = (unsigned)(n * 2 * CO);   // below 2^32: fewer than 2^26 voxels
        typedef __attribute__((address_space(3))) void* lds_ptr;
        auto stage = [&](int slot) {
            u16* to = sm + slot * SLOT;
            const auto ra = raw_buffer(a0 + it.cube * n * 32, (int)bytes);
            const auto rb = raw_buffer(dz0 + it.cube * n * CO, (int)bytesb);
            const int x0 = it.tx * kWgX, y0 = it.ty * kWgY, v0 = (it.z * ny + y0) * nx + x0;
            // columns x0 - 1 + [xl, xh) and rows of planes z - 1 .. z + 1 that lie in the cube
            const unsigned xl = x0 == 0 ? 1 : 0, xh = min(kWgLX, nx - x0 + 1);
            const unsigned rows = ((1u << min(kWgLY, ny - y0 + 1)) - 1) & (y0 == 0 ? ~1u : ~0u);
            const unsigned in = (it.z > 0 ? rows : 0) | rows << kWgLY | (it.z + 1 < nz ? rows << (2 * kWgLY) : 0);
            const unsigned inb = (1u << min(kWgY, ny - y0)) - 1, xhb = min(kWgX, nx - x0);
#pragma unroll
            for (int k = 0; k < KA; ++k) {
                const bool ok = col[k] - xl < xh - xl && (bit[k] & in);
                const unsigned off = ok ? (unsigned)v0 * 64u + rel[k] : bytes;
                if (192 * (k + 1) <= QA || lt + 192 * k < QA)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_ptr)(to + (64 * lw + 192 * k) * 8), 16, off, 0, 0, 0);
            }
            if constexpr (NB == 2) {
#pragma unroll
                for (int k = 0; k < KB; ++k) {
                    const bool ok = colb[k] < xhb && (bitb[k] & inb);
                    const unsigned off = ok ? (unsigned)v0 * 64u + relb[k] : bytesb;
                    if (192 * (k + 1) <= QB || 64 * lw + 192 * k < QB)
                        __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_ptr)(to + B0 + (64 * lw + 192 * k) * 8), 16, off, 0, 0, 0);
                }
            } else if (lw < 2) {                             // voxels 64 lw + lane
                const int r = 2 * lw + (lane >> 5), x = lane & 31;
                const unsigned off = x < (int)xhb && (inb >> r & 1) ? (unsigned)(v0 + r * nx + x) * 2u : bytesb;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_ptr)(to + B0 + 128 * lw), 2, off, 0, 0, 0);
            }
            if (it.step()) it.next_run();
        };
        // loads that a unit takes of this wavefront: KA, and of the gradient (NB = 2) 3, 3
        // and 2, (NB = 1) 1, 1 and 0
        __builtin_amdgcn_s_setprio(2);
        int ahead = 0;                                       // units whole or under way past the one consumed
        for (; ahead < 2 && it.more(); ++ahead) stage(ahead);
        for (int slot = 0; ahead > 0; slot = slot == 2 ? 0 : slot + 1) {
            if (ahead == 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            else if (lw == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(KA + (NB == 2 ? 2 : 0)) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(KA + (NB == 2 ? 3 : 1)) : "memory");
            barrier();                                       // the unit in `slot` is whole, the one before it done
            --ahead;
            if (it.more()) {
                stage(slot == 0 ? 2 : slot - 1);
                ++ahead;
            }
        }
        return;
    }
    if (w == MW) {
        __builtin_amdgcn_s_setprio(2);
        float bsum = 0.0f;
        for (int slot = 0; it.more(); slot = slot == 2 ? 0 : slot + 1) {
            barrier();
            wg_bias<NB>(sm + slot * SLOT + B0, lane, &bsum);
            if (it.step()) {
                if (lane < CO) part[it.run * PART + 27 * 32 * CO + lane] = bsum;
                bsum = 0.0f;
                it.next_run();
            }
        }
        return;
    }
    const int ms = w & 1, p = (w >> 1) % 3, nb = w / 6, i = lane & 15, kg = lane >> 4;
    f32x4 acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    int lo[3], hi[3];                                        // this lane's place in a fragment shifted by dx
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
        lo[dx] = p * kWgPlA + wg_half(8 * kg + i / 4 + dx, ms) + 4 * (i & 3);
        hi[dx] = p * kWgPlA + wg_half(8 * kg + i / 4 + dx + 4, ms) + 4 * (i & 3);
    }
    const int gl = B0 + wg_grad_lane<NB>(lane, nb);
    // fragment m: input row j = m / 3 (the unit's row - 1), shift dx = m % 3
    constexpr int FR = kWgAhead + 1;
    bf16x8 b[kWgY], f[FR];
    for (int slot = 0; it.more(); slot = slot == 2 ? 0 : slot + 1) {
        barrier();
        const u16* S = sm + slot * SLOT;
        auto load = [&](auto mc) {
            constexpr int m = decltype(mc)::value, r = m / 3 * kWgLX * 32;
            if constexpr (m < 18) f[m % FR] = tr_frag(S + lo[m % 3] + r, S + hi[m % 3] + r);
        };
        b[0] = wg_grad_frag<NB>(S + gl, 0);
        static_for<kWgAhead>(load);
        static_for<18>([&](auto mc) {
            constexpr int m = decltype(mc)::value, j = m / 3, dx = m % 3;
            if constexpr (dx == 0 && j + 1 < kWgY) b[j + 1] = wg_grad_frag<NB>(S + gl, j + 1);
            load(std::integral_constant<int, m + kWgAhead>{});
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
                if (j - dy >= 0 && j - dy < kWgY)
                    acc[3 * dy + dx] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[m % FR], b[j - dy], acc[3 * dy + dx], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        });
        if (it.step()) {
            float* P = part + it.run * PART;
#pragma unroll
            for (int t = 0; t < 9; ++t) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (NB == 2 || i == 0)
                        P[((9 * p + t) * 32 + 16 * ms + 4 * kg + e) * CO + (NB == 2 ? 16 * nb + i : 0)] = acc[t][e];
                acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
            it.next_run();
        }
    }
}

// One input channel and 32 output channels (NB = 2) or one: M = the 27 taps (padded to
// 32), N = output channels, K = 32 voxels of a row; a workgroup per run.  Wavefront (m,
// nb) owns 16 taps and 16 channels, the last one the bias sums too.  The input's planes
// are staged three times, shifted by dx, so a lane's 8 values are one aligned read.
// Bound by the bias chain and reading dz: four 96^3 cubes 67 us (4 x 143 before).
constexpr int kWg1Threads = 256;
constexpr int kWg1Row = 40;                                  // u16 per staged input row (32, padded to spread the banks)
constexpr int kWg1Copy = kWgLY * kWg1Row, kWg1Pl = 3 * kWg1Copy;
template <int NB>
__global__ void __launch_bounds__(kWg1Threads)
k_wgrad1(const u16* __restrict__ a0, const u16* __restrict__ dz0, float* __restrict__ part, int nx, int ny, int nz,
         int ntx, int nty, int groups, int runs) {
    constexpr int CO = NB == 2 ? 32 : 1;
    __shared__ __attribute__((aligned(16))) u16 Qs[3 * kWg1Pl + kWgY * kWg1Row];   // + zeros
    __shared__ __attribute__((aligned(16))) u16 Bs[wg_grad(NB)];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = w & 1, nb = w >> 1;
    const int i = lane & 15, kg = lane >> 4;
    for (int k = tid; k < kWgY * kWg1Row; k += kWg1Threads) Qs[3 * kWg1Pl + k] = 0;
    const int t = 16 * m + i;                                // this lane's tap
    const u16* Qa = Qs + (t < 27 ? t / 9 * kWg1Pl + t % 3 * kWg1Copy + t / 3 % 3 * kWg1Row : 3 * kWg1Pl) + 8 * kg;
    const u16* Ba = Bs + wg_grad_lane<NB>(lane, nb);
    WgUnits it(ntx, nty, nz, groups, runs);
    const long cube = it.cube * ((long)nx * ny * nz);
    const u16 *a = a0 + cube, *dz = dz0 + cube * CO;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float bsum = 0.0f;

    constexpr int KA = (3 * kWgLX * kWgLY + kWg1Threads - 1) / kWg1Threads, KB = NB == 2 ? 2 : 1;
    u16 sa[KA];
    uint4 sb[KB];
    auto fetch = [&]() {
        const int x0 = it.tx * kWgX, y0 = it.ty * kWgY;
#pragma unroll
        for (int k = 0; k < KA; ++k) {
            const int q = tid + kWg1Threads * k;
            const int x = x0 + q % kWgLX - 1, y = y0 + q / kWgLX % kWgLY - 1, z = it.z + q / (kWgLX * kWgLY) - 1;
            const bool ok = q < 3 * kWgLX * kWgLY && x >= 0 && x < nx && y >= 0 && y < ny && z >= 0 && z < nz;
            sa[k] = ok ? a[((long)z * ny + y) * nx + x] : (u16)0;
        }
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            const int q = tid + kWg1Threads * k, vox = NB == 2 ? q >> 2 : q & (kWgX * kWgY - 1);
            const int x = x0 + vox % kWgX, y = y0 + vox / kWgX;
            const long v = ((long)it.z * ny + y) * nx + x;
            sb[k] = make_uint4(0, 0, 0, 0);
            if (x < nx && y < ny) {
                if constexpr (NB == 2) sb[k] = *reinterpret_cast<const uint4*>(dz + v * 32 + 8 * (q & 3));
                else sb[k].x = dz[v];
            }
        }
    };
    auto put = [&]() {
#pragma unroll
        for (int k = 0; k < KA; ++k) {
            const int q = tid + kWg1Threads * k, x = q % kWgLX, r = q / kWgLX % kWgLY, p = q / (kWgLX * kWgLY);
            if (q < 3 * kWgLX * kWgLY)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
                    if (x - dx >= 0 && x - dx < kWgX) Qs[p * kWg1Pl + dx * kWg1Copy + r * kWg1Row + x - dx] = sa[k];
        }
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            const int q = tid + kWg1Threads * k;
            if constexpr (NB == 2) reinterpret_cast<uint4*>(Bs)[q ^ (q >> 4 & 2)] = sb[k];   // (wg_half)
            else if (q < kWgX * kWgY) reinterpret_cast<unsigned*>(Bs)[q] = sb[k].x;
        }
    };
    fetch();
    for (bool last = false; !last;) {
        put();
        __syncthreads();
        last = it.step();
        if (!last) fetch();
        if (nb < NB)
#pragma unroll
            for (int r = 0; r < kWgY; ++r) {
                const bf16x8 f = *reinterpret_cast<const bf16x8*>(Qa + r * kWg1Row);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, wg_grad_frag<NB>(Ba, r), acc, 0, 0, 0);
            }
        if (w == 3) wg_bias<NB>(Bs, lane, &bsum);
        __syncthreads();
    }
    float* P = part + it.run * (28L * CO);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int tt = 16 * m + 4 * kg + e;
        if (tt < 27 && nb < NB && (NB == 2 || i == 0)) P[tt * CO + (NB == 2 ? 16 * nb + i : 0)] = acc[e];
    }
    if (w == 3 && lane < CO) P[27 * CO + lane] = bsum;
}

// dW[j] (j < lenw) and db[j - lenw] (+)= the cubes' gradients in order, a cube's the
// sum over its nwg runs of part[run][j]: quarter q of the runs, [q nwg/4, (q+1)
// nwg/4), in order (eight loads in flight), then the quarters in order.  Sixteen
// wavefronts take four cubes at a time, each a quarter for 64 consecutive j.  Bound by
// reading the partials: 2 x 57 MB of two 96^3 cubes in 20 us.
__global__ void __launch_bounds__(1024)
k_wgrad_fold(const float* __restrict__ part, long nwg, int cubes, long lenw, long len, float* __restrict__ dW,
             float* __restrict__ db, int accumulate) {
    __shared__ float sh[16][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, q = w & 3;
    const long j = (long)blockIdx.x * 64 + lane;
    const long k0 = q * nwg / 4, k1 = (q + 1) * nwg / 4;
    float* d = j < lenw ? dW + j : db + (j - lenw);
    float g = w == 0 && j < len && accumulate ? *d : 0.0f;
    for (int c0 = 0; c0 < cubes; c0 += 4) {
        const int c = c0 + (w >> 2);
        float s = 0.0f;
        if (c < cubes && j < len) {
            const float* p = part + c * nwg * len + j;
            long k = k0;
            for (; k + 8 <= k1; k += 8) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = p[(k + u) * len];
#pragma unroll
                for (int u = 0; u < 8; ++u) s += v[u];
            }
            for (; k < k1; ++k) s += p[k * len];
        }
        sh[w][lane] = s;
        __syncthreads();
        if (w == 0)
            for (int e = 0; e < min(4, cubes - c0); ++e) {
                const float t = ((sh[4 * e][lane] + sh[4 * e + 1][lane]) + sh[4 * e + 2][lane]) + sh[4 * e + 3][lane];
                g = accumulate || c0 + e > 0 ? g + t : t;
            }
        __syncthreads();
    }
    if (w == 0 && j < len) *d = g;
}

// ---------------------------------------------------------- loss, inputs
// x (FP32 cube) -> 1-channel bf16 activation
__global__ void k_to_bf16(const float* __restrict__ x, u16* __restrict__ a, long n) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) a[i] = f2bf(x[i]);
}

// dy = (2/N_total) (y - t) as bf16 (1 channel); per-workgroup FP64 loss partial
__global__ void __launch_bounds__(256)
k_mse(const float* __restrict__ y, const float* __restrict__ t, long n, double scale, u16* __restrict__ dy,
      double* __restrict__ part) {
    __shared__ double sh[256];
    double s = 0.0;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256) {
        const double r = (double)y[i] - (double)t[i];
        s += r * r;
        if (dy) dy[i] = f2bf((float)(2.0 * scale * r));
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// ---------------------------------------------------------- optimiser
// Gradient clipping by global norm: FP64 sum of squares of the gradient per
// workgroup, then one workgroup folds the partials in a fixed order and writes the
// factor min(1, max_norm / ||g||) (1 when max_norm <= 0).
__global__ void __launch_bounds__(256)
k_sumsq(const float* __restrict__ g, long n, double* __restrict__ part) {
    __shared__ double sh[256];
    double s = 0.0;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256) {
        const double v = g[i];
        s += v * v;
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}
__global__ void __launch_bounds__(256)
k_clip_factor(const double* __restrict__ part, int nparts, float max_norm, float* __restrict__ factor,
              double* __restrict__ norm_out) {
    __shared__ double sh[256];
    double s = 0.0;
    for (int k = threadIdx.x; k < nparts; k += 256) s += part[k];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    const double nrm = sqrt(sh[0]);
    *norm_out = nrm;
    *factor = (max_norm > 0.0f && nrm > (double)max_norm) ? (float)((double)max_norm / nrm) : 1.0f;
}

// Adam on FP32 master parameters (bias-corrected), grads scaled by *gscale.
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, long n, float lr, float b1, float b2, float eps, float bc1, float bc2,
                       const float* __restrict__ gscale) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i] * *gscale;
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

// Pack FP32 weights W[27][cin][cout] into the B-fragment layout.
//   mode 0 (forward):  B_t[k = c][n = o]               = W[t][c][o]
//   mode 1 (input gradient): B_t[k = o][n = c]         = W[26 - t][c][o]
// For a 1-channel K (cin == 1 in mode 0, cout == 1 in mode 1) the taps are K.
__device__ __forceinline__ void pack_one(const float* __restrict__ W, int cin, int cout, int mode, int q,
                                         bf16x8* __restrict__ out) {
    const int kin = mode == 0 ? cin : cout, nout = mode == 0 ? cout : cin;
    const int NB = (nout + 15) / 16;
    const int ntap_blocks = kin == 1 ? 1 : 27;
    const int total = ntap_blocks * NB * 64;
    if (q >= total) return;
    const int lane = q % 64, nb = (q / 64) % NB, tb = q / (64 * NB);
    const int n = 16 * nb + (lane & 15);
    bf16x8 r;
    for (int e = 0; e < 8; ++e) {
        const int k = 8 * (lane >> 4) + e;
        float val = 0.0f;
        if (n < nout) {
            if (kin == 1) {              // k is the tap
                if (k < 27) {
                    const int t = mode == 0 ? k : 26 - k;
                    val = mode == 0 ? W[(t * cin + 0) * cout + n] : W[(t * cin + n) * cout + 0];
                }
            } else if (k < kin) {
                const int t = mode == 0 ? tb : 26 - tb;
                val = mode == 0 ? W[(t * cin + k) * cout + n] : W[(t * cin + n) * cout + k];
            }
        }
        r[e] = __builtin_bit_cast(__bf16, f2bf(val));
    }
    out[q] = r;
}
__global__ void k_pack(const float* __restrict__ W, int cin, int cout, int mode, bf16x8* __restrict__ out) {
    pack_one(W, cin, cout, mode, blockIdx.x * 256 + threadIdx.x, out);
}
// Every layer of a network in both forms in one launch (blockIdx.y = 2 layer + mode).
constexpr int kMaxLayers = 64;
struct PackAll {
    int layers;
    bf16x8* out[2 * kMaxLayers];
};
__global__ void k_pack_all(const float* __restrict__ params, PackAll a) {
    const int l = blockIdx.y >> 1, mode = blockIdx.y & 1;
    const int cin = l == 0 ? 1 : 32, cout = l + 1 == a.layers ? 1 : 32;
    // parameters: layer by layer, W[27][cin][cout] then b[cout]
    const long off = l == 0 ? 0 : 27L * 32 + 32 + (l - 1) * (27L * 1024 + 32);
    pack_one(params + off, cin, cout, mode, blockIdx.x * 256 + threadIdx.x, a.out[blockIdx.y]);
}

}  // namespace igs

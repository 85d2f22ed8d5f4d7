// Convolution and fully connected layers as an implicit GEMM whose operand tiles are copied from memory to LDS by the
// load unit itself (buffer_load_dwordx4 ... lds), without passing through registers.
//
//   D[k, m] = sum_j Wp[k, j] * A[m, j]        k: output channel, m: output pixel (n, p, q), j: (r, s, c)
//
// Wp is the filter bank packed as [n_pad][k_pad], A the im2col matrix, never materialised: eight consecutive j with
// C % 8 == 0 are eight channels of one input pixel, one 16-byte piece of the NHWC tensor or, in the padding halo, an
// out-of-range offset for which the load delivers zeros.
//
// What bounds it: a stage of 64 reduction elements passes through load unit, LDS and matrix cores; staging it through
// registers (the form before) cost a chain of load, wait, LDS write, barrier, LDS read and matrix instructions per 64
// elements, and padded LDS rows.  Here NBUF stages of LDS are in flight, one barrier per stage waits for the oldest, and rows
// are 128 bytes without padding, their 16-byte columns permuted so that operand reads use all 64 banks (conflicts per LDS
// cycle 0.5 with a permutation over 8 rows, 0.0 with the one over 16).  MI355X, us before / now, launch gap included:
//   3x3, 256 -> 256 on 8 x 56 x 56 (59 GFLOP)  52.0 / 32.7      3x3, 512 -> 512 on 8 x 28 x 28  47.5 / 34.4
//   1x1, 1024 -> 512 on 64 x 14 x 14           28.4 / 20.0      1x1, 512 -> 2048 on 64 x 7 x 7   20.3 / 15.0
//   1x1, 768 -> 192 on 5 x 17 x 17              9.9 /  5.3      3x3, 64 -> 64 on 56 x 56          5.4 /  4.6
// fp32 rows hold 32 elements and a piece feeds four v_mfma_f32_*x2 / x4; at 128 multiply-adds per cycle and unit the matrix cores
// bound the larger layers (4 x 28 x 28, 3x3, 128 -> 128: 21.1 us from registers, 16.8 on 64 x 32 tiles, 7.7 us of it matrix instructions).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <type_traits>
#include <utility>

#include "internal.h"
#include "device_types.h"
#include "mfma.h"

namespace mt {

// How a row of A is gathered: TG_POINT 1x1 windows without padding and C % 64 == 0 (a row is contiguous), TG_TAP
// C % 64 == 0 (64 consecutive j lie inside one filter tap), TG_CHUNK C % 8 == 0 (every 16-byte piece has its own tap).  Which taps
// of a window are inside the image is a mask of 15 rows and 16 columns; TG_FAR is TG_CHUNK for larger windows and compares.
constexpr int TG_POINT = 0, TG_TAP = 1, TG_CHUNK = 2, TG_FAR = 3;

namespace {

constexpr int TK = 64;                          // reduction elements of one LDS row (128 bytes) of a 16-bit type
template <typename T> constexpr int ROW = 128 / (int)sizeof(T);    // the same of any type
constexpr int XCDS = 8;
constexpr uint32_t OUT_OF_RANGE = 0x80000000u;  // beyond any tensor: the load delivers zeros

// 64 lanes x 16 bytes from rsrc + voff (per lane) + soff to LDS at `lds` + 16 * lane.  The instruction takes the LDS address from m0;
// the compiler puts it there, so it knows what m0 holds, and the wait state the load needs after that follows.  It needs five after a vector
// instruction that writes one of its scalars (v_readlane, v_readfirstlane), which nothing adds inside inline assembly: the scalars come from
// arguments and scalar arithmetic, none of the kernels spills any, and the host tests look for such a pair in the built kernels.  (Five states
// in front of every load make ResNet-50 at batch 64 0.5 %, Inception-v3 and AlexNet at batch 5 1 % slower.)
__device__ __forceinline__ void load_to_lds(u32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds) {
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"{m0}"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}

// The same with 4 bytes a lane.  Once per tile: its descriptor may come out of vector registers (v_readlane) just before, and the five wait
// states between a vector instruction that writes scalar registers and a load that reads them are not added inside inline assembly.
__device__ __forceinline__ void load_words_to_lds(u32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds) {
    asm volatile("s_nop 4\n\tbuffer_load_dword %1, %2, %3 offen lds" ::"{m0}"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}

// All but the N youngest loads of this wave have landed, its LDS reads are done, and the other waves got here as well.
template <int N>
__device__ __forceinline__ void wait_and_meet() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// The same when `later` stages (at most MAX) of L loads each were requested after the one waited for.
template <int L, int MAX>
__device__ __forceinline__ void wait_for_stage(int later) {
    if constexpr (MAX > 0) {
        if (later < MAX) return wait_for_stage<L, MAX - 1>(later);
    }
    wait_and_meet<MAX * L>();
}

// All but the youngest `later` rows (at most MAX) of L loads each have landed; this wave's loads only.
template <int L, int MAX>
__device__ __forceinline__ void wait_for_row(int later) {
    if constexpr (MAX > 0) {
        if (later < MAX) return wait_for_row<L, MAX - 1>(later);
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(MAX * L) : "memory");
}

__device__ __forceinline__ u32x4 raw_buffer(const void *p, uint32_t bytes) {
    const uint64_t b = (uint64_t)p;
    return u32x4{(uint32_t)b, (uint32_t)(b >> 32) & 0xffffu, bytes, 0x00027000u};
}

}  // namespace

// Whether the taps of this layer can be read from a patch in LDS (patch_body).
bool patch_stageable(const OpArgs &a) {
    return a.kind == MT_CONV && a.dtype != MT_F32 && a.groups <= 1 && a.R == 3 && a.S == 3 && a.sh == 1 && a.sw == 1 && a.ph == 1 && a.pw == 1 && a.C % TK == 0 && a.H <= 1024;
}

// ---- epilogues ----------------------------------------------------------------------------------------------------
// On small maps the epilogue is a chain of trips: partial sums through LDS to one wave group, from there through LDS to the threads that
// store, and in between a trip to memory for bias and residual (0.6 to 0.9 of a layer's 4 us).  Here the threads that store add
// the sums up themselves and asked for bias and residual before the reduction began.  us, before / now: ResNet-18 at one image
// 108.6 / 105.8, ResNet-101, Inception-v3, MobileNetV2 and AlexNet together 535 / 518, eight ResNet-50 at batch 16 2689 / 2640.
// Bias and residual of V consecutive channels of one output pixel.
template <typename T, int V>
struct Addend {
    typedef std::conditional_t<sizeof(T) * V == 8, uint64_t, u32x4> Raw;     // V elements; fp32 only ever takes four of them
    float bias[V];
    Raw res;

    __device__ __forceinline__ void load(const OpArgs &a, int m, int k, bool vec_ok) {
#pragma unroll
        for (int v = 0; v < V; v += 4) *reinterpret_cast<float4 *>(&bias[v]) = *reinterpret_cast<const float4 *>(a.bias + k + v);   // padded to n_pad
        res = Raw{};
        if (a.res != nullptr && !a.pool2 && vec_ok && m >= 0 && k < a.K) res = *reinterpret_cast<const Raw *>((const T *)a.res + (int64_t)m * a.res_ct + k);
    }
};

// Whether V channels can be loaded and stored in one access: then they are also all inside the layer or all outside.
template <int V>
__device__ __forceinline__ bool whole_packs(const OpArgs &a) {
    return (a.K % V == 0) & (a.y_ct % V == 0) & (a.y_coff % V == 0) & (a.res_ct % V == 0);
}

// Finished sums of V channels from k on of output pixel m, and of the pixels beside it: bias, residual, activation, one rounding,
// store.  Pooling: the four pixels of a window are STRIDE lanes apart and m is the pooled pixel of all four.
template <typename T, int V, int STRIDE>
__device__ __forceinline__ void finish_pixel(const OpArgs &a, float (&v)[V], const Addend<T, V> &add, int m, int k, bool vec_ok, bool first_of_window) {
#pragma unroll
    for (int t = 0; t < V; ++t) v[t] += add.bias[t];
    if (a.pool2) {
#pragma unroll
        for (int t = 0; t < V; ++t) {
            v[t] = fmaxf(v[t], -INFINITY);                 // a window without a number has no maximum, as in the pooling kernels
            v[t] = fmaxf(v[t], __shfl_xor(v[t], STRIDE));
            v[t] = fmaxf(v[t], __shfl_xor(v[t], 2 * STRIDE));
        }
        if (!first_of_window) return;
    }
    if (m < 0 || k >= a.K) return;
    const Results y = results_in(a.y);
    const uint32_t at = (uint32_t)m * (uint32_t)a.y_ct + (uint32_t)(a.y_coff + k);
    if (vec_ok) {
        if (a.res != nullptr && !a.pool2) {
            const Pack<T, V> rp = __builtin_bit_cast(Pack<T, V>, add.res);
#pragma unroll
            for (int t = 0; t < V; ++t) v[t] += to_f32(rp.e[t]);
        }
#pragma unroll
        for (int t = 0; t < V; ++t) v[t] = apply_act(v[t], a.act);
        store_pack<T, V>(y, at, v);
    } else {
#pragma unroll
        for (int t = 0; t < V; ++t) {
            if (k + t >= a.K) continue;
            float f = v[t];
            if (a.res != nullptr && !a.pool2) f += to_f32(((const T *)a.res)[(int64_t)m * a.res_ct + k + t]);
            store_one<T>(y, at + (uint32_t)t, apply_act(f, a.act));
        }
    }
}

// Place of channels 4 * c .. + 3 of pixel p in a [pixels][BN] block of partial sums in LDS, in floats: written by 16 lanes with
// consecutive pixels and read by 16 lanes with consecutive channels, both without bank conflicts.
template <int BN>
__device__ __forceinline__ uint32_t sum_at(int p, int c) {
    constexpr int SHARE = BN < 64 ? 64 / BN : 1;           // rows that fill the 64 banks
    return (uint32_t)(p * BN + ((c ^ ((p / SHARE) & (BN / 4 - 1))) * 4));
}

// What follows the main loop where WK wave groups share the reduction: every group puts its partial sums into LDS, and the threads
// that store add them up, in group order, with bias and residual already at hand.  A group's block of sums is BLOCK floats
// after the one before it.
template <int BN, int MF, int SUBN, int SUBM, typename Acc, int TN, int TM>
__device__ __forceinline__ void publish_sums(const Acc (&acc)[TN][TM], float *sums, int wn, int wm, int frow, int fgrp) {
    constexpr int GROUPS = MF == 32 ? 4 : 1;
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int g = 0; g < GROUPS; ++g)
                *reinterpret_cast<float4 *>(&sums[sum_at<BN>(wm * SUBM + j * MF + frow, (wn * SUBN + i * MF) / 4 + (MF == 32 ? 2 * g + fgrp : fgrp))]) =
                    make_float4(acc[i][j][g * 4], acc[i][j][g * 4 + 1], acc[i][j][g * 4 + 2], acc[i][j][g * 4 + 3]);
}

template <int BN, int V, int WK>
__device__ __forceinline__ void add_up(const float *sums, int block, int p, int c, float (&v)[V]) {
    float4 part[WK][V / 4];
#pragma unroll
    for (int w = 0; w < WK; ++w)
#pragma unroll
        for (int h = 0; h < V / 4; ++h) part[w][h] = *reinterpret_cast<const float4 *>(&sums[w * block + sum_at<BN>(p, c * (V / 4) + h)]);
#pragma unroll
    for (int h = 0; h < V / 4; ++h) {
        float4 s = part[0][h];
#pragma unroll
        for (int w = 1; w < WK; ++w) { s.x += part[w][h].x; s.y += part[w][h].y; s.z += part[w][h].z; s.w += part[w][h].w; }
        v[4 * h] = s.x; v[4 * h + 1] = s.y; v[4 * h + 2] = s.z; v[4 * h + 3] = s.w;
    }
}

// Split reduction: publishes this workgroup's partial sums; the last workgroup of the tile to arrive adds them in split order into acc, the
// others are done (false).  GT threads (the owners) hold the sums.  Device-coherent 16-byte accesses (sc1).
template <int BN, int BM, int GT, typename Acc, int TN, int TM>
__device__ __forceinline__ bool meet_splits(const OpArgs &a, Acc (&acc)[TN][TM], int *s_last, int tile, int z, bool owner, int gtid) {
    if (a.walk.split.d == 1) return true;
    constexpr int GROUPS = sizeof(Acc) / 16, SC1 = 16;
    const int parts = a.split_k;
    const __amdgpu_buffer_rsrc_t ws = __builtin_amdgcn_make_buffer_rsrc(a.ws + (int64_t)tile * parts * (BN * BM), 0, parts * (BN * BM * 4), 0x00027000);
    if (owner) {
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int g = 0; g < GROUPS; ++g) {
                    const f32x4 v{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), ws, gtid * 16, z * (BN * BM * 4) + ((i * TM + j) * GROUPS + g) * (GT * 16), SC1);
                }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned old = __hip_atomic_fetch_add(&a.counters[tile], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *s_last = (old == (unsigned)parts - 1u);
    }
    __syncthreads();
    if (!*s_last) return false;
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = Acc{};
    constexpr int AT_ONCE = TN * TM * GROUPS <= 4 ? 4 : 1; // parts whose loads are in flight together
    for (int z0 = 0; owner && z0 < parts; z0 += AT_ONCE) {
        u32x4 part[AT_ONCE][TN][TM][GROUPS];
#pragma unroll
        for (int b = 0; b < AT_ONCE; ++b)
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int j = 0; j < TM; ++j)
#pragma unroll
                    for (int g = 0; g < GROUPS; ++g)
                        part[b][i][j][g] = __builtin_amdgcn_raw_buffer_load_b128(ws, gtid * 16, min(z0 + b, parts - 1) * (BN * BM * 4) + ((i * TM + j) * GROUPS + g) * (GT * 16), SC1);
#pragma unroll
        for (int b = 0; b < AT_ONCE; ++b) {
            if (z0 + b >= parts) continue;
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int j = 0; j < TM; ++j)
#pragma unroll
                    for (int g = 0; g < GROUPS; ++g)
#pragma unroll
                        for (int t = 0; t < 4; ++t) acc[i][j][4 * g + t] += __uint_as_float(part[b][i][j][g][t]);
        }
    }
    if (threadIdx.x == 0) __hip_atomic_store(&a.counters[tile], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

// Bias, residual, activation and store straight from the accumulators, for channel counts and offsets that 16-byte pieces do not fit.
// k0: first channel of the wave's products; m: output pixel of this lane in each of them, negative for none.
template <typename T, int MF, typename Acc, int TN, int TM>
__device__ __forceinline__ void store_lanes(const OpArgs &a, const Acc (&acc)[TN][TM], int k0, const int (&m)[TM], int fgrp) {
    const Results y = results_in(a.y);
    const T *res = (const T *)a.res;
    const bool vec_ok = (a.y_ct % 4 == 0) && (a.y_coff % 4 == 0) && (a.res_ct % 4 == 0);
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) {
            if (m[j] < 0) continue;
#pragma unroll
            for (int g = 0; g < (MF == 32 ? 4 : 1); ++g) {
                const int k = k0 + i * MF + ((MF == 32) ? (8 * g + 4 * fgrp) : (4 * fgrp));
                if (k >= a.K) continue;
                const float4 b = *reinterpret_cast<const float4 *>(a.bias + k);    // padded to n_pad
                float v[4] = {acc[i][j][g * 4] + b.x, acc[i][j][g * 4 + 1] + b.y, acc[i][j][g * 4 + 2] + b.z, acc[i][j][g * 4 + 3] + b.w};
                if (vec_ok && k + 4 <= a.K) {
                    if (res) {
                        float rv[4];
                        load_pack<T, 4>(res + (int64_t)m[j] * a.res_ct + k, rv);
#pragma unroll
                        for (int t = 0; t < 4; ++t) v[t] += rv[t];
                    }
#pragma unroll
                    for (int t = 0; t < 4; ++t) v[t] = apply_act(v[t], a.act);
                    store_pack<T, 4>(y, (uint32_t)m[j] * (uint32_t)a.y_ct + (uint32_t)(a.y_coff + k), v);
                } else {
                    for (int t = 0; t < 4 && k + t < a.K; ++t) {
                        float f = v[t];
                        if (res) f += to_f32(res[(int64_t)m[j] * a.res_ct + k + t]);
                        store_one<T>(y, (uint32_t)m[j] * (uint32_t)a.y_ct + (uint32_t)(a.y_coff + k + t), apply_act(f, a.act));
                    }
                }
            }
        }
}

// The wide forms of the 16-bit types: a wave finishes its CT x TM products of 32 channels x 32 pixels by itself.  Bias, residual and
// activation in the layout of the accumulators, one rounding, and 32 pixels at a time through a block of LDS of its own, so that
// every store is a row of channels; no barrier.  The residual takes the same way in the other direction.  Through an fp32 tile in LDS that
// all waves write and read, with bias and residual fetched in between and a branch on pooling and residual at every four channels, this took
// 2.3 to 4.2 us of a workgroup's time and 200 to 234 registers; 1.1 us (2 with a residual) here, and 171 registers on the 128x128 tile, 184 and
// 230 on the 128-wide patches.  ResNet-50 at batch 64 1412 -> 1387 us, eight at batch 16 2610 -> 2572, on disjoint eighths of the units
// 6135 -> 6010, ResNet-101 with three others at one image 514 -> 501.
// m_lane: output pixel of row lane % 32 of each 32 pixels, negative for rows without one; pooling: the pooled pixel.
template <typename T, int CT, int TM>
struct WaveTile {
    static constexpr int COLS = 32 * CT, SLD = COLS + 8, LPR = COLS / 8, RPI = 64 / LPR, IT = 32 / RPI;   // staging row; lanes a row; rows and accesses
    static constexpr int BYTES = 32 * SLD * 2;
    int m_lane[TM];
    uint32_t k;                               // channel of this lane's 16-byte piece
    u32x4 res[TM][IT];

    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void *p, uint32_t bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000);
    }
    __device__ __forceinline__ void load_res(const OpArgs &a, int lane) {
        const __amdgpu_buffer_rsrc_t r = buffer(a.res, a.walk.pixels * (uint32_t)a.res_ct * 2u);
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int m = __shfl(m_lane[j], lane / LPR + RPI * it);
                res[j][it] = __builtin_amdgcn_raw_buffer_load_b128(r, m >= 0 && k < (uint32_t)a.K ? ((uint32_t)m * (uint32_t)a.res_ct + k) * 2u : OUT_OF_RANGE, 0, 0);
            }
    }
    static __device__ __forceinline__ void fence() {      // the block is the wave's own and LDS serves its accesses in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // Residual and pooling are decided once: a branch at every four channels keeps the compiler from having several accesses to LDS under way.
    template <bool RES, bool POOL, typename Acc>
    __device__ __forceinline__ void finish_as(const OpArgs &a, const Acc (&acc)[CT][TM], uint16_t *sg, const float *bias, int lane) {
        const int frow = lane & 31, fgrp = lane >> 5, srow = lane / LPR, scol = (lane % LPR) * 8;
        const __amdgpu_buffer_rsrc_t out = buffer(a.y, (POOL ? a.walk.pixels / 4 : a.walk.pixels) * (uint32_t)a.y_ct * 2u);
        auto store = [&](int row, int m) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(&sg[row * SLD + scol]);
            __builtin_amdgcn_raw_buffer_store_b128(v, out, m >= 0 && k < (uint32_t)a.K ? ((uint32_t)m * (uint32_t)a.y_ct + (uint32_t)a.y_coff + k) * 2u : OUT_OF_RANGE, 0, THROUGH);
        };
        float4 b[CT][4];
#pragma unroll
        for (int i = 0; i < CT; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g) b[i][g] = *reinterpret_cast<const float4 *>(&bias[i * 32 + 8 * g + 4 * fgrp]);
        uint16_t *mine = &sg[(POOL ? frow >> 2 : frow) * SLD + 4 * fgrp];
#pragma unroll
        for (int j = 0; j < TM; ++j) {
            Pack<T, 4> r[CT][4];
            if (RES) {
#pragma unroll
                for (int it = 0; it < IT; ++it) *reinterpret_cast<u32x4 *>(&sg[(srow + RPI * it) * SLD + scol]) = res[j][it];
                fence();
#pragma unroll
                for (int i = 0; i < CT; ++i)
#pragma unroll
                    for (int g = 0; g < 4; ++g) r[i][g] = *reinterpret_cast<const Pack<T, 4> *>(&mine[i * 32 + 8 * g]);
            }
            Pack<T, 4> o[CT][4];
#pragma unroll
            for (int i = 0; i < CT; ++i)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    float v[4] = {acc[i][j][g * 4] + b[i][g].x, acc[i][j][g * 4 + 1] + b[i][g].y, acc[i][j][g * 4 + 2] + b[i][g].z, acc[i][j][g * 4 + 3] + b[i][g].w};
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        if (RES) v[t] += to_f32(r[i][g].e[t]);
                        if (POOL) {                        // the maximum over the four lanes of a window; without a number there is none
                            v[t] = fmaxf(v[t], -INFINITY);
                            v[t] = fmaxf(v[t], __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v[t]), 0xB1, 0xf, 0xf, true)));
                            v[t] = fmaxf(v[t], __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v[t]), 0x4E, 0xf, 0xf, true)));
                        }
                        from_f32(apply_act(v[t], a.act), o[i][g].e[t]);
                    }
                }
            if (!POOL || (frow & 3) == 0) {
#pragma unroll
                for (int i = 0; i < CT; ++i)
#pragma unroll
                    for (int g = 0; g < 4; ++g) *reinterpret_cast<Pack<T, 4> *>(&mine[i * 32 + 8 * g]) = o[i][g];
            }
            fence();
            if (POOL) {
                const int m = __shfl(m_lane[j], (srow & 7) * 4);
                if (RPI == 8 || srow < 8) store(srow, m);
            } else {
#pragma unroll
                for (int it = 0; it < IT; ++it) store(srow + RPI * it, __shfl(m_lane[j], srow + RPI * it));
            }
            fence();
        }
    }
    template <typename Acc>
    __device__ __forceinline__ void finish(const OpArgs &a, const Acc (&acc)[CT][TM], uint16_t *sg, const float *bias, int lane) {
        if (a.pool2) finish_as<false, true>(a, acc, sg, bias, lane);
        else if (a.res != nullptr) {
            load_res(a, lane);
            finish_as<true, false>(a, acc, sg, bias, lane);
        }
        else finish_as<false, false>(a, acc, sg, bias, lane);
    }
};

// What follows the main loop otherwise: the wave groups' partial sums meet, then those of the workgroups that share the tile, then
// bias, residual, activation, one rounding and the store.  pixel(ml) is the output pixel of tile row ml (the pooled pixel
// of its window when the epilogue pools), negative for rows without one.
template <typename T, int BN, int BM, int WN, int WM, int WK, int MF, typename Acc, int TN, int TM, typename Pixel>
__device__ __forceinline__ void finish_tile(const OpArgs &a, Acc (&acc)[TN][TM], uint8_t *smem, int *s_last, int n0, int tile, int z, Pixel pixel) {
    constexpr int GT = 64 * WN * WM, NT = GT * WK;
    constexpr int SUBN = BN / WN, SUBM = BM / WM, ACC = MF == 32 ? 16 : 4, GROUPS = ACC / 4, ELD = BN + 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wk = wave / (WN * WM), wn = (wave % (WN * WM)) % WN, wm = (wave % (WN * WM)) / WN;
    const int frow = lane % MF, fgrp = lane / MF;

    // ---- wave groups: groups 1 .. WK-1 hand their accumulators to group 0, which adds them in group order
    const bool owner = wk == 0;
    const int gtid = tid % GT;
    constexpr int NACC = TN * TM * ACC;
    if constexpr (WK > 1) {
        float *red = reinterpret_cast<float *>(&smem[0]);
        if (!owner) {
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int j = 0; j < TM; ++j)
#pragma unroll
                    for (int g = 0; g < GROUPS; ++g)
                        *reinterpret_cast<float4 *>(&red[(((wk - 1) * (NACC / 4) + (i * TM + j) * GROUPS + g) * GT + gtid) * 4]) =
                            make_float4(acc[i][j][g * 4], acc[i][j][g * 4 + 1], acc[i][j][g * 4 + 2], acc[i][j][g * 4 + 3]);
        }
        __syncthreads();
        if (owner) {
            for (int w = 1; w < WK; ++w)
#pragma unroll
                for (int i = 0; i < TN; ++i)
#pragma unroll
                    for (int j = 0; j < TM; ++j)
#pragma unroll
                        for (int g = 0; g < GROUPS; ++g) {
                            const float4 v = *reinterpret_cast<const float4 *>(&red[(((w - 1) * (NACC / 4) + (i * TM + j) * GROUPS + g) * GT + gtid) * 4]);
                            acc[i][j][g * 4] += v.x; acc[i][j][g * 4 + 1] += v.y; acc[i][j][g * 4 + 2] += v.z; acc[i][j][g * 4 + 3] += v.w;
                        }
        }
    }

    if (!meet_splits<BN, BM, GT>(a, acc, s_last, tile, z, owner, gtid)) return;

    // ---- epilogue: bias, residual, activation, one rounding, NHWC store
    const Results y = results_in(a.y);
    const T *res = (const T *)a.res;
    const bool vec8_ok = (a.K % 8 == 0) && (a.y_ct % 8 == 0) && (a.y_coff % 8 == 0) && (a.res_ct % 8 == 0);
    if (vec8_ok) {
        float *et = reinterpret_cast<float *>(&smem[0]);
        constexpr int CPR = BN / 8;
        constexpr int EP_IT = (BM * CPR + NT - 1) / NT;
        // (16-bit types: a register quad, not a struct, which costs the wide tiles 12 to 32 registers and the tenants beside them 2 %)
        typedef std::conditional_t<sizeof(T) == 2, u32x4, Pack<T, 8>> Raw;
        static_assert(NT % CPR == 0, "a thread stores the same channels of several pixels");
        float bias[8];
        const int k = n0 + (tid % CPR) * 8;
        *reinterpret_cast<float4 *>(&bias[0]) = *reinterpret_cast<const float4 *>(a.bias + k);     // padded to n_pad
        *reinterpret_cast<float4 *>(&bias[4]) = *reinterpret_cast<const float4 *>(a.bias + k + 4);
        Raw res_raw[EP_IT];
        const bool add_res = res != nullptr && !a.pool2;
        if (add_res) {
#pragma unroll
            for (int it = 0; it < EP_IT; ++it) {
                const int c = tid + it * NT;
                const int m = pixel(min(c / CPR, BM - 1));
                const bool live = (c < BM * CPR) & (m >= 0) & (k < a.K);
                res_raw[it] = live ? *reinterpret_cast<const Raw *>(res + (int64_t)m * a.res_ct + k) : Raw{};
            }
        }
        __syncthreads();
        if (owner) {
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int j = 0; j < TM; ++j)
#pragma unroll
                    for (int g = 0; g < GROUPS; ++g) {
                        const int ml = wm * SUBM + j * MF + frow;
                        const int kl = wn * SUBN + i * MF + ((MF == 32) ? (8 * g + 4 * fgrp) : (4 * fgrp));
                        *reinterpret_cast<float4 *>(&et[ml * ELD + kl]) =
                            make_float4(acc[i][j][g * 4 + 0], acc[i][j][g * 4 + 1], acc[i][j][g * 4 + 2], acc[i][j][g * 4 + 3]);
                    }
        }
        __syncthreads();
        if (a.pool2) {
            for (int c = tid; c < (BM / 4) * CPR; c += NT) {
                const int r4 = c / CPR, col = (c % CPR) * 8;
                const int m = pixel(r4 * 4);
                if (m < 0 || k >= a.K) continue;
                float v[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) v[t] = -INFINITY;
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const float4 lo = *reinterpret_cast<const float4 *>(&et[(r4 * 4 + rr) * ELD + col]);
                    const float4 hi = *reinterpret_cast<const float4 *>(&et[(r4 * 4 + rr) * ELD + col + 4]);
                    v[0] = fmaxf(v[0], lo.x); v[1] = fmaxf(v[1], lo.y); v[2] = fmaxf(v[2], lo.z); v[3] = fmaxf(v[3], lo.w);
                    v[4] = fmaxf(v[4], hi.x); v[5] = fmaxf(v[5], hi.y); v[6] = fmaxf(v[6], hi.z); v[7] = fmaxf(v[7], hi.w);
                }
#pragma unroll
                for (int t = 0; t < 8; ++t) v[t] = apply_act(v[t] + bias[t], a.act);
                store_pack<T, 8>(y, (uint32_t)m * (uint32_t)a.y_ct + (uint32_t)(a.y_coff + k), v);
            }
            return;
        }
#pragma unroll
        for (int it = 0; it < EP_IT; ++it) {
            const int c = tid + it * NT;
            const int row = c / CPR, col = (c % CPR) * 8;
            const int m = pixel(min(row, BM - 1));
            if (c >= BM * CPR || m < 0 || k >= a.K) continue;
            float v[8];
            const float4 lo = *reinterpret_cast<const float4 *>(&et[row * ELD + col]);
            const float4 hi = *reinterpret_cast<const float4 *>(&et[row * ELD + col + 4]);
            v[0] = lo.x; v[1] = lo.y; v[2] = lo.z; v[3] = lo.w; v[4] = hi.x; v[5] = hi.y; v[6] = hi.z; v[7] = hi.w;
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t] += bias[t];
            if (add_res) {
                const Pack<T, 8> rp = __builtin_bit_cast(Pack<T, 8>, res_raw[it]);
#pragma unroll
                for (int t = 0; t < 8; ++t) v[t] += to_f32(rp.e[t]);
            }
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t] = apply_act(v[t], a.act);
            store_pack<T, 8>(y, (uint32_t)m * (uint32_t)a.y_ct + (uint32_t)(a.y_coff + k), v);
        }
        return;
    }
    if (!owner) return;
    int m[TM];
#pragma unroll
    for (int j = 0; j < TM; ++j) m[j] = pixel(wm * SUBM + j * MF + frow);
    store_lanes<T, MF>(a, acc, n0 + wn * SUBN, m, fgrp);
}

// Image and top left input pixel of the window of output pixel m (walked window by window when the epilogue pools).
__device__ __forceinline__ void window_origin(const OpArgs &a, uint32_t m, int &n, int &ih0, int &iw0) {
    const uint32_t mq = a.pool2 ? m >> 2 : m;
    n = (int)divide(mq, a.walk.pq);
    const uint32_t rem = mq - (uint32_t)n * a.walk.pq.d;
    int p = (int)divide(rem, a.walk.q);
    int q = (int)(rem - (uint32_t)p * a.walk.q.d);
    if (a.pool2) {
        p = 2 * p + (int)((m >> 1) & 1u);
        q = 2 * q + (int)(m & 1u);
    }
    ih0 = p * a.sh - a.ph;
    iw0 = q * a.sw - a.pw;
}

// Bit r: filter row r reads inside the image for this pixel; bit 16 + s: so does filter column s.
__device__ __forceinline__ uint32_t window_mask(const OpArgs &a, int ih0, int iw0) {
    auto range = [](int first, int extent, int window) {
        const int lo = min(max(-first, 0), window), hi = min(max(extent - first, 0), window);
        return ((1u << hi) - 1u) & ~((1u << lo) - 1u);
    };
    return range(ih0, a.H, a.R) | range(iw0, a.W, a.S) << 16;
}

// A workgroup's arguments, all in one trip.  fetch_walk only asks for them together and leaves the compiler free to keep what it likes; held, they are two trips
// in the kernels of one operator with narrow tiles (the scalar registers run out).  us a layer, f16, asked for together / held: 1x7 192 -> 192 on 17 x 17 (ring)
// 3.46 / 3.57, 3x3 256 -> 256 on 16 x 14 x 14 (64x64 patch) 8.61 / 8.69, 512 -> 512 on 8 x 14 x 14 13.15 / 13.29; rings on rectangles as much either way; 128x64 patch
// 128 -> 128 on 112 x 112 7.55 / 7.51, on 16 x 28 x 28 7.61 / 7.57.  Launches of several operators hold them as well, for 0.3 % less: eight ResNet-50 at batch 16, two to a
// launch, 2178 / 2183 us a pass.
__device__ __forceinline__ void fetch_walk(const OpArgs &a) {
    const TileWalk &w = a.walk;
    asm volatile("" ::"s"(a.x), "s"(a.w), "s"(w.total), "s"(w.per_xcd), "s"(w.pixels), "s"(w.x_bytes), "s"(w.w_bytes), "s"(w.flat), "s"(w.units), "s"(w.per),
                 "s"(w.split.d), "s"(w.split.m), "s"(w.tiles.d), "s"(w.tiles.m), "s"(w.tiles.s1), "s"(w.tiles.s2), "s"(w.pq.d), "s"(w.pq.m), "s"(w.pq.s1), "s"(w.pq.s2),
                 "s"(w.q.d), "s"(w.q.m), "s"(w.q.s1), "s"(w.q.s2), "s"(a.tile_order), "s"(a.pool2), "s"(a.k_pad), "s"(a.x_ct), "s"(a.x_coff), "s"(a.H));
    asm volatile("" ::"s"(w.c.d), "s"(w.c.m), "s"(w.c.s1), "s"(w.c.s2), "s"(w.adv_t), "s"(w.adv_c), "s"(w.inv_s), "s"(a.W), "s"(a.C), "s"(a.R), "s"(a.S), "s"(a.sh), "s"(a.sw),
                 "s"(a.ph), "s"(a.pw), "s"(a.N), "s"(a.P), "s"(a.Q), "s"(a.panel), "s"(a.prio), "s"(a.K), "s"(a.res_ct), "s"(a.y_coff), "s"(a.y_ct), "s"(a.bias), "s"(a.res));
}
// The same for ring_patch_body: fewer, so that they are one trip there too (with the ones above the compiler ran out of scalar registers
// and asked for the epilogue's in a second trip, 0.1 us).
__device__ __forceinline__ void fetch_rect_walk(const OpArgs &a) {
    const TileWalk &w = a.walk;
    asm volatile("" ::"s"(a.x), "s"(a.w), "s"(w.total), "s"(w.per_xcd), "s"(w.x_bytes), "s"(w.w_bytes), "s"(w.units), "s"(w.tiles.d), "s"(w.tiles.m), "s"(w.tiles.s1), "s"(w.tiles.s2),
                 "s"(w.pq.d), "s"(w.pq.m), "s"(w.pq.s1), "s"(w.pq.s2), "s"(w.q.d), "s"(w.q.m), "s"(w.q.s1), "s"(w.q.s2), "s"(a.tile_order), "s"(a.pool2), "s"(a.x_ct), "s"(a.x_coff), "s"(a.H),
                 "s"(a.W), "s"(a.P), "s"(a.Q), "s"(a.panel), "s"(a.prio));
    asm volatile("" ::"s"(a.K), "s"(a.res_ct), "s"(a.y_coff), "s"(a.y_ct), "s"(a.bias), "s"(a.res));
}
// TAPS: the window has more than one tap, or the map is walked image by image
template <bool TAPS>
__device__ __forceinline__ void hold_walk(OpArgs &a) {
    TileWalk &w = a.walk;
    hold(a.x, a.w, w.total, w.per_xcd, w.pixels, w.x_bytes, w.w_bytes, w.flat, w.units, w.per, w.split.d, w.split.m, w.split.s1, w.split.s2, w.tiles.d, w.tiles.m, w.tiles.s1, w.tiles.s2,
         w.pq.d, w.pq.m, w.pq.s1, w.pq.s2, w.q.d, w.q.m, w.q.s1, w.q.s2, a.tile_order, a.pool2, a.k_pad, a.x_ct, a.x_coff, a.H, a.W, a.sh, a.sw, a.ph, a.pw, a.prio, a.K, a.res_ct, a.y_coff, a.y_ct, a.bias, a.res);
    if constexpr (TAPS) hold(w.c.d, w.c.m, w.c.s1, w.c.s2, w.adv_t, w.adv_c, w.inv_s, a.C, a.R, a.S);
    else hold(a.gemm_k);
}

// Tiles of the 16-bit types whose filters are packed in operand order and go straight to registers, a kilobyte a load and requested as many stages ahead
// as pixels; waves share a tile such that no filter is loaded twice.  With both operands in LDS these tiles spend three to four times as many cycles on LDS
// as on matrix instructions and leave room for one or two workgroups a unit.  A wait for filters leaves the (NBUF - 1) * W youngest requests under way, and as the
// compiler does not count requests for pixels these are the pixels and filters of fewer stages: one to two of the two to four.  us a layer, both in LDS / this, f16:
//   128x64   1x1 512 -> 512 on 16 x 14 x 14  6.31 / 5.88     1x1 768 -> 768 on 5 x 17 x 17  7.52 / 6.74     3x3, stride 2, 192 -> 384 on 8 x 27 x 27  20.1 / 16.8
//   64x64    1x1 1024 -> 256 on 16 x 14 x 14  8.04 / 7.84 (a pass of one layer)     2048 -> 512 on 32 x 7 x 7  11.2 / 10.3
//            1x1 256 -> 256 on 16 x 14 x 14   3.85 / 4.25, 512 -> 256 6.24 / 6.66 alone: four groups of waves have twice the sums to exchange.  But beside others these
//            gain as well: four ResNet-50 at batch 4, us a pass, 625 with both in LDS up to 640 elements, 588 without.
// Eight ResNet-50 at batch 16, us a pass: 2467 with both in LDS, 2210 so (patches with packed filters included).  128x128 tiles lose: 1x1 1024 -> 1024 on 16 x 14 x 14
// 12.4 / 11.0, but ResNet-50 at batch 64 1278 / 1290, eight at batch 16 2234 / 2314.  64x64 of short reductions (one row a stage) and 64x32 are no matter of course: 64 -> 256 on
// 56 x 56 2.89 / 3.18; 2048 -> 512 on 16 x 7 x 7 9.16 / 8.32 and 512 -> 512 4.18 / 4.39.
constexpr bool filters_packed(int bn, int bm, int kd) { return (bn == 128 && bm == 64) || (bn == 64 && bm == 64 && kd == 2); }

// This workgroup's tile, as (channel tile, pixel tile), and its part of a split reduction.  False: a workgroup without work.
// slot: position in the XCD's range of tiles.
__device__ __forceinline__ bool find_tile(const OpArgs &a, uint32_t slot, int &tile, int &z, int &tn_idx, int &tm_idx) {
    const TileWalk &w = a.walk;
    const uint32_t vid = (blockIdx.x % XCDS) * w.per_xcd + slot;
    if (vid >= w.total) return false;
    const uint32_t t = w.split.d == 1 ? vid : divide(vid, w.split);
    z = (int)(vid - t * w.split.d);
    tile = (int)t;
    const int slow = (int)divide(t, w.tiles), fast = (int)(t - (uint32_t)slow * w.tiles.d);
    tn_idx = a.tile_order ? slow : fast;
    tm_idx = a.tile_order ? fast : slow;
    return true;
}

// BN output channels x BM pixels per workgroup; WN x WM waves over the tile, WK such groups that share the reduction;
// KD 64-deep slices of the reduction per stage, NBUF stages in LDS.
template <typename T, int BN, int BM, int WN, int WM, int WK, int KD, int NBUF, int MODE, bool HELD, int ROOM = 0>
__device__ __forceinline__ void tile_body(const OpArgs &args, uint32_t slot) {
    OpArgs a = args;
    if constexpr (HELD) hold_walk<MODE != TG_POINT>(a);
    else fetch_walk(a);
    set_wave_priority(a.prio);
    constexpr int NW = WN * WM * WK;
    constexpr int SUBN = BN / WN, SUBM = BM / WM;
    constexpr int MF = (SUBN % 32 == 0 && SUBM % 32 == 0) ? 32 : 16;
    constexpr int TN = SUBN / MF, TM = SUBM / MF;
    static_assert(TN >= 1 && TM >= 1, "wave tile smaller than one matrix instruction");
    constexpr int ES = sizeof(T), RK = ROW<T>, EPP = 16 / ES;   // bytes of an element, elements of an LDS row and of a 16-byte piece
    constexpr int PPS = MF == 32 ? 2 : 4;                  // pieces of a row per step
    constexpr int STEPS = KD * 8 / PPS;                    // steps per stage
    static_assert(STEPS % WK == 0, "the wave groups share a stage evenly");
    constexpr int MY_STEPS = STEPS / WK;
    constexpr int ACC = MF == 32 ? 16 : 4;
    constexpr bool PACKED = ES == 2 && filters_packed(BN, BM, KD);     // filters go straight to registers
    constexpr int W = MY_STEPS * TN, SETS = NBUF - 1;      // such loads of a wave per stage, stages of them in registers
    constexpr int WQ = PACKED ? 0 : KD * BN / 8 / NW, XQ = KD * BM / 8 / NW;   // loads of a wave to LDS per stage: 8 rows of 128 bytes each
    static_assert((PACKED || WQ * NW * 8 == KD * BN) && XQ * NW * 8 == KD * BM, "the waves share the loads of a stage evenly");
    static_assert(!PACKED || WM == 1, "no filter is loaded twice");
    constexpr int L = PACKED ? W + XQ : WQ + XQ;
    constexpr int W_BYTES = PACKED ? 0 : KD * BN * 128, X_BYTES = KD * BM * 128, STAGE = W_BYTES + X_BYTES;
    constexpr bool WIDE = ES == 2 && MF == 32 && WK == 1;  // every wave finishes its own part of the tile
    constexpr int RED_BYTES = (WK > 1 ? WK : 0) * BN * BM * 4, EP_BYTES = WIDE ? NW * WaveTile<T, TN, TM>::BYTES : BM * (BN + 4) * 4;
    constexpr int COUNTED = ROOM > 0 ? 160 * 1024 / (ROOM + 1) + 1 : 0;      // a compute unit holds no more workgroups than are counted on
    constexpr int BIAS = std::max({NBUF * STAGE, RED_BYTES, EP_BYTES, COUNTED + 15 & ~15}), LDS_BYTES = BIAS + (WIDE ? BN * 4 : 0);
    typedef typename Mma<T, MF>::Acc Acc;
    __shared__ __attribute__((aligned(1024))) uint8_t smem[LDS_BYTES];
    __shared__ int s_last;

    int tid = threadIdx.x;
    if (ROOM > 0) asm volatile("" : "+v"(tid));            // what a lane's place decides is worked out for every tile: kept, it is more registers than there are
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave / (WN * WM), wn = (wave % (WN * WM)) % WN, wm = (wave % (WN * WM)) / WN;
    const int frow = lane % MF, fgrp = lane / MF;          // operand row and reduction group of this lane

    int tile, z, tn_idx, tm_idx;
    if (!find_tile(a, slot, tile, z, tn_idx, tm_idx)) return;
    const int M = (int)a.walk.pixels;
    const int n0 = tn_idx * BN, m0 = tm_idx * BM;

    // Epilogue of this form: from the accumulators themselves where a wave has one 16 x 16 product, from the sums in LDS where wave groups
    // share the reduction.  Bias and residual are requested ahead of the operands (in front of them, so that the waits of the
    // reduction count the same loads) if a thread has one piece of the tile to store.
    constexpr bool DIRECT = WK == 1 && MF == 16 && TN == 1 && TM == 1, SUMS = WK > 1;
    constexpr int NT = 64 * NW, V = !DIRECT && ES == 2 && BN * BM >= 8 * NT ? 8 : 4, PIECES = BN / V, STORING = DIRECT ? NT : std::min(NT, BN * BM / V);
    constexpr int EP_IT = DIRECT ? 1 : BN * BM / V / STORING;
    constexpr bool AHEAD = DIRECT || (SUMS && EP_IT == 1);
    const bool unsplit = a.walk.split.d == 1, vec_ok = whole_packs<V>(a), storing = STORING == NT || tid < STORING;
    auto pixel = [&](int ml) {
        const int m = m0 + ml;
        return m < M ? (a.pool2 ? m >> 2 : m) : -1;
    };
    auto my_row = [&](int it) { return DIRECT ? frow : (tid + it * NT) / PIECES; };
    const int my_k = n0 + (DIRECT ? wn * 16 + 4 * fgrp : (tid % PIECES) * V);
    Addend<T, V> add;
    if (AHEAD && unsplit && storing) add.load(a, pixel(my_row(0)), my_k, vec_ok);
    if (WIDE && wave < BN / 64)
        load_words_to_lds(raw_buffer(a.bias, (uint32_t)(n0 + BN) * 4u), (uint32_t)(n0 + lane) * 4u, (uint32_t)wave * 256u,
                          (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem + BIAS + (uint32_t)wave * 256u);

    const int st0 = z * (int)a.walk.per;
    const int ns = min((int)a.walk.units, st0 + (int)a.walk.per) - st0;

    const int XS = a.x_ct;
    const T *x = (const T *)a.x + a.x_coff;
    const u32x4 rsrc_x = raw_buffer(x, a.walk.x_bytes - (uint32_t)a.x_coff * ES);
    const u32x4 rsrc_w = raw_buffer(a.w, a.walk.w_bytes);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;

    // A load covers 8 rows; lane l delivers 16-byte column l % 8 of row l / 8.  Column c of LDS row r holds piece
    // c ^ (r / 2 % 8) of that row: 16 lanes reading one piece of 16 rows touch each of the 64 banks once.  The groups of 8
    // rows a wave loads are all even or all odd, as the wave is.
    static_assert(NW % 2 == 0 && BN % 16 == 0 && BM % 16 == 0, "a wave's row groups have one parity");
    const int lrow = lane >> 3, piece = (lane & 7) ^ ((wave & 1) * 4 + (lrow >> 1));

    const uint32_t wv = (uint32_t)((n0 + lrow) * a.k_pad + piece * EPP) * ES;
    uint32_t ws[std::max(WQ, 1)];                          // scalar part of each filter load
#pragma unroll
    for (int i = 0; i < WQ; ++i) {
        const int q = i * NW + wave, kd = q / (BN / 8), rg = q % (BN / 8);
        ws[i] = (uint32_t)(rg * 8 * a.k_pad + (st0 * KD + kd) * RK) * ES;
    }
    // Packed filters: [32 channels][row of 64 elements][16 elements][lane][16 bytes]
    const __amdgpu_buffer_rsrc_t packed = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w), 0, (int)a.walk.w_bytes, 0x00027000);
    uint32_t wtile[TN];                                    // this wave's part of the stage requested next, per 32 channels
#pragma unroll
    for (int i = 0; i < TN; ++i) wtile[i] = (uint32_t)(((n0 / 32 + wn * TN + i) * (a.k_pad / TK) + st0 * KD) * 4 + wk * MY_STEPS) * 1024u;
    u32x4 w[PACKED ? SETS : 1][MY_STEPS][TN];
    auto load_filters = [&](int set, int step, uint32_t voff) {
#pragma unroll
        for (int i = 0; i < TN; ++i) {
            w[set][step][i] = __builtin_amdgcn_raw_buffer_load_b128(packed, voff + (uint32_t)(step % 4) * 1024u, wtile[i] + (uint32_t)(step / 4) * 4096u, 0);
            if (step == MY_STEPS - 1) wtile[i] += KD * 4096;
        }
    };
    constexpr int NP = KD == 1 ? 1 : XQ;                   // positions along j tracked (loads of one 64-slice share one)
    constexpr bool PIECEWISE = MODE == TG_CHUNK || MODE == TG_FAR;   // every 16-byte piece has a tap of its own
    uint32_t xoff[XQ], xmask[XQ];
    int first_row[XQ], first_col[XQ];                      // TG_FAR: first row and column of the window
    int ptap[NP], pch[NP];                                 // tap and channel of each position (TG_TAP: wave-uniform)
    uint32_t xs = (uint32_t)(st0 * KD) * 128u;          // TG_POINT: scalar offset
    const uint32_t x_end = (uint32_t)a.gemm_k * ES;
#pragma unroll
    for (int i = 0; i < XQ; ++i) {
        const int q = i * NW + wave, kd = q / (BM / 8), rg = q % (BM / 8);
        const int m = m0 + rg * 8 + lrow;
        const bool ok = m < M;
        int n = 0, ih0 = 0, iw0 = m;
        if (MODE != TG_POINT || !a.walk.flat) window_origin(a, ok ? (uint32_t)m : 0u, n, ih0, iw0);
        xoff[i] = (uint32_t)(((n * a.H + ih0) * a.W + iw0) * XS + (PIECEWISE ? 0 : piece * EPP)) * ES;
        if constexpr (MODE == TG_POINT) {
            xoff[i] = ok ? xoff[i] + (uint32_t)(kd * 128) : OUT_OF_RANGE;
        } else if constexpr (MODE == TG_FAR) {
            first_row[i] = ok ? ih0 : INT32_MIN / 2;            // beyond the last pixel: outside the image at every tap
            first_col[i] = iw0;
        } else {
            xmask[i] = ok ? window_mask(a, ih0, iw0) : 0u;
        }
        if (MODE != TG_POINT && i < NP) {
            const int j0 = (st0 * KD + (KD == 1 ? 0 : kd)) * RK + (PIECEWISE ? piece * EPP : 0);
            ptap[i] = (int)divide((uint32_t)j0, a.walk.c);
            pch[i] = j0 - ptap[i] * a.C;
        }
    }
    const int adv_t = (int)a.walk.adv_t, adv_c = (int)a.walk.adv_c;
    const uint32_t inv_s = a.walk.inv_s;

    auto issue = [&](int buf, bool some = true) {           // some: false for a stage beyond the reduction
        const uint32_t base = lds0 + (uint32_t)(buf * STAGE);
#pragma unroll
        for (int i = 0; i < WQ; ++i) {
            load_to_lds(rsrc_w, wv, ws[i], base + (uint32_t)((i * NW + wave) * 1024));
            ws[i] += KD * 128;
        }
        uint32_t toff[NP], trow[NP], tcol[NP];
        if constexpr (MODE != TG_POINT) {
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int tr = a.S == 1 ? ptap[i] : (int)__umulhi((uint32_t)ptap[i], inv_s);
                const int tc = ptap[i] - tr * a.S;
                toff[i] = (uint32_t)((tr * a.W + tc) * XS + pch[i]) * ES;
                if constexpr (MODE == TG_FAR) {
                    trow[i] = (uint32_t)(tr < a.R ? tr : INT32_MIN / 2);   // beyond the window: outside every image
                    tcol[i] = (uint32_t)tc;
                } else {
                    trow[i] = (uint32_t)min(tr, 15);       // beyond the window (padding of the reduction): a bit that is never set
                    tcol[i] = (uint32_t)(16 + tc);
                }
                ptap[i] += adv_t;
                pch[i] += adv_c;
                const bool carry = pch[i] >= a.C;
                pch[i] -= carry ? a.C : 0;
                ptap[i] += carry ? 1 : 0;
            }
        }
#pragma unroll
        for (int i = 0; i < XQ; ++i) {
            const uint32_t dst = base + (uint32_t)(W_BYTES + (i * NW + wave) * 1024);
            if constexpr (MODE == TG_POINT) {
                // Slices of the last stage that lie beyond the reduction (C is not a multiple of KD rows) hold the next pixel's channels:
                // the filters are zero there, but zero times infinity or NaN is NaN
                const uint32_t slice = (uint32_t)((i * NW + wave) / (BM / 8) * 128);
                load_to_lds(rsrc_x, some && (KD == 1 || xs + slice < x_end) ? xoff[i] : OUT_OF_RANGE, xs, dst);
            } else {
                const int pi = KD == 1 ? 0 : i;
                bool inside;
                if constexpr (MODE == TG_FAR) inside = ((uint32_t)first_row[i] + trow[pi] < (uint32_t)a.H) & ((uint32_t)first_col[i] + tcol[pi] < (uint32_t)a.W);
                else inside = (xmask[i] >> trow[pi]) & (xmask[i] >> tcol[pi]) & 1u;
                load_to_lds(rsrc_x, some && inside ? xoff[i] + toff[pi] : OUT_OF_RANGE, 0u, dst);
            }
        }
        xs += KD * 128;
    };

    Acc acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int v = 0; v < ACC; ++v) acc[i][j][v] = 0.f;

    struct Frag { u32x4 w[PACKED ? 1 : TN], x[TM]; };
    const uint32_t wrow = (uint32_t)((wn * SUBN + frow) * 128), xrow = (uint32_t)(W_BYTES + (wm * SUBM + frow) * 128);
    const uint32_t swz = (uint32_t)((frow >> 1) & 7);
    auto load_frag = [&](uint32_t buf, int s, Frag &f) {   // s: step of the stage
        const int kd = s / (8 / PPS), c0 = (s % (8 / PPS)) * PPS;
        const uint32_t col = ((uint32_t)(c0 + fgrp) ^ swz) * 16u;
#pragma unroll
        for (int i = 0; !PACKED && i < TN; ++i)
            f.w[PACKED ? 0 : i] = *reinterpret_cast<const u32x4 *>(&smem[buf + (uint32_t)(kd * BN * 128 + i * MF * 128) + wrow + col]);
#pragma unroll
        for (int j = 0; j < TM; ++j)
            f.x[j] = *reinterpret_cast<const u32x4 *>(&smem[buf + (uint32_t)(kd * BM * 128 + j * MF * 128) + xrow + col]);
    };
    // One stage; SET: where its packed filters are.  Those of the stage NBUF - 1 ahead, at voff, take their place step by step if there may be MORE.
    auto compute = [&]<int SET, bool MORE>(int buf, uint32_t voff) {
        const uint32_t b = (uint32_t)(buf * STAGE);
        Frag f[2];
        const int s0 = wk * MY_STEPS;
        load_frag(b, s0, f[0]);
#pragma unroll
        for (int s = 0; s < MY_STEPS; ++s) {
            if (s + 1 < MY_STEPS) load_frag(b, s0 + s + 1, f[(s + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);             // the next step's operands are requested before this one multiplies
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int j = 0; j < TM; ++j) acc[i][j] = Mma<T, MF>::run(PACKED ? w[SET][s][i] : f[s & 1].w[PACKED ? 0 : i], f[s & 1].x[j], acc[i][j]);
            if constexpr (PACKED && MORE) {
                __builtin_amdgcn_sched_barrier(0);
                load_filters(SET, s, voff);
            }
        }
    };

    int rbuf = 0, ibuf = NBUF - 1;
    if constexpr (PACKED) {
        // Stages beyond the reduction are requested out of range: with a branch around a request the compiler would not know how many are under way and
        // wait for all of them.
        auto filters_at = [&](int t) { return t < ns ? (uint32_t)lane * 16u : OUT_OF_RANGE; };
        [&]<int... S>(std::integer_sequence<int, S...>) {
            auto request = [&]<int SET>() {
                issue(SET, SET < ns);
#pragma unroll
                for (int s = 0; s < MY_STEPS; ++s) {
                    load_filters(SET, s, filters_at(SET));
                    __builtin_amdgcn_sched_barrier(0);     // in the order in which they are waited for
                }
            };
            (request.template operator()<S>(), ...);
            // Whole rounds, then what is left: a loop left from the middle is rewritten such that its ways out run into its way round, where the compiler
            // then does not know how many filters are under way and waits for all of them once a round: 3x3 96 -> 96 on 8 x 35 x 35 (128x64) 10.9 / 9.6 us,
            // 2048 -> 512 on 32 x 7 x 7 (64x64) 10.8 / 10.4, eight ResNet-50 at batch 16 2216 / 2204.
            int t = 0;
            auto stage = [&]<int SET>() {
                wait_and_meet<(NBUF - 2) * L + W>();       // requested after this stage's pixels: its filters, and NBUF - 2 stages
                issue(ibuf, t + NBUF - 1 < ns);
                compute.template operator()<SET, true>(rbuf, filters_at(t + NBUF - 1));
                rbuf = rbuf + 1 == NBUF ? 0 : rbuf + 1;
                ibuf = ibuf + 1 == NBUF ? 0 : ibuf + 1;
                ++t;
            };
            for (int rounds = ns / SETS; rounds > 0; --rounds) (stage.template operator()<S>(), ...);
            auto rest = [&]<int SET>() {                   // nothing is requested any more
                if (t + SET >= ns) return;
                wait_and_meet<(NBUF - 2 - SET) * L + W>();
                compute.template operator()<SET, false>(rbuf, 0u);
                rbuf = rbuf + 1 == NBUF ? 0 : rbuf + 1;
            };
            [&]<int... R>(std::integer_sequence<int, R...>) { (rest.template operator()<R>(), ...); }(std::make_integer_sequence<int, SETS - 1>{});
        }(std::make_integer_sequence<int, SETS>{});
    } else {
        for (int s = 0; s < NBUF - 1; ++s)
            if (s < ns) issue(s);
        for (int t = 0; t < ns; ++t) {
            // stages issued after stage t: NBUF - 2 of them, fewer at the end
            wait_for_stage<L, NBUF - 2>(min(ns - 1 - t, NBUF - 2));
            if (t + NBUF - 1 < ns) issue(ibuf);
            compute.template operator()<0, false>(rbuf, 0u);
            rbuf = rbuf + 1 == NBUF ? 0 : rbuf + 1;
            ibuf = ibuf + 1 == NBUF ? 0 : ibuf + 1;
        }
    }
    if constexpr (DIRECT) {
        if (unsplit) {
            float v[4] = {acc[0][0][0], acc[0][0][1], acc[0][0][2], acc[0][0][3]};
            return finish_pixel<T, 4, 1>(a, v, add, pixel(frow), my_k, vec_ok, (frow & 3) == 0);
        }
    }
    wait_and_meet<0>();                                    // the tile buffers are free
    if constexpr (WIDE) {
        if (!meet_splits<BN, BM, NT>(a, acc, &s_last, tile, z, true, tid)) return;
        WaveTile<T, TN, TM> mine;
        mine.k = (uint32_t)(n0 + wn * SUBN + (lane % mine.LPR) * 8);
#pragma unroll
        for (int j = 0; j < TM; ++j) mine.m_lane[j] = pixel(wm * SUBM + j * 32 + frow);
        if (whole_packs<8>(a)) mine.finish(a, acc, reinterpret_cast<uint16_t *>(&smem[wave * mine.BYTES]), reinterpret_cast<const float *>(&smem[BIAS]) + wn * SUBN, lane);
        else store_lanes<T, MF>(a, acc, n0 + wn * SUBN, mine.m_lane, fgrp);
        return;
    }
    if constexpr (SUMS) {
        if (unsplit) {
            float *sums = reinterpret_cast<float *>(&smem[0]);
            Addend<T, V> adds[EP_IT];
            if constexpr (AHEAD) adds[0] = add;
#pragma unroll
            for (int it = 0; !AHEAD && it < EP_IT; ++it) adds[it].load(a, pixel(my_row(it)), my_k, vec_ok);
            publish_sums<BN, MF, SUBN, SUBM>(acc, sums + wk * (BN * BM), wn, wm, frow, fgrp);
            __syncthreads();
            if (!storing) return;
#pragma unroll
            for (int it = 0; it < EP_IT; ++it) {
                const int row = my_row(it);
                float v[V];
                add_up<BN, V, WK>(sums, BN * BM, row, tid % PIECES, v);
                finish_pixel<T, V, PIECES>(a, v, adds[it], pixel(row), my_k, vec_ok, (row & 3) == 0);
            }
            return;
        }
    }
    if constexpr (!WIDE) finish_tile<T, BN, BM, WN, WM, WK, MF>(a, acc, smem, &s_last, n0, tile, z, pixel);
}

// Small maps: a workgroup owns BN output channels x 16 pixels and its WK waves deal the rows of the reduction (128 bytes
// each) out between them.  A wave's operands are nobody else's, so every wave has D rows in LDS of its own and waits for its
// own loads only: the reduction has no barrier, and WK * D rows of it are in flight after one trip to memory.  The partial sums
// meet once at the end.
//
// What bounds it: launch, one trip to memory and the operand bytes of a tile at the 64 bytes per cycle a compute unit copies to
// LDS; tile_body with the same tile needs a barrier per stage (0.24 us each).  MI355X, bf16, one image, us, 64 x 16 tiles with a
// split reduction / this: 3x3 256 -> 256 on 14 x 14 6.9 / 5.8, 512 -> 512 on 7 x 7 7.9 / 7.4, 1x7 192 -> 192 on 17 x 17 6.3 / 5.1,
// 1x1 1024 -> 256 on 14 x 14 4.9 / 3.9; 2048 -> 192 on 8 x 8 with waves that load to registers 6.5, 4.6 here.
// Rings hold 64 to 72 KB, not what fits: with 128 to 144 KB a layer alone is up to 0.6 us faster, but its workgroups wait for an empty
// compute unit when other tenants run (ResNet-101, Inception-v3, MobileNetV2 and AlexNet together: 665 us, 587 with these).
template <typename T, int BN, int WK, int D, int MODE, bool HELD>
__device__ __forceinline__ void ring_body(const OpArgs &args) {
    OpArgs a = args;
    if constexpr (HELD) hold_walk<MODE != TG_POINT>(a);
    else fetch_walk(a);
    set_wave_priority(a.prio);
    constexpr int ES = sizeof(T), RK = ROW<T>, EPP = 16 / ES, BM = 16, TN = BN / 16;
    constexpr int WQ = BN / 8, XQ = BM / 8, L = WQ + XQ;   // loads of a row: 8 operand rows of 128 bytes each
    constexpr int ROW_BYTES = (BN + BM) * 128;
    static_assert(D * ROW_BYTES >= BN * BM * 4, "a wave's sums fit its ring");
    typedef typename Mma<T, 16>::Acc Acc;
    __shared__ __attribute__((aligned(1024))) uint8_t smem[WK * D * ROW_BYTES];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int tile, z, tn_idx, tm_idx;
    if (!find_tile(a, blockIdx.x / XCDS, tile, z, tn_idx, tm_idx)) return;
    const int M = (int)a.walk.pixels;
    const int n0 = tn_idx * BN, m0 = tm_idx * BM;

    // Four channels of a pixel per storing thread; bias and residual are requested ahead of the operands
    constexpr int STORING = BN / 16;                       // waves that store
    const int my_row = (int)threadIdx.x / (BN / 4), my_piece = (int)threadIdx.x % (BN / 4), my_k = n0 + 4 * my_piece;
    const int my_m = m0 + my_row < M ? (a.pool2 ? (m0 + my_row) >> 2 : m0 + my_row) : -1;
    const bool vec_ok = whole_packs<4>(a);
    Addend<T, 4> add;
    if (wave < STORING) add.load(a, my_m, my_k, vec_ok);

    const int first = wave, end = (int)a.walk.units;
    const int mine = first < end ? (end - first + WK - 1) / WK : 0;    // this wave's rows: first, first + WK, ...

    const int XS = a.x_ct;
    const T *x = (const T *)a.x + a.x_coff;
    const u32x4 rsrc_x = raw_buffer(x, a.walk.x_bytes - (uint32_t)a.x_coff * ES);
    const u32x4 rsrc_w = raw_buffer(a.w, a.walk.w_bytes);
    const uint32_t ring = (uint32_t)wave * (D * ROW_BYTES);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem + ring;

    // columns of the LDS rows permuted as in tile_body: column c of operand row r holds piece c ^ (r / 2 % 8)
    const int lrow = lane >> 3;
    uint32_t wv[WQ], xoff[XQ], xmask[XQ];
    int piece[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) piece[i] = (lane & 7) ^ (i * 4 + (lrow >> 1));
#pragma unroll
    for (int i = 0; i < WQ; ++i) wv[i] = (uint32_t)((n0 + i * 8 + lrow) * a.k_pad + piece[i & 1] * EPP) * ES;
    constexpr int NP = MODE == TG_CHUNK ? XQ : 1;          // positions along j: of every load, or of the row
    int ptap[NP], pch[NP];
#pragma unroll
    for (int i = 0; i < XQ; ++i) {
        const int m = m0 + i * 8 + lrow;
        const bool ok = m < M;
        int n = 0, ih0 = 0, iw0 = m;
        if (MODE != TG_POINT || !a.walk.flat) window_origin(a, ok ? (uint32_t)m : 0u, n, ih0, iw0);
        xoff[i] = (uint32_t)(((n * a.H + ih0) * a.W + iw0) * XS + (MODE == TG_CHUNK ? 0 : piece[i & 1] * EPP)) * ES;
        if constexpr (MODE == TG_POINT) xoff[i] = ok ? xoff[i] : OUT_OF_RANGE;
        else xmask[i] = ok ? window_mask(a, ih0, iw0) : 0u;
        if (MODE != TG_POINT && i < NP) {
            const int j0 = first * RK + (MODE == TG_CHUNK ? piece[i & 1] * EPP : 0);
            ptap[i] = (int)divide((uint32_t)j0, a.walk.c);
            pch[i] = j0 - ptap[i] * a.C;
        }
    }
    const int adv_t = (int)a.walk.adv_t, adv_c = (int)a.walk.adv_c;
    const uint32_t inv_s = a.walk.inv_s;
    uint32_t at = (uint32_t)first * 128u;                  // byte of the row requested next

    auto issue = [&](int slot) {
        const uint32_t base = lds0 + (uint32_t)(slot * ROW_BYTES);
#pragma unroll
        for (int i = 0; i < WQ; ++i) load_to_lds(rsrc_w, wv[i], at, base + (uint32_t)(i * 1024));
        uint32_t toff[NP], trow[NP], tcol[NP];
        if constexpr (MODE != TG_POINT) {
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int tr = a.S == 1 ? ptap[i] : (int)__umulhi((uint32_t)ptap[i], inv_s);
                const int tc = ptap[i] - tr * a.S;
                toff[i] = (uint32_t)((tr * a.W + tc) * XS + pch[i]) * ES;
                trow[i] = (uint32_t)min(tr, 15);           // beyond the window (padding of the reduction): a bit that is never set
                tcol[i] = (uint32_t)(16 + tc);
                ptap[i] += adv_t;
                pch[i] += adv_c;
                const bool carry = pch[i] >= a.C;
                pch[i] -= carry ? a.C : 0;
                ptap[i] += carry ? 1 : 0;
            }
        }
#pragma unroll
        for (int i = 0; i < XQ; ++i) {
            const uint32_t dst = base + (uint32_t)(WQ * 1024 + i * 1024);
            if constexpr (MODE == TG_POINT) {
                load_to_lds(rsrc_x, xoff[i], at, dst);
            } else {
                const int pi = MODE == TG_CHUNK ? i : 0;
                const uint32_t off = (xmask[i] >> trow[pi]) & (xmask[i] >> tcol[pi]) & 1u ? xoff[i] + toff[pi] : OUT_OF_RANGE;
                load_to_lds(rsrc_x, off, 0u, dst);
            }
        }
        at += WK * 128;
    };

    Acc acc[TN][1];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[i][0][v] = 0.f;

    const int frow = lane & 15, fgrp = lane >> 4;
    const uint32_t swz = (uint32_t)((frow >> 1) & 7);
#pragma unroll
    for (int s = 0; s < D; ++s)
        if (s < mine) issue(s);
    int slot = 0;
    for (int t = 0; t < mine; ++t) {
        wait_for_row<L, D - 1>(min(mine - 1 - t, D - 1));
        u32x4 fw[2][TN], fx[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const uint32_t col = ((uint32_t)(s * 4 + fgrp) ^ swz) * 16u;
            const uint32_t b = ring + (uint32_t)(slot * ROW_BYTES) + (uint32_t)(frow * 128) + col;
#pragma unroll
            for (int i = 0; i < TN; ++i) fw[s][i] = *reinterpret_cast<const u32x4 *>(&smem[b + (uint32_t)(i * 16 * 128)]);
            fx[s] = *reinterpret_cast<const u32x4 *>(&smem[b + (uint32_t)(BN * 128)]);
        }
        if (t + D < mine) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");         // the row has been read: its place can be filled again
            issue(slot);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int i = 0; i < TN; ++i) acc[i][0] = Mma<T, 16>::run(fw[s][i], fx[s], acc[i][0]);
        slot = slot + 1 == D ? 0 : slot + 1;
    }
    // a wave's sums go into its own ring, whose loads have all landed and been read
    publish_sums<BN, 16, BN, 16>(acc, reinterpret_cast<float *>(&smem[ring]), 0, 0, frow, fgrp);
    __syncthreads();
    if (wave >= STORING) return;
    float v[4];
    add_up<BN, 4, WK>(reinterpret_cast<const float *>(&smem[0]), D * ROW_BYTES / 4, my_row, my_piece, v);
    finish_pixel<T, 4, BN / 4>(a, v, add, my_m, my_k, vec_ok, (my_row & 3) == 0);
}

// 3x3 windows, stride 1, padding 1 on the rings: a wave's part of the reduction is not rows of 64 elements but chunks of 64 bytes of channels with
// all nine taps.  The tile is a rectangle of 2 x 8 or 4 x 4 pixels, so a wave copies the 4 x 10 or 6 x 6 input pixels of a chunk to LDS once
// and every tap reads its operand there, and the filters, packed in operand order ([channel tile][chunk][tap][lane][16 bytes]), go straight to
// registers, a kilobyte a load.  Two chunks of a wave are in flight after one trip to memory.
//
// What bounds it: a compute unit copies 64 bytes a cycle, and ring_body copies every input pixel nine times: 147 KB and 5200 cycles for 16 channels
// x 16 pixels of 256 channels, of which 4300 wait for copies.  98 KB here, and a third to two thirds of the LDS.  us a layer, ring_body / this, f16 at one
// image: 128 -> 128 on 28 x 28 4.0 / 3.4, 256 -> 256 on 14 x 14 4.0 / 3.6, 512 -> 512 on 14 x 14 7.2 / 5.6, on 7 x 7 5.2 / 4.3; ResNet-18 98.4 / 95.0,
// ResNet-101, Inception-v3, MobileNetV2 and AlexNet together 458 / 446.
template <typename T, int TN, int WK, bool HELD>
__device__ __forceinline__ void ring_patch_body(const OpArgs &args) {
    OpArgs a = args;
    if constexpr (HELD)
        hold(a.x, a.w, a.walk.total, a.walk.per_xcd, a.walk.x_bytes, a.walk.w_bytes, a.walk.units, a.walk.tiles.d, a.walk.tiles.m, a.walk.tiles.s1, a.walk.tiles.s2, a.walk.pq.d, a.walk.pq.m,
             a.walk.pq.s1, a.walk.pq.s2, a.walk.q.d, a.walk.q.m, a.walk.q.s1, a.walk.q.s2, a.tile_order, a.pool2, a.x_ct, a.x_coff, a.H, a.W, a.P, a.Q, a.panel, a.prio, a.K, a.res_ct, a.y_coff,
             a.y_ct, a.bias, a.res);
    else fetch_rect_walk(a);
    set_wave_priority(a.prio);
    constexpr int ES = sizeof(T), BN = 16 * TN, D = 2;
    constexpr int PIXELS = 48, PATCH = PIXELS * 64, XL = PIXELS / 16;  // a load covers 16 pixels of 64 bytes
    constexpr int REGION = std::max(D * PATCH, BN * 16 * 4);           // LDS of a wave: its patches, then its sums
    typedef typename Mma<T, 16>::Acc Acc;
    __shared__ __attribute__((aligned(1024))) uint8_t smem[WK * REGION];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int tile, z, tn_idx, tm_idx;
    if (!find_tile(a, blockIdx.x / XCDS, tile, z, tn_idx, tm_idx)) return;
    const int rect = -a.panel, PW = rect + 2;              // columns of the rectangle and of its patch
    const bool wide = rect == 8;
    const int n0 = tn_idx * BN;
    const int img = (int)divide((uint32_t)tm_idx, a.walk.pq), in_img = tm_idx - img * (int)a.walk.pq.d;
    const int trow = (int)divide((uint32_t)in_img, a.walk.q), tcol = in_img - trow * (int)a.walk.q.d;
    const int p0 = trow * (wide ? 2 : 4), q0 = tcol * rect;

    // Place of tile row j in the rectangle: four consecutive rows are a 2 x 2 window, so that the epilogue can pool.
    auto place = [&](int j, int &dy, int &dx) {
        dy = (wide ? 0 : 2 * (j >> 3)) + ((j >> 1) & 1);
        dx = 2 * (wide ? j >> 2 : (j >> 2) & 1) + (j & 1);
    };
    // Four channels of a pixel per storing thread; bias and residual are requested ahead of the operands
    constexpr int STORING = BN / 16;                       // waves that store
    const int my_row = (int)threadIdx.x / (BN / 4), my_piece = (int)threadIdx.x % (BN / 4), my_k = n0 + 4 * my_piece;
    int my_m = -1;
    {
        int dy, dx;
        place(my_row, dy, dx);
        const int p = p0 + dy, q = q0 + dx;
        if (a.pool2) my_m = (p >> 1) < (a.P >> 1) && (q >> 1) < (a.Q >> 1) ? (img * (a.P >> 1) + (p >> 1)) * (a.Q >> 1) + (q >> 1) : -1;
        else my_m = p < a.P && q < a.Q ? (img * a.P + p) * a.Q + q : -1;
    }
    const bool vec_ok = whole_packs<4>(a);
    Addend<T, 4> add;
    if (wave < STORING) add.load(a, my_m, my_k, vec_ok);

    const T *x = (const T *)a.x + a.x_coff;
    const u32x4 rsrc_x = raw_buffer(x, a.walk.x_bytes - (uint32_t)a.x_coff * ES);
    const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w), 0, (int)a.walk.w_bytes, 0x00027000);
    const uint32_t region = (uint32_t)wave * REGION;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem + region;

    // Lane l of load i delivers 16-byte column l % 4 of patch pixel 16 i + l / 4; column c of pixel r holds piece c ^ (r / 4 % 4).
    uint32_t xoff[XL];
    const int need = (wide ? 4 : 6) * PW;
    const uint32_t inv = wide ? 6554u : 10923u;            // 2^16 over PW, rounded up
#pragma unroll
    for (int i = 0; i < XL; ++i) {
        const int r = i * 16 + (lane >> 2), pr = (int)(((uint32_t)r * inv) >> 16), pc = r - pr * PW;
        const int ih = p0 - 1 + pr, iw = q0 - 1 + pc, piece = (lane ^ (r >> 2)) & 3;
        const bool ok = (r < need) & ((uint32_t)ih < (uint32_t)a.H) & ((uint32_t)iw < (uint32_t)a.W);
        xoff[i] = ok ? (uint32_t)(((img * a.H + ih) * a.W + iw) * a.x_ct) * ES + (uint32_t)piece * 16u : OUT_OF_RANGE;
    }
    const int chunks = (int)a.walk.units;
    uint32_t wtile[TN];                                    // filters of a channel tile
#pragma unroll
    for (int i = 0; i < TN; ++i) wtile[i] = (uint32_t)((tn_idx * TN + i) * chunks) * 9216u;

    const int frow = lane & 15, fgrp = lane >> 4;
    int dy, dx;
    place(frow, dy, dx);
    const int first_pixel = dy * PW + dx;                  // patch pixel of tap (0, 0)

    Acc acc[TN][1];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[i][0][v] = 0.f;

    u32x4 w[D][9][TN];
    auto copy_patch = [&](int c, int d) {
#pragma unroll
        for (int i = 0; i < XL; ++i) load_to_lds(rsrc_x, xoff[i], (uint32_t)c * 64u, lds0 + (uint32_t)(d * PATCH + i * 1024));
    };
    auto load_filters = [&](int c, int d) {
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int i = 0; i < TN; ++i)
                w[d][t][i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, (uint32_t)lane * 16u + (uint32_t)(t % 3) * 1024u, wtile[i] + (uint32_t)c * 9216u + (uint32_t)(t / 3) * 3072u, 0);
    };
    auto multiply = [&](int d) {
        u32x4 fx[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const uint32_t r = (uint32_t)(first_pixel + (t / 3) * PW + t % 3);
            fx[t] = *reinterpret_cast<const u32x4 *>(&smem[region + (uint32_t)(d * PATCH) + r * 64u + (((uint32_t)fgrp ^ (r >> 2)) & 3u) * 16u]);
        }
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int i = 0; i < TN; ++i) acc[i][0] = Mma<T, 16>::run(w[d][t][i], fx[t], acc[i][0]);
    };
    // This wave's chunks: wave, wave + WK, ...
    for (int c = wave; c < chunks; c += D * WK) {
        const bool two = c + WK < chunks;
        if (c != wave) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the patches have been read: their place can be filled again
        copy_patch(c, 0);
        if (two) {
            copy_patch(c + WK, 1);
            load_filters(c, 0);
            load_filters(c + WK, 1);
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(D * 9 * TN) : "memory");
            multiply(0);
            multiply(1);
        } else {
            load_filters(c, 0);
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(9 * TN) : "memory");
            multiply(0);
        }
    }
    // a wave's sums go into its own region, whose patches have all landed and been read
    publish_sums<BN, 16, BN, 16>(acc, reinterpret_cast<float *>(&smem[region]), 0, 0, frow, fgrp);
    __syncthreads();
    if (wave >= STORING) return;
    float v[4];
    add_up<BN, 4, WK>(reinterpret_cast<const float *>(&smem[0]), REGION / 4, my_row, my_piece, v);
    finish_pixel<T, 4, BN / 4>(a, v, add, my_m, my_k, vec_ok, (my_row & 3) == 0);
}

// LDS that the bodies of one kernel share.
template <int BYTES>
__device__ __forceinline__ uint8_t *lds_place() {
    __shared__ __attribute__((aligned(1024))) uint8_t place[BYTES];
    return place;
}

// 3x3 windows, stride 1, padding 1, C % 64 == 0: the nine taps of a 64-channel chunk read the same input pixels, so those
// are staged once per chunk as a patch and every tap reads its operand rows at a shifted position.
// The map is cut into panels of `panel` columns; inside a panel pixels are numbered row by row through all images, and a
// tile is BM consecutive ones.  Its patch holds the rows from the one above its first to the one below its last, each
// panel + 2 pixels wide, with an empty row between two images; what lies outside an image is loaded out of range, i.e. zero.
// The filter bank is packed in operand order ([32 channels][chunk][tap][16 elements][lane][16 bytes]) and goes straight to registers, a kilobyte a
// load, so LDS holds only the patches and the waves meet once per chunk.  Up to DW steps ahead: requests that belong to the next chunk stand behind a branch, the
// compiler does not know whether they are under way, and its waits fall to none by the end of a chunk.  Without the branch (out of range after the last chunk) a layer
// alone is faster, 64x64 256 -> 256 on 16 x 14 x 14 8.7 / 7.8 us, 128x64 512 -> 512 on 64 x 7 x 7 19.4 / 17.9, but ResNet-18, VGG-16 and MobileNetV2 beside each other take 222 us
// instead of 219, in four stages 287 instead of 283: VGG-16's layers leave the other two less.
//
// What bounds it: matrix instructions (with loads of both operands left out a 128x128 tile of 512 channels takes 25.5 us, with them 31.6) and,
// at short reductions, the first patch and the finish.  Filters that pass through LDS, as they did before, are two thirds of the bytes written to it and half of
// those read, with a barrier per tap, and their three stages kept a second workgroup from the unit: 64x64 and 128x64 tiles now leave room for one.
// The wave groups divide the four steps of a tap such that no filter is loaded twice on 64 channels (two waves, four groups) and on the 128x64
// tile (four waves, two groups); on the 128x128 tile two waves load the same filters, the second from the L1, which costs nothing (two waves and four
// groups: 31.6 / 32.4 us).  The 128x256 tile has one group of waves up to four chunks, of which four load the same filters: two groups' exchange of sums takes
// longer there than the filters do.  From five chunks on it has two groups.  us a layer, filters through LDS / this, f16, 3x3:
//   128x64   128 -> 128 on 16 x 28 x 28  8.73 / 7.78     512 -> 512 on 64 x 7 x 7    22.7 / 19.5     64 -> 128 on 112 x 112  6.59 / 6.10
//   64x64    256 -> 256 on 16 x 14 x 14  9.06 / 8.66     512 -> 512 on 8 x 14 x 14   14.5 / 13.7     256 -> 256 on 56 x 56   9.04 / 8.66
//   64x32    256 -> 512 -> 256 on 28 x 28 (64x64 and split the way back)  10.1 / 8.9
//   128x128  256 -> 256 on 64 x 14 x 14  18.4 / 17.2     512 -> 512 on 8 x 28 x 28   30.9 / 29.5
//   128x256  (in brackets the other number of groups)
//            128 -> 128 on 8 x 112 x 112 34.9 / 34.9 (38.5)     on 54 x 28 x 28  17.0 / 16.4 (17.5)     256 -> 256 on 8 x 56 x 56  29.1 / 28.0 (28.5)
//            448 -> 448 on 32 x 28 x 28  90.9 / 91.6 (93.5)     512 -> 512  104 / 105 (108)             on 64 x 14 x 14  52.4 / 51.0 (53.0)
template <typename T, int BN, int BM, int WN, int WM, int WK, int DW, int PC, bool HELD, int ROOM = 0, int PLACE = 0>
__device__ __forceinline__ void patch_body(const OpArgs &args, uint32_t slot) {
    OpArgs a = args;
    if constexpr (HELD)
        hold(a.x, a.w, a.walk.total, a.walk.per_xcd, a.walk.x_bytes, a.walk.w_bytes, a.walk.units, a.walk.per, a.walk.split.d, a.walk.split.m, a.walk.split.s1, a.walk.split.s2, a.walk.tiles.d,
             a.walk.tiles.m, a.walk.tiles.s1, a.walk.tiles.s2, a.walk.pq.d, a.walk.pq.m, a.walk.pq.s1, a.walk.pq.s2, a.walk.q.d, a.walk.q.m, a.walk.q.s1, a.walk.q.s2, a.walk.panel_tiles.d,
             a.walk.panel_tiles.m, a.walk.panel_tiles.s1, a.walk.panel_tiles.s2, a.walk.inv_pw, a.walk.inv_h, a.tile_order, a.pool2, a.k_pad, a.x_ct, a.x_coff, a.H, a.W, a.N, a.P, a.Q, a.panel, a.prio, a.K, a.res_ct, a.y_coff,
             a.y_ct, a.bias, a.res);
    else fetch_walk(a);
    set_wave_priority(a.prio);
    constexpr int NW = WN * WM * WK, MF = 32;
    constexpr int SUBN = BN / WN, SUBM = BM / WM, TN = SUBN / MF, TM = SUBM / MF;
    static_assert(TN >= 1 && TM >= 1 && 4 % WK == 0, "the wave groups share the four 16-element steps of a tap");
    constexpr int ACC = 16, MY = 4 / WK, SPC = 9 * MY;     // a wave's steps per tap and per chunk
    static_assert(SPC % DW == 0, "registers of a step");
    constexpr int PL = PC / 8 / NW;                        // loads of a wave per patch
    static_assert(PL * NW * 8 == PC && PL < SPC, "the waves share a patch evenly, and it is requested during a chunk's steps");
    constexpr int P_BYTES = PC * 128;
    constexpr bool WIDE = WK <= 2, SUMS = !WIDE;           // every wave finishes its part of the tile, of two groups half of it
    constexpr int CT = WK == 2 ? 1 : TN, OWN = WK == 2 ? TN * TM / 2 : TM;     // products of 32 x 32 in it: CT * 32 channels x OWN * 32 pixels
    static_assert(WK != 2 || (TN * TM % 2 == 0 && TM % OWN == 0), "the half is a row of products");
    constexpr int XCH = WK == 2 ? NW * OWN * 4096 : 0, RED_BYTES = WIDE ? XCH + NW * WaveTile<T, CT, OWN>::BYTES : WK * BN * BM * 4, EP_BYTES = WIDE ? 0 : BM * (BN + 4) * 4;
    constexpr int COUNTED = ROOM > 0 ? 160 * 1024 / (ROOM + 1) + 1 : 0;      // a compute unit holds no more workgroups than are counted on
    constexpr int BIAS = std::max({2 * P_BYTES, RED_BYTES, EP_BYTES, COUNTED + 15 & ~15}), LDS_BYTES = BIAS + (WIDE ? BN * 4 : 0);
    static_assert(PLACE == 0 || LDS_BYTES <= PLACE, "LDS shared with another body");
    typedef typename Mma<T, MF>::Acc Acc;
    uint8_t *const smem = lds_place<std::max(LDS_BYTES, PLACE)>();
    __shared__ int s_last;

    int tid = threadIdx.x;
    if (ROOM > 0) asm volatile("" : "+v"(tid));            // what a lane's place decides is worked out for every tile: kept, it is more registers than there are
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave / (WN * WM), wn = (wave % (WN * WM)) % WN, wm = (wave % (WN * WM)) / WN;

    const int Wt = a.panel, PW = Wt + 2;
    int tile, z, tn_idx, tm_idx;
    if (!find_tile(a, slot, tile, z, tn_idx, tm_idx)) return;
    const int ppx = a.N * a.P * Wt;                        // pixels of a panel
    const int pn = (int)divide((uint32_t)tm_idx, a.walk.panel_tiles);
    const int n0 = tn_idx * BN, m0 = (tm_idx - pn * (int)a.walk.panel_tiles.d) * BM;
    const int c_begin = z * (int)a.walk.per;
    const int nc = min((int)a.walk.units, c_begin + (int)a.walk.per) - c_begin;    // chunks of this workgroup (>= 1 by construction)

    // image row (through all images) and column of pixel i of the panel; divisors: panel width, rows of the map (halved when pooling)
    auto locate = [&](uint32_t i, int &row, int &img, int &col) {
        const uint32_t mq = a.pool2 ? i >> 2 : i;
        const uint32_t rr = divide(mq, a.walk.q);
        img = (int)divide(rr, a.walk.pq);
        row = (int)(rr - (uint32_t)img * a.walk.pq.d);
        col = (int)(mq - rr * a.walk.q.d);
        if (a.pool2) {
            row = 2 * row + (int)((i >> 1) & 1u);
            col = 2 * col + (int)(i & 1u);
        }
    };
    int row_a, img_a, row_b, img_b, col_u;
    locate((uint32_t)m0, row_a, img_a, col_u);
    locate((uint32_t)(min(m0 + BM, ppx) - 1), row_b, img_b, col_u);
    const int need = ((img_b - img_a) * (a.H + 1) + row_b - row_a + 3) * PW;   // patch pixels in use

    const int XS = a.x_ct;
    const T *x = (const T *)a.x + a.x_coff;
    const u32x4 rsrc_x = raw_buffer(x, a.walk.x_bytes - (uint32_t)a.x_coff * 2u);
    const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w), 0, (int)a.walk.w_bytes, 0x00027000);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    // Columns of the LDS rows as in tile_body; a patch row's key is its pixel's number without the two border columns of the
    // rows above it, so that 16 consecutive pixels of a tile have 16 consecutive keys wherever a map row ends among them.
    static_assert(NW % 2 == 0 && BN % 16 == 0, "a wave's row groups have one parity");
    const int lrow = lane >> 3;

    uint32_t wtile[TN];                                    // this wave's part of the filters of 32 channels, chunk by chunk
#pragma unroll
    for (int i = 0; i < TN; ++i) wtile[i] = (((uint32_t)(n0 / 32 + wn * TN + i) * a.walk.units + (uint32_t)c_begin) * 36u + (uint32_t)(wk * MY)) * 1024u;
    uint32_t xoff[PL];
    const uint32_t inv_pw = a.walk.inv_pw, inv_h = a.walk.inv_h;
#pragma unroll
    for (int i = 0; i < PL; ++i) {
        const uint32_t px = (uint32_t)((i * NW + wave) * 8 + lrow);
        const int prow = (int)((px * inv_pw) >> 20), pcol = (int)px - prow * PW;
        const int piece = (lane & 7) ^ ((int)((px >> 1) - (uint32_t)prow) & 7);
        const int d = row_a - 1 + prow;                    // row counted from the top of the first image, one empty row per image
        const int di = d < 0 ? 0 : (int)(((uint32_t)d * inv_h) >> 20);
        const int ih = d - di * (a.H + 1), n = img_a + di, iw = pn * Wt - 1 + pcol;
        const bool ok = ((int)px < need) & ((uint32_t)ih < (uint32_t)a.H) & ((uint32_t)iw < (uint32_t)a.W) & (n < a.N);
        xoff[i] = ok ? (uint32_t)(((n * a.H + ih) * a.W + iw) * XS + piece * 8) * 2u : OUT_OF_RANGE;
    }
    uint32_t xs = (uint32_t)(c_begin * TK) * 2u;           // channel offset of the patch requested next

    auto issue_patch = [&](int i, int buf) {
        load_to_lds(rsrc_x, xoff[i], xs, lds0 + (uint32_t)(buf * P_BYTES + (i * NW + wave) * 1024));
    };
    // Step j of a chunk: 16 elements of tap j / MY
    u32x4 w[DW][TN];
    auto load_filters = [&](int c, int j) {
#pragma unroll
        for (int i = 0; i < TN; ++i)
            w[j % DW][i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, (uint32_t)lane * 16u + (uint32_t)(j % MY) * 1024u, wtile[i] + (uint32_t)c * 36864u + (uint32_t)(j / MY) * 4096u, 0);
    };

    Acc acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int v = 0; v < ACC; ++v) acc[i][j][v] = 0.f;

    const int frow = lane % MF, fgrp = lane / MF;
    int ppos[TM], prow[TM];                                          // patch pixel of tap (0, 0) for this lane's pixels
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        int row, img, col;
        locate((uint32_t)min(m0 + wm * SUBM + j * MF + frow, ppx - 1), row, img, col);
        prow[j] = (img - img_a) * (a.H + 1) + row - row_a;
        ppos[j] = prow[j] * PW + col;
    }

    u32x4 fx[2][TM];
    auto load_pixels = [&](int j, int pb, u32x4 (&x)[TM]) {
        const int tap = j / MY, c0 = (wk * MY + j % MY) * 2;
        const int shift = (tap / 3) * PW + tap % 3;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const uint32_t rr = (uint32_t)(ppos[i] + shift);
            const uint32_t col = ((uint32_t)(c0 + fgrp) ^ (((rr >> 1) - (uint32_t)(prow[i] + tap / 3)) & 7u)) * 16u;
            x[i] = *reinterpret_cast<const u32x4 *>(&smem[(uint32_t)(pb * P_BYTES) + rr * 128u + col]);
        }
    };

    if (WIDE && wave < BN / 64)
        load_words_to_lds(raw_buffer(a.bias, (uint32_t)(n0 + BN) * 4u), (uint32_t)(n0 + lane) * 4u, (uint32_t)wave * 256u, lds0 + BIAS + (uint32_t)wave * 256u);
#pragma unroll
    for (int i = 0; i < PL; ++i) issue_patch(i, 0);
#pragma unroll
    for (int j = 0; j < DW; ++j) load_filters(0, j);
    wait_and_meet<DW * TN>();
    load_pixels(0, 0, fx[0]);
    for (int c = 0; c < nc; ++c) {
        const bool last = c + 1 == nc;
        xs += TK * 2;
#pragma unroll
        for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(ppos[i]));     // the addresses of all steps, kept from chunk to chunk, are more registers than there are
#pragma unroll
        for (int j = 0; j < SPC; ++j) {
            if (j < PL && !last) issue_patch(j, (c + 1) & 1);
            if (j + 1 < SPC) {
                load_pixels(j + 1, c & 1, fx[(j + 1) & 1]);
            } else if (!last) {
                wait_and_meet<(SPC - PL) * TN>();          // the filters requested after the last piece of the patch may be under way
                load_pixels(0, (c + 1) & 1, fx[(j + 1) & 1]);
            }
            __builtin_amdgcn_sched_barrier(0);             // the next step's operands are requested before this one multiplies
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int m = 0; m < TM; ++m) acc[i][m] = Mma<T, MF>::run(w[j % DW][i], fx[j & 1][m], acc[i][m]);
            __builtin_amdgcn_sched_barrier(0);
            if (j + DW < SPC) load_filters(c, j + DW);
            else if (!last) load_filters(c + 1, j + DW - SPC);
        }
        if constexpr (SPC % 2 != 0) {
#pragma unroll
            for (int m = 0; m < TM; ++m) fx[0][m] = fx[1][m];
        }
    }
    auto pixel = [&](int ml) {
        const int i = m0 + ml;
        int row, img, col;
        locate((uint32_t)min(i, ppx - 1), row, img, col);
        const int q = pn * Wt + col;
        if (i >= ppx || q >= a.Q) return -1;
        return a.pool2 ? (img * (a.P >> 1) + (row >> 1)) * (a.Q >> 1) + (q >> 1) : (img * a.P + row) * a.Q + q;
    };
    wait_and_meet<0>();
    if constexpr (WIDE) {
        auto complete = [&](Acc (&sums)[CT][OWN], int c0, int p0) {
            if (!meet_splits<BN, BM, 64 * NW>(a, sums, &s_last, tile, z, true, tid)) return;
            WaveTile<T, CT, OWN> part;
            static_assert(XCH + NW * part.BYTES <= BIAS, "exchanged sums and staging blocks fit");
            part.k = (uint32_t)(n0 + c0 + (lane % part.LPR) * 8);
#pragma unroll
            for (int j = 0; j < OWN; ++j) part.m_lane[j] = pixel(p0 + j * 32 + frow);
            if (whole_packs<8>(a)) part.finish(a, sums, reinterpret_cast<uint16_t *>(&smem[XCH + wave * part.BYTES]), reinterpret_cast<const float *>(&smem[BIAS]) + c0, lane);
            else store_lanes<T, MF>(a, sums, n0 + c0, part.m_lane, fgrp);
        };
        if constexpr (WK == 1) {
            complete(acc, wn * SUBN, wm * SUBM);
        } else {
            // each group hands the other the sums of half of its products and finishes the other half.  Each on a path of its own: picked lane by lane the
            // sums take four cycles a register twice (128x256 tile: 0.4 us of a layer's 18).
            float *xch = reinterpret_cast<float *>(&smem[0]) + lane * 4;
            const int other = wave ^ (WN * WM);
            Acc mine[1][OWN];
            auto hand_over = [&]<int GROUP>() {
#pragma unroll
                for (int q = 0; q < OWN; ++q) {
                    const int h = OWN + q;
                    const Acc &given = GROUP == 0 ? acc[h / TM][h % TM] : acc[0][q], &kept = GROUP == 0 ? acc[0][q] : acc[h / TM][h % TM];
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        *reinterpret_cast<float4 *>(&xch[(wave * OWN * 4 + 4 * q + g) * 256]) = make_float4(given[4 * g], given[4 * g + 1], given[4 * g + 2], given[4 * g + 3]);
                    mine[0][q] = kept;
                }
                asm volatile("; group %0" ::"n"(GROUP) : "memory");        // keeps the two paths apart
            };
            if (wk == 0) hand_over.template operator()<0>();
            else hand_over.template operator()<1>();
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 4 * OWN; ++q) {
                const float4 v = *reinterpret_cast<const float4 *>(&xch[(other * OWN * 4 + q) * 256]);
                Acc &to = mine[0][q / 4];
                to[4 * (q % 4)] += v.x; to[4 * (q % 4) + 1] += v.y; to[4 * (q % 4) + 2] += v.z; to[4 * (q % 4) + 3] += v.w;
            }
            complete(mine, wn * SUBN + wk * OWN / TM * 32, wm * SUBM + wk * OWN % TM * 32);
        }
        return;
    }
    if constexpr (SUMS) {
        if (a.walk.split.d == 1) {
            constexpr int NT = 64 * NW, V = BN * BM >= 8 * NT ? 8 : 4, PIECES = BN / V, EP_IT = BN * BM / V / NT;
            const bool vec_ok = whole_packs<V>(a);
            const int my_k = n0 + (tid % PIECES) * V;
            float *sums = reinterpret_cast<float *>(&smem[0]);
            int m[EP_IT];
            Addend<T, V> add[EP_IT];
#pragma unroll
            for (int it = 0; it < EP_IT; ++it) {
                m[it] = pixel((tid + it * NT) / PIECES);
                add[it].load(a, m[it], my_k, vec_ok);
            }
            publish_sums<BN, MF, SUBN, SUBM>(acc, sums + wk * (BN * BM), wn, wm, frow, fgrp);
            __syncthreads();
#pragma unroll
            for (int it = 0; it < EP_IT; ++it) {
                const int row = (tid + it * NT) / PIECES;
                float v[V];
                add_up<BN, V, WK>(sums, BN * BM, row, tid % PIECES, v);
                finish_pixel<T, V, PIECES>(a, v, add[it], m[it], my_k, vec_ok, (row & 3) == 0);
            }
            return;
        }
    }
    if constexpr (!WIDE) finish_tile<T, BN, BM, WN, WM, WK, MF>(a, acc, smem, &s_last, n0, tile, z, pixel);
}

// Waves per SIMD the registers have to leave room for: two workgroups per compute unit of the widest tile, whose LDS fits twice.
constexpr int tile_waves_per_simd(int bn, int bm, int nbuf) { return bn * bm >= 128 * 128 && nbuf == 2 ? 2 : 1; }
template <typename T, int BN, int BM, int WN, int WM, int WK, int KD, int NBUF, int MODE>
__global__ void __launch_bounds__(64 * WN * WM * WK, tile_waves_per_simd(BN, BM, NBUF)) tile_kernel(OpArgs a) {
    tile_body<T, BN, BM, WN, WM, WK, KD, NBUF, MODE, sizeof(T) == 2 && BM / WM >= 32 && WK == 1>(a, blockIdx.x / XCDS);
    results_stored();
}

// Workgroups of a walking kernel that a compute unit holds: by LDS (made to hold no more) and by registers, which the launch bounds have the
// compiler leave for as many.
constexpr int tile_room(int bn, int bm, int kd) { return kd == 1 && bn * bm <= 128 * 64 ? 3 : kd == 2 && bm == 64 ? 1 : 2; }
constexpr int patch_room(int bn, int bm) { return bn * bm <= 128 * 64 ? 2 : 1; }

// The OpArgs a kernel was launched with, as its only parameter.  What is read through one call is not kept for the next.
__device__ __forceinline__ const OpArgs &kernel_arguments() {
    typedef const OpArgs __attribute__((address_space(4))) InConstant;
    uint64_t at = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(at));
    return *(const OpArgs *)(InConstant *)at;
}

// The same with fewer workgroups than tiles: a workgroup takes every walk.step-th tile of its XCD's range.  Where two queues share a dispatch
// pipe the pipe is taken until the last workgroup of a launch has found room: launches that fit their queue's units at once let
// the other queue's run beside them.  Queues on 32 units each, two to a pipe, us a kernel (four queues in brackets): 37 us of short workgroups 89 (39),
// 50 us of resident ones 86 (54).  Eight ResNet-50 on disjoint eighths of the units, us: batch 4 3397 / 2972, 16 5452 / 3979
// (in eight stages 5988 / 4464), 64 13997 / 9700; four and fewer have a pipe each and run the kernel above.
// The arguments are read anew for every tile: kept across the loop they are more scalars than there are, and the compiler puts 70 to 146 of them
// into lanes of vector registers (f16 64x32 tile: 129 registers, one more than two workgroups leave each; 126 to 128 so).  Eight ResNet-50 at
// batch 16 in eight stages 4597 / 4500 us, runs of one side 4 % apart.
template <typename T, int BN, int BM, int WN, int WM, int WK, int KD, int NBUF, int MODE>
__global__ void __launch_bounds__(64 * WN * WM * WK, tile_room(BN, BM, KD) * WN * WM * WK / 4) tile_walk_kernel(OpArgs) {
    for (uint32_t slot = blockIdx.x / XCDS;;) {
        const OpArgs &a = kernel_arguments();
        tile_body<T, BN, BM, WN, WM, WK, KD, NBUF, MODE, true, tile_room(BN, BM, KD)>(a, slot);
        slot += a.walk.step;
        if (slot >= a.walk.per_xcd) break;
        __syncthreads();                                   // every wave is done with the tile's LDS
    }
    results_stored();
}

template <typename T, int BN, int BM, int WN, int WM, int WK, int KD, int NBUF, int MODE>
__global__ void __launch_bounds__(64 * WN * WM * WK, tile_waves_per_simd(BN, BM, NBUF)) tile_pair_kernel(OpArgsPair p) {
    tile_body<T, BN, BM, WN, WM, WK, KD, NBUF, MODE, true>(p.a[blockIdx.y], blockIdx.x / XCDS);
    results_stored();
}

template <typename T, int BN, int WK, int D, int MODE>
__global__ void __launch_bounds__(64 * WK) ring_kernel(OpArgs a) {
    ring_body<T, BN, WK, D, MODE, false>(a);
    results_stored();
}

template <typename T, int BN, int WK, int D, int MODE>
__global__ void __launch_bounds__(64 * WK) ring_pair_kernel(OpArgsPair p) {
    ring_body<T, BN, WK, D, MODE, true>(p.a[blockIdx.y]);
    results_stored();
}

template <typename T, int TN, int WK>
__global__ void __launch_bounds__(64 * WK) ring_patch_kernel(OpArgs a) {
    ring_patch_body<T, TN, WK, false>(a);
    results_stored();
}

template <typename T, int TN, int WK>
__global__ void __launch_bounds__(64 * WK) ring_patch_pair_kernel(OpArgsPair p) {
    ring_patch_body<T, TN, WK, true>(p.a[blockIdx.y]);
    results_stored();
}

template <typename T, int BN, int BM, int WN, int WM, int WK, int DW, int PC>
__global__ void __launch_bounds__(64 * WN * WM * WK) patch_kernel(OpArgs a) {
    patch_body<T, BN, BM, WN, WM, WK, DW, PC, BN == 128>(a, blockIdx.x / XCDS);
    results_stored();
}

// The walking kernel of the widest tile has both its bodies.
constexpr uint32_t LONG_PATCHES = 4;                       // chunks of the reduction beyond which that tile has two groups of waves (patch_body)
constexpr int WIDEST_LDS = 152064;
template <typename T, int BN, int BM, int WN, int WM, int WK, int DW, int PC>
__global__ void __launch_bounds__(64 * WN * WM * WK, patch_room(BN, BM) * WN * WM * WK / 4) patch_walk_kernel(OpArgs) {
    constexpr int AHEAD = BN == 64 && BM == 64 ? 3 : BM == 256 ? 2 : DW;     // filters further ahead are more registers than there are
    for (uint32_t slot = blockIdx.x / XCDS;;) {
        const OpArgs &a = kernel_arguments();
        if constexpr (BM == 256) {                         // both in the same LDS; what they share the compiler would move ahead of the branch, and that is more scalars than there are
            if (a.walk.units <= LONG_PATCHES) {
                asm volatile("; one group");
                patch_body<T, BN, BM, WN, WM * WK, 1, 4, PC, true, 1, WIDEST_LDS>(kernel_arguments(), slot);
            } else {
                asm volatile("; two groups");
                patch_body<T, BN, BM, WN, WM, WK, AHEAD, PC, true, 1, WIDEST_LDS>(kernel_arguments(), slot);
            }
        } else patch_body<T, BN, BM, WN, WM, WK, AHEAD, PC, true, patch_room(BN, BM)>(a, slot);
        slot += a.walk.step;
        if (slot >= a.walk.per_xcd) break;
        __syncthreads();
    }
    results_stored();
}

template <typename T, int BN, int BM, int WN, int WM, int WK, int DW, int PC>
__global__ void __launch_bounds__(64 * WN * WM * WK) patch_pair_kernel(OpArgsPair p) {
    patch_body<T, BN, BM, WN, WM, WK, DW, PC, true>(p.a[blockIdx.y], blockIdx.x / XCDS);
    results_stored();
}

// ---- choice of form -----------------------------------------------------------------------------------------------
namespace {

// Time of a launch in us on MI355X: start + wave * (n - 1) + ns * (stage + crowd * (n - 1)), and split_once + split_each *
// split if the reduction is split over workgroups (16-bit types only, and rings never are: a split costs them more than it gives); n: workgroups per compute unit, ns: stages of a workgroup.  Fitted to timings of the
// distinct convolutions and classifiers of nine networks at batches 1 to 64 (fp32: 1 to 8), launch gap included.  Sum over
// those layers, us, without the ring forms / picking by the estimate / the fastest measured form of every layer: bf16 at batch 1
// 593 / 531 / 519, batch 5 839 / 805 / 767.  The timings are of the kernels before TileWalk and WaveTile, which took up to 1.25 us from every start and 1 to
// 2 us from the wide forms; sums and numbers have not been fitted again (a fit to launches that have the chip to themselves picked forms that
// made tenants beside each other slower, and was not kept).  fp32, operands from memory to registers (kernels_dconv.hip) / picking here /
// fastest: batch 1 1219 / 930 / 900, batch 4 1526 / 1220 / 1160.
struct TileCost {
    double start, wave, stage, crowd, split_once, split_each;
};
struct TileForm {
    int bn, bm, kd, rows, threads, patch_pixels;           // rows: LDS rows of the reduction per stage; patch_pixels 0: tile_body or ring_body
    int ring;                                              // waves of ring_body that share the reduction, 0: another body
    TileCost half, single;                                 // of the 16-bit types and of fp32 (NONE: not built)
};
constexpr TileCost NONE = {0, 0, 0, 0, 0, 0};

constexpr TileForm FORMS[] = {
    {128, 128, 1, 1, 256, 0, 0, {5.33, 2.29, 0.537, 0.350, 1.98, 0.995}, NONE},
    {128, 64, 1, 1, 256, 0, 0, {4.17, 1.29, 0.372, 0.209, 1.49, 0.726}, NONE},
    {64, 64, 1, 1, 256, 0, 0, {3.68, 0.965, 0.285, 0.133, 1.52, 0.375}, {3.92, 0.653, 0.582, 0.569, 0, 0}},
    {64, 64, 2, 2, 512, 0, 0, {3.66, 2.50, 0.402, 0.515, 2.07, 0.218}, {4.58, 2.09, 0.888, 1.61, 0, 0}},
    {64, 32, 2, 2, 512, 0, 0, {3.63, 1.11, 0.323, 0.235, 1.35, 0.266}, {3.89, 0.912, 0.613, 0.635, 0, 0}},
    {64, 16, 2, 2, 256, 0, 0, {2.79, 0.723, 0.295, 0.166, 1.60, 0.140}, {2.99, 0.671, 0.437, 0.306, 0, 0}},
    {128, 256, 1, 1, 512, 384, 0, {9.21, 5.92, 0.545, 0.823, 2.20, 1.36}, NONE},
    {128, 128, 1, 1, 512, 256, 0, {7.59, 6.90, 0.331, 0.357, 2.31, 0.748}, NONE},
    {128, 64, 1, 1, 512, 192, 0, {5.83, 4.94, 0.219, 0.238, 1.52, 0.602}, NONE},
    {64, 64, 3, 3, 512, 192, 0, {4.96, 3.74, 0.413, 0.438, 1.53, 0.284}, NONE},
    {64, 32, 1, 1, 512, 128, 0, {4.56, 1.38, 0.118, 0.109, 1.38, 0.252}, NONE},
    {32, 32, 2, 2, 512, 0, 0, NONE, {3.32, 0.897, 0.395, 0.402, 0, 0}},
    {16, 16, 1, 8, 512, 0, 8, {3.30, 1.82, 0.283, 0.480, 0, 0}, {3.19, 1.88, 0.453, 0.528, 0, 0}},
    {32, 16, 1, 4, 256, 0, 4, {3.35, 0.9, 0.28, 0.25, 0, 0}, {3.3, 0.95, 0.37, 0.4, 0, 0}},
    {16, 16, 1, 4, 256, 0, 4, {3.19, 0.568, 0.193, 0.175, 0, 0}, {3.03, 0.652, 0.259, 0.209, 0, 0}},
};
bool far_window(const OpArgs &a) { return a.R > 15 || a.S > 15; }
bool far_form(int form) { return form >= 1 && form <= 5; }    // built for such windows; few layers have them
constexpr int N_FORMS = sizeof(FORMS) / sizeof(FORMS[0]), FORM_64x16 = 5, FORM_RING4 = 14;
constexpr int MAX_SPLIT = 8, TARGET_WGS = 768, UNITS = 256;

int cdiv(int a, int b) { return (a + b - 1) / b; }

// Columns of a panel for a map of P x Q pixels and N images: the fewest tiles whose patches all fit PC pixels, then the
// narrowest patch; 0 if there is none.
int patch_panel(int N, int P, int Q, int BM, int PC, bool pool) {
    int best = 0;
    int64_t best_tiles = 0;
    int best_need = 0;
    for (int wt = pool ? 2 : 1; wt <= Q && 3 * (wt + 2) <= PC; wt += pool ? 2 : 1) {
        const int panels = (Q + wt - 1) / wt;
        const int64_t ppx = (int64_t)N * P * wt, tiles = (ppx + BM - 1) / BM;
        if (best && tiles * panels > best_tiles) continue;
        int need = 0;
        for (int64_t t = 0; t < tiles && need <= PC; ++t) {
            // first and last image row of the tile, counted with one empty row between images
            auto at = [&](int64_t i) {
                const int64_t row = pool ? i / 4 / (wt / 2) * 2 + (i >> 1 & 1) : i / wt;
                return row / P * (P + 1) + row % P;
            };
            need = std::max<int>(need, (int)(at(std::min(t * BM + BM, ppx) - 1) - at(t * BM) + 3) * (wt + 2));
        }
        if (need > PC) continue;
        if (!best || tiles * panels < best_tiles || need < best_need) {
            best = wt;
            best_tiles = tiles * panels;
            best_need = need;
        }
    }
    return best;
}

// Columns of the rectangles a ring's tiles are for this layer: the shape of which fewer cover the map; 0: tiles of consecutive pixels.  Rectangles
// that stick out at the edges are work for nothing, and a tenant beside it pays for that: where they are 14 and 23 % more than tiles of consecutive
// pixels (14 x 14 and 7 x 7 maps at batch 4) the layer alone is 1.5 to 5 us faster, but ResNet-18 + MobileNetV2 in fp32 take 388 us instead of 376,
// four networks at batch 8 842 instead of 836.  At one image (14 x 14: 8 % more) both gain.
int ring_rect(const OpArgs &a) {
    const int chunk = 64 / (a.dtype == MT_F32 ? 4 : 2);
    if (a.kind != MT_CONV || a.groups > 1 || a.R != 3 || a.S != 3 || a.sh != 1 || a.sw != 1 || a.ph != 1 || a.pw != 1 || a.C % chunk != 0) return 0;
    const int flat = cdiv(a.N * a.P * a.Q, 16), wide = a.N * cdiv(a.P, 2) * cdiv(a.Q, 8), square = a.N * cdiv(a.P, 4) * cdiv(a.Q, 4);
    if (10 * std::min(wide, square) > 11 * flat) return 0;
    return wide < square ? 8 : 4;
}
// Pixel tiles of a form: over the flattened map, per panel, or rectangles (panel < 0).
int pixel_tiles(const TileForm &f, const OpArgs &a, int panel) {
    if (panel < 0) return a.N * cdiv(a.P, 16 / -panel) * cdiv(a.Q, -panel);
    if (f.patch_pixels == 0) return cdiv(a.N * a.P * a.Q, f.bm);
    return cdiv(a.Q, panel) * cdiv(a.N * a.P * panel, f.bm);
}

void set_walk(OpArgs &a) {
    const TileForm &t = FORMS[a.form];
    const uint32_t es = a.dtype == MT_F32 ? 4 : 2, row = 128 / es, half = a.pool2 ? 2 : 1;
    const uint32_t q = (uint32_t)(a.panel > 0 ? a.panel : a.Q) / half, p = (uint32_t)a.P / half;
    const uint32_t tiles_m = (uint32_t)pixel_tiles(t, a, a.panel), tiles_n = (uint32_t)(a.n_pad / t.bn);
    const uint32_t advance = row * (uint32_t)(t.ring ? t.ring : t.kd);   // reduction elements from one stage, or row of a wave, to the next
    TileWalk &w = a.walk;
    w.total = tiles_m * tiles_n * (uint32_t)a.split_k;
    w.per_xcd = (w.total + XCDS - 1) / XCDS;
    w.pixels = (uint32_t)(a.N * a.P * a.Q);
    w.x_bytes = (uint32_t)((uint64_t)a.N * a.H * a.W * a.x_ct * es);
    w.w_bytes = (uint32_t)((uint64_t)a.n_pad * a.k_pad * es);
    w.flat = a.R == 1 && a.S == 1 && a.sh == 1 && a.sw == 1 && a.ph == 0 && a.pw == 0 && !a.pool2;
    w.units = a.panel < 0 ? (uint32_t)a.C / (row / 2) : t.patch_pixels > 0 ? (uint32_t)(a.C / TK) : (uint32_t)a.k_pad / (row * (uint32_t)t.kd);
    w.per = (w.units + (uint32_t)a.split_k - 1) / (uint32_t)a.split_k;
    w.split = divisor((uint32_t)a.split_k);
    w.tiles = divisor(a.tile_order ? tiles_m : tiles_n);
    w.q = divisor(a.panel < 0 ? (uint32_t)cdiv(a.Q, -a.panel) : q);
    w.pq = divisor(a.panel < 0 ? (uint32_t)(cdiv(a.Q, -a.panel) * cdiv(a.P, 16 / -a.panel)) : a.panel > 0 ? p : p * q);
    a.divq_m = w.q.m; a.divq_s1 = w.q.s1; a.divq_s2 = w.q.s2;            // for the fused 1x1 + depthwise kernels
    a.divpq_m = w.pq.m; a.divpq_s1 = w.pq.s1; a.divpq_s2 = w.pq.s2;
    w.c = divisor((uint32_t)a.C);
    w.adv_t = advance / (uint32_t)a.C;
    w.adv_c = advance % (uint32_t)a.C;
    w.inv_s = (uint32_t)((0x100000000ull + (uint32_t)a.S - 1) / (uint32_t)a.S);
    if (a.panel > 0) {
        w.panel_tiles = divisor((uint32_t)cdiv(a.N * a.P * a.panel, t.bm));
        w.inv_pw = ((1u << 20) + (uint32_t)a.panel + 1) / (uint32_t)(a.panel + 2);
        w.inv_h = ((1u << 20) + (uint32_t)a.H) / (uint32_t)(a.H + 1);
    }
}

}  // namespace

// Form, split and launch shape of a convolution (a fully connected layer is a 1x1 one) with C % 8 == 0 (fp32: C % 4 == 0 and a
// window of at most 15 x 15): a pure function of the layer's shape and of `choice` (see TileChoice).
bool plan_tile(OpArgs &a, TileChoice choice) {
    const int only = choice == TILE_NARROW ? FORM_64x16 : choice == TILE_RING4 ? FORM_RING4 : -1;
    const bool unsplit = choice == TILE_UNSPLIT;
    const bool f32 = a.dtype == MT_F32;
    const int row = f32 ? ROW<float> : TK;
    const bool far = far_window(a);
    if (a.C % (row / 8) != 0) return false;
    if (far && (f32 || (int64_t)a.R * a.S * a.S >= (int64_t)1 << 32)) return false;    // the division of a tap by S is exact below
    // fp32 with few output channels: the tiles would be half padding (144 -> 24 on 4 x 56 x 56 7.4 us, 5.7 with operands from
    // memory; 288 -> 32 on 4 x 149 x 149 41 / 37; short reductions are bound by their input: 32 -> 16 on 4 x 112 x 112 7.9 / 20)
    if (f32 && a.K <= 32 && a.gemm_k >= 128) return false;
    const bool patch_ok = patch_stageable(a);
    int panels[N_FORMS] = {};                               // of the patch forms; 0: no panel fits the patch
    bool patch_fits = false;
    for (int f = 0; patch_ok && f < N_FORMS; ++f) {
        if (FORMS[f].patch_pixels == 0) continue;
        panels[f] = patch_panel(a.N, a.P, a.Q, FORMS[f].bm, FORMS[f].patch_pixels, false);
        patch_fits = patch_fits || (panels[f] > 0 && FORMS[f].bm >= 64);
    }
    // Layers of K_PCONV's size run on a patch wherever one of 64 pixels or more fits: the estimate, fitted to all layers,
    // sometimes puts another tile first there, and it is the slower one.  us, measured with the kernels the estimate was fitted to, patch / tile of least estimate: 8 x 28 x 28
    // 128 -> 128 7.6 / 8.7, 56 x 56 128 -> 256 7.5 / 8.7, 112 x 112 64 -> 128 7.8 / 8.1, 5 x 35 x 35 64 -> 96 6.2 / 6.8, 40 x 7 x 7
    // 64 -> 320 6.2 / 6.7, 60 x 7 x 7 128 -> 256 7.7 / 8.6.  On maps of a few pixels a tile touches more images than such a patch
    // holds, and the estimate chooses among all forms (700 x 2 x 2, 512 -> 512: 64 x 32 patch 33.0, 128 x 64 tile 27.8).
    if (a.kernel_id == K_PCONV && !patch_fits) a.kernel_id = K_IGEMM_64x64;
    double best = 0;
    int form = -1, split = 1, panel = 0;
    for (int f = 0; f < N_FORMS; ++f) {
        const TileForm &t = FORMS[f];
        const TileCost &c = f32 ? t.single : t.half;
        if (c.start == 0) continue;
        if ((only >= 0 && f != only) || (far && !far_form(f))) continue;
        if (t.patch_pixels == 0 && a.kernel_id == K_PCONV) continue;
        if (t.bn > 64 && a.K <= t.bn / 2) continue;         // more than half of the tile would be padding
        const int w = panels[f];
        if (t.patch_pixels > 0 && w == 0) continue;
        const int tiles = pixel_tiles(t, a, w) * cdiv(a.K, t.bn);
        const int units = t.patch_pixels > 0 ? a.C / TK : cdiv(a.gemm_k, row * t.kd);     // what a split cuts
        for (int s = 1; s <= (unsplit || t.ring ? 1 : MAX_SPLIT); ++s) {
            if (s > 1 && (tiles * s > TARGET_WGS || (t.patch_pixels > 0 ? s > units : 2 * s * t.rows > units * t.kd))) break;
            const int per = cdiv(units, s);
            if (cdiv(units, per) != s) continue;            // an empty split
            const int ns = t.patch_pixels > 0 ? per * 9 / t.kd : cdiv(per * t.kd, t.rows), n = cdiv(tiles * s, UNITS);
            const double us = c.start + c.wave * (n - 1) + ns * (c.stage + c.crowd * (n - 1)) + (s > 1 ? c.split_once + c.split_each * s : 0.0);
            if (form < 0 || us < best) { best = us; form = f; split = s; panel = w; }
        }
    }
    if (form < 0) return false;
    const TileForm &t = FORMS[form];
    a.form = form;
    a.panel = panel = t.ring ? -ring_rect(a) : panel;
    a.split_k = split;
    a.block = t.threads;
    a.n_pad = cdiv(a.K, t.bn) * t.bn;
    a.k_pad = t.patch_pixels > 0 || panel < 0 ? a.gemm_k : cdiv(a.gemm_k, row * t.kd) * row * t.kd;
    // Consecutive tiles run on one XCD: they walk the channel tiles of one pixel tile when the activations are the larger
    // operand, the pixel tiles of one channel tile otherwise.
    a.tile_order = ((double)a.K * a.gemm_k > (double)a.N * a.H * a.W * a.C) ? 1 : 0;
    a.grid_x = cdiv(pixel_tiles(t, a, panel) * (a.n_pad / t.bn) * split, XCDS) * XCDS;
    a.grid_y = a.grid_z = 1;
    set_walk(a);
    return true;
}

bool tile_packs_filters(const OpArgs &a) {
    return a.form >= 0 && a.dtype != MT_F32 && a.panel == 0 && FORMS[a.form].ring == 0 && filters_packed(FORMS[a.form].bn, FORMS[a.form].bm, FORMS[a.form].kd);
}

// One ascending pass over the reduction on 64 x 16 tiles.
bool tile_is_narrow(const OpArgs &a) { return a.form == FORM_64x16 && a.split_k == 1; }

void describe_tile(const OpArgs &a, mt_op_form *out) {
    const TileForm &t = FORMS[a.form];
    std::snprintf(out->name, sizeof(out->name), "%s_%dx%d", t.ring ? "ring" : t.patch_pixels ? "patch" : "tile", t.bn, t.bm);
    out->tile_channels = t.bn;
    out->tile_pixels = t.bm;
    out->stage_slices = t.kd;
    out->ring_waves = t.ring;
    out->panel_columns = std::max(a.panel, 0);
}

void tile_workspace(const OpArgs &a, size_t *tiles, size_t *floats) {
    const TileForm &t = FORMS[a.form];
    *tiles = (size_t)pixel_tiles(t, a, a.panel) * (a.n_pad / t.bn);
    *floats = (size_t)a.split_k * t.bn * t.bm;
}

// The plan of the same convolution with a 2x2 max pooling in its epilogue.  False: the patch form has no panel of an even
// width for this map.
bool plan_tile_pooled(OpArgs &a) {
    const TileForm &t = FORMS[a.form];
    a.pool2 = 1;
    if (a.panel > 0) {
        const int was = pixel_tiles(t, a, a.panel);
        a.panel = patch_panel(a.N, a.P, a.Q, t.bm, t.patch_pixels, true);
        if (a.panel == 0 || (a.split_k > 1 && pixel_tiles(t, a, a.panel) > was)) return false;   // the workspace is laid out for `was`
        a.grid_x = cdiv(pixel_tiles(t, a, a.panel) * (a.n_pad / t.bn) * a.split_k, XCDS) * XCDS;
    }
    set_walk(a);
    return true;
}

template <typename T>
static int launch_tile_typed(const OpArgs &a, hipStream_t st, const OpArgs *mate, int n_mates) {
    const dim3 grid(a.grid_x), block(a.block);
    auto by_gather = [&](auto go) {
        if (a.C % ROW<T> != 0) go.template operator()<TG_CHUNK>();
        else if (a.R == 1 && a.S == 1 && a.ph == 0 && a.pw == 0) go.template operator()<TG_POINT>();
        else go.template operator()<TG_TAP>();
    };
    // Workgroups of a launch that has to fit a.units compute units at once, `room` of them per unit; 0: it fits, or need not.  Rings and 64x16 tiles, rows
    // gathered by 16-byte pieces (C not a multiple of 64, windows over 15), fp32 and launches of several tenants have no such form.
    OpArgs walked = a;
    auto walkers = [&](int room) {
        const uint32_t fit = (uint32_t)(a.units * room) / XCDS;
        if (a.units == 0 || mate || fit >= a.walk.per_xcd) return 0u;
        walked.walk.step = fit;
        count_launch(&LaunchRecorder::walked);
        return fit * XCDS;
    };
    auto tile = [&]<int BN, int BM, int WN, int WM, int WK, int KD, int NBUF>() {
        auto go = [&]<int MODE>() {
            if constexpr (sizeof(T) == 2 && (MODE == TG_POINT || MODE == TG_TAP) && BM > 16) {
                if (const uint32_t g = walkers(tile_room(BN, BM, KD)))
                    return launch((tile_walk_kernel<T, BN, BM, WN, WM, WK, KD, NBUF, MODE>), dim3(g), block, 0, st, walked);
            }
            if constexpr (std::is_same_v<T, float>) launch((tile_kernel<T, BN, BM, WN, WM, WK, KD, NBUF, MODE>), grid, block, 0, st, a);
            else MT_LAUNCH((tile_kernel<T, BN, BM, WN, WM, WK, KD, NBUF, MODE>), (tile_pair_kernel<T, BN, BM, WN, WM, WK, KD, NBUF, MODE>), grid, block, st, a, mate);
        };
        by_gather(go);
    };
    auto ring = [&]<int BN, int WK, int D>() {
        if (a.panel < 0) {
            if constexpr (std::is_same_v<T, float>) launch((ring_patch_kernel<T, BN / 16, WK>), grid, block, 0, st, a);
            else MT_LAUNCH((ring_patch_kernel<T, BN / 16, WK>), (ring_patch_pair_kernel<T, BN / 16, WK>), grid, block, st, a, mate);
            return;
        }
        auto go = [&]<int MODE>() {
            if constexpr (std::is_same_v<T, float>) launch((ring_kernel<T, BN, WK, D, MODE>), grid, block, 0, st, a);
            else MT_LAUNCH((ring_kernel<T, BN, WK, D, MODE>), (ring_pair_kernel<T, BN, WK, D, MODE>), grid, block, st, a, mate);
        };
        by_gather(go);
    };
    // The widest tiles have two stages of LDS (128x64 with filters in registers: three), so that two workgroups, or another tenant's, fit beside them; a launch that
    // has the chip to itself and at most one workgroup per unit waits for memory at every stage that way (0.75 us, matrix instructions 0.2) and takes four (five).
    // The order of the sums is the same.  us, two / four, both operands in LDS: ResNet-50 alone at batch 16, 32, 64 619 / 607, 903 / 862,
    // 1434 / 1401; used always: batch 64 1438 (layers of 392 workgroups and more), eight tenants at batch 16 2582 / 2712.
    const bool deep = a.alone && !mate && a.walk.total <= (uint32_t)UNITS;
    auto patch = [&]<int BN, int BM, int WN, int WM, int WK, int DW, int PC>() {
        if (const uint32_t g = walkers(patch_room(BN, BM)))
            return launch((patch_walk_kernel<T, BN, BM, WN, BM == 256 ? 2 : WM, BM == 256 ? 2 : WK, BM == 256 ? 3 : DW, PC>), dim3(g), block, 0, st, walked);
        MT_LAUNCH((patch_kernel<T, BN, BM, WN, WM, WK, DW, PC>), (patch_pair_kernel<T, BN, BM, WN, WM, WK, DW, PC>), grid, block, st, a, mate);
    };
    auto wide = [&]<int BN, int BM, int WN, int WM, int NBUF>() {
        count_launch(&LaunchRecorder::deep);
        by_gather([&]<int MODE>() { launch((tile_kernel<T, BN, BM, WN, WM, 1, 1, NBUF, MODE>), grid, block, 0, st, a); });
    };
    constexpr bool f32 = std::is_same_v<T, float>;
    if (far_window(a)) {
        if constexpr (!f32) {
            // us, element-wise gather / this: 17x17, 64 -> 64 on 40 x 40 66.7 / 17.5, 1x31, 64 -> 128 on 8 x 56 x 56 75.6 / 24.2, 16x3,
            // 128 -> 256 on 16 x 28 x 28 213 / 62.7
            auto far = [&]<int BN, int BM, int WN, int WM, int WK, int KD, int NBUF>() {
                MT_LAUNCH((tile_kernel<T, BN, BM, WN, WM, WK, KD, NBUF, TG_FAR>), (tile_pair_kernel<T, BN, BM, WN, WM, WK, KD, NBUF, TG_FAR>), grid, block, st, a, mate);
            };
            switch (a.form) {
                case 1: far.template operator()<128, 64, 4, 1, 1, 1, 3>(); break;
                case 2: far.template operator()<64, 64, 2, 2, 1, 1, 3>(); break;
                case 3: far.template operator()<64, 64, 2, 1, 4, 2, 4>(); break;
                case 4: far.template operator()<64, 32, 2, 1, 4, 2, 3>(); break;
                case 5: far.template operator()<64, 16, 4, 1, 1, 2, 3>(); break;
                default: return (int)hipErrorInvalidValue;
            }
            return (int)hipGetLastError();
        }
        return (int)hipErrorInvalidValue;
    }
    switch (a.form) {
        case 2: tile.template operator()<64, 64, 2, 2, 1, 1, 3>(); break;
        case 3: if constexpr (f32) tile.template operator()<64, 64, 2, 2, 2, 2, 3>(); else tile.template operator()<64, 64, 2, 1, 4, 2, 4>(); break;
        case 4: tile.template operator()<64, 32, 2, 1, 4, 2, 3>(); break;
        case 5: tile.template operator()<64, 16, 4, 1, 1, 2, 3>(); break;
        case 12: ring.template operator()<16, 8, 2>(); break;
        case 13: ring.template operator()<32, 4, 3>(); break;
        case 14: ring.template operator()<16, 4, 4>(); break;
        default:
            if constexpr (f32) {
                if (a.form != 11) return (int)hipErrorInvalidValue;
                tile.template operator()<32, 32, 2, 2, 2, 2, 4>();
            } else {
                switch (a.form) {
                    case 0: if (deep) wide.template operator()<128, 128, 2, 2, 4>(); else tile.template operator()<128, 128, 2, 2, 1, 1, 2>(); break;
                    case 1: if (deep) wide.template operator()<128, 64, 4, 1, 5>(); else tile.template operator()<128, 64, 4, 1, 1, 1, 3>(); break;
                    case 6: if (a.walk.units <= LONG_PATCHES) patch.template operator()<128, 256, 2, 4, 1, 4, 384>(); else patch.template operator()<128, 256, 2, 2, 2, 3, 384>(); break;
                    case 7: patch.template operator()<128, 128, 2, 2, 2, 6, 256>(); break;
                    case 8: patch.template operator()<128, 64, 4, 1, 2, 9, 192>(); break;
                    case 9: patch.template operator()<64, 64, 2, 1, 4, 9, 192>(); break;
                    case 10: patch.template operator()<64, 32, 2, 1, 4, 9, 128>(); break;
                    default: return (int)hipErrorInvalidValue;
                }
            }
    }
    return (int)hipGetLastError();
}

int launch_tile(const OpArgs &a, void *stream, const OpArgs *mate, int n_mates) {
    if (mate && (n_mates < 1 || n_mates >= COISSUE_MAX || a.groups > 1)) return (int)hipErrorInvalidValue;
    if (a.dtype == MT_F32) return mate ? (int)hipErrorInvalidValue : launch_tile_typed<float>(a, (hipStream_t)stream, nullptr, 0);
    if (a.dtype == MT_F16) return launch_tile_typed<f16>(a, (hipStream_t)stream, mate, n_mates);
    if (a.dtype == MT_BF16) return launch_tile_typed<bf16>(a, (hipStream_t)stream, mate, n_mates);
    return (int)hipErrorInvalidValue;
}

}  // namespace mt

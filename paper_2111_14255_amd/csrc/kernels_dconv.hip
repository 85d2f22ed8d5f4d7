// fp32 convolutions whose matrix-core operands come straight from memory: no LDS tiles, no barrier in the reduction.  They are the
// ones the tile kernels (kernels_tile.hip) do not take: channel counts that are no multiple of 4, windows of more than 15 rows
// or columns, few output channels.
//
// A wave owns TN x TM tiles of 16 output channels x 16 pixels.  A reduction step is 16 elements of a filter row and of an
// im2col row: lane l loads the four elements of row l % 16 that start at 4 * (l / 16), which feed four
// v_mfma_f32_16x16x4_f32 (instruction e multiplies element e of every 16-byte piece, so the four lane groups hold the reduction
// elements e, 4 + e, 8 + e, 12 + e: the same for both operands, and any order of the sum is a correct one).  D steps are
// in flight in registers; the one consumed is refilled at once.  Pixels outside the image and steps beyond the end get
// an out-of-range offset, for which the buffer load returns zeros.
//
// WK > 1: WK waves share the tile and split the reduction into contiguous ranges; their sums meet in LDS and are added in
// range order.  That is the form for small maps: the whole reduction of a tile is in flight after one trip to memory.
//
// The matrix cores need 32 cycles per instruction, so operands from the L1 keep up with them; the kernel replaces
// one thread per output element (MI355X, ResNet-18 + MobileNetV2 at batch 4 with every layer on it: 6609 us before, 552 us).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.h"
#include "device_types.h"
#include "mfma.h"

namespace mt {

namespace {

constexpr uint32_t DC_OOB = 0x80000000u;     // beyond any tensor: buffer loads return zeros
constexpr int DC_TABLE = 2048;               // reduction elements of the element-wise gather (a table entry each)

// How an im2col row is gathered.  Tap-uniform: the channels are a multiple of a step, so a step lies inside one filter
// tap.  Piecewise: they are a multiple of 16 bytes, every lane group has a tap of its own.  Element-wise: any channel
// count (first layers), offsets from a table in LDS.
constexpr int DC_ELEMENT = 0, DC_PIECE = 1, DC_UNIFORM = 2;

template <int TN, int TM, int WN, int WM, int WK, int D, int MODE>
__global__ void __launch_bounds__(64 * WN * WM * WK) dconv_kernel(OpArgs args) {
    OpArgs a = args;
    hold(a.x, a.w, a.walk.total, a.walk.per_xcd, a.walk.pixels, a.N, a.walk.tiles.d, a.walk.tiles.m, a.walk.tiles.s1, a.walk.tiles.s2, a.walk.split.d, a.walk.split.m,
         a.walk.split.s1, a.walk.split.s2, a.walk.c.d, a.walk.c.m, a.walk.c.s1, a.walk.c.s2, a.tile_order, a.k_pad, a.x_ct, a.x_coff, a.H, a.W, a.C, a.S, a.sh, a.sw, a.ph, a.pw, a.P, a.Q, a.prio, a.K,
         a.act, a.res_ct, a.y_coff, a.y_ct, a.bias, a.res, a.y, a.gemm_k, a.n_pad, a.divq_m, a.divq_s1, a.divq_s2, a.divpq_m, a.divpq_s1, a.divpq_s2);
    set_wave_priority(a.prio);
    constexpr int ES = 4, KST = 16, EPV = 4;
    constexpr int NW = WN * WM * WK, BN = 16 * TN * WN, BM = 16 * TM * WM, F = TN * TM;
    __shared__ __attribute__((aligned(16))) f32x4 red[WK > 1 ? NW * F * 64 : 1];
    __shared__ int2 table[MODE == DC_ELEMENT ? DC_TABLE : 1];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave / (WN * WM), wn = wave % WN, wm = (wave / WN) % WM;
    const int row = lane & 15, grp = lane >> 4;

    const int M = (int)a.walk.pixels;
    const uint32_t vid = (blockIdx.x % 8) * a.walk.per_xcd + blockIdx.x / 8;   // each XCD's L2 serves a contiguous tile range
    if (vid >= a.walk.total) return;                                   // the whole workgroup
    const int slow = (int)divide(vid, a.walk.tiles), fast = (int)(vid - (uint32_t)slow * a.walk.tiles.d);
    const int tn_idx = a.tile_order ? slow : fast, tm_idx = a.tile_order ? fast : slow;
    const int n0 = tn_idx * BN + wn * 16 * TN, m0 = tm_idx * BM + wm * 16 * TM;

    if constexpr (MODE == DC_ELEMENT) {
        for (int j = tid; j < a.k_pad; j += 64 * NW) {
            const int rs = (int)divide((uint32_t)j, a.walk.c), c = j - rs * a.C, r = (int)divide((uint32_t)rs, a.walk.split), s = rs - r * a.S;
            table[j] = j < a.gemm_k ? int2{((r * a.W + s) * a.x_ct + c) * ES, r << 16 | s} : int2{0, 0x7fff << 16};
        }
        __syncthreads();
    }

    const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void *>(a.x), 0, (int)((int64_t)a.N * a.H * a.W * a.x_ct * ES), 0x00027000);
    const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void *>(a.w), 0, (int)((int64_t)a.n_pad * a.k_pad * ES), 0x00027000);

    // pixel rows of this lane
    int ih0[TM], iw0[TM], xbase[TM];
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        const int m = m0 + 16 * j + row;
        const bool ok = m < M;
        const uint32_t mm = ok ? (uint32_t)m : 0u;
        const uint32_t t1 = __umulhi(a.divpq_m, mm);
        const int n = (int)((t1 + ((mm - t1) >> a.divpq_s1)) >> a.divpq_s2);
        const uint32_t rem = mm - (uint32_t)n * (uint32_t)(a.P * a.Q);
        const uint32_t t2 = __umulhi(a.divq_m, rem);
        const int p = (int)((t2 + ((rem - t2) >> a.divq_s1)) >> a.divq_s2);
        const int q = (int)(rem - (uint32_t)p * (uint32_t)a.Q);
        ih0[j] = ok ? p * a.sh - a.ph : -0x10000;                      // a pixel beyond the last one is outside the image at every tap
        iw0[j] = q * a.sw - a.pw;
        xbase[j] = ((n * a.H + (ok ? p * a.sh - a.ph : 0)) * a.W + iw0[j]) * a.x_ct * ES + a.x_coff * ES;
    }
    uint32_t wrow[TN];
#pragma unroll
    for (int i = 0; i < TN; ++i) wrow[i] = (uint32_t)(((n0 + 16 * i + row) * a.k_pad + grp * EPV) * ES);   // rows beyond n_pad read zeros

    const int nsteps = (a.gemm_k + KST - 1) / KST;
    const int per = (nsteps + WK - 1) / WK;
    const int s_begin = wk * per, s_end = min(nsteps, s_begin + per);

    // position of the next step to load: tap and channel of its first element
    int u_r = 0, u_s = 0, u_c = 0;
    if constexpr (MODE == DC_UNIFORM) {
        const int j0 = s_begin * KST, rs = (int)divide((uint32_t)j0, a.walk.c);
        u_c = j0 - rs * a.C;
        u_r = (int)divide((uint32_t)rs, a.walk.split);
        u_s = rs - u_r * a.S;
    } else if constexpr (MODE == DC_PIECE) {
        const int j0 = s_begin * KST + grp * EPV, rs = (int)divide((uint32_t)j0, a.walk.c);
        u_c = j0 - rs * a.C;
        u_r = (int)divide((uint32_t)rs, a.walk.split);
        u_s = rs - u_r * a.S;
    }
    u32x4 fa[D][TN], fb[D][TM];
    auto load_step = [&](int s, u32x4 (&wa)[TN], u32x4 (&xb)[TM]) {
        const bool live = s < s_end;
#pragma unroll
        for (int i = 0; i < TN; ++i)
            wa[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, live ? wrow[i] : DC_OOB, (uint32_t)(s * 64), 0);
        if constexpr (MODE == DC_ELEMENT) {
            const int j0 = s * KST + grp * EPV;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int2 t = live ? table[j0 + e] : int2{0, 0x7fff << 16};
                const int r = t.y >> 16, sx = t.y & 0xffff;
#pragma unroll
                for (int j = 0; j < TM; ++j) {
                    const bool v = ((uint32_t)(ih0[j] + r) < (uint32_t)a.H) & ((uint32_t)(iw0[j] + sx) < (uint32_t)a.W);
                    xb[j][e] = __builtin_amdgcn_raw_buffer_load_b32(rsrc_x, v ? (uint32_t)(xbase[j] + t.x) : DC_OOB, 0, 0);
                }
            }
        } else {
            const int off = MODE == DC_UNIFORM ? ((u_r * a.W + u_s) * a.x_ct + u_c) * ES + grp * 16 : ((u_r * a.W + u_s) * a.x_ct + u_c) * ES;
            const bool tap = live & (u_r < a.R);
#pragma unroll
            for (int j = 0; j < TM; ++j) {
                const bool v = tap & ((uint32_t)(ih0[j] + u_r) < (uint32_t)a.H) & ((uint32_t)(iw0[j] + u_s) < (uint32_t)a.W);
                xb[j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, v ? (uint32_t)(xbase[j] + off) : DC_OOB, 0, 0);
            }
            u_c += KST;
            if constexpr (MODE == DC_UNIFORM) {
                if (u_c >= a.C) {                                      // scalar
                    u_c = 0;
                    if (++u_s == a.S) { u_s = 0; ++u_r; }
                }
            } else {
                while (u_c >= a.C) {                                   // channels may be fewer than a step
                    u_c -= a.C;
                    if (++u_s == a.S) { u_s = 0; ++u_r; }
                }
            }
        }
    };

    f32x4 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < D; ++d) load_step(s_begin + d, fa[d], fb[d]);
    for (int s0 = s_begin; s0 < s_end; s0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (s0 + d < s_end) {
#pragma unroll
                for (int i = 0; i < TN; ++i)
#pragma unroll
                    for (int j = 0; j < TM; ++j) acc[i][j] = Mma<float, 16>::run(fa[d][i], fb[d][j], acc[i][j]);
            }
            if (s0 + D < s_end) load_step(s0 + d + D, fa[d], fb[d]);
        }
    }

    // ---- epilogue: bias, residual, activation.  A lane holds 4 consecutive channels of one pixel.
    const Results y = results_in(a.y);
    const float *res = (const float *)a.res;
    const bool vec_ok = (a.y_ct % 4 == 0) & (a.y_coff % 4 == 0) & (a.res_ct % 4 == 0);
    auto finish = [&](f32x4 v4, int i, int j) {
        const int m = m0 + 16 * j + row, k = n0 + 16 * i + 4 * grp;
        const bool live = (m < M) & (k < a.K);
        const float4 b = live ? *reinterpret_cast<const float4 *>(a.bias + k) : float4{0.f, 0.f, 0.f, 0.f};    // padded to n_pad
        float v[4] = {v4[0] + b.x, v4[1] + b.y, v4[2] + b.z, v4[3] + b.w};
        if (!live) return;
        if (vec_ok && k + 4 <= a.K) {
            if (res) {
                float rv[4];
                load_pack<float, 4>(res + (int64_t)m * a.res_ct + k, rv);
#pragma unroll
                for (int t = 0; t < 4; ++t) v[t] += rv[t];
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = apply_act(v[t], a.act);
            store_pack<float, 4>(y, (uint32_t)m * (uint32_t)a.y_ct + (uint32_t)(a.y_coff + k), v);
        } else {
            for (int t = 0; t < 4 && k + t < a.K; ++t) {
                float f = v[t];
                if (res) f += res[(int64_t)m * a.res_ct + k + t];
                store_one<float>(y, (uint32_t)m * (uint32_t)a.y_ct + (uint32_t)(a.y_coff + k + t), apply_act(f, a.act));
            }
        }
    };
    if constexpr (WK == 1) {
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j) finish(acc[i][j], i, j);
    } else {
        f32x4 *mine = red + (size_t)wave * F * 64;
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j) mine[(i * TM + j) * 64 + lane] = acc[i][j];
        __syncthreads();
        // the waves of a tile deal its 16 x 16 pieces out between them; every piece is added in range order
#pragma unroll
        for (int f = 0; f < F; ++f) {
            if (f % WK != wk) continue;
            f32x4 v = red[((size_t)(wn + WN * wm) * F + f) * 64 + lane];
#pragma unroll
            for (int g = 1; g < WK; ++g) {
                const f32x4 p = red[((size_t)(g * WN * WM + wn + WN * wm) * F + f) * 64 + lane];
                v += p;
            }
            finish(v, f / TM, f % TM);
        }
    }
    results_stored();
}

// The tilings, widest first: channels x pixels of a workgroup, waves along the reduction.
struct DcTile { int bn, bm, wk, waves; };
constexpr DcTile DC_F32[] = {{64, 64, 1, 4}, {32, 32, 4, 4}, {32, 16, 4, 4}, {16, 16, 8, 8}};

}  // namespace

// The tiling of least estimated time, 0 if the element-wise gather's table is too small for the layer (it then
// stays with one thread per output).  Estimate in cycles of a compute unit: the matrix instructions of its workgroups, or
// the operand bytes of its workgroups at 64 per cycle, whichever is longer, plus the exchange of the partial sums.  256
// units; with fewer workgroups than units the time is that of one workgroup.
int dconv_f32_plan(int M, int K, int gemm_k, int C) {
    if (C % 4 != 0 && (gemm_k + 15) / 16 * 16 > DC_TABLE) return 0;
    double best = 0;
    int pick = 0;
    for (int i = 0; i < (int)(sizeof(DC_F32) / sizeof(DC_F32[0])); ++i) {
        const DcTile &t = DC_F32[i];
        const int64_t tiles = (int64_t)((M + t.bm - 1) / t.bm) * ((K + t.bn - 1) / t.bn);
        const double rounds = (double)((tiles + 255) / 256);
        const double mfma = rounds * (double)t.bn * t.bm * gemm_k / 256.0, feed = rounds * (double)(t.bn + t.bm) * gemm_k * 4 / 64.0;
        const double c = std::max(mfma, feed) + (t.wk > 1 ? 300.0 : 0.0);
        if (pick == 0 || c < best) { best = c; pick = i + 1; }
    }
    return pick;
}
void dconv_f32_tile(int form, int *channels, int *pixels) {
    *channels = DC_F32[form - 1].bn;
    *pixels = DC_F32[form - 1].bm;
}
int dconv_f32_grid(int form, int M, int K) {
    const DcTile &t = DC_F32[form - 1];
    return (((M + t.bm - 1) / t.bm) * ((K + t.bn - 1) / t.bn) + 7) / 8 * 8;
}

// walk.tiles: workgroup -> (slow, fast) tile index; walk.c, split: divisors of the reduction index by the channels and of a tap by S.
void plan_dconv_f32(OpArgs &a) {
    const DcTile &t = DC_F32[a.wk - 1];
    TileWalk &w = a.walk;
    w.pixels = (uint32_t)(a.N * a.P * a.Q);
    const uint32_t tiles_m = (w.pixels + (uint32_t)t.bm - 1) / (uint32_t)t.bm, tiles_n = (uint32_t)((a.K + t.bn - 1) / t.bn);
    w.total = tiles_m * tiles_n;
    w.per_xcd = (w.total + 7) / 8;
    w.tiles = divisor(a.tile_order ? tiles_m : tiles_n);
    w.c = divisor((uint32_t)a.C);
    w.split = divisor((uint32_t)a.S);
}

int launch_dconv_f32(const OpArgs &a, void *stream) {
    hipStream_t st = (hipStream_t)stream;
    const dim3 grid(a.grid_x);
    auto go = [&]<int MODE>() {
        switch (a.wk) {
            case 1: launch((dconv_kernel<2, 2, 2, 2, 1, 4, MODE>), grid, dim3(256), 0, st, a); break;
            case 2: launch((dconv_kernel<2, 2, 1, 1, 4, 4, MODE>), grid, dim3(256), 0, st, a); break;
            case 3: launch((dconv_kernel<2, 1, 1, 1, 4, 6, MODE>), grid, dim3(256), 0, st, a); break;
            default: launch((dconv_kernel<1, 1, 1, 1, 8, 8, MODE>), grid, dim3(512), 0, st, a); break;
        }
    };
    if (a.C % 16 == 0) go.template operator()<DC_UNIFORM>();
    else if (a.C % 4 == 0) go.template operator()<DC_PIECE>();
    else go.template operator()<DC_ELEMENT>();
    return (int)hipGetLastError();
}

}  // namespace mt

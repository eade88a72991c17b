// conv_f32.h -- FP32 convolution (Methodology, Table 2: the FP32 Conv2D row)
// on the bf16 matrix cores, C_in a multiple of 32: every float as three bf16
// terms, eight products kept (f32_split.h).  Compiled as a part of
// k_gemm_nt.hip.
//
//  1. Prep: x NCHW -> a zero-bordered NHWC image of split values,
//     xs [N][H+2p][W+2p][Ci/32][3][32] bf16 (a pixel's 32 channels: h, m, l,
//     192 contiguous bytes), and w OIHW -> ws [Cop][Kd/32][3][32] with
//     k = (kh*KW + kw)*Ci + ci; both times kSplitScale.
//  2. Contraction: a K tile is 32 channels of one kernel tap, gathered per
//     pixel straight from the image into LDS (direct-to-LDS loads, a ring of
//     stages).  A wave whose sums are not all finite contracts its tile again
//     on the fp32 matrix cores from x and w.  Few tiles split K over
//     workgroups; the partial outputs are added in split order.
//
// Bound (8x64x56x56 -> 128, 3x3): 392 tiles on 256 CUs, so 17 us of matrix
// products on the busiest SIMDs; the kernel takes about 31 us of the 38 (46 on
// the fp32 matrix cores).  Tiles of 128 x 128 (eight waves, three stages) and
// six stages of 64 x 64 gained nothing there (measured with six products a
// multiply-add), and the former lose where C_out is not a multiple of 128.
#pragma once

#include <algorithm>
#include <type_traits>

#include "f32_split.h"
#include "qx_internal.h"

namespace qx {

typedef float f16x __attribute__((ext_vector_type(16)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// Blocks of 64 consecutive bordered positions of one image and 32 channels
// (a thread splits eight channels of a position, coalesced over positions;
// LDS turns the result into rows of 192 bytes), then blocks of 256 threads of
// eight channels of one weight tap.
__global__ __launch_bounds__(256) void k_conv_prep_f32(const ConvF32Params p) {
    constexpr int ROW = 192 + 16;
    __shared__ __align__(16) unsigned char t[64 * ROW];
    const ConvGeom& g = p.g;
    const int tid = threadIdx.x;
    const bool image = (int)blockIdx.x < p.xblocks;
    const int nc = g.Ci / 32;
    const int Hp = g.H + 2 * g.pad, Wp = g.W + 2 * g.pad, pos_n = Hp * Wp;
    const int per_img = (pos_n + 63) / 64;
    float v[8] = {};
    int img = 0, chunk = 0, pos0 = 0, co = 0;
    int64_t wv = 0;
    if (image) {
        chunk = blockIdx.x % nc;
        const int ib = blockIdx.x / nc;
        img = ib / per_img;
        pos0 = (ib - img * per_img) * 64;
        const int pos = pos0 + (tid & 63), hp = pos / Wp, h = hp - g.pad, w = pos - hp * Wp - g.pad;
        if (h >= 0 && h < g.H && w >= 0 && w < g.W) {
            const int64_t hw = (int64_t)g.H * g.W;
            const float* src = p.x + ((int64_t)img * g.Ci + chunk * 32 + (tid >> 6) * 8) * hw + (int64_t)h * g.W + w;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = src[e * hw];
        }
    } else {
        wv = (int64_t)((int)blockIdx.x - p.xblocks) * 256 + tid;
        const int kc = p.Kd / 8;
        co = (int)(wv / kc);
        const int k0 = (int)(wv - (int64_t)co * kc) * 8, tap = k0 / g.Ci, ci = k0 - tap * g.Ci;
        if (co < p.Co) {
            const int taps = g.KH * g.KW;
            const float* src = p.w + ((int64_t)co * g.Ci + ci) * taps + tap;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = src[e * taps];
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] *= kSplitScale;
    b8 h, m, l;
    split3(v, h, m, l);
    if (!image) {
        if (co >= p.Cop) return;
        unsigned char* dst = p.ws + (wv / 4 * 3) * 64 + (wv & 3) * 16;   // 32-channel chunk wv / 4
        *(b8*)dst = h;
        *(b8*)(dst + 64) = m;
        *(b8*)(dst + 128) = l;
        return;
    }
    unsigned char* row = &t[(tid & 63) * ROW + (tid >> 6) * 16];
    *(b8*)row = h;
    *(b8*)(row + 64) = m;
    *(b8*)(row + 128) = l;
    __syncthreads();
    unsigned char* dst = p.xs + (((int64_t)img * pos_n + pos0) * nc + chunk) * 192;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int q = tid + 256 * i, r = q / 12, c = q - r * 12;
        if (pos0 + r < pos_n) *(u4*)(dst + (int64_t)r * nc * 192 + c * 16) = *(const u4*)&t[r * ROW + c * 16];
    }
}

// s_waitcnt vmcnt(N), N in [0, 63]
template <int N>
__device__ __forceinline__ void wait_loads() {
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// BM output channels x BN pixels per workgroup, waves of 64 x WN.  An LDS row
// is the 192 bytes of a pixel (or weight row) of the K tile; within each
// 64-byte plane the 16-byte chunks are swizzled by (row >> 2) & 3, so the 16
// rows of one ds_read_b128 phase fall on 64 different banks.
template <int BM, int BN, int WN, int STAGES>
__global__ __launch_bounds__(BM * BN / WN) void k_conv_f32(const ConvF32Params p) {
    constexpr int NTH = BM * BN / WN;
    constexpr int WAVES_N = BN / WN, TN = WN / 32;
    constexpr int AL = BM * 12 / NTH, BL = BN * 12 / NTH, LPT = AL + BL;
    static_assert(AL * NTH == BM * 12 && BL * NTH == BN * 12, "whole loads");
    __shared__ __align__(16) unsigned char As[STAGES][BM * 192];
    __shared__ __align__(16) unsigned char Bs[STAGES][BN * 192];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, hh = lane >> 5;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    // consecutive ids go to different XCDs: give each XCD a contiguous range
    // of pixel tiles (all channel tiles of a pixel tile next to each other)
    const int total = gridDim.x, xcd = blockIdx.x & 7;
    const int pid = xcd * (total >> 3) + min(xcd, total & 7) + ((int)blockIdx.x >> 3);
    const int tiles_m = (p.Co + BM - 1) / BM;
    const int m0 = pid % tiles_m * BM, n0 = pid / tiles_m * BN;
    const ConvGeom& g = p.g;
    const int Wp = g.W + 2 * g.pad, Hp = g.H + 2 * g.pad;
    const int pix_bytes = g.Ci * 6;

    unsigned oa[AL], ob[BL];
#pragma unroll
    for (int i = 0; i < AL; ++i) {
        const int q = tid + NTH * i, row = q / 12, pc = q - row * 12;
        oa[i] = (unsigned)row * (unsigned)(p.Kd * 6) + (pc >> 2) * 64 + ((pc & 3) ^ ((row >> 2) & 3)) * 16;
    }
#pragma unroll
    for (int i = 0; i < BL; ++i) {
        const int q = tid + NTH * i, row = q / 12, pc = q - row * 12;
        int pix = n0 + row;
        if (pix >= p.P) pix = 0;     // never stored
        const int img = pix / p.hw, rem = pix - img * p.hw;
        const int oh = rem / g.Wo, ow = rem - oh * g.Wo;
        ob[i] = (unsigned)(((int64_t)(img * Hp + oh * g.stride) * Wp + ow * g.stride) * pix_bytes) + (pc >> 2) * 64 +
                ((pc & 3) ^ ((row >> 2) & 3)) * 16;
    }
    const unsigned char* a_panel = p.ws + (int64_t)m0 * p.Kd * 6;
    int tap_h = 0, tap_w = 0, tap_c = 0;
    const unsigned wave_u = __builtin_amdgcn_readfirstlane(wave);
    const unsigned lds_a0 = (unsigned)(uintptr_t)&As[0][0] + wave_u * 1024;
    const unsigned lds_b0 = (unsigned)(uintptr_t)&Bs[0][0] + wave_u * 1024;
    // load i of tile t (A rows first); `next` moves to the tile after
    const int tile0 = blockIdx.y * p.tiles_per_split;    // K tiles [tile0, tile0 + ktiles) of the sum
    const int ktiles = min(p.tiles_per_split, p.Kd / 32 - tile0);
    {
        const int chunks = g.Ci / 32, tap = tile0 / chunks;
        tap_c = (tile0 - tap * chunks) * 192;
        tap_h = tap / g.KW;
        tap_w = tap - tap_h * g.KW;
    }
    const unsigned char *ab = a_panel + (int64_t)tile0 * 192, *bb = p.xs + (int64_t)(tap_h * Wp + tap_w) * pix_bytes + tap_c;
    auto load = [&](int t, int i) {
        const int s = t % STAGES;
        if (i < AL)
            asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                         :: "v"(oa[i < AL ? i : 0]), "s"(ab), "s"(lds_a0 + s * BM * 192 + NTH * 16 * i) : "memory", "m0");
        else
            asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                         :: "v"(ob[i < AL ? 0 : i - AL]), "s"(bb), "s"(lds_b0 + s * BN * 192 + NTH * 16 * (i - AL))
                         : "memory", "m0");
    };
    auto next = [&]() {
        ab += 192;
        tap_c += 192;
        if (tap_c == pix_bytes) {
            tap_c = 0;
            if (++tap_w == g.KW) {
                tap_w = 0;
                ++tap_h;
            }
        }
        bb = p.xs + (int64_t)(tap_h * Wp + tap_w) * pix_bytes + tap_c;
    };

    f16x acc[2][TN], low[2][TN];   // sums of the h h products and of the smaller ones
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = low[i][j] = f16x{};
    struct Frag {
        b8 a[2][3], b[TN][3];
    };
    const int arow = wm * 64 + l32, brow = wn * WN + l32, swz = (l32 >> 2) & 3;
    auto read = [&](int t, int ks, Frag& f) {
        const int c = ((2 * ks + hh) ^ swz) * 16;
        const unsigned char* A0 = &As[t % STAGES][arow * 192 + c];
        const unsigned char* B0 = &Bs[t % STAGES][brow * 192 + c];
#pragma unroll
        for (int q = 2; q >= 0; --q) {
#pragma unroll
            for (int i = 0; i < 2; ++i) f.a[i][q] = *(const b8*)(A0 + i * 32 * 192 + q * 64);
#pragma unroll
            for (int j = 0; j < TN; ++j) f.b[j][q] = *(const b8*)(B0 + j * 32 * 192 + q * 64);
        }
    };
    auto term = [&](const Frag& f, int pa, int pb) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                f16x& sum = pa + pb ? low[i][j] : acc[i][j];
                sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i][pa], f.b[j][pb], sum, 0, 0, 0);
            }
    };
    // smallest products first
    constexpr int TERMS = 8, PA[TERMS] = {2, 1, 2, 1, 0, 1, 0, 0}, PB[TERMS] = {1, 2, 0, 1, 2, 0, 1, 0};

    // Each 16-k step's fragments are read while the step before is
    // multiplied, and a tile's loads are issued between the products of the
    // second step, once every wave has read the tile they overwrite.
#pragma unroll
    for (int s = 0; s < STAGES; ++s)
        if (s < ktiles) {
#pragma unroll
            for (int i = 0; i < LPT; ++i) load(s, i);
            next();
        }
    if (ktiles >= STAGES) wait_loads<(STAGES - 1) * LPT>();
    else wait_loads<0>();
    __syncthreads();
    Frag f0, f1;
    read(0, 0, f0);
    // (tile t of those with a tile t + STAGES to load: `more`)
    auto step = [&](int t, auto more) {
        read(t, 1, f1);
#pragma unroll
        for (int e = 0; e < TERMS; ++e) term(f0, PA[e], PB[e]);
        // tile t + 1 has landed
        if (t + STAGES - 1 < ktiles) wait_loads<(STAGES - 2) * LPT>();
        else wait_loads<0>();
        __syncthreads();
        read(t + 1, 0, f0);
#pragma unroll
        for (int e = 0; e < TERMS; ++e) {
            term(f1, PA[e], PB[e]);
            if constexpr (decltype(more)::value) {
#pragma unroll
                for (int i = e * LPT / TERMS; i < (e + 1) * LPT / TERMS; ++i) load(t + STAGES, i);
            }
        }
        if constexpr (decltype(more)::value) next();
    };
    int tile = 0;
    for (; tile + STAGES < ktiles; ++tile) step(tile, std::true_type{});
    for (; tile + 1 < ktiles; ++tile) step(tile, std::false_type{});
    read(tile, 1, f1);
#pragma unroll
    for (int e = 0; e < TERMS; ++e) term(f0, PA[e], PB[e]);
#pragma unroll
    for (int e = 0; e < TERMS; ++e) term(f1, PA[e], PB[e]);

    const int taps = g.KH * g.KW, img_px = g.H * g.W;
    float* out = p.part ? p.part + (int64_t)blockIdx.y * p.part_stride : p.y;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int gn = n0 + wn * WN + j * 32 + l32, pix = min(gn, p.P - 1);
        const int n_img = pix / p.hw, n_pix = pix - n_img * p.hw;
        bool redo = false;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[i][j][r] = (acc[i][j][r] + low[i][j][r]) * (1.f / (kSplitScale * kSplitScale));
                redo |= !(fabsf(acc[i][j][r]) < INFINITY);
            }
        if (__ballot(redo) != 0) {
            const int oh = n_pix / g.Wo, ow = n_pix - oh * g.Wo;
            const float* xi = p.x + ((int64_t)n_img * g.Ci + hh) * img_px;
            const float* wi[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                wi[i] = p.w + ((int64_t)min(m0 + wm * 64 + i * 32 + l32, p.Co - 1) * g.Ci + hh) * taps;
                acc[i][j] = f16x{};
            }
            const int chunks = g.Ci / 32;
            int tap = tile0 / chunks, ci = (tile0 - tap * chunks) * 32, kh = tap / g.KW, kw = tap - kh * g.KW;
            // A K tile at a time, its loads in flight together.  8x64x56x56 ->
            // 128 with every wave here 165 us, with one of them 92 (183 and
            // 111 with half a tile and divisions for every element).
            for (int t = 0; t < ktiles; ++t) {
                const int ih = oh * g.stride + kh - g.pad, iw = ow * g.stride + kw - g.pad;
                const bool in = ih >= 0 && ih < g.H && iw >= 0 && iw < g.W;
                const float* xs = xi + (int64_t)ci * img_px + (in ? ih * g.W + iw : 0);
                float bv[16], av[2][16];
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    bv[e] = xs[(unsigned)(2 * e) * (unsigned)img_px];
#pragma unroll
                    for (int i = 0; i < 2; ++i) av[i][e] = wi[i][((int64_t)ci + 2 * e) * taps + tap];
                }
#pragma unroll
                for (int e = 0; e < 16; ++e)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i][e], in ? bv[e] : 0.f, acc[i][j], 0, 0, 0);
                if ((ci += 32) == g.Ci) {
                    ci = 0;
                    ++tap;
                    if (++kw == g.KW) {
                        kw = 0;
                        ++kh;
                    }
                }
            }
        }
        if (gn >= p.P) continue;
        float* y = out + (int64_t)n_img * p.Co * p.hw + n_pix;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int gm = m0 + wm * 64 + i * 32 + 8 * (r >> 2) + 4 * hh + (r & 3);
                if (gm < p.Co) __builtin_nontemporal_store(acc[i][j][r], &y[(int64_t)gm * p.hw]);
            }
    }
}

// Tiles of 64 x 128 (four waves, two workgroups per CU) from 256 of them on;
// below, tiles of 64 x 64 (two waves, three workgroups per CU), K split until
// the grid fills three workgroups per CU or a split has six K tiles (a tile
// takes about 0.7 us of a lone workgroup; the reduction launch about 4 us).
// Steps, FP32 matrix cores before / these: 8x64x56x56 -> 128 3x3 44.6 / 32 us
// (64 x 64 tiles 44); 4x64x112x112 -> 64 96 / 40 (64 x 64 48); 1x256x7x7 ->
// 256 93 / 17 (one split 51); 8x256x14x14 -> 256 99 / 30 (53); 1x1 over 256
// channels of 2x28x28 21 / 13.6 (two splits of four tiles 15.7).
void conv_f32_shape(int64_t Co, int64_t P, int64_t Kd, int* bn, int64_t* splits, int64_t* per) {
    const int64_t tm = (Co + 63) / 64, kt = Kd / 32;
    *bn = tm * ((P + 127) / 128) >= 256 ? 128 : 64;
    const int64_t tiles = tm * ((P + *bn - 1) / *bn);
    const int64_t s = *bn == 128 ? 1 : std::max<int64_t>(1, std::min(768 / tiles, kt / 6));
    *per = (kt + s - 1) / s;
    *splits = (kt + *per - 1) / *per;
}

void build_conv_f32(const ConvF32Params& p0, int bn, int splits, LaunchRec* prep, LaunchRec* rec) {
    ConvF32Params p = p0;
    const ConvGeom& g = p.g;
    const int64_t pos = (int64_t)(g.H + 2 * g.pad) * (g.W + 2 * g.pad);
    p.xblocks = (int32_t)((pos + 63) / 64 * p.nimg * (g.Ci / 32));
    const int64_t wblocks = ((int64_t)p.Cop * (p.Kd / 8) + 255) / 256;
    prep->fn = (const void*)k_conv_prep_f32;
    prep->grid = dim3((unsigned)(p.xblocks + wblocks), 1, 1);
    prep->block = dim3(256, 1, 1);
    prep->name = "conv_prep_nhwc_f32";
    prep->set_params(p);
    rec->fn = bn == 128 ? (const void*)k_conv_f32<64, 128, 32, 2> : (const void*)k_conv_f32<64, 64, 32, 2>;
    rec->grid = dim3((unsigned)((p.Co + 63) / 64 * ((p.P + bn - 1) / bn)), (unsigned)splits, 1);
    rec->block = dim3((unsigned)(2 * bn), 1, 1);
    rec->name = bn == 128 ? "conv_f32_64x128" : "conv_f32_64x64";
    rec->set_params(p);
}

}  // namespace qx

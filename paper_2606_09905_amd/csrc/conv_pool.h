// conv_pool.h -- the LeNet pipeline's two convolutions (5x5, smul24), each
// fused with its ReLU and 2x2 average, on the int8 matrix cores.  Compiled as
// a part of k_reduce.hip.
//
// An activation word is read as three limbs, a = s0 + 2^8 s1 + 2^16 s2 + C with
// C = 32896 (the bytes of its low 24 bits xor 0x8080, as signed bytes), and a
// weight as four, b = t0 + 2^8 t1 + 2^16 t2 + 2^24 t3 (signed bytes, t3 in
// {0, 1}: what a balanced t2 carries out).  With no offset in b the correction
// is C times the sum of a channel's weights, one constant per channel:
//   sum a b = sum_{i+j<=3} 2^(8(i+j)) sum s_i t_j + C sum b   (mod 2^32),
// nine int8 products, summed from the highest shift down, so one accumulator
// is shifted left by 8 three times.
//
// The weights are the A operand and stay in registers; the windows are the B
// operand, so a lane ends with channels of one output position in its
// registers and the four pixels of a 2x2 block are pooled inside the lane:
// floor of the exact sum of the four ReLUs over 4.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qx_internal.h"

namespace qx {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef uint32_t u2v __attribute__((ext_vector_type(2)));

constexpr int CP_WAVES = 4, CP_THREADS = CP_WAVES * 64;
constexpr uint32_t CP_OFFSET = 32896u;

// limbs t0..t3 of sext24(x) as bytes
__device__ __forceinline__ uint32_t weight_limbs(int32_t x) {
    const int32_t b = (int32_t)((uint32_t)x << 8) >> 8;
    const int32_t t0 = (int8_t)b, r1 = (b - t0) >> 8, t1 = (int8_t)r1, r2 = (r1 - t1) >> 8, t2 = (int8_t)r2;
    return ((uint32_t)t0 & 0xFFu) | (((uint32_t)t1 & 0xFFu) << 8) | (((uint32_t)t2 & 0xFFu) << 16) |
           (((uint32_t)(r2 - t2) >> 8) << 24);
}

// byte j of four words
__device__ __forceinline__ uint32_t pack_byte(uint32_t a, uint32_t b, uint32_t c, uint32_t d, int j) {
    const uint32_t sel = (uint32_t)j | ((uint32_t)(4 + j) << 8) | (0x0C0Cu << 16);
    return __builtin_amdgcn_perm(__builtin_amdgcn_perm(d, c, sel), __builtin_amdgcn_perm(b, a, sel), 0x05040100u);
}

// relu(a) + relu(b), below 2^32
__device__ __forceinline__ uint32_t relu_sum(int a, int b) { return (uint32_t)max(a, 0) + (uint32_t)max(b, 0); }
// floor((a + b) / 4), the sum in 33 bits
__device__ __forceinline__ int quarter(uint32_t a, uint32_t b) { return (int)(((uint64_t)a + b) >> 2); }

// conv 1x32x32 -> 6x28x28, pooled to 6x14x14.  A position is a pooled pixel:
// its 6x6 input window is a 48-byte operand column (six rows of eight bytes)
// for the 32 operand rows 8 px + channel, px the pixel of its 2x2 block: two
// steps of v_mfma_i32_32x32x32_i8 per product, the last 16 k empty.  Lane
// (position, h) ends with channels 4h..4h+3 of pixel r/4 in register r.
//
// Batch 4096, 22 us: the matrix products are 14 100 cycles of each SIMD (6.4
// us), the vector ALU 15 400 (the shifts between limbs, the byte shifts of
// windows that start at odd pairs, the pooling), 36 MB read and written 7 us.
__global__ __launch_bounds__(CP_THREADS) void k_conv1_pool(const ConvPoolParams p) {
    constexpr int IMG = 1024, POS = 196;
    __shared__ __align__(16) unsigned char ws[2][4][64 * 16];   // [step][limb][lane]
    __shared__ int32_t wsum[2][64];
    extern __shared__ __align__(16) unsigned char cp_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, h = lane >> 5;
    const int img0 = (int)blockIdx.x * p.imgs, cnt = min(p.imgs, p.nimg - img0);
    const int plane = p.imgs * IMG + 16;

    // four pixels a load, four loads in flight (past the end: the last ones again)
    const v4i* src = (const v4i*)(p.x + (int64_t)img0 * IMG);
    for (int i0 = tid; i0 < cnt * 256; i0 += CP_THREADS * 4) {
        v4i v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = src[min(i0 + u * CP_THREADS, cnt * 256 - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = min(i0 + u * CP_THREADS, cnt * 256 - 1);
#pragma unroll
            for (int j = 0; j < 3; ++j)
                *(uint32_t*)&cp_lds[j * plane + i * 4] =
                    pack_byte(v[u][0], v[u][1], v[u][2], v[u][3], j) ^ (j < 2 ? 0x80808080u : 0u);
        }
    }
    if (wave < 2) {
        // wave s makes the weight operand of step s: row l32 = 8 px + channel;
        // chunk c = 2 s + h holds window rows 2c, 2c + 1, eight bytes each.
        // Every load unconditional (all in flight), then the empty ones cleared.
        const int co = l32 & 7, dy = l32 >> 4, dx = l32 >> 3 & 1, r0 = 4 * wave + 2 * h - dy;
        uint32_t t[16];
        int32_t sum = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q)
            t[q] = (uint32_t)p.w[min(co, 5) * 25 + min(max(r0 + (q >> 3), 0), 4) * 5 + min(max((q & 7) - dx, 0), 4)];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int kh = r0 + (q >> 3), kw = (q & 7) - dx;
            t[q] &= co < 6 && kh >= 0 && kh < 5 && kw >= 0 && kw < 5 ? ~0u : 0u;
            sum += (int32_t)(t[q] << 8) >> 8;
            t[q] = weight_limbs((int32_t)t[q]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v4i o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (int)pack_byte(t[4 * e], t[4 * e + 1], t[4 * e + 2], t[4 * e + 3], j);
            *(v4i*)&ws[wave][j][lane * 16] = o;
        }
        wsum[wave][lane] = sum;
    }
    __syncthreads();
    v4i a[4][2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j][s] = *(const v4i*)&ws[s][j][lane * 16];
    uint32_t corr[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int r = 4 * h + e;
        corr[e] = CP_OFFSET * (uint32_t)(wsum[0][r] + wsum[0][32 + r] + wsum[1][r] + wsum[1][32 + r]);
    }

    for (int t = wave; t * 32 < cnt * POS; t += CP_WAVES) {
        const int pos = t * 32 + l32, ps = min(pos, cnt * POS - 1);
        const int img = ps / POS, rem = ps - img * POS, ph = rem / 14, pw = rem - ph * 14;
        const unsigned char* base = &cp_lds[img * IMG + ph * 64 + (pw >> 1) * 4];
        const uint32_t sh = (uint32_t)(pw & 1) * 2;
        v4i b[3][2];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    // window row 4s + 2h + r; the empty rows 6 and 7 read row 4 and 5
                    const uint32_t* w = (const uint32_t*)(base + j * plane + (min(4 * s + 2 * h, 4) + r) * 32);
                    const uint32_t w0 = w[0], w1 = w[1], w2 = w[2];
                    b[j][s][2 * r] = (int)__builtin_amdgcn_alignbyte(w1, w0, sh);
                    b[j][s][2 * r + 1] = (int)__builtin_amdgcn_alignbyte(w2, w1, sh);
                }
        v16i acc = v16i{};
#pragma unroll
        for (int g = 3; g >= 0; --g) {
            if (g < 3) acc <<= 8;
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (g - j >= 0 && g - j < 4)
#pragma unroll
                    for (int s = 0; s < 2; ++s)
                        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[g - j][s], b[j][s], acc, 0, 0, 0);
        }
        if (pos >= cnt * POS) continue;
        int32_t* y = p.y + ((int64_t)(img0 + img) * 6 + 4 * h) * POS + rem;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e < 2 || h == 0)
                y[e * POS] = quarter(relu_sum((int)((uint32_t)acc[e] + corr[e]), (int)((uint32_t)acc[4 + e] + corr[e])),
                                     relu_sum((int)((uint32_t)acc[8 + e] + corr[e]), (int)((uint32_t)acc[12 + e] + corr[e])));
    }
}

// conv 6x14x14 -> 16x10x10, pooled to 16x5x5.  The images are staged as limb
// planes of eight bytes per pixel (six channels, two unused: their weights
// are 0), so two neighbouring taps of a window row are 16 contiguous bytes:
// five rows of six taps (the last unused) are 15 operand chunks of 16, four
// steps of v_mfma_i32_16x16x64_i8.  A lane ends with channels 4g..4g+3 of its
// position, g = lane / 16, for each pixel of the 2x2 block in turn.
//
// Batch 4096, 19 us: the matrix products are 14 400 cycles of each SIMD (6.5
// us); the rest is the start of a workgroup (weights, images) and the waits of
// each tile on its 24 window reads.
__global__ __launch_bounds__(CP_THREADS, 2) void k_conv2_pool(const ConvPoolParams p) {
    constexpr int IMG = 196 * 8, POS = 25;
    __shared__ __align__(16) unsigned char ws[4][4][64 * 16];   // [step][limb][lane]
    __shared__ int32_t wsum[4][64];
    extern __shared__ __align__(16) unsigned char cp_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, g = lane >> 4;
    const int img0 = (int)blockIdx.x * p.imgs, cnt = min(p.imgs, p.nimg - img0);
    const int plane = p.imgs * IMG + 16;

    {
        // wave s makes the weight operand of step s: channel l16, chunk 4 s + g
        const int c = 4 * wave + g, kh = c / 3, kw0 = (c - 3 * kh) * 2;
        uint32_t t[16];
        int32_t sum = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q)
            t[q] = (uint32_t)p.w[(l16 * 6 + min(q & 7, 5)) * 25 + min(kh, 4) * 5 + min(kw0 + (q >> 3), 4)];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            t[q] &= c < 15 && (q & 7) < 6 && kw0 + (q >> 3) < 5 ? ~0u : 0u;
            sum += (int32_t)(t[q] << 8) >> 8;
            t[q] = weight_limbs((int32_t)t[q]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v4i o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (int)pack_byte(t[4 * e], t[4 * e + 1], t[4 * e + 2], t[4 * e + 3], j);
            *(v4i*)&ws[wave][j][lane * 16] = o;
        }
        wsum[wave][lane] = sum;
    }
    // two pixels a thread in flight (past the end: the last one again)
    const int32_t* src = p.x + (int64_t)img0 * 6 * 196;
    for (int i0 = tid; i0 < cnt * 196; i0 += CP_THREADS * 2) {
        uint32_t v[2][6];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int i = min(i0 + u * CP_THREADS, cnt * 196 - 1), img = i / 196, pix = i - img * 196;
#pragma unroll
            for (int c = 0; c < 6; ++c) v[u][c] = (uint32_t)src[(img * 6 + c) * 196 + pix];
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int i = min(i0 + u * CP_THREADS, cnt * 196 - 1);
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const uint32_t x = j < 2 ? 0x80808080u : 0u;
                *(u2v*)&cp_lds[j * plane + i * 8] =
                    u2v{pack_byte(v[u][0], v[u][1], v[u][2], v[u][3], j) ^ x,
                        pack_byte(v[u][4], v[u][5], v[u][4], v[u][5], j) ^ x};
            }
        }
    }
    __syncthreads();
    v4i a[4][4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j][s] = *(const v4i*)&ws[s][j][lane * 16];
    uint32_t corr[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        int32_t sum = 0;
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int k = 0; k < 4; ++k) sum += wsum[s][k * 16 + 4 * g + r];
        corr[r] = CP_OFFSET * (uint32_t)sum;
    }
    int off[4];                      // this lane's chunk of each step, from the window's first byte
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int c = min(4 * s + g, 14), kh = c / 3;
        off[s] = (kh * 14 + (c - 3 * kh) * 2) * 8;
    }
    for (int t = wave; t * 16 < cnt * POS; t += CP_WAVES) {
        const int pos = t * 16 + l16, ps = min(pos, cnt * POS - 1);
        const int img = ps / POS, rem = ps - img * POS, ph = rem / 5, pw = rem - ph * 5;
        const unsigned char* base = &cp_lds[img * IMG + (ph * 28 + pw * 2) * 8];
        uint32_t upper[4] = {}, sum[4] = {};
#pragma unroll 1
        for (int dy = 0; dy < 2; ++dy) {
            // the row's two pixels together: two independent chains of products
            v4i b[2][3][4];
#pragma unroll
            for (int dx = 0; dx < 2; ++dx)
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        const u2v* w = (const u2v*)(base + j * plane + (dy * 14 + dx) * 8 + off[s]);
                        const u2v lo = w[0], hi = w[1];
                        b[dx][j][s] = v4i{(int)lo[0], (int)lo[1], (int)hi[0], (int)hi[1]};
                    }
            v4i acc[2] = {v4i{}, v4i{}};
#pragma unroll
            for (int k = 3; k >= 0; --k) {
                if (k < 3) {
                    acc[0] <<= 8;
                    acc[1] <<= 8;
                }
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    if (k - j >= 0 && k - j < 4)
#pragma unroll
                        for (int s = 0; s < 4; ++s)
#pragma unroll
                            for (int dx = 0; dx < 2; ++dx)
                                acc[dx] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[k - j][s], b[dx][j][s], acc[dx], 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                upper[r] = sum[r];
                sum[r] = relu_sum((int)((uint32_t)acc[0][r] + corr[r]), (int)((uint32_t)acc[1][r] + corr[r]));
            }
        }
        if (pos >= cnt * POS) continue;
        int32_t* out = p.y + ((int64_t)(img0 + img) * 16 + 4 * g) * POS + rem;
#pragma unroll
        for (int r = 0; r < 4; ++r) out[r * POS] = quarter(upper[r], sum[r]);
    }
}

}  // namespace qx

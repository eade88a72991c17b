// k_attn.hip -- the single-head attention core O = (Q K^T) V on matrix cores
// (Methodology: attention operator of the form O = (Q K^T) V; Table 2,
// attention rows), without scale, softmax or mask, and the FP32 softmax form
// (the attention baseline of Table 2's footnote).
//
// All kernels keep S on chip.  A wave owns 32 queries; per block of 32 keys
// it forms S^T = K_blk Q^T with one MFMA chain, whose 32x32 accumulator
// (lane = query, 16 registers = 16 keys) is exactly the A operand layout of
// the second product O += S V once the V operand is gathered with the same
// key permutation (the order of a contraction's terms is free).  Keys are
// split across workgroups; partial results are combined in a fixed order.
//
//  * FP32: operands as three bf16 terms on v_mfma_f32_32x32x16_bf16, six
//    products kept (k_attn_b3, which also is the softmax attention); per-split
//    partials are reduced in split order, so repeated runs are bit-identical.
//  * INT32 (|q|,|k|,|v| <= 127 and d*max^2 < 2^23): S^T on
//    v_mfma_i32_32x32x32_i8; every S is read as three offset int8 limbs,
//    S = s0 + 2^8 s1 + 2^16 s2 + 32896, where the limbs are the bytes of
//    S xor 0x8080; O gets three int8 products mod 2^32 plus 32896 * colsum(V).
//    Integer partials from different splits are added with atomics (exact
//    and order-independent mod 2^32).
#include "f32_split.h"
#include "qx_internal.h"

namespace qx {

typedef float f16x __attribute__((ext_vector_type(16)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // a caller's output may be 4-byte aligned
typedef int i16x __attribute__((ext_vector_type(16)));
typedef int i4 __attribute__((ext_vector_type(4)));

constexpr int AT = 256;      // 4 waves
constexpr int AQW = 32;      // queries per wave
constexpr int AQ = 4 * AQW;  // queries per workgroup
constexpr int AKB = 32;      // keys per block

// Sum of the splits' partials in split order, four outputs a thread.
__global__ __launch_bounds__(AT) void k_reduce_splits(const ReduceParams p) {
    const int64_t i = ((int64_t)blockIdx.x * AT + threadIdx.x) * 4;
    if (i >= p.n) return;
    f4 s = *(const f4*)(p.part + i);
#pragma unroll 4
    for (int k = 1; k < p.splits; ++k) s += *(const f4*)(p.part + (int64_t)k * p.stride + i);
    if (i + 4 <= p.n) {
        *(f4u*)(p.out + i) = s;
    } else {
        for (int e = 0; e < 3 && i + e < p.n; ++e) p.out[i + e] = s[e];
    }
}

// ---------------------------------------------------------------------------
// INT32 through int8 matrix cores
// ---------------------------------------------------------------------------
// Byte j of four words, packed into one word (a, b, c, d -> bytes 0..3).
__device__ __forceinline__ uint32_t gather_byte(uint32_t a, uint32_t b, uint32_t c, uint32_t d, int j) {
    const uint32_t sel = (uint32_t)j | ((uint32_t)(4 + j) << 8) | (0x0C0Cu << 16);
    const uint32_t lo = __builtin_amdgcn_perm(b, a, sel);   // (a_j, b_j, 0, 0)
    const uint32_t hi = __builtin_amdgcn_perm(d, c, sel);   // (c_j, d_j, 0, 0)
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);      // (a_j, b_j, c_j, d_j)
}

template <int D>
__global__ __launch_bounds__(AT) void k_attn_i32(const AttnParams p) {
    constexpr int NTO = D / 32;
    constexpr int KCH = D / 16;                 // 16-byte chunks per key row (int8)
    constexpr int KW = AKB * D / 4 / AT;        // packed K words per thread
    __shared__ i4 Ks8[AKB][KCH];                // int8 K rows
    __shared__ uint32_t Vt8[D][AKB / 4 + 1];    // int8 V^T: [column][keys], padded

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, l32 = lane & 31;
    const int q0 = blockIdx.x * AQ + wave * AQW;
    const int split = blockIdx.y;
    const int key_lo = split * p.keys_per_split;
    const int key_hi = min(p.L, key_lo + p.keys_per_split);
    const int32_t* Q = (const int32_t*)p.Q;
    const int32_t* Kp = (const int32_t*)p.K;
    const int32_t* Vp = (const int32_t*)p.V;

    auto pack4 = [](i4 v) -> uint32_t {
        return ((uint32_t)v[0] & 0xFFu) | (((uint32_t)v[1] & 0xFFu) << 8) |
               (((uint32_t)v[2] & 0xFFu) << 16) | ((uint32_t)v[3] << 24);
    };
    // Q fragment: lane (query, half h), MFMA t: Q[query][32t + 16h + e], e < 16.
    i4 qf[NTO];
    {
        const int q = q0 + l32;
#pragma unroll
        for (int t = 0; t < NTO; ++t) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const i4 v = (q < p.L) ? *(const i4*)(Q + (int64_t)q * D + 32 * t + 16 * h + 4 * w) : i4{};
                qf[t][w] = (int)pack4(v);
            }
        }
    }
    i16x o[3][NTO];
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int n = 0; n < NTO; ++n) o[j][n] = i16x{};

    // Column sums of V over this split's keys, for the offset correction.
    __shared__ uint32_t vsum[D];
    if (tid < D) vsum[tid] = 0u;
    __syncthreads();
    uint32_t vpart[KW];
#pragma unroll
    for (int i = 0; i < KW; ++i) vpart[i] = 0u;

    uint32_t rk[KW], rv[KW];
    auto load = [&](int kb) {
#pragma unroll
        for (int i = 0; i < KW; ++i) {
            const int v = tid + AT * i;
            // K: word v covers key v/(D/4), columns 4*(v%(D/4)) .. +3
            const int krow = v / (D / 4), kc = v % (D / 4);
            const int key = kb + krow;
            rk[i] = key < key_hi ? pack4(*(const i4*)(Kp + (int64_t)key * D + kc * 4)) : 0u;
            // V^T: word v covers column v % D, keys 4*(v / D) .. +3
            const int col = v % D, kq = v / D;
            uint32_t w = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int key2 = kb + kq * 4 + e;
                const uint32_t x = key2 < key_hi ? (uint32_t)Vp[(int64_t)key2 * D + col] : 0u;
                w |= (x & 0xFFu) << (8 * e);
                vpart[i] += x;
            }
            rv[i] = w;
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int i = 0; i < KW; ++i) {
            const int v = tid + AT * i;
            const int krow = v / (D / 4), kc = v % (D / 4);
            ((uint32_t*)&Ks8[krow][0])[kc] = rk[i];
            Vt8[v % D][v / D] = rv[i];
        }
    };

    if (key_lo < key_hi) load(key_lo);
    for (int kb = key_lo; kb < key_hi; kb += AKB) {
        __syncthreads();
        stash();
        __syncthreads();
        if (kb + AKB < key_hi) load(kb + AKB);
        i16x s = i16x{};
#pragma unroll
        for (int t = 0; t < NTO; ++t)
            s = __builtin_amdgcn_mfma_i32_32x32x32_i8(Ks8[l32][2 * t + h], qf[t], s, 0, 0, 0);
        // Offset limbs: bytes 0..2 of S ^ 0x8080.  K-slot (h, e) of the
        // second product is key 8*(e/4) + 4*h + e%4, as the S^T layout gives.
        uint32_t x[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = (uint32_t)s[r] ^ 0x8080u;
        i4 limb[3];
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int w = 0; w < 4; ++w)
                limb[j][w] = (int)gather_byte(x[4 * w], x[4 * w + 1], x[4 * w + 2], x[4 * w + 3], j);
#pragma unroll
        for (int n = 0; n < NTO; ++n) {
            i4 vb;
#pragma unroll
            for (int w = 0; w < 4; ++w) vb[w] = (int)Vt8[n * 32 + l32][2 * w + h];
#pragma unroll
            for (int j = 0; j < 3; ++j)
                o[j][n] = __builtin_amdgcn_mfma_i32_32x32x32_i8(limb[j], vb, o[j][n], 0, 0, 0);
        }
    }

#pragma unroll
    for (int i = 0; i < KW; ++i) atomicAdd(&vsum[(tid + AT * i) % D], vpart[i]);
    __syncthreads();

    int32_t* O = (int32_t*)p.O;
#pragma unroll
    for (int n = 0; n < NTO; ++n) {
        const int c = n * 32 + l32;
        // every split adds 32896 * sum over its own keys of V[key][c]
        const uint32_t corr = 32896u * vsum[c];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int q = q0 + 8 * (r >> 2) + 4 * h + (r & 3);
            if (q >= p.L) continue;
            const uint32_t v = (uint32_t)o[0][n][r] + ((uint32_t)o[1][n][r] << 8) +
                               ((uint32_t)o[2][n][r] << 16) + corr;
            if (p.splits > 1) atomicAdd(O + (int64_t)q * D + c, (int)v);
            else O[(int64_t)q * D + c] = (int32_t)v;
        }
    }
}

// ---------------------------------------------------------------------------
// INT32 with resident key splits.  A prep launch writes int8 copies of K
// (rows) and V^T (rows of keys, each 32-key block reordered as in the V
// operand gather below) into the workspace and clears O; then each workgroup
// loads its whole key split -- kps keys of K8 and of V8 -- into LDS with
// direct-to-LDS loads in one batch, and runs every key block from LDS with
// no further global loads or barriers.  The S^T tile and the limb split are
// those of k_attn_i32.
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(AT) void k_attn_i32_prep(const AttnParams p) {
    const int64_t i = (int64_t)blockIdx.x * AT + threadIdx.x;
    const int32_t* Kp = (const int32_t*)p.K;
    const int32_t* Vp = (const int32_t*)p.V;
    auto pack4 = [](i4 v) -> uint32_t {
        return ((uint32_t)v[0] & 0xFFu) | (((uint32_t)v[1] & 0xFFu) << 8) |
               (((uint32_t)v[2] & 0xFFu) << 16) | ((uint32_t)v[3] << 24);
    };
    if (i < p.prep_k) {
        // 16 consecutive d of one key row
        const int key = (int)(i / (D / 16)), c0 = (int)(i % (D / 16)) * 16;
        i4 o = i4{};
        if (key < p.L) {
#pragma unroll
            for (int w = 0; w < 4; ++w) o[w] = (int)pack4(*(const i4*)(Kp + (int64_t)key * D + c0 + 4 * w));
        }
        *(i4*)((int8_t*)p.k8 + (int64_t)key * D + c0) = o;
        return;
    }
    const int64_t iv = i - p.prep_k;
    if (iv < p.prep_v) {
        // column c, half-block hb (16 keys): byte 4w + e holds key
        // 32*(hb/2) + 8w + 4*(hb%2) + e
        const int c = (int)(iv % D);
        const int hb = (int)(iv / D);
        const int kb = (hb >> 1) * 32 + 4 * (hb & 1);
        i4 o;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            uint32_t x = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int key = kb + 8 * w + e;
                const uint32_t v = key < p.L ? (uint32_t)Vp[(int64_t)key * D + c] : 0u;
                x |= (v & 0xFFu) << (8 * e);
            }
            o[w] = (int)x;
        }
        int8_t* dst = p.v_blocks ? (int8_t*)p.v8 + ((int64_t)(hb >> 1) * D + c) * 32 + 16 * (hb & 1)
                                 : (int8_t*)p.v8 + (int64_t)c * p.Lp + 16 * (int64_t)hb;
        *(i4*)dst = o;
        return;
    }
    const int64_t iq = iv - p.prep_v;
    if (iq < p.prep_q) {
        // 16 consecutive d of one query row
        const int q = (int)(iq / (D / 16)), c0 = (int)(iq % (D / 16)) * 16;
        const int32_t* Qp = (const int32_t*)p.Q;
        i4 o;
#pragma unroll
        for (int w = 0; w < 4; ++w) o[w] = (int)pack4(*(const i4*)(Qp + (int64_t)q * D + c0 + 4 * w));
        *(i4*)((int8_t*)p.q8 + (int64_t)q * D + c0) = o;
        return;
    }
    const int64_t io = iq - p.prep_q;
    if (p.clear_o && io < (int64_t)p.L * D / 4) ((i4*)p.O)[io] = i4{};
}

// chunk swizzles of the resident tiles: K rows of D bytes (16 lanes of one
// ds_read_b128 read 16 rows at one chunk: spread them over the 64 banks), and
// V rows of kps bytes (swizzle within the largest power-of-two group of
// chunks that divides the row, at most 16)
template <int D>
__device__ __forceinline__ int swz_k(int row) { return (row / (256 / D)) & (D / 16 - 1); }
__device__ __forceinline__ int swz_v(int row, int vmask) { return row & vmask; }

template <int D>
__global__ __launch_bounds__(AT) void k_attn_i32r(const AttnParams p) {
    constexpr int NTO = D / 32;
    constexpr int CK = D / 16;                   // 16-byte chunks per K row
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int kps = p.keys_per_split;
    char* Ks = smem;                             // [kps][D] int8
    char* Vs = smem + (int64_t)kps * D;          // [D][kps] int8
    __shared__ uint32_t vsum[D];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, l32 = lane & 31;
    const int q0 = blockIdx.x * AQ + wave * AQW;
    const int split = blockIdx.y;
    const int key_lo = split * kps;
    const int CV = kps / 16;                     // 16-byte chunks per V row
    const int vmask = min(CV & -CV, 16) - 1;
    const unsigned wave_u = __builtin_amdgcn_readfirstlane(wave);

    // the split's K8 rows and V8 columns, 1 KB per wave instruction
    {
        const char* k8 = (const char*)p.k8 + (int64_t)key_lo * D;
        const char* v8 = (const char*)p.v8 + key_lo;
        const unsigned lds_k = (unsigned)(uintptr_t)Ks, lds_v = (unsigned)(uintptr_t)Vs;
        const int nk = kps * D / 1024, nv = D * kps / 1024;
        for (int I = (int)wave_u; I < nk; I += 4) {
            const int q = I * 64 + lane, row = q / CK, pos = q % CK;
            const unsigned off = (unsigned)(row * D + ((pos ^ swz_k<D>(row)) * 16));
            asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                         :: "v"(off), "s"(k8), "s"(lds_k + I * 1024) : "memory", "m0");
        }
        for (int I = (int)wave_u; I < nv; I += 4) {
            const int q = I * 64 + lane, row = q / CV, pos = q % CV;
            const unsigned off = (unsigned)(row * p.Lp + ((pos ^ swz_v(row, vmask)) * 16));
            asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                         :: "v"(off), "s"(v8), "s"(lds_v + I * 1024) : "memory", "m0");
        }
    }
    const int32_t* Q = (const int32_t*)p.Q;
    auto pack4 = [](i4 v) -> uint32_t {
        return ((uint32_t)v[0] & 0xFFu) | (((uint32_t)v[1] & 0xFFu) << 8) |
               (((uint32_t)v[2] & 0xFFu) << 16) | ((uint32_t)v[3] << 24);
    };
    i4 qf[NTO];
    {
        const int q = q0 + l32;
#pragma unroll
        for (int t = 0; t < NTO; ++t) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const i4 v = (q < p.L) ? *(const i4*)(Q + (int64_t)q * D + 32 * t + 16 * h + 4 * w) : i4{};
                qf[t][w] = (int)pack4(v);
            }
        }
    }
    if (tid < D) vsum[tid] = 0u;
    __builtin_amdgcn_s_waitcnt(0x0070);          // vmcnt(0), lgkmcnt(0): the tiles have landed
    __syncthreads();
    // column sums of V over the split's keys (padding keys are zero)
    {
        constexpr int TPR = AT / D;              // threads per V row
        const int row = tid / TPR, part = tid % TPR;
        const uint32_t* vr = (const uint32_t*)(Vs + (int64_t)row * kps);
        // thread `part` sums words [part*per, (part+1)*per), visited in an
        // order rotated by the row so that lanes on different rows (whose
        // rows start in the same bank) read different banks
        const int per = kps / 4 / TPR;
        int acc = 0;
        for (int i = 0; i < per; ++i)
            acc = __builtin_amdgcn_sdot4((int)vr[part * per + (i + row) % per], 0x01010101, acc, false);
        atomicAdd(&vsum[row], (uint32_t)acc);
    }

    i16x o[3][NTO];
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int n = 0; n < NTO; ++n) o[j][n] = i16x{};
    for (int blk = 0; blk < kps / 32; ++blk) {
        const int krow = blk * 32 + l32;
        i16x s = i16x{};
#pragma unroll
        for (int t = 0; t < NTO; ++t) {
            const i4 kf = *(const i4*)(Ks + (int64_t)krow * D + (((2 * t + h) ^ swz_k<D>(krow)) * 16));
            s = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf, qf[t], s, 0, 0, 0);
        }
        uint32_t x[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = (uint32_t)s[r] ^ 0x8080u;
        i4 limb[3];
#pragma unroll
        for (int jj = 0; jj < 3; ++jj)
#pragma unroll
            for (int w = 0; w < 4; ++w)
                limb[jj][w] = (int)gather_byte(x[4 * w], x[4 * w + 1], x[4 * w + 2], x[4 * w + 3], jj);
#pragma unroll
        for (int n = 0; n < NTO; ++n) {
            const int vrow = n * 32 + l32;
            const i4 vb = *(const i4*)(Vs + (int64_t)vrow * kps + (((2 * blk + h) ^ swz_v(vrow, vmask)) * 16));
#pragma unroll
            for (int jj = 0; jj < 3; ++jj)
                o[jj][n] = __builtin_amdgcn_mfma_i32_32x32x32_i8(limb[jj], vb, o[jj][n], 0, 0, 0);
        }
    }
    __syncthreads();                             // vsum complete

    int32_t* O = (int32_t*)p.O;
#pragma unroll
    for (int n = 0; n < NTO; ++n) {
        const int c = n * 32 + l32;
        const uint32_t corr = 32896u * vsum[c];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int q = q0 + 8 * (r >> 2) + 4 * h + (r & 3);
            if (q >= p.L) continue;
            const uint32_t v = (uint32_t)o[0][n][r] + ((uint32_t)o[1][n][r] << 8) +
                               ((uint32_t)o[2][n][r] << 16) + corr;
            if (p.splits > 1) atomicAdd(O + (int64_t)q * D + c, (int)v);
            else O[(int64_t)q * D + c] = (int32_t)v;
        }
    }
}

// ---------------------------------------------------------------------------
// INT32, streaming.  A workgroup of eight waves takes QT query tiles of 32
// queries and one key split, cut into KQ = 8 / QT key parts: wave w holds
// query tile w % QT over key part w / QT.  Per 32-key block: S^T on the int8
// matrix cores, the offset limb split of S, three limb products into O, and
// the block's V column sums (for the offset correction) from the same V
// registers.  The KQ partial outputs of a query tile are added through LDS,
// each wave adding a slice of the tile, and one wrapping int32 atomic per
// output joins the key splits (exact mod 2^32 in any order).
// ---------------------------------------------------------------------------
template <int D, int QT>
struct AttnStream {
    static constexpr int NTO = D / 32;
    static constexpr int KQ = 8 / QT;                    // key parts
    static constexpr int BLK = 2 * NTO * 1024;           // bytes of one block's K and V
    static constexpr int PER_PAIR = 4 * NTO;             // 1 KB loads per pair of blocks
    static constexpr int PW = PER_PAIR / QT;             // of them issued by each wave
    static constexpr int R0 = (128 * 1024) / (KQ * 2 * BLK);
    static constexpr int R = R0 > 8 ? 8 : R0;            // ring depth in pairs
    static_assert(PER_PAIR % QT == 0 && R >= 2 && (R & (R - 1)) == 0, "ring geometry");
    static_assert(PW * (R - 2) < 64, "loads in flight fit the vmcnt counter");
    static constexpr int KEYS = 64 * KQ;                 // keys_per_split is a multiple of this
};

// s_waitcnt vmcnt(N) (expcnt and lgkmcnt left alone), N in [0, 63]
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
// wait until at most STEP * n of this wave's vector memory loads are in flight,
// n in [0, NMAX] (the immediate is a constant: dispatch on n)
template <int STEP, int NMAX>
__device__ __forceinline__ void wait_vmcnt_steps(int n) {
    if constexpr (NMAX <= 0) {
        wait_vmcnt<0>();
    } else {
        if (n >= NMAX) wait_vmcnt<STEP * NMAX>();
        else wait_vmcnt_steps<STEP, NMAX - 1>(n);
    }
}

template <int D, int QT>
__global__ __launch_bounds__(512) void k_attn_i32s(const AttnParams p) {
    using G = AttnStream<D, QT>;
    constexpr int NTO = G::NTO, KQ = G::KQ, BLK = G::BLK, PW = G::PW, R = G::R;
    // per key part a ring of R pairs of blocks; after the loop the ring
    // carries the partial outputs between the waves of a query tile
    __shared__ __attribute__((aligned(16))) char ring[KQ][R][2][BLK];
    __shared__ __attribute__((aligned(16))) char qs[8][NTO * 1024];

    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: block addresses stay scalar
    const int qw = wave % QT, kp = wave / QT;
    const int q0 = blockIdx.x * (32 * QT) + qw * 32;
    const int kps = p.keys_per_split;            // a multiple of G::KEYS
    const int npair = kps / G::KEYS;             // pairs of 32-key blocks per key part
    const int blk0 = (int)(((int64_t)blockIdx.y * kps + (int64_t)kp * (kps / KQ)) / 32);
    const char* K8 = (const char*)p.k8;          // [Lp][D]
    const char* V8 = (const char*)p.v8;          // [Lp/32][D][32]

    // The QT waves of a key part stage its blocks in the part's ring with
    // direct-to-LDS loads, R-1 pairs ahead, each wave PW of the 1 KB loads
    // of every pair.  A lane's 16 bytes land where the MFMA operand layout
    // reads them (lane (key | column l32, half h): K row chunk 2t + h, V 16
    // keys of column n*32 + l32), which is the same for every query tile,
    // so the ring reads are contiguous.
    const unsigned koff = (unsigned)(l32 * D + h * 16), voff = (unsigned)(l32 * 32 + h * 16);
    auto issue = [&](int pr) {
        const unsigned lds = (unsigned)(uintptr_t)&ring[kp][pr & (R - 1)][0][0];
#pragma unroll
        for (int u = 0; u < PW; ++u) {
            const int l = qw * PW + u;                           // 0 .. PER_PAIR-1
            const int e = l / (2 * NTO), part = l % (2 * NTO);   // block of the pair, 1 KB part
            const int64_t bg = blk0 + 2 * pr + e;
            const unsigned dst = lds + (unsigned)(e * BLK + part * 1024);
            if (part < NTO) {
                const char* kb = K8 + bg * 32 * D;
                asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                             :: "v"(koff + part * 32), "s"(kb), "s"(dst) : "memory", "m0");
            } else {
                const char* vb = V8 + bg * D * 32;
                asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                             :: "v"(voff + (part - NTO) * 1024), "s"(vb), "s"(dst) : "memory", "m0");
            }
        }
    };
    // this wave's Q rows as int8 (written by the prep launch), staged the
    // same way ahead of the key blocks: lane (query l32, half h), MFMA t
    // reads Q[query][32t + 16h + e]; rows past L repeat the last row
    {
        const int qr = min(q0, p.L - 1);         // a tile past L (last workgroup) reads row L-1
        const char* qb = (const char*)p.q8 + (int64_t)qr * D;
        const unsigned qoff = (unsigned)((min(q0 + l32, p.L - 1) - qr) * D + 16 * h);
        const unsigned dst = (unsigned)(uintptr_t)&qs[wave][0];
#pragma unroll
        for (int t = 0; t < NTO; ++t)
            asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                         :: "v"(qoff + 32 * t), "s"(qb), "s"(dst + t * 1024) : "memory", "m0");
    }
    for (int pr = 0; pr < R - 1 && pr < npair; ++pr) issue(pr);

    i16x o[3][NTO];
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int n = 0; n < NTO; ++n) o[j][n] = i16x{};
    int vs[NTO];                                 // V column n*32 + l32, keys of half h
#pragma unroll
    for (int n = 0; n < NTO; ++n) vs[n] = 0;
    i4 qf[NTO];

    // the offset limbs of S (bytes of S ^ 0x8080, read as int8): K-slot
    // (h, e) of the second product is key 8*(e/4) + 4*h + e%4, as the S^T
    // accumulator layout gives.  Per four elements a, b, c, d a byte
    // transpose: (a0 b0 a1 b1), (c0 d0 c1 d1), (a2 b2 - -), (c2 d2 - -), then
    // limb j = (a_j b_j c_j d_j); the XOR with 0x80 of bytes 0 and 1 is done
    // on the transposed words.
    auto limbs = [](const i16x& s, i4 (&limb)[3]) {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const uint32_t a = (uint32_t)s[4 * w], b = (uint32_t)s[4 * w + 1];
            const uint32_t c = (uint32_t)s[4 * w + 2], d = (uint32_t)s[4 * w + 3];
            const uint32_t ab01 = __builtin_amdgcn_perm(b, a, 0x05010400u);
            const uint32_t cd01 = __builtin_amdgcn_perm(d, c, 0x05010400u);
            const uint32_t ab2 = __builtin_amdgcn_perm(b, a, 0x0C0C0602u);
            const uint32_t cd2 = __builtin_amdgcn_perm(d, c, 0x0C0C0602u);
            limb[0][w] = (int)(__builtin_amdgcn_perm(cd01, ab01, 0x05040100u) ^ 0x80808080u);
            limb[1][w] = (int)(__builtin_amdgcn_perm(cd01, ab01, 0x07060302u) ^ 0x80808080u);
            limb[2][w] = (int)__builtin_amdgcn_perm(cd2, ab2, 0x05040100u);
        }
    };
    // Software pipeline: the second block's limb products of pair pr run at
    // the start of pair pr+1, beside its S^T chains and first limb split
    // (zero limbs stand in before the first pair: they add nothing).
    i4 lp[3] = {i4{}, i4{}, i4{}};
    i4 vp[NTO];
#pragma unroll
    for (int n = 0; n < NTO; ++n) vp[n] = i4{};
    for (int pr = 0; pr < npair; ++pr) {
        // this wave's loads of pair pr (and, before them, its Q rows) have
        // landed once no more than those of the later pairs are in flight
        wait_vmcnt_steps<PW, R - 2>(npair - 1 - pr);
        __syncthreads();                         // every part landed; slot of pair pr-1 read by all
        if (pr + R - 1 < npair) issue(pr + R - 1);
        if (pr == 0) {
#pragma unroll
            for (int t = 0; t < NTO; ++t) qf[t] = *(const i4*)(&qs[wave][t * 1024 + lane * 16]);
        }
        const char* st0 = &ring[kp][pr & (R - 1)][0][0];
        const char* st1 = &ring[kp][pr & (R - 1)][1][0];
        i4 kf0[NTO], kf1[NTO], vf0[NTO], vf1[NTO];
#pragma unroll
        for (int t = 0; t < NTO; ++t) {
            kf0[t] = *(const i4*)(st0 + t * 1024 + lane * 16);
            kf1[t] = *(const i4*)(st1 + t * 1024 + lane * 16);
        }
#pragma unroll
        for (int n = 0; n < NTO; ++n) {
            vf0[n] = *(const i4*)(st0 + (NTO + n) * 1024 + lane * 16);
            vf1[n] = *(const i4*)(st1 + (NTO + n) * 1024 + lane * 16);
        }
        // both S^T chains first (pinned: left alone, the scheduler ran the
        // second chain after the first block's products, so every limb split
        // waited on its own chain)
        i16x s0 = i16x{}, s1 = i16x{};
#pragma unroll
        for (int t = 0; t < NTO; ++t) {
            s0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf0[t], qf[t], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf1[t], qf[t], s1, 0, 0, 0);
        }
        asm volatile("" : "+v"(s1));
        __builtin_amdgcn_sched_barrier(0);
        // the previous pair's second-block products beside this pair's first
        // limb split
        i4 l0[3], l1[3];
#pragma unroll
        for (int n = 0; n < NTO; ++n)
#pragma unroll
            for (int jj = 0; jj < 3; ++jj)
                o[jj][n] = __builtin_amdgcn_mfma_i32_32x32x32_i8(lp[jj], vp[n], o[jj][n], 0, 0, 0);
        limbs(s0, l0);
#pragma unroll
        for (int g = 0; g < 3 * NTO; ++g) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 36 / (3 * NTO), 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        // the first block's products beside the second block's limb split
#pragma unroll
        for (int n = 0; n < NTO; ++n)
#pragma unroll
            for (int jj = 0; jj < 3; ++jj)
                o[jj][n] = __builtin_amdgcn_mfma_i32_32x32x32_i8(l0[jj], vf0[n], o[jj][n], 0, 0, 0);
        limbs(s1, l1);
#pragma unroll
        for (int g = 0; g < 3 * NTO; ++g) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
            __builtin_amdgcn_sched_group_barrier(0x002, 36 / (3 * NTO), 1);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < NTO; ++n)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                vs[n] = __builtin_amdgcn_sdot4(vf0[n][w], 0x01010101, vs[n], false);
                vs[n] = __builtin_amdgcn_sdot4(vf1[n][w], 0x01010101, vs[n], false);
            }
#pragma unroll
        for (int jj = 0; jj < 3; ++jj) lp[jj] = l1[jj];
#pragma unroll
        for (int n = 0; n < NTO; ++n) vp[n] = vf1[n];
    }
#pragma unroll
    for (int n = 0; n < NTO; ++n)
#pragma unroll
        for (int jj = 0; jj < 3; ++jj)
            o[jj][n] = __builtin_amdgcn_mfma_i32_32x32x32_i8(lp[jj], vp[n], o[jj][n], 0, 0, 0);

    // recombine the limbs and add the offset correction of this wave's keys
    uint32_t v[NTO][16];
#pragma unroll
    for (int n = 0; n < NTO; ++n) {
        const uint32_t cs = (uint32_t)(vs[n] + __shfl_xor(vs[n], 32, 64));
        const uint32_t corr = 32896u * cs;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            v[n][r] = (uint32_t)o[0][n][r] + ((uint32_t)o[1][n][r] << 8) + ((uint32_t)o[2][n][r] << 16) + corr;
    }
    // the partial outputs of the KQ key parts, [QT][KQ][32][D], through the
    // ring once every wave is done reading it
    uint32_t* red = (uint32_t*)&ring[0][0][0][0];
    static_assert(8 * 32 * D * 4 <= (int)sizeof(ring), "partial outputs fit the ring");
    __syncthreads();
    {
        uint32_t* mine = red + (qw * KQ + kp) * (32 * D);
#pragma unroll
        for (int n = 0; n < NTO; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                mine[(8 * (r >> 2) + 4 * h + (r & 3)) * D + n * 32 + l32] = v[n][r];
    }
    __syncthreads();
    // wave (qw, kp) adds slice kp of query tile qw: 64 consecutive outputs
    // (row-major, query by column) per step, one atomic per output
    constexpr int PERW = 32 * D / 64 / KQ;
    const uint32_t* tile = red + qw * KQ * (32 * D);
    int32_t* dst = (int32_t*)p.O;
#pragma unroll
    for (int i = 0; i < PERW; ++i) {
        const int e = (kp * PERW + i) * 64 + lane;
        uint32_t t = 0;
#pragma unroll
        for (int k = 0; k < KQ; ++k) t += tile[k * 32 * D + e];
        const int q = q0 + e / D, c = e % D;
        if (q >= p.L) continue;
        // splits add into the output cleared by the prep launch:
        // wrapping int32 atomics, exact mod 2^32 in any order
        if (p.splits > 1) atomicAdd(dst + (int64_t)q * D + c, (int)t);
        else dst[(int64_t)q * D + c] = (int32_t)t;
    }
}

// ---------------------------------------------------------------------------
// FP32 attention on split operands (f32_split.h): the core O = (Q K^T) V (SM = false) and the
// softmax form (SM = true).  NW waves of 32 queries; blocks of 32 keys are
// split once per workgroup while they are staged: K planes by key (rows of D),
// V planes transposed (a column's 32 keys, in the order in which the lanes
// hold S).  S^T = K Q^T leaves lane (query l32, half h) with keys
// 8*(r/4) + 4*h + r%4 of register r; split again, those registers are the B
// operand of O^T += V^T S^T, so O stays by query too and the softmax's factors
// never change lanes.  One barrier per block; a block's loads are in flight
// for a whole block before it is staged.
//
// Scales: the core takes Q, K and V times kSplitScale and S down to S times it;
// the softmax form takes V and its probabilities times it (scores need no more
// than their absolute error, a probability down to 2^-126 all of its bits).
//
// Bound: the matrix cores; per 32x32 block and wave 2048 matrix cycles against
// about 1450 of vector ALU (exponentials, splits).  32 causal heads x 4096 x
// 64: 430 us, 16 x 2048 x 128 235 (616 and 302 on v_mfma_f32_32x32x2f32); the
// core at L = 4096, d = 64 38.5 us (43), 300 x 64 9.1 (9.3), 2048 x 128 31 (32);
// errors a third of theirs.  Without the products m l and l m and with one
// running sum (338, 195 and 33 us) a sum of one product was up to 1.4 ulp off.
//
// PIPE, a software pipeline over the blocks, is the core's for d <= 64 with one
// wave per SIMD and at least eight blocks a split (L = 4096, d = 64 40.1 us
// without it, 38.5 with; short calls would stage blocks that are not there, 208 x
// 64 10.5 us with it, 8.7 without; the softmax form lost 4%).
//
// Softmax: per block the running maximum m (base-2 exponent domain,
// t = scale*log2(e)*s) and the running sum are updated online.  With key
// splits every split writes unnormalised O, its maximum and its sum;
// k_sdpa_combine merges them in split order (the core: k_reduce_splits adds
// the partials in split order), so repeated runs are bit-identical.
// RAG: d < D, columns d..D-1 read as zeros and are not written.
// ---------------------------------------------------------------------------
template <int D, int NW, bool SM, bool RAG, bool PIPE = false>
__global__ __launch_bounds__(NW * 64) void k_attn_b3(const SdpaParams p) {
    constexpr int NTH = NW * 64;
    constexpr int QW = 32 * NW;              // queries per workgroup
    constexpr int KS = D / 16;               // 16-k steps of Q K^T
    constexpr int NTO = D / 32;              // output row tiles of O^T
    constexpr int KP = 2 * D + 16;           // bytes of a K row and of a V column in LDS (padded:
    constexpr int VP = 2 * AKB + 16;         // 16 rows of one chunk fall on 64 different banks)
    constexpr bool FROM_ZERO = SM || (D <= 64 && !PIPE);
    static_assert(!PIPE || !SM, "the pipeline has no place for the running maximum");
    constexpr int KB = AKB * KP, VB = D * VP;            // bytes of one plane
    constexpr int NI = (8 * D + NTH - 1) / NTH;          // staging items (8 elements) per thread
    __shared__ __align__(16) unsigned char lds[2][3 * (KB + VB)];
    __shared__ int large_k;

    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wave64 = wave * 64;
    // Under the mask a query block's work grows with its index: the dispatch
    // order (x fastest, then z) hands out the longest blocks of every head
    // first, so that the short ones fill in behind them.
    int qblk = blockIdx.x;
    int64_t head = blockIdx.z;
    if (SM && p.causal) {
        const int id = (int)blockIdx.x + (int)gridDim.x * (int)blockIdx.z;
        qblk = (int)gridDim.x - 1 - id / (int)gridDim.z;
        head = id % (int)gridDim.z;
    }
    const bool causal = SM && p.causal;
    const int qb = qblk * QW;
    const int q0 = qb + wave * AQW;
    const int split = blockIdx.y;
    const int d = RAG ? p.d : D;
    const int key_lo = split * p.keys_per_split;
    int key_hi = min(p.L, key_lo + p.keys_per_split);
    if (causal) key_hi = min(key_hi, qb + QW);
    const int64_t hoff = head * p.L * d;
    const float* Q = p.Q + hoff;
    const float* Kp = p.K + hoff;
    const float* Vp = p.V + hoff;

    // eight elements c8.. of the row that starts at base + row; past d they
    // read as the row's last element (zero: as 0)
    auto ld8 = [&](const float* base, unsigned row, int c8, bool zero, float (&v)[8]) {
        const float* src = base + row;
        if (!RAG || c8 + 8 <= d) {
            const f4u a = *(const f4u*)(src + c8), b = *(const f4u*)(src + c8 + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[e] = a[e]; v[4 + e] = b[e]; }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                v[e] = src[min(c8 + e, d - 1)];
                if (zero && c8 + e >= d) v[e] = 0.f;
            }
        }
    };

    const int q = q0 + l32;           // this lane's query
    // Softmax: Q is taken pre-multiplied by c = scale*log2(e), so the scores
    // come out of the MFMAs already in the base-2 exponent domain.
    const float c = SM ? p.c : kSplitScale;
    b8 qh[KS], qm[KS], ql[KS];        // k-slot (h, e) of step t is d-index 16 t + 8 h + e
    float qmax = 0.f, kmax = 0.f;     // largest |q c|, |k| this thread has split
    {
#pragma unroll
        for (int t = 0; t < KS; ++t) {
            float v[8] = {};
            if (q < p.L) ld8(Q, (unsigned)q * d, 16 * t + 8 * h, true, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                v[e] *= c;
                if (SM) qmax = fmaxf(qmax, fabsf(v[e]));
            }
            split3(v, qh[t], qm[t], ql[t]);
        }
        if (SM) asm volatile("" : "+v"(qmax));   // found here, not from values kept to the end
    }
    f16x o[NTO];
#pragma unroll
    for (int n = 0; n < NTO; ++n) o[n] = f16x{};
    float m = -INFINITY;              // running maximum of t for query q
    float lsum = 0.f;                 // this half's share of the running sum

    const int nblk = max(0, (key_hi - key_lo + AKB - 1) / AKB);
    // blocks this wave contracts: under the mask, those with a key at or before its last query
    const int nact = causal ? max(0, min(nblk, (q0 + 2 * AQW - 1 - key_lo) / AKB)) : nblk;
    // Staging items: 4 D of K (row, eight columns), then 4 D of V (column,
    // eight keys); 4 D is a multiple of 64, so a wave's items are of one kind.
    // Keys past key_hi read as the last key and columns past d as the last
    // column, so no load is guarded: the scores of such keys are masked, Q is
    // 0 in such columns and O's are not written.
    typedef float Stage[NI][8];
    auto load = [&](Stage& st, int jk, int jv) {   // block jk of K, jv of V
        const int kk = key_lo + jk * AKB, kv = key_lo + jv * AKB;
        const float* Kb = Kp + (int64_t)kk * d;
        const float* Vb = Vp + (int64_t)kv * d;
        const int last_k = key_hi - 1 - kk, last_v = key_hi - 1 - kv;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int iw = wave64 + NTH * i, it = iw + lane;
            if (NI * NTH != 8 * D && iw >= 8 * D) break;
            if (iw < 4 * D) {
                ld8(Kb, (unsigned)(min(it / (D / 8), last_k) * d), it % (D / 8) * 8, false, st[i]);
            } else {
                const int iv = it - 4 * D, sh = iv / D, k0 = 16 * (sh >> 1) + 4 * (sh & 1);
                const unsigned col = RAG ? min(iv % D, d - 1) : iv % D;
                if (last_v >= AKB - 1) {
                    const float* src = Vb + (k0 * d + col);
#pragma unroll
                    for (int e = 0; e < 8; ++e) st[i][e] = src[(8 * (e >> 2) + (e & 3)) * d];
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        st[i][e] = Vb[(unsigned)min(k0 + 8 * (e >> 2) + (e & 3), last_v) * d + col];
                }
            }
        }
    };
    // block j into buffer j & 1
    auto stash = [&](const Stage& st, int jk, int jv) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int iw = wave64 + NTH * i, it = iw + lane, iv = it - 4 * D;
            if (NI * NTH != 8 * D && iw >= 8 * D) break;
            const bool is_k = iw < 4 * D;
            float v[8];
            const float scale = SM && is_k ? 1.f : kSplitScale;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                v[e] = st[i][e] * scale;
                if (SM && is_k) kmax = fmaxf(kmax, fabsf(v[e]));
            }
            b8 a, b, l;
            split3(v, a, b, l);
            unsigned char* dst = &lds[(is_k ? jk : jv) & 1][is_k ? (it / (D / 8)) * KP + it % (D / 8) * 16 : 3 * KB + (iv % D) * VP + iv / D * 16];
            const int plane = is_k ? KB : VB;
            *(b8*)dst = a;
            *(b8*)(dst + plane) = b;
            *(b8*)(dst + 2 * plane) = l;
        }
    };
    // S^T of block j: the h h products in one sum, the smaller ones in another
    auto scores = [&](int j, f16x& s) {
        const unsigned char* Ks = &lds[j & 1][l32 * KP + 16 * h];
        f16x slow = f16x{};
        s = f16x{};
#pragma unroll
        for (int t = 0; t < KS; ++t) {
            const b8 kh = *(const b8*)(Ks + 32 * t), km = *(const b8*)(Ks + KB + 32 * t),
                     kl = *(const b8*)(Ks + 2 * KB + 32 * t);
#define QX_S(S_, K_, Q_) S_ = __builtin_amdgcn_mfma_f32_32x32x16_bf16(K_, Q_[t], S_, 0, 0, 0);
            QX_S(slow, kl, qm) QX_S(slow, km, ql) QX_S(slow, kl, qh) QX_S(slow, km, qm) QX_S(slow, kh, ql)
            QX_S(slow, km, qh) QX_S(slow, kh, qm) QX_S(s, kh, qh)
#undef QX_S
        }
        s += slow;
        if (D > 64) __builtin_amdgcn_sched_barrier(0);
    };
    // the same from the caller's arrays, on the fp32 matrix cores
    auto scores_f32 = [&](int j, f16x& s) {
        const int key = key_lo + j * AKB + l32;
        const unsigned kr = (unsigned)min(key, key_hi - 1) * d;
        unsigned qr = (unsigned)min(q, p.L - 1) * d;
        asm volatile("" : "+v"(qr));      // read again: Q's values are not kept from the start for this
        s = f16x{};
#pragma unroll 2
        for (int t = 0; t < D; t += 16) {
            float kv[8], qv[8];
            ld8(Kp, kr, t + 8 * h, true, kv);
            ld8(Q, qr, t + 8 * h, true, qv);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[e], SM ? qv[e] * c : qv[e], s, 0, 0, 0);
        }
    };
    // Register r holds key kb + 8*(r/4) + 4*h + r%4.  In a block that
    // reaches past key_hi or (causal) past a query of this wave, keys at or
    // past key_lim are set to -inf, whose exponential is 0, or (no softmax)
    // to 0.
    auto mask = [&](int j, f16x& s) {
        const int kb = key_lo + j * AKB;
        if (kb + AKB > key_hi || (causal && kb + AKB - 1 > q0)) {
            const int key_lim = causal ? min(key_hi, q + 1) : key_hi;
            const int kl = key_lim - kb - 4 * h;    // register r is kept iff 8*(r/4) + r%4 < kl
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (8 * (r >> 2) + (r & 3) >= kl) s[r] = SM ? -INFINITY : 0.f;
        }
    };
    float alpha = 1.f, m_use = 0.f;   // the block's rescale factor and subtracted maximum
    auto maximum = [&](const f16x& s) {
        float mx = fmaxf(fmaxf(s[0], s[1]), s[2]);
#pragma unroll
        for (int r = 3; r < 15; r += 2) mx = fmaxf(fmaxf(mx, s[r]), s[r + 1]);
        mx = fmaxf(mx, s[15]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m, mx);
        m_use = m_new == -INFINITY ? 0.f : m_new;
        // v_exp_f32 directly: arguments are <= 0 here, results below 2^-126
        // flush to 0, which no sum of a row with its maximum term 1 can see
        alpha = __builtin_amdgcn_exp2f(m - m_use);
        m = m_new;
    };
    auto exponentials = [&](f16x& s, float scale) {
        float ps = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            s[r] = __builtin_amdgcn_exp2f(s[r] - m_use) * scale;
            ps += s[r];
        }
        lsum = lsum * alpha + ps;
    };
    auto split_s = [&](const f16x& s, b8 (&ph)[2], b8 (&pm)[2], b8 (&pl)[2]) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            float pv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) pv[e] = SM ? s[8 * t + e] : s[8 * t + e] * (1.f / kSplitScale);
            split3(pv, ph[t], pm[t], pl[t]);
        }
    };
    // O^T = alpha O^T + V^T S^T of block j, the smaller products and the h h
    // ones summed apart, each from zero.  The core adds the latter straight to
    // O in long sums and where registers are short (d >= 96): a matrix step
    // cuts its addend at 2^-25 of its largest product, which a short sum that
    // cancels shows (160 x 32: largest error 1.1e-6 of the rms so, 3.9e-7 from
    // zero; 6.6e-7 on the fp32 matrix cores).
    auto accumulate = [&](int j, const b8 (&ph)[2], const b8 (&pm)[2], const b8 (&pl)[2]) {
        const unsigned char* Vs = &lds[j & 1][3 * KB + l32 * VP + 16 * h];
        if (D > 64) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < NTO; ++n) {
            f16x high_sum = f16x{}, ls = f16x{};
            f16x& hs = FROM_ZERO ? high_sum : o[n];
            b8 vh[2];
#define QX_PV(S_, V_, P_) S_ = __builtin_amdgcn_mfma_f32_32x32x16_bf16(V_, P_[t], S_, 0, 0, 0);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const unsigned char* src = Vs + n * 32 * VP + 32 * t;
                vh[t] = *(const b8*)src;
                const b8 vm = *(const b8*)(src + VB), vl = *(const b8*)(src + 2 * VB);
                QX_PV(ls, vl, pm) QX_PV(ls, vm, pl) QX_PV(ls, vl, ph) QX_PV(ls, vm, pm) QX_PV(ls, vh[t], pl)
                QX_PV(ls, vm, ph) QX_PV(ls, vh[t], pm)
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) QX_PV(hs, vh[t], ph)
#undef QX_PV
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float low = SM ? fmaf(o[n][r], alpha, ls[r]) : o[n][r] + ls[r];
                o[n][r] = FROM_ZERO ? low + hs[r] : low;
            }
            if (D > 64) __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto accumulate_f32 = [&](int j, const f16x& s) {
        const int kb = key_lo + j * AKB + 4 * h;
#pragma unroll
        for (int n = 0; n < NTO; ++n) {
            const unsigned col = RAG ? min(n * 32 + l32, d - 1) : n * 32 + l32;
            float v[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = kb + 8 * (r >> 2) + (r & 3);
                v[r] = Vp[(unsigned)min(key, key_hi - 1) * d + col];
                if (key >= key_hi) v[r] = 0.f;
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) o[n] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[r], s[r], o[n], 0, 0, 0);
        }
    };

    b8 ph[2], pm[2], pl[2];
    Stage st;
    if constexpr (PIPE) {
        // Pass j splits the scores of block j beside the score products of
        // block j + 1, then stages K of block j + 2 and V of block j + 1 beside
        // the O products of block j.  (Past the last block the last one is
        // staged again; the last pass's scores are not used.)
        const int end = nblk - 1;
        Stage st1;
        load(st, 0, 0);
        load(st1, min(1, end), min(1, end));
        stash(st, 0, 0);
        stash(st1, 1, 1);
        load(st, min(2, end), min(1, end));
        __syncthreads();
        f16x s0, s1;
        scores(0, s0);
        mask(0, s0);
        __syncthreads();                     // pass 0 stages over K of block 0
        auto pass = [&](int j, f16x& s, f16x& sn) {
            scores(j + 1, sn);
            split_s(s, ph, pm, pl);
            // all of it before the mask's branch, beside the scores
#pragma unroll
            for (int t = 0; t < 2; ++t) asm volatile("" : "+v"(ph[t]), "+v"(pm[t]), "+v"(pl[t]));
            mask(j + 1, sn);
            accumulate(j, ph, pm, pl);
            stash(st, j + 2, j + 1);
            load(st, min(j + 3, end), min(j + 2, end));
            __syncthreads();
        };
        for (int j = 0; j < nblk; j += 2) {
            pass(j, s0, s1);
            if (j + 1 < nblk) pass(j + 1, s1, s0);
        }
    } else {
        if (nblk > 0) {
            load(st, 0, 0);
            stash(st, 0, 0);
            if (nblk > 1) load(st, 1, 1);
            __syncthreads();
        }
        for (int j = 0; j < nblk; ++j) {
            if (j < nact) {
                f16x s;
                scores(j, s);
                mask(j, s);
                if (SM) {
                    maximum(s);
                    exponentials(s, kSplitScale);
                }
                split_s(s, ph, pm, pl);
                // (before the products, which do not wait for it)
                if (j + 1 < nblk) stash(st, j + 1, j + 1);
                accumulate(j, ph, pm, pl);
            } else if (j + 1 < nblk) {
                stash(st, j + 1, j + 1);
            }
            if (j + 1 == nblk) break;
            if (j + 2 < nblk) load(st, j + 2, j + 2);
            __syncthreads();
        }
    }
    // Split values are finite only where the products are (f32_split.h): an
    // output that is not starts its wave again on the fp32 matrix cores (where
    // every wave does, 32 causal heads x 4096 x 64 take 1330 us and the core at
    // L = 4096, d = 64 101; 1880 and 129 with each load waited for by itself).
    // A score too low for fp32 would end as a probability of 0, so the softmax
    // form also holds |q| and |k| below 2^60.
    bool redo = SM && !(qmax < 0x1p60f && fabsf(lsum) < INFINITY);
#pragma unroll
    for (int n = 0; n < NTO; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) redo |= !(fabsf(o[n][r]) < INFINITY);
    redo = __ballot(redo) != 0;
    if (SM) {
        if (tid == 0) large_k = 0;
        __syncthreads();
        if (!(kmax < 0x1p60f)) large_k = 1;
        __syncthreads();
        redo |= large_k != 0;
    }
    // what the sums are multiplied by
    float lscale = SM ? kSplitScale : 1.f, oscale = kSplitScale * kSplitScale;
    if (redo) {
        lscale = oscale = 1.f;
#pragma unroll
        for (int n = 0; n < NTO; ++n) o[n] = f16x{};
        m = -INFINITY;
        lsum = 0.f;
        for (int j = 0; j < nact; ++j) {
            f16x s;
            scores_f32(j, s);
            mask(j, s);
            if (SM) {
                maximum(s);
#pragma unroll
                for (int n = 0; n < NTO; ++n)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[n][r] *= alpha;
                exponentials(s, 1.f);
            }
            accumulate_f32(j, s);
        }
    }

    // lane (q, h), register r of tile n: column 32 n + 8*(r/4) + 4*h + r%4
    const float l = SM ? lsum + __shfl_xor(lsum, 32) : 1.f;
    float f = 1.f / oscale;
    float* dst = p.O + hoff;
    if (p.splits > 1) {
        const int64_t rows = (int64_t)p.BH * p.L;
        dst = p.part + ((int64_t)split * rows + head * p.L) * d;
        if (SM && h == 0 && q < p.L) {
            float* stt = p.stat + ((int64_t)split * rows + head * p.L + q) * 2;
            stt[0] = m;
            stt[1] = l * (1.f / lscale);
        }
    } else if (SM) {
        f = l > 0.f ? 1.f / l * (lscale / oscale) : 0.f;
    }
    if (q >= p.L) return;
    dst += (int64_t)q * d;
#pragma unroll
    for (int n = 0; n < NTO; ++n)
#pragma unroll
        for (int r = 0; r < 16; r += 4) {
            const int col = 32 * n + 8 * (r >> 2) + 4 * h;
            const f4 v = f4{o[n][r] * f, o[n][r + 1] * f, o[n][r + 2] * f, o[n][r + 3] * f};
            if (!RAG) *(f4u*)(dst + col) = v;
            else
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (col + e < d) dst[col + e] = v[e];
        }
}

// Merge of the key splits, one thread per output element, splits in order:
// O = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s with M = max_s m_s.
__global__ __launch_bounds__(AT) void k_sdpa_combine(const SdpaCombineParams p) {
    const int64_t i = (int64_t)blockIdx.x * AT + threadIdx.x;
    if (i >= p.rows * p.d) return;
    const int64_t row = i / p.d;
    float M = -INFINITY;
    for (int s = 0; s < p.splits; ++s) M = fmaxf(M, p.stat[((int64_t)s * p.rows + row) * 2]);
    float num = 0.f, den = 0.f;
    for (int s = 0; s < p.splits; ++s) {
        const float* st = p.stat + ((int64_t)s * p.rows + row) * 2;
        const float w = exp2f(st[0] - M);
        num += w * p.part[(int64_t)s * p.rows * p.d + i];
        den += w * st[1];
    }
    p.O[i] = num / den;
}

// ---------------------------------------------------------------------------
// Builders
// ---------------------------------------------------------------------------
bool build_attn_i32(const AttnParams& p, LaunchRec* rec) {
    switch (p.d) {
    case 32: rec->fn = (const void*)k_attn_i32<32>; break;
    case 64: rec->fn = (const void*)k_attn_i32<64>; break;
    case 96: rec->fn = (const void*)k_attn_i32<96>; break;
    case 128: rec->fn = (const void*)k_attn_i32<128>; break;
    default: return false;
    }
    rec->name = "attn_i32";
    rec->grid = dim3((unsigned)((p.L + AQ - 1) / AQ), (unsigned)p.splits, 1);
    rec->block = dim3(AT, 1, 1);
    rec->set_params(p);
    return true;
}

bool resident_attn_i32(int64_t d, int64_t kps) {
    return (d == 32 || d == 64 || d == 128) && kps % 32 == 0 && (kps * d) % 4096 == 0 && 2 * kps * d <= 49152;
}

bool build_attn_i32_prep(const AttnParams& p, LaunchRec* rec) {
    switch (p.d) {
    case 32: rec->fn = (const void*)k_attn_i32_prep<32>; break;
    case 64: rec->fn = (const void*)k_attn_i32_prep<64>; break;
    case 128: rec->fn = (const void*)k_attn_i32_prep<128>; break;
    default: return false;
    }
    const int64_t items = p.prep_k + p.prep_v + p.prep_q + (p.clear_o ? (int64_t)p.L * p.d / 4 : 0);
    rec->name = "attn_i32_prep";
    rec->grid = dim3((unsigned)((items + AT - 1) / AT), 1, 1);
    rec->block = dim3(AT, 1, 1);
    rec->set_params(p);
    return true;
}

bool build_attn_i32r(const AttnParams& p, LaunchRec* rec) {
    switch (p.d) {
    case 32: rec->fn = (const void*)k_attn_i32r<32>; break;
    case 64: rec->fn = (const void*)k_attn_i32r<64>; break;
    case 128: rec->fn = (const void*)k_attn_i32r<128>; break;
    default: return false;
    }
    rec->name = "attn_i32_resident";
    rec->grid = dim3((unsigned)((p.L + AQ - 1) / AQ), (unsigned)p.splits, 1);
    rec->block = dim3(AT, 1, 1);
    rec->shmem = (uint32_t)(2 * (int64_t)p.keys_per_split * p.d);
    rec->set_params(p);
    return true;
}

bool build_attn_i32s(const AttnParams& p, LaunchRec* rec) {
    int keys = 0;
#define QX_ATTN_S(DD, QQ) \
    if (p.d == DD && p.qt == QQ) { rec->fn = (const void*)k_attn_i32s<DD, QQ>; keys = AttnStream<DD, QQ>::KEYS; }
    QX_ATTN_S(32, 2) QX_ATTN_S(64, 2)
#undef QX_ATTN_S
    if (keys == 0 || p.keys_per_split % keys != 0 || !p.v_blocks) return false;
    rec->name = "attn_i32_stream";
    rec->grid = dim3((unsigned)((p.L + 32 * p.qt - 1) / (32 * p.qt)), (unsigned)p.splits, 1);
    rec->block = dim3(512, 1, 1);
    rec->set_params(p);
    return true;
}

void build_reduce(const ReduceParams& p, LaunchRec* rec) {
    rec->fn = (const void*)k_reduce_splits;
    rec->grid = dim3((unsigned)((p.n + 4 * AT - 1) / (4 * AT)), 1, 1);
    rec->block = dim3(AT, 1, 1);
    rec->name = "reduce_splits";
    rec->set_params(p);
}

template <int D, bool SM>
static const void* attn_b3_fn(int queries, bool rag, bool pipe) {
    if constexpr (!SM && D <= 64)
        if (pipe) return (const void*)k_attn_b3<D, 4, false, false, true>;
    if (queries == 256) return rag ? (const void*)k_attn_b3<D, 8, SM, SM> : (const void*)k_attn_b3<D, 8, SM, false>;
    return rag ? (const void*)k_attn_b3<D, 4, SM, SM> : (const void*)k_attn_b3<D, 4, SM, false>;
}

bool build_attn_b3(const SdpaParams& p, bool softmax, int queries, LaunchRec* rec) {
    const int D = (p.d + 31) / 32 * 32;
    const bool rag = p.d != D;
    if (rag && !softmax) return false;
    const bool pipe = !softmax && queries == 128 && p.keys_per_split >= 8 * AKB && p.L >= 8 * AKB;
    switch (D) {
    case 32: rec->fn = softmax ? attn_b3_fn<32, true>(queries, rag, pipe) : attn_b3_fn<32, false>(queries, rag, pipe); break;
    case 64: rec->fn = softmax ? attn_b3_fn<64, true>(queries, rag, pipe) : attn_b3_fn<64, false>(queries, rag, pipe); break;
    case 96: rec->fn = softmax ? attn_b3_fn<96, true>(queries, rag, pipe) : attn_b3_fn<96, false>(queries, rag, pipe); break;
    case 128: rec->fn = softmax ? attn_b3_fn<128, true>(queries, rag, pipe) : attn_b3_fn<128, false>(queries, rag, pipe); break;
    default: return false;
    }
    rec->name = softmax ? "sdpa_f32" : "attn_f32";
    rec->grid = dim3((unsigned)((p.L + queries - 1) / queries), (unsigned)p.splits, (unsigned)p.BH);
    rec->block = dim3((unsigned)(2 * queries), 1, 1);
    rec->set_params(p);
    return true;
}

void build_sdpa_combine(const SdpaCombineParams& p, LaunchRec* rec) {
    rec->fn = (const void*)k_sdpa_combine;
    rec->grid = dim3((unsigned)((p.rows * p.d + AT - 1) / AT), 1, 1);
    rec->block = dim3(AT, 1, 1);
    rec->name = "sdpa_combine";
    rec->set_params(p);
}

}  // namespace qx

// Large-M forward: the prompt prefill that fills the KV cache before the
// first draft (Algorithm 2 starts from a cache holding the prompt), and
// long forwards in general.  With hundreds of rows the linear layers are
// dense contractions, 2 M N K flops per N K weight bytes, so they run on
// matrix cores:
//   - k_pf_gemm: C = A W^T with the float32 activations as X_TERMS bfloat16
//     terms (exact for float32 values), v_mfma 16x16x32 bf16 on tiles of
//     256 x 256 down to 128 x 64, every operand loaded straight into LDS in
//     MFMA fragment order; tiles are ordered so the work-groups one XCD
//     runs together share their weight and activation slices in that XCD's
//     L2; residual updates split the reduction into partials
//     (the QKV product's epilogue rotates q and k and appends to the cache, the
//     gate/up product's applies the SwiGLU);
//   - k_pf_thin: the same products for up to 64 rows, bound by the weight
//     stream;
//   - k_pf_attn128 and k_pf_attn_terms: causal attention for head_dim 128, 128
//     query rows of a head sharing 64-key stages through LDS, split over chunks
//     of the keys, and the chunks combined;
//   - k_pf_attn: causal attention for head_dim 32 and 64, one wave per 16 query
//     rows of a head, 32-key blocks;
//     both with scores and the weighted sum of values on matrix cores, an online
//     softmax, and the longest row blocks dispatched first;
//   - small row kernels between them: embedding, and RMSNorm into terms (adding
//     a residual update's partials first).
#include "sd_internal.h"

#include <algorithm>
#include <type_traits>

namespace sdk {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

__device__ __forceinline__ f32x4_t mfma16(u32x4_t a, u32x4_t b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b),
                                                   c, 0, 0, 0);
}

// Terms of eight consecutive values, each packed as 8 bf16 (one 16-byte word).
__device__ __forceinline__ void split8(const float (&x)[8], u32x4_t (&t)[X_TERMS]) {
    uint16_t h[X_TERMS][8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        uint16_t s[X_TERMS];
        split3(x[u], s);
#pragma unroll
        for (int i = 0; i < X_TERMS; ++i)
            h[i][u] = s[i];
    }
#pragma unroll
    for (int i = 0; i < X_TERMS; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            t[i][j] = (uint32_t)h[i][2 * j] | ((uint32_t)h[i][2 * j + 1] << 16);
}

// ---------------------------------------------------------------------------
// GEMM inputs
//
// A float32 activation is held as X_TERMS bfloat16 terms, which reproduce it
// exactly, and the weights are multiplied as stored, so every product is exact
// and only the float32 accumulation rounds.  (Two float16 terms of the row times
// a power of two take two thirds of the matrix instructions, but hold 22 bits,
// fewer below 2^-18 of the row's largest: MLP channels 2^24 and 2^30 times the
// others, undone by their down weights, moved logits by 0.39 of their deviation.)

// Terms of elements k .. k + 7 of row m (K of them): from x, one 16-byte word a term.
__device__ __forceinline__ void store_terms8(const PfTerms &o, int m, int k, int K, const float (&x)[8]) {
    u32x4_t t[X_TERMS];
    split8(x, t);
    uint16_t *p = o.at(m, k, K);
#pragma unroll
    for (int i = 0; i < X_TERMS; ++i)
        *reinterpret_cast<u32x4_t *>(p + i * o.step()) = t[i];
}

// The same of four elements (k a multiple of 4).
__device__ __forceinline__ void store_terms4(const PfTerms &o, int m, int k, int K, f32x4_t x) {
    uint16_t h[4][X_TERMS];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        split3(x[u], h[u]);
    uint16_t *p = o.at(m, k, K);
#pragma unroll
    for (int i = 0; i < X_TERMS; ++i)
        *reinterpret_cast<u32x2_t *>(p + i * o.step()) =
            u32x2_t{(uint32_t)h[0][i] | ((uint32_t)h[1][i] << 16), (uint32_t)h[2][i] | ((uint32_t)h[3][i] << 16)};
}

// Row i of 16-row weight tile t of a QKV product: eight elements of the first
// half of a head (i < 8), then their rotary partners, half = head_dim / 2 on.
__device__ __forceinline__ int qkv_row(int t, int i, int head_dim) {
    const int half = head_dim >> 1, per_head = half >> 3;
    const int head = t / per_head, p = (t - head * per_head) * 8 + (i & 7);
    return head * head_dim + (i < 8 ? p : half + p);
}

// Elements i .. i + 3 of tile t (y0) and their partners (y1) of row m: rotated q
// into q [M][ldq], rotated k and v into the cache (bfloat16).
__device__ __forceinline__ void store_qkv4(const PfRope &a, int t, int i, int m, f32x4_t y0, f32x4_t y1, float *q,
                                           int64_t ldq) {
    const int dh = a.head_dim, half = dh >> 1, per_head = half >> 3;
    const int head = t / per_head, e = (t - head * per_head) * 8 + i, pos = a.start + m;
    if (head < a.n_heads + a.n_kv_heads) {
        const float *cs = reinterpret_cast<const float *>(a.table + (int64_t)pos * half + e);
        const f32x4_t c01 = reinterpret_cast<const f32x4_t *>(cs)[0], c23 = reinterpret_cast<const f32x4_t *>(cs)[1];
        const float cx[4] = {c01[0], c01[2], c23[0], c23[2]}, cy[4] = {c01[1], c01[3], c23[1], c23[3]};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float r0 = y0[j] * cx[j] - y1[j] * cy[j];
            const float r1 = y1[j] * cx[j] + y0[j] * cy[j];
            y0[j] = r0;
            y1[j] = r1;
        }
    }
    if (head < a.n_heads) {
        float *o = q + (int64_t)m * ldq + head * dh + e;
        *reinterpret_cast<f32x4_t *>(o) = y0;
        *reinterpret_cast<f32x4_t *>(o + half) = y1;
    } else {
        const bool is_k = head < a.n_heads + a.n_kv_heads;
        const int g = head - a.n_heads - (is_k ? 0 : a.n_kv_heads);
        uint16_t *c = (is_k ? a.kcache : a.vcache) + (int64_t)g * a.kv_head_stride + (int64_t)pos * dh + e;
        u32x2_t w0, w1;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            w0[j] = (uint32_t)bf16_rne_bits(y0[2 * j]) | ((uint32_t)bf16_rne_bits(y0[2 * j + 1]) << 16);
            w1[j] = (uint32_t)bf16_rne_bits(y1[2 * j]) | ((uint32_t)bf16_rne_bits(y1[2 * j + 1]) << 16);
        }
        *reinterpret_cast<u32x2_t *>(c) = w0;
        *reinterpret_cast<u32x2_t *>(c + half) = w1;
    }
}

// ---------------------------------------------------------------------------
// GEMM
//
// C = A W^T on tiles of BM activation rows x BN weight rows, NWN x NWM waves,
// 32-k stages through LDS.  Every 16 x 32 MFMA operand block is 1 KB of LDS
// with lane l's 16 bytes at 16 l, so a fragment read is one contiguous 1 KB
// read.  All operands go from global memory straight into LDS
// (global_load_lds_dwordx4: lane l's 16 bytes to 16 l), P stages ahead in
// P + 1 stage buffers.  The barrier is a bare s_barrier: a release fence before
// it would also wait for the loads of the coming stages.

// s_waitcnt immediate (gfx9 layout: vmcnt bits 3:0 and 15:14, expcnt 6:4,
// lgkmcnt 11:8) that waits for vmcnt n and leaves the other counters alone
constexpr int wait_vmcnt(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// Sixteen bytes per lane from g to LDS at l + 16 lane (l the same in every
// lane).  The compiler does not see these loads: it would wait for all of them
// before it reads or writes LDS anywhere, as they might overlap.  The kernel
// counts them itself (wait_vmcnt).  They have no register result; M0 holds the
// LDS address and needs one wait state before the load.
__device__ __forceinline__ void load_to_lds16(const uint16_t *g, uint16_t *l) {
    const uint32_t off = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t *)l;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(
                     __builtin_amdgcn_readfirstlane(off)),
                 "v"(g)
                 : "memory", "m0");
}

template <int EPI, int BN, int BM, int NWN, int NWM, int P, int WPS>
__global__ __launch_bounds__(64 * NWN * NWM, WPS) void k_pf_gemm(PfGemmArgs a) {
    constexpr int T = X_TERMS, NW = NWN * NWM;
    constexpr int WN = BN / NWN, WM = BM / NWM;          // a wave's share
    constexpr int NT = WN / 16, MT = WM / 16;            // 16 x 16 output tiles per wave
    constexpr int NBW = BN / 16, NB = NBW + T * BM / 16; // blocks per stage: weights, then activation terms
    constexpr int PW = (NB + NW - 1) / NW;               // load instructions per wave and stage
    static_assert(NT * 16 == WN && MT * 16 == WM, "tile split");
    static_assert(EPI == EPI_STORE || EPI == EPI_PARTIAL || EPI == EPI_SWIGLU || EPI == EPI_QKV, "epilogue");
    constexpr bool SWI = EPI == EPI_SWIGLU, QKV = EPI == EPI_QKV;
    __shared__ __attribute__((aligned(1024))) uint16_t lds[(P + 1) * NB * 512];

    constexpr int BC = SWI ? BN / 2 : BN;                // output columns per tile
    const int M = a.M, N = a.N, K = a.K, F = N / 2;
    const int NC = SWI ? F : N;                          // output columns
    // Tile and k-split of this work-group.  Work-groups are dealt to the 8
    // XCDs in turn, so each XCD gets a contiguous range of tile indices, and
    // the range is walked in groups of 4 row tiles: the tiles one XCD runs
    // at a time form a compact block whose operand slices its L2 holds.
    const int TM = (M + BM - 1) / BM, TN = (NC + BC - 1) / BC, TT = TM * TN * a.splits;
    const int per = (TT + 7) / 8;
    int L = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || L >= TT)
        return;  // uniform over the work-group
    const int split = L % a.splits;
    L /= a.splits;
    const int GM = TM < 4 ? TM : 4;
    const int grp_i = L / (GM * TN), first = grp_i * GM, gm = min(TM - first, GM);
    const int in = L - grp_i * GM * TN;
    const int m0 = (first + in % gm) * BM, n0 = in / gm * BC;  // SWI: n0 is the first f
    // the split's stages (possibly none: its partial tile is then zeros)
    const int S_all = (K + 31) / 32, S_per = (S_all + a.splits - 1) / a.splits;
    const int s_begin = split * S_per, S = max(0, min(S_all - s_begin, S_per));

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wn = wave % NWN, wm = wave / NWN, col = lane & 15, grp = lane >> 4;

    // Weight block b holds rows n0 + 16 b .., with SWI eight gate rows
    // f = n0 + 8 b .. and then the up rows of the same f, with QKV eight rows of
    // the first half of a head and then their rotary partners; block NBW + c term
    // c / (BM / 16) of activation rows m0 + 16 (c % (BM / 16)) ...  Lane l loads
    // row l % 16, k chunk l / 16 (rows past the end read the last one: never
    // stored; where the blocks do not come out even, waves share the last one).
    const uint16_t *src[PW];
#pragma unroll
    for (int i = 0; i < PW; ++i) {
        const int b = min(wave + NW * i, NB - 1);
        if (b < NBW) {
            int row;
            if constexpr (SWI)
                row = (col < 8 ? 0 : F) + min(n0 + 8 * b + (col & 7), F - 1);
            else if constexpr (QKV)
                row = qkv_row(min(n0 / 16 + b, N / 16 - 1), col, a.rope.head_dim);
            else
                row = min(n0 + 16 * b + col, N - 1);
            src[i] = a.W + (int64_t)row * K + 8 * grp;
        } else {
            const int c = b - NBW, t = c / (BM / 16), rg = c % (BM / 16);
            src[i] = a.A + t * a.a_term + (int64_t)min(m0 + 16 * rg + col, M - 1) * K + 8 * grp;
        }
    }
    // stages past the end load the last one again (into buffers no one reads),
    // so every wave has the same number of loads in flight
    auto issue = [&](int stage, int buf) {
        const int k0 = (s_begin + min(stage, S - 1)) * 32;
        uint16_t *dst = lds + buf * NB * 512;
        if (k0 + 32 <= K) {
#pragma unroll
            for (int i = 0; i < PW; ++i)
                load_to_lds16(src[i] + k0, dst + min(wave + NW * i, NB - 1) * 512);
        } else {  // zeros past K
#pragma unroll
            for (int i = 0; i < PW; ++i)
                load_to_lds16(k0 + 8 * grp < K ? src[i] + k0 : a.zero, dst + min(wave + NW * i, NB - 1) * 512);
        }
    };

    // Where two waves per SIMD leave the registers, the second and third terms
    // have sums of their own: the large sum is then rounded once per stage and
    // not three times (the same time; keys and values of the first layer that
    // round to another bfloat16 than the float64 ones, 13B, 100 rows: 580 -> 339).
    constexpr int SUMS = WPS == 2 ? 2 : 1;
    f32x4_t acc[SUMS][NT][MT];
#pragma unroll
    for (int q = 0; q < SUMS; ++q)
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < MT; ++j)
                acc[q][i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    if (S > 0) {
#pragma unroll
        for (int p = 0; p < P; ++p)
            issue(p, p);
    }
    for (int s = 0, buf = 0; s < S; ++s) {
        // This wave's blocks of stage s have landed: at most the loads issued
        // after them are in flight.  Then everyone's have, and every read of
        // stage s - 1, whose buffer the next loads fill, has returned.
        __builtin_amdgcn_s_waitcnt(wait_vmcnt((P - 1) * PW));
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (P > 1 || s + 1 < S)
            issue(s + P, buf == 0 ? P : buf - 1);
        const uint16_t *ws = lds + buf * NB * 512, *as = ws + NBW * 512;
        buf = buf == P ? 0 : buf + 1;
        u32x4_t wf[NT], af[MT][T];
#pragma unroll
        for (int i = 0; i < NT; ++i)
            wf[i] = *reinterpret_cast<const u32x4_t *>(&ws[(wn * NT + i) * 512 + lane * 8]);
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int t = 0; t < T; ++t)
                af[j][t] = *reinterpret_cast<const u32x4_t *>(&as[(t * (BM / 16) + wm * MT + j) * 512 + lane * 8]);
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < MT; ++j) {
                    f32x4_t &c = acc[t ? SUMS - 1 : 0][i][j];
                    c = mfma16(wf[i], af[j][t], c);
                }
    }
    __builtin_amdgcn_s_waitcnt(wait_vmcnt(0));  // no load into LDS outlives the work-group
    f32x4_t(&sum)[NT][MT] = acc[0];
    if constexpr (SUMS == 2) {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < MT; ++j)
                sum[i][j] += acc[1][i][j];
    }

    // lane holds C^T[n0 + wn WN + 16 i + 4 grp + v][m0 + wm WM + 16 j + col]
    // (EPI_PARTIAL: of the split's partial sum, part[split][m][n])
    if constexpr (SWI || QKV) {
        // Block rows 0-7 and 8-15 are a pair's two rows (gate and up; a rotary
        // pair): lanes 0-31 hold the first, lanes 32-63 the second of the same
        // eight pairs.  Swapping the lane halves of two tiles leaves both rows
        // of the first tile's pairs in lanes 0-31 and of the second's in lanes
        // 32-63.
#pragma unroll
        for (int i = 0; i < NT; i += 2) {
            const int i2 = i + 1 < NT ? i + 1 : i;
            const int bl = wn * NT + (lane < 32 ? i : i2);
            const bool own = lane < 32 || i2 != i;
#pragma unroll
            for (int j = 0; j < MT; ++j) {
                const int m = m0 + wm * WM + 16 * j + col;
                f32x4_t y0, y1;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum[i][j][v]),
                                                                    __float_as_uint(sum[i2][j][v]), false, false);
                    y0[v] = __uint_as_float(r[0]);
                    y1[v] = __uint_as_float(r[1]);
                }
                if (m >= M || !own)
                    continue;
                if constexpr (SWI) {
                    const int f = n0 + 8 * bl + 4 * (grp & 1);
                    if (f >= F)  // F % 8 == 0
                        continue;
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        y0[v] = y0[v] / (1.0f + expf(-y0[v])) * y1[v];
                    store_terms4(a.out, m, f, F, y0);
                } else if (n0 + 16 * bl < N) {
                    store_qkv4(a.rope, n0 / 16 + bl, 4 * (grp & 1), m, y0, y1, a.C, a.ldc);
                }
            }
        }
    } else {
        float *C = EPI == EPI_PARTIAL ? a.part + (int64_t)split * M * a.ldc : a.C;
        const bool vec = (a.ldc & 3) == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0;
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const int n = n0 + wn * WN + 16 * i + 4 * grp;
#pragma unroll
            for (int j = 0; j < MT; ++j) {
                const int m = m0 + wm * WM + 16 * j + col;
                if (m >= M || n >= N)
                    continue;
                float *c = C + (int64_t)m * a.ldc + n;
                if (vec && n + 3 < N) {
                    *reinterpret_cast<f32x4_t *>(c) = sum[i][j];
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (n + u < N)
                            c[u] = sum[i][j][u];
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// GEMM for few rows (17 to 64): bound by the weight stream, with 2 M flops per
// weight byte on top.  A work-group owns TN tiles of 16 weight rows, over all
// MB blocks of 16 activation rows; its NW waves take every NW-th 64-element
// k-step and meet in LDS at the end, so nothing is shared and no wave waits
// for another inside the loop (the tile kernel above spends 0.4 us per 32-k
// stage on its barrier chain at these sizes, whatever the tile).  A wave loads
// its weights coalesced (eight lanes per 128-byte row slice) and transposes
// them through a private LDS tile whose 16-byte chunks are XOR-swizzled by row.
// The activation terms come in fragment order (thin_off), each operand one
// contiguous 1 KB load.

template <int EPI>
__device__ __forceinline__ int thin_row(int t, int i, const PfThinArgs &a) {
    if constexpr (EPI == EPI_QKV) {
        return qkv_row(t, i, a.rope.head_dim);
    } else if constexpr (EPI == EPI_SWIGLU) {  // eight gate rows and their up rows
        const int f = min(t * 8 + (i & 7), (a.N >> 1) - 1);
        return i < 8 ? f : (a.N >> 1) + f;
    } else {
        return min(t * 16 + i, a.N - 1);
    }
}

template <int EPI, int MB, int NW, int TN>
__global__ __launch_bounds__(64 * NW, 2) void k_pf_thin(PfThinArgs a) {
    constexpr int T = X_TERMS;
    constexpr int WL = TN * 16 * 64;          // elements of a wave's staging tile
    constexpr int RC = MB * 16 + 1;           // pitch of the reduction rows
    constexpr size_t SMEM_W = (size_t)NW * WL * 2, SMEM_R = (size_t)NW * 16 * RC * 4;
    __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM_W > SMEM_R ? SMEM_W : SMEM_R];
    __shared__ float fin[EPI == EPI_QKV || EPI == EPI_SWIGLU ? 16 * RC : 1];
    const int S = EPI == EPI_PARTIAL ? a.splits : 1;
    const int grp = blockIdx.x / S, sp = blockIdx.x - grp * S;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, kg = lane >> 4;
    const int M = a.M, n_tiles = a.n_tiles;
    uint16_t *wl = reinterpret_cast<uint16_t *>(smem) + wave * WL;
    // load instruction ii of tile j reads rows 8 ii + lane / 8, 16-byte chunk
    // lane % 8 of the k-step's 128-byte slice
    const int lrow = lane >> 3, lch = lane & 7;
    uint32_t woff[TN][2];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int ii = 0; ii < 2; ++ii)
            woff[j][ii] = ((uint32_t)thin_row<EPI>(min(grp * TN + j, n_tiles - 1), 8 * ii + lrow, a) * (uint32_t)a.K +
                           lch * 8) * 2;  // bytes (below 2^32: checked by the launcher)
    const int KS_all = a.K >> 6;
    const int ks0 = (int)(((int64_t)KS_all * sp) / S), ks1 = (int)(((int64_t)KS_all * (sp + 1)) / S);

    f32x4_t acc[TN][MB];
    u32x4_t wv[TN][2], xv[2][MB][T];
    // (a uniform base and a 32-bit offset per lane)
    auto load_w = [&](int q) {
        const char *base = reinterpret_cast<const char *>(a.W) + ((int64_t)q << 7);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int ii = 0; ii < 2; ++ii)
                wv[j][ii] =
                    __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(base + woff[j][ii]));
    };
    const uint32_t xoff = lane * 16;
    auto load_x = [&](int q, int i) {
        const char *base = reinterpret_cast<const char *>(a.X) + (int64_t)(2 * q + i) * (T * MB * 1024);
#pragma unroll
        for (int b = 0; b < MB; ++b)
#pragma unroll
            for (int t = 0; t < T; ++t)
                xv[i][b][t] = *reinterpret_cast<const u32x4_t *>(base + (t * MB + b) * 1024 + xoff);
    };
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int b = 0; b < MB; ++b)
            acc[j][b] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    int q = ks0 + wave;
    if (q < ks1) {
        load_w(q);
        load_x(q, 0);
        load_x(q, 1);
    }
    // One k-step, requesting the next one's operands if there is one.  The
    // last is peeled: where the loads are under a branch, the compiler waits at
    // the join for what may have been issued, that is for everything in flight.
    auto kstep = [&](int q, auto more) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int ii = 0; ii < 2; ++ii) {
                const int row = 8 * ii + lrow;
                *reinterpret_cast<u32x4_t *>(wl + j * 1024 + row * 64 + ((lch ^ (row & 7)) << 3)) = wv[j][ii];
            }
        if constexpr (decltype(more)::value)
            load_w(q + NW);
        // the staging tile is private to this wave, whose LDS accesses run in
        // program order; the fences only keep the compiler from reordering them
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const u32x4_t wf =
                    *reinterpret_cast<const u32x4_t *>(wl + j * 1024 + r16 * 64 + (((4 * i + kg) ^ (r16 & 7)) << 3));
#pragma unroll
                for (int t = 0; t < T; ++t)
#pragma unroll
                    for (int b = 0; b < MB; ++b)
                        acc[j][b] = mfma16(wf, xv[i][b][t], acc[j][b]);
            }
            // one set of registers per half step: its next activations (cache
            // hits) are requested once its MFMAs have read these
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (decltype(more)::value)
                load_x(q + NW, i);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    for (; q + NW < ks1; q += NW)
        kstep(q, std::true_type{});
    if (q < ks1)
        kstep(q, std::false_type{});

    // acc: lane holds rows 4 kg + v of tile j, activation row 16 b + r16.
    // Tile by tile the waves' sums meet in LDS and are added in wave order.
    float *red = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int t = grp * TN + j;
        if (t >= n_tiles)
            break;  // uniform over the work-group
        __syncthreads();
#pragma unroll
        for (int b = 0; b < MB; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                red[(wave * 16 + 4 * kg + v) * RC + 16 * b + r16] = acc[j][b][v];
        __syncthreads();
        // consecutive threads take consecutive weight rows of one activation row
        for (int o = tid; o < 16 * M; o += 64 * NW) {
            const int ni = o & 15, m = o >> 4;
            float v = red[ni * RC + m];
#pragma unroll
            for (int w = 1; w < NW; ++w)
                v += red[(w * 16 + ni) * RC + m];
            if constexpr (EPI == EPI_QKV || EPI == EPI_SWIGLU) {
                fin[ni * RC + m] = v;
            } else {
                const int n = t * 16 + ni;
                float *C = EPI == EPI_PARTIAL ? a.C + (int64_t)sp * M * a.ldc : a.C;
                if (n < a.N)
                    C[(int64_t)m * a.ldc + n] = v;
            }
        }
        if constexpr (EPI == EPI_SWIGLU || EPI == EPI_QKV) {
            __syncthreads();
            for (int o = tid; o < 2 * M; o += 64 * NW) {
                const int i = 4 * (o & 1), m = o >> 1;
                f32x4_t y0, y1;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    y0[v] = fin[(i + v) * RC + m];
                    y1[v] = fin[(i + v + 8) * RC + m];
                }
                if constexpr (EPI == EPI_QKV) {
                    store_qkv4(a.rope, t, i, m, y0, y1, a.C, a.ldc);
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        y0[v] = y0[v] / (1.0f + expf(-y0[v])) * y1[v];
                    store_terms4(a.out, m, t * 8 + i, a.N >> 1, y0);  // F is a multiple of 8
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Causal attention.  Work-group (64-row block, head): wave w takes query rows
// r0 .. r0 + 15 and walks the keys [0, start + its last row] in blocks of
// 32.  Score tile t, row i holds key kb + 16 t + 4 (i % 4) + i / 4, so lane
// group G ends up with keys kb + 16 t + 4 v + G, which are exactly the
// reduction slots 8 G + 4 t + v that the lane supplies to the value MFMA:
// the probabilities never leave their lanes.  Values are staged in the
// wave's LDS tile (row pitch head_dim + 16, conflict-free) and gathered in
// that key order.

constexpr int PA_KB = 32;

template <int DH>
__global__ __launch_bounds__(256) void k_pf_attn(PfAttnArgs a, PfTerms out) {
    constexpr int T = X_TERMS;
    constexpr int ES = DH / 32;     // 32-wide slices of head_dim (score MFMAs)
    constexpr int ET = DH / 16;     // 16-wide tiles of head_dim (value MFMAs)
    constexpr int VP = DH + 16;     // LDS pitch of a value row, bf16
    constexpr int LPR = DH / 8;     // lanes per value row (16-byte loads)
    constexpr int RPI = 64 / LPR;   // value rows per load instruction
    constexpr int NVJ = PA_KB / RPI;
    __shared__ __attribute__((aligned(16))) uint16_t vt[4][PA_KB * VP];

    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
    // Work-group i takes head i % H and row block TM - 1 - i / H: the
    // longest row blocks (most keys) start first, and consecutive indices,
    // which the dispatcher deals to the 8 XCDs in turn, carry the same mix of
    // row blocks on every XCD.  (With the row block as the fast grid index,
    // row blocks x and x + 8 of every head landed on one XCD: the one holding
    // the last row blocks had 2.4 times the work of the lightest.)
    const int TM = (a.M + 63) / 64;
    const int head = (int)(blockIdx.x % a.n_heads), g = head / (a.n_heads / a.n_kv_heads);
    const int r0 = (TM - 1 - (int)(blockIdx.x / a.n_heads)) * 64 + wave * 16;
    if (r0 >= a.M)
        return;  // uniform over the wave; the waves never synchronise
    const bool qok = r0 + col < a.M;
    const int rq = min(r0 + col, a.M - 1);
    const int qpos = a.start + rq;
    const int kend = a.start + min(r0 + 15, a.M - 1) + 1;  // keys some row of the wave sees
    const uint16_t *Kg = a.kcache + (int64_t)g * a.kv_head_stride;
    const uint16_t *Vg = a.vcache + (int64_t)g * a.kv_head_stride;
    uint16_t *vs = vt[wave];

    // query terms: B operand of the score MFMAs (dims x queries)
    u32x4_t qf[ES][T];
    {
        const float *qs = a.q + (int64_t)rq * a.ldq + (int64_t)head * DH + 8 * grp;
        const float scale = 1.0f / sqrtf((float)DH);
#pragma unroll
        for (int s = 0; s < ES; ++s) {
            const f32x4_t lo = reinterpret_cast<const f32x4_t *>(qs + 32 * s)[0];
            const f32x4_t hi = reinterpret_cast<const f32x4_t *>(qs + 32 * s)[1];
            float x[8];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                x[u] = lo[u] * scale;
                x[4 + u] = hi[u] * scale;
            }
            split8(x, qf[s]);
        }
    }

    float m_run = -INFINITY, l_run = 0.0f;
    f32x4_t oacc[ET];
#pragma unroll
    for (int et = 0; et < ET; ++et)
        oacc[et] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

    for (int kb = 0; kb < kend; kb += PA_KB) {
        // keys past kend read the last key inside it: their scores are
        // masked and their weights are zero
        u32x4_t kf[2][ES], vr[NVJ];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int key = min(kb + 16 * t + 4 * (col & 3) + (col >> 2), kend - 1);
            const uint16_t *kp = Kg + (int64_t)key * DH + 8 * grp;
#pragma unroll
            for (int s = 0; s < ES; ++s)
                kf[t][s] = *reinterpret_cast<const u32x4_t *>(kp + 32 * s);
        }
#pragma unroll
        for (int j = 0; j < NVJ; ++j) {
            const int key = min(kb + j * RPI + lane / LPR, kend - 1);
            vr[j] = *reinterpret_cast<const u32x4_t *>(Vg + (int64_t)key * DH + 8 * (lane % LPR));
        }
        __builtin_amdgcn_sched_barrier(0);

        f32x4_t sacc[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            sacc[t] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int s = 0; s < ES; ++s)
#pragma unroll
                for (int i = 0; i < T; ++i)
                    sacc[t] = mfma16(kf[t][s], qf[s][i], sacc[t]);
        }
        // online softmax; slot u = 4 t + v of this lane is key kb + 16 t + 4 v + grp
        float sv[8], bm = -INFINITY;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int key = kb + 16 * (u >> 2) + 4 * (u & 3) + grp;
            sv[u] = key <= qpos ? sacc[u >> 2][u & 3] : -INFINITY;
            bm = fmaxf(bm, sv[u]);
        }
        bm = fmaxf(bm, __shfl_xor(bm, 16, 64));
        bm = fmaxf(bm, __shfl_xor(bm, 32, 64));
        const float m_new = fmaxf(m_run, bm);  // finite: key 0 is in the first block
        const float sc = expf(m_run - m_new);
        float p[8], ls = 0.0f;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            p[u] = expf(sv[u] - m_new);
            ls += p[u];
        }
        ls += __shfl_xor(ls, 16, 64);
        ls += __shfl_xor(ls, 32, 64);
        l_run = l_run * sc + ls;
        m_run = m_new;
        u32x4_t pf[T];
        split8(p, pf);

        // values of the block into the wave's tile (after the previous
        // block's reads), then O^T += V^T P^T tile by tile
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int j = 0; j < NVJ; ++j)
            *reinterpret_cast<u32x4_t *>(vs + (j * RPI + lane / LPR) * VP + 8 * (lane % LPR)) = vr[j];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int et = 0; et < ET; ++et) {
            // A operand V^T: lane (col, grp) needs column 16 et + col of keys
            // kb + 16 (u >> 2) + 4 (u & 3) + grp, u = 0..7 (the score slots).
            // ds_read_b64_tr_b16 hands lane l of each 16-lane group element
            // l % 4 of the 8 bytes that lanes l / 4 + 4 k (k = 0..3) point at,
            // so lane r points at key kb + 16 I + 4 (r >> 2) + grp, columns
            // 16 et + 4 (r & 3) ..: two reads give the eight keys in order.
            uint32_t w[4];
#pragma unroll
            for (int I = 0; I < 2; ++I) {
                const uint16_t *src = vs + (16 * I + 4 * (col >> 2) + grp) * VP + 16 * et + 4 * (col & 3);
                const s16x4_t r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)src);
                w[2 * I] = (uint32_t)(uint16_t)r[0] | ((uint32_t)(uint16_t)r[1] << 16);
                w[2 * I + 1] = (uint32_t)(uint16_t)r[2] | ((uint32_t)(uint16_t)r[3] << 16);
            }
            const u32x4_t vf = {w[0], w[1], w[2], w[3]};
            oacc[et] *= sc;
#pragma unroll
            for (int i = 0; i < T; ++i)
                oacc[et] = mfma16(vf, pf[i], oacc[et]);
        }
    }

    // lane holds O^T[16 et + 4 grp + v][query col]
    if (!qok)
        return;
    const float inv = 1.0f / l_run;
#pragma unroll
    for (int et = 0; et < ET; ++et)
        store_terms4(out, rq, head * DH + 16 * et + 4 * grp, a.n_heads * DH, oacc[et] * inv);
}

// ---------------------------------------------------------------------------
// Row kernels (one work-group per row)

__device__ __forceinline__ void load8bf(const uint16_t *p, float (&x)[8]) {
    const u32x4_t w = *reinterpret_cast<const u32x4_t *>(p);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        x[2 * j] = __uint_as_float(w[j] << 16);
        x[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
    }
}

__global__ __launch_bounds__(256) void k_pf_embed(const uint16_t *E, int d, const int32_t *tokens, float *h) {
    const int m = blockIdx.x, k = (blockIdx.y * 256 + threadIdx.x) * 8;  // d is a multiple of 8
    if (k >= d)
        return;
    float x[8];
    load8bf(E + (int64_t)tokens[m] * d + k, x);
    f32x4_t *o = reinterpret_cast<f32x4_t *>(h + (int64_t)m * d + k);
    o[0] = f32x4_t{x[0], x[1], x[2], x[3]};
    o[1] = f32x4_t{x[4], x[5], x[6], x[7]};
}

// Threads of a row kernel: a row's loads in one or two steps of latency where
// there are few rows, smaller work-groups where rows fill the chip.
constexpr int PF_FEW_ROWS = 256;

__device__ __forceinline__ void load8f(const float *p, float (&x)[8]) {
    const f32x4_t a = reinterpret_cast<const f32x4_t *>(p)[0], b = reinterpret_cast<const f32x4_t *>(p)[1];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        x[j] = a[j];
        x[4 + j] = b[j];
    }
}

// g * h / rms(h) of every row as terms.  With splits > 0 the partials of a
// residual update are added into h first, in split order:
// h[m] += part[0][m] + part[1][m] + ...
template <int NT>
__global__ __launch_bounds__(NT) void k_pf_norm_split(float *h, const float *part, int splits, int64_t stride, int K,
                                                       const uint16_t *gain, float eps, PfTerms out) {
    __shared__ float red[NT / 64];
    const int m = blockIdx.x, tid = threadIdx.x;
    float *x = h + (int64_t)m * K;
    const float *p = part + (int64_t)m * K;
    float ss = 0.0f;
    // 16-byte loads (K is a multiple of 8): with 4-byte loads this pass over
    // the row and three partial planes took 40 us per 13B call
    for (int k = 8 * tid; k < K; k += 8 * NT) {
        float v[8];
        load8f(x + k, v);
        if (splits) {
            float w[8];
            load8f(p + k, w);
            for (int s = 1; s < splits; ++s) {
                float w2[8];
                load8f(p + (int64_t)s * stride + k, w2);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    w[j] += w2[j];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
                v[j] += w[j];
            reinterpret_cast<f32x4_t *>(x + k)[0] = f32x4_t{v[0], v[1], v[2], v[3]};
            reinterpret_cast<f32x4_t *>(x + k)[1] = f32x4_t{v[4], v[5], v[6], v[7]};
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            ss = fmaf(v[j], v[j], ss);
    }
    ss = wave_sum_all(ss);
    if ((tid & 63) == 0)
        red[tid >> 6] = ss;
    __syncthreads();
    ss = 0.0f;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w)
        ss += red[w];
    const float inv = 1.0f / sqrtf(ss / (float)K + eps);
    // (re-reads what this thread wrote or read above)
    for (int k = 8 * tid; k < K; k += 8 * NT) {
        float v[8], g[8];
        load8f(x + k, v);
        load8bf(gain + k, g);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            v[j] = g[j] * (v[j] * inv);
        store_terms8(out, m, k, K, v);
    }
}

// ---------------------------------------------------------------------------
// Causal attention, head_dim 128.  A work-group takes 128 query rows of one
// head, 32 per wave, over one chunk of the keys, in stages of 64 keys whose K
// and V rows all four waves read from LDS (loaded straight there, one stage
// ahead).  With every wave loading its own K and V for 16 rows, as k_pf_attn
// does, 1000 rows over 8000 keys read 11 GB through the L2s per 13B layer and
// spent most of their issue slots on the softmax: 1082 us a layer; this kernel
// 480 us.  It is bound by its matrix instructions (three bfloat16 terms of q
// and of the probabilities).
//
// 32 keys at a time: scores S^T = K q as 32x32x16 MFMAs leave lane (col, half)
// the keys 8 (v / 4) + 4 half + v % 4, v = 0..15, of query col; the values
// v = 8 j .. 8 j + 7 are the operand slots (half, u) of the j-th 16-key value
// MFMA, so the probabilities stay in their lanes and V^T is read to match.
// Scores are in units of log2: q carries the factor log2(e) / sqrt(128).
//
// LDS rows are 256 bytes; row r keeps its 16-byte chunk c at c ^ swz(r), so
// that a K read (32 rows, one chunk) and a transposed V read (four rows, four
// adjacent chunks) touch every bank once.  The loads permute the chunks of a
// row on the way in, within the row's own cache lines.
//
// Each (chunk, row, head) leaves its unnormalised output and (max, sum), which
// k_pf_attn_terms combines in chunk order.  Work-group i takes head i % H (the
// work-groups of a head run on one XCD when H is a multiple of 8), the longest
// row blocks first.

constexpr int PA2_ROWS = 128;  // query rows per work-group
constexpr int PA2_KB = 64;     // keys per stage

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2v_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x16_t mfma32(u32x4_t a, u32x4_t b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                   0, 0, 0);
}
__device__ __forceinline__ uint32_t cvt_pk_bf16(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2v_t{a, b}), bf16x2_t));
}
// The three bf16 terms of two values, packed (the conversion rounds to nearest even).
__device__ __forceinline__ void split3_pk(float a, float b, uint32_t (&t)[X_TERMS]) {
    t[0] = cvt_pk_bf16(a, b);
    const float a1 = a - __uint_as_float(t[0] << 16), b1 = b - __uint_as_float(t[0] & 0xffff0000u);
    t[1] = cvt_pk_bf16(a1, b1);
    t[2] = cvt_pk_bf16(a1 - __uint_as_float(t[1] << 16), b1 - __uint_as_float(t[1] & 0xffff0000u));
}

__global__ __launch_bounds__(256, 2) void k_pf_attn128(PfAttnArgs a) {
    constexpr int DH = 128, T = X_TERMS;
    __shared__ __attribute__((aligned(1024))) uint16_t kv[2][2][PA2_KB * DH];  // [stage % 2][K, V]
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
    const int RB = (a.M + PA2_ROWS - 1) / PA2_ROWS;
    const int head = (int)(blockIdx.x % a.n_heads), g = head / (a.n_heads / a.n_kv_heads);
    const int unit = (int)(blockIdx.x / a.n_heads);
    const int chunk = unit % a.chunks, rb = RB - 1 - unit / a.chunks;
    const int w0 = rb * PA2_ROWS, r0 = w0 + wave * 32;
    const int kend = a.start + min(w0 + PA2_ROWS, a.M);  // keys some row of the work-group sees
    const int k_lo = chunk * a.chunk_keys, k_hi = min(kend, k_lo + a.chunk_keys);
    if (k_lo >= k_hi)
        return;  // uniform over the work-group: k_pf_attn_terms leaves this chunk out
    const int rq = min(r0 + col, a.M - 1), qpos = a.start + rq;
    const int q_min = a.start + r0;                          // the wave's first row sees keys up to here
    const int q_max = a.start + min(r0 + 31, a.M - 1);       // and its last row up to here

    // query terms: B operand of the score MFMAs
    u32x4_t qf[8][T];
    {
        const float *qs = a.q + (int64_t)rq * a.ldq + (int64_t)head * DH + 8 * half;
        const float scale = 1.4426950408889634f / sqrtf((float)DH);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            float x[8];
            load8f(qs + 16 * s, x);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t t[T];
                split3_pk(x[2 * j] * scale, x[2 * j + 1] * scale, t);
#pragma unroll
                for (int i = 0; i < T; ++i)
                    qf[s][i][j] = t[i];
            }
        }
    }

    const uint16_t *Kg = a.kcache + (int64_t)g * a.kv_head_stride, *Vg = a.vcache + (int64_t)g * a.kv_head_stride;
    auto swz = [](int r) { return ((r & 3) << 2) | ((r >> 2) & 3); };
    // load instruction i of a wave fills rows 16 wave + 4 i .. + 3 of K or V
    auto load_stage = [&](int kb, int buf) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 16 * wave + 4 * i + (lane >> 4), key = min(kb + r, kend - 1);
            const int64_t o = (int64_t)key * DH + 8 * ((lane & 15) ^ swz(r));
            load_to_lds16(Kg + o, &kv[buf][0][(16 * wave + 4 * i) * DH]);
            load_to_lds16(Vg + o, &kv[buf][1][(16 * wave + 4 * i) * DH]);
        }
    };

    float m_run = -INFINITY, l_run = 0.0f;
    f32x16_t oacc[4];
#pragma unroll
    for (int et = 0; et < 4; ++et)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            oacc[et][v] = 0.0f;

    load_stage(k_lo, 0);
    int buf = 0;
    for (int kb = k_lo; kb < k_hi; kb += PA2_KB, buf ^= 1) {
        // this wave's loads of the stage have landed, then everyone's; every
        // read of the other buffer has returned
        __builtin_amdgcn_s_waitcnt(wait_vmcnt(0));
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (kb + PA2_KB < k_hi)
            load_stage(kb + PA2_KB, buf ^ 1);
        const uint16_t *ks = kv[buf][0], *vs = kv[buf][1];
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
            const int k0 = kb + 32 * h;
            if (k0 > q_max || k0 >= k_hi)
                break;  // uniform over the wave: no row of it sees these keys
            f32x16_t s;
#pragma unroll
            for (int v = 0; v < 16; ++v)
                s[v] = 0.0f;
            const int kr = 32 * h + col;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const u32x4_t kf =
                    *reinterpret_cast<const u32x4_t *>(ks + kr * DH + 8 * ((2 * e + half) ^ swz(kr)));
#pragma unroll
                for (int i = 0; i < T; ++i)
                    s = mfma32(kf, qf[e][i], s);
            }
            if (k0 + 31 > q_min || k0 + 31 >= k_hi) {
                // keys a row does not see, and keys past the chunk
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int key = k0 + 8 * (v >> 2) + 4 * half + (v & 3);
                    s[v] = key <= qpos && key < k_hi ? s[v] : -INFINITY;
                }
            }
            float mx = s[0];
#pragma unroll
            for (int v = 1; v < 16; ++v)
                mx = fmaxf(mx, s[v]);
            {
                const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
                mx = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
            }
            if (__any(mx > m_run)) {
                // (a row that has seen no key yet keeps zeros)
                const float m_new = fmaxf(m_run, mx);
                const float sc = m_run == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m_run - m_new);
                l_run *= sc;
#pragma unroll
                for (int et = 0; et < 4; ++et)
                    oacc[et] *= sc;
                m_run = m_new;
            }
            const float m_use = m_run == -INFINITY ? 0.0f : m_run;
            // (the running sum is rounded once per block: weight by weight, equal
            // ones err the same way, 2.9e-5 of the sum over 7600 keys a lane)
            float p[16], sum = 0.0f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                p[v] = __builtin_amdgcn_exp2f(s[v] - m_use);
                sum += p[v];
            }
            l_run += sum;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                u32x4_t pf[T];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    uint32_t t[T];
                    split3_pk(p[8 * j + 2 * u], p[8 * j + 2 * u + 1], t);
#pragma unroll
                    for (int i = 0; i < T; ++i)
                        pf[i][u] = t[i];
                }
                // A operand V^T: lane (col, half) needs column 32 et + col of
                // keys 16 j + 8 (u / 4) + 4 half + u % 4.  ds_read_b64_tr_b16
                // hands lane l of each 16-lane group element l % 4 of the 8
                // bytes that lanes l / 4 + 4 k (k = 0..3) point at: lane l
                // points at key 16 j + 8 I + 4 half + l / 4 % 4, columns 32 et +
                // 16 (l / 16 % 2) + 4 (l % 4) ...
#pragma unroll
                for (int et = 0; et < 4; ++et) {
                    u32x4_t vf;
#pragma unroll
                    for (int I = 0; I < 2; ++I) {
                        const int r = 32 * h + 16 * j + 8 * I + 4 * half + ((lane >> 2) & 3);
                        const int c = 4 * et + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
                        const uint16_t *src = vs + r * DH + 8 * (c ^ swz(r)) + 4 * (lane & 1);
                        const s16x4_t x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)src);
                        const u32x2_t y = __builtin_bit_cast(u32x2_t, x);
                        vf[2 * I] = y[0];
                        vf[2 * I + 1] = y[1];
                    }
#pragma unroll
                    for (int i = 0; i < T; ++i)
                        oacc[et] = mfma32(vf, pf[i], oacc[et]);
                }
            }
        }
    }

    // lane holds O^T[32 et + 8 (v / 4) + 4 half + v % 4][query col]
    const auto lr = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
    const float l = __uint_as_float(lr[0]) + __uint_as_float(lr[1]);
    if (r0 + col < a.M) {
        const int64_t row = (int64_t)chunk * a.M + rq;
        float *o = a.out + row * a.ldo + (int64_t)head * DH + 4 * half;
#pragma unroll
        for (int et = 0; et < 4; ++et)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<f32x4_t *>(o + 32 * et + 8 * q) =
                    f32x4_t{oacc[et][4 * q], oacc[et][4 * q + 1], oacc[et][4 * q + 2], oacc[et][4 * q + 3]};
        if (half == 0)
            a.ml[row * a.n_heads + head] = make_float2(m_run, l);
    }
}

// The chunks of k_pf_attn128 combined in order and normalised, one work-group
// per row, as terms.  LDS: the chunks' weights [H][chunks].
template <int NT>
__global__ __launch_bounds__(NT) void k_pf_attn_terms(PfAttnArgs a, PfTerms out) {
    extern __shared__ __attribute__((aligned(16))) float wt[];
    const int m = blockIdx.x, tid = threadIdx.x, H = a.n_heads, hd = H * 128;
    // chunks some row of this row's work-group saw keys of
    const int kend = a.start + min((m / PA2_ROWS + 1) * PA2_ROWS, a.M);
    const int nc = min(a.chunks, (kend + a.chunk_keys - 1) / a.chunk_keys);
    for (int h = tid; h < H; h += NT) {
        float mx = -INFINITY, L = 0.0f;
        for (int c = 0; c < nc; ++c)
            mx = fmaxf(mx, a.ml[((int64_t)c * a.M + m) * H + h].x);
        for (int c = 0; c < nc; ++c) {
            const float2 v = a.ml[((int64_t)c * a.M + m) * H + h];
            const float w = v.x == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(v.x - mx);
            wt[h * nc + c] = w;
            L = fmaf(w, v.y, L);
        }
        const float inv = 1.0f / L;
        for (int c = 0; c < nc; ++c)
            wt[h * nc + c] *= inv;
    }
    __syncthreads();
    for (int k = 8 * tid; k < hd; k += 8 * NT) {
        const float *w = wt + (k >> 7) * nc, *p = a.out + (int64_t)m * a.ldo + k;
        float v[8] = {};
        for (int c = 0; c < nc; ++c) {
            float x[8];
            load8f(p + (int64_t)c * a.M * a.ldo, x);
#pragma unroll
            for (int j = 0; j < 8; ++j)
                v[j] += w[c] * x[j];
        }
        store_terms8(out, m, k, hd, v);
    }
}

}  // namespace

hipError_t launch_pf_embed(const uint16_t *emb, int d, const int32_t *tokens, int M, float *h, hipStream_t s) {
    hipLaunchKernelGGL(k_pf_embed, dim3(M, (d + 2047) / 2048), dim3(256), 0, s, emb, d, tokens, h);
    return hipGetLastError();
}

hipError_t launch_pf_norm_split(float *h, const float *part, int splits, int K, int M, const uint16_t *gain, float eps,
                                const PfTerms &t, hipStream_t s) {
    if (K % 8 || (t.blocks && K % 32) || splits < 0 || splits > PF_MAX_SPLITS)
        return hipErrorInvalidValue;
    auto kern = M <= PF_FEW_ROWS ? k_pf_norm_split<1024> : k_pf_norm_split<256>;
    hipLaunchKernelGGL(kern, dim3(M), dim3(M <= PF_FEW_ROWS ? 1024 : 256), 0, s, h, part, splits, (int64_t)M * K, K,
                       gain, eps, t);
    return hipGetLastError();
}

namespace {

template <int BN, int BM, int NWN, int NWM, int P, int WPS>
hipError_t launch_tile(const PfGemmArgs &a, int epi, hipStream_t s) {
    const int bc = epi == EPI_SWIGLU ? BN / 2 : BN, nc = epi == EPI_SWIGLU ? a.N / 2 : a.N;
    const int tiles = ((nc + bc - 1) / bc) * ((a.M + BM - 1) / BM) * a.splits;
    const dim3 grid(8 * ((tiles + 7) / 8)), block(64 * NWN * NWM);
    if (epi == EPI_STORE)
        hipLaunchKernelGGL((k_pf_gemm<EPI_STORE, BN, BM, NWN, NWM, P, WPS>), grid, block, 0, s, a);
    else if (epi == EPI_RESID)
        hipLaunchKernelGGL((k_pf_gemm<EPI_PARTIAL, BN, BM, NWN, NWM, P, WPS>), grid, block, 0, s, a);
    else if (epi == EPI_SWIGLU)
        hipLaunchKernelGGL((k_pf_gemm<EPI_SWIGLU, BN, BM, NWN, NWM, P, WPS>), grid, block, 0, s, a);
    else if (epi == EPI_QKV)
        hipLaunchKernelGGL((k_pf_gemm<EPI_QKV, BN, BM, NWN, NWM, P, WPS>), grid, block, 0, s, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

template <int EPI, int NW, int TN>
hipError_t launch_thin_mb(const PfThinArgs &a, hipStream_t s) {
    const dim3 grid((a.n_tiles + TN - 1) / TN * (EPI == EPI_PARTIAL ? a.splits : 1)), block(64 * NW);
    switch ((a.M + 15) / 16) {
    case 1:
    case 2:
        hipLaunchKernelGGL((k_pf_thin<EPI, 2, NW, TN>), grid, block, 0, s, a);
        break;
    case 3:
        if constexpr (TN > 4)
            return hipErrorInvalidValue;
        else
            hipLaunchKernelGGL((k_pf_thin<EPI, 3, NW, TN>), grid, block, 0, s, a);
        break;
    case 4:
        if constexpr (TN > 4)
            return hipErrorInvalidValue;
        else
            hipLaunchKernelGGL((k_pf_thin<EPI, 4, NW, TN>), grid, block, 0, s, a);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int NW, int TN>
hipError_t launch_thin_nw(const PfThinArgs &a, int epi, hipStream_t s) {
    switch (epi) {
    case EPI_STORE:
        return launch_thin_mb<EPI_STORE, NW, TN>(a, s);
    case EPI_PARTIAL:
        return launch_thin_mb<EPI_PARTIAL, NW, TN>(a, s);
    case EPI_SWIGLU:
        return launch_thin_mb<EPI_SWIGLU, NW, TN>(a, s);
    case EPI_QKV:
        return launch_thin_mb<EPI_QKV, NW, TN>(a, s);
    default:
        return hipErrorInvalidValue;
    }
}

}  // namespace

namespace {

// The tiles of k_pf_gemm: weight rows, activation rows, and the time of one
// 32-k stage of a work-group (ns, one work-group per CU with the chip full;
// 13B and 7B shapes, random operands, weights not in cache).  The larger tiles
// read fewer operand bytes per product: 256 x 256 multiplies 1.9 times as fast
// per CU as 128 x 64.  Tiles of 224 save an eighth of the columns and 2 to 4%
// of the time, as the power limit sets the clock: they are for layers they
// fill the rounds of better (13B gate/up, 1000 rows: 496 of 512 work-group
// slots and 752 us, 432 and 770 us with 256).
struct PfTile {
    int bn, bm, ns;
};
constexpr PfTile PF_TILES[PF_TILE_COUNT] = {
    {256, 256, 2500}, {224, 256, 2400}, {256, 128, 1340}, {128, 128, 960}, {128, 64, 600}};

}  // namespace

// The tile and the split of the reduction with the least time by that table:
// rounds of one work-group per CU, times the stages of a split, plus the
// writing and reading of the partial sums at 5 TB/s.
int pf_gemm_tile(int M, int N, int K, int epi, int *splits) {
    const int stages = (K + 31) / 32;
    // partial planes: PF_MAX_SPLITS of them, and in all 4 x PF_ROWS rows
    const int most = epi == EPI_RESID ? std::min(PF_MAX_SPLITS, PF_PART_ROWS / M) : 1;
    double best = 0.0;
    int tile = -1;
    for (int i = 0; i < PF_TILE_COUNT; ++i) {
        const PfTile &t = PF_TILES[i];
        const int bc = epi == EPI_SWIGLU ? t.bn / 2 : t.bn, nc = epi == EPI_SWIGLU ? N / 2 : N;
        const int64_t tiles = (int64_t)((nc + bc - 1) / bc) * ((M + t.bm - 1) / t.bm);
        for (int s = 1; s <= most && (s == 1 || stages >= 8 * s); ++s) {
            const double rounds = (double)((tiles * s + 255) / 256);
            const double ns =
                rounds * ((stages + s - 1) / s) * t.ns + (epi == EPI_RESID ? s * 8.0e-3 / 5 * M * N : 0.0);
            if (tile < 0 || ns < best) {
                best = ns;
                tile = i;
                *splits = s;
            }
        }
    }
    return tile;
}

hipError_t launch_pf_gemm_tile(const PfGemmArgs &a, int epi, int tile, hipStream_t s) {
    if (a.M < 1 || a.N < 1 || a.K < 8 || a.K % 8 || a.M > PF_ROWS || !a.zero || a.splits < 1 ||
        a.splits > (epi == EPI_RESID ? PF_MAX_SPLITS : 1) || a.splits * a.M > PF_PART_ROWS)
        return hipErrorInvalidValue;
    if (epi == EPI_SWIGLU ? (a.N % 16 || !a.out.x || a.out.blocks) : epi == EPI_RESID ? !a.part
        : epi == EPI_QKV ? (a.rope.head_dim % 16 || a.N % 16) : epi != EPI_STORE)
        return hipErrorInvalidValue;
    // Waves, and stages in flight: as many as LDS takes for one work-group per
    // CU, but two of them for 128 x 64 (13B, 1023 rows, QKV: 256 x 128 two
    // stages ahead 439 us, one and two work-groups per CU 473; 128 x 64 in four
    // waves 757, in eight 900).
    switch (tile) {
    case 0:
        return launch_tile<256, 256, 4, 4, 1, 4>(a, epi, s);
    case 1:
        return launch_tile<224, 256, 2, 8, 1, 4>(a, epi, s);
    case 2:
        return launch_tile<256, 128, 4, 2, 2, 2>(a, epi, s);
    case 3:
        return launch_tile<128, 128, 4, 2, 2, 2>(a, epi, s);
    case 4:
        return launch_tile<128, 64, 2, 2, 3, 2>(a, epi, s);
    default:
        return hipErrorInvalidValue;
    }
}

hipError_t launch_pf_gemm(const PfGemmArgs &a, int epi, hipStream_t s, int *out) {
    if (a.M < 1 || a.N < 1 || a.K < 8 || a.M > PF_ROWS || (epi == EPI_RESID && !out))
        return hipErrorInvalidValue;
    PfGemmArgs b = a;
    const int tile = pf_gemm_tile(a.M, a.N, a.K, epi, &b.splits);
    if (epi == EPI_RESID)
        *out = b.splits;
    return launch_pf_gemm_tile(b, epi, tile, s);
}

bool pf_thin_ok(int M, int64_t N, int K) { return M <= PF_THIN_ROWS && K % 64 == 0 && N * K < ((int64_t)1 << 31); }

hipError_t launch_pf_thin(const PfThinArgs &a0, int epi, hipStream_t s, int *out) {
    PfThinArgs a = a0;
    if (a.M < 1 || a.N < 1 || !pf_thin_ok(a.M, a.N, a.K))
        return hipErrorInvalidValue;
    a.splits = 1;
    if (epi == EPI_SWIGLU) {
        if (a.N % 16 || !a.out.x)
            return hipErrorInvalidValue;
        a.n_tiles = a.N / 16;
    } else if (epi == EPI_QKV) {
        if (a.rope.head_dim % 16)
            return hipErrorInvalidValue;
        a.n_tiles = a.N / 16;
    } else {
        a.n_tiles = (a.N + 15) / 16;
    }
    // Tiles per work-group: four, or three where that takes an eighth off the
    // tiles of the busiest CU (us, 33 rows: 7B gate/up, 6 for 8, 60.6 -> 51.4,
    // QKV, 3 for 4, 32.6 -> 30.0; not 13B gate/up, 9 for 8, 75.3 and 91.7).
    // Up to 32 rows seven where that is one group per CU (13B gate/up, 20 rows:
    // 67.0 -> 55.2; at 33 rows there are no registers for them).
    int tn = 4;
    if (epi != EPI_RESID) {
        tn = 8 * mfma_busiest(3, a.n_tiles) <= 7 * mfma_busiest(4, a.n_tiles) ? 3 : 4;
        if (a.M <= 32 && mfma_busiest(7, a.n_tiles) == 7 && mfma_busiest(tn, a.n_tiles) > 7)
            tn = 7;
    }
    const int groups = (a.n_tiles + tn - 1) / tn;
    if (epi == EPI_RESID) {
        if (!out)
            return hipErrorInvalidValue;
        // output projections: as many splits of the reduction as fill the CUs
        // with one work-group (33 rows: 13B, 80 groups, O 21.2, 17.2 and 21.6 us
        // with 2, 3 and 4 splits, down 48.1, 38.2 and 49.0; 7B, 64 groups, O 13.5,
        // 11.7 and 15.4 with 3, 4 and 5)
        a.splits = std::max(1, std::min({PF_MAX_SPLITS, 256 / groups, a.K / 512}));
        *out = a.splits;
        epi = EPI_PARTIAL;
    }
    // (four waves: eight of them lose up to 5% at the same number of tiles)
    return tn == 3 ? launch_thin_nw<4, 3>(a, epi, s)
           : tn == 4 ? launch_thin_nw<4, 4>(a, epi, s) : launch_thin_nw<8, 7>(a, epi, s);
}

// Chunks of the keys per row block: enough work-groups for PA_UNITS of them,
// chunks of at least 256 keys, and no more partial rows than the scratch holds.
constexpr int PA_UNITS = 1280;

hipError_t launch_pf_attention(const PfAttnArgs &a0, const PfTerms &t, hipStream_t s) {
    PfAttnArgs a = a0;
    if (a.M < 1 || a.n_heads < 1 || a.n_kv_heads < 1 || a.n_heads % a.n_kv_heads)
        return hipErrorInvalidValue;
    const int hd = a.n_heads * a.head_dim;
    // head_dim 128 with more than 64 heads (none of the shapes here) runs on
    // k_pf_attn: us of 64 heads on this kernel and 66 on that one, 1000 rows over
    // 4000 keys 437 and 812, 600 from position 0 44 and 45, 200 from position 0 22
    // and 17.
    if (a.head_dim == 128 && hd <= 8192) {
        const int units = ((a.M + PA2_ROWS - 1) / PA2_ROWS) * a.n_heads, keys = a.start + a.M;
        const int most = std::min({PF_PART_ROWS / a.M, keys / 256, 16384 / a.n_heads});
        a.chunks = std::max(1, std::min(most, (PA_UNITS + units - 1) / units));
        a.chunk_keys = ((keys + a.chunks - 1) / a.chunks + PA2_KB - 1) / PA2_KB * PA2_KB;
        a.chunks = (keys + a.chunk_keys - 1) / a.chunk_keys;
        hipLaunchKernelGGL(k_pf_attn128, dim3(units * a.chunks), dim3(256), 0, s, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        auto kern = a.M <= PF_FEW_ROWS ? k_pf_attn_terms<1024> : k_pf_attn_terms<256>;
        hipLaunchKernelGGL(kern, dim3(a.M), dim3(a.M <= PF_FEW_ROWS ? 1024 : 256),
                           (size_t)a.n_heads * a.chunks * sizeof(float), s, a, t);
        return hipGetLastError();
    }
    const dim3 grid(((a.M + 63) / 64) * a.n_heads), block(256);
    switch (a.head_dim) {
    case 32:
        hipLaunchKernelGGL(k_pf_attn<32>, grid, block, 0, s, a, t);
        break;
    case 64:
        hipLaunchKernelGGL(k_pf_attn<64>, grid, block, 0, s, a, t);
        break;
    case 128:
        hipLaunchKernelGGL(k_pf_attn<128>, grid, block, 0, s, a, t);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace sdk

// For the tests: what pf_gemm_tile picks for a shape (weight rows and
// activation rows of the tile), and one product on a given tile.
extern "C" int32_t sdk_prefill_tile(int32_t M, int32_t N, int32_t K, int32_t epi, int32_t *bn, int32_t *bm,
                                    int32_t *splits) {
    if (M < 1 || M > sdk::PF_ROWS || N < 1 || K < 8)
        return -1;
    const int tile = sdk::pf_gemm_tile(M, N, K, epi, splits);
    *bn = sdk::PF_TILES[tile].bn;
    *bm = sdk::PF_TILES[tile].bm;
    return tile;
}

extern "C" int32_t sdk_prefill_gemm(int32_t tile, int32_t epi, int32_t splits, int32_t M, int32_t N, int32_t K,
                                    const uint16_t *W, const uint16_t *A, int64_t a_term, const uint16_t *zero,
                                    float *C, int64_t ldc, uint16_t *out, int64_t out_term, const float2 *table,
                                    uint16_t *kcache, uint16_t *vcache, int64_t kv_head_stride, int32_t start,
                                    int32_t n_heads, int32_t n_kv_heads, int32_t head_dim, hipStream_t s) {
    sdk::PfGemmArgs g{};
    g.W = W;
    g.A = A;
    g.a_term = a_term;
    g.zero = zero;
    g.C = C;
    g.ldc = ldc;
    g.M = M;
    g.N = N;
    g.K = K;
    g.part = C;
    g.splits = splits;
    g.out = sdk::PfTerms{out, out_term, 0};
    g.rope = sdk::PfRope{table, kcache, vcache, kv_head_stride, start, n_heads, n_kv_heads, head_dim};
    return (int32_t)sdk::launch_pf_gemm_tile(g, epi, tile, s);
}

// And the attention of M rows, its output as row-major terms.
extern "C" int32_t sdk_prefill_attention(int32_t M, int32_t start, int32_t n_heads, int32_t n_kv_heads,
                                         int32_t head_dim, const float *q, const uint16_t *kcache,
                                         const uint16_t *vcache, int64_t kv_head_stride, float *part, float2 *ml,
                                         uint16_t *out, int64_t out_term, hipStream_t s) {
    sdk::PfAttnArgs a{};
    a.q = q;
    a.ldq = a.ldo = (int64_t)n_heads * head_dim;
    a.kcache = kcache;
    a.vcache = vcache;
    a.kv_head_stride = kv_head_stride;
    a.out = part;
    a.ml = ml;
    a.M = M;
    a.start = start;
    a.n_heads = n_heads;
    a.n_kv_heads = n_kv_heads;
    a.head_dim = head_dim;
    return (int32_t)sdk::launch_pf_attention(a, sdk::PfTerms{out, out_term, 0}, s);
}

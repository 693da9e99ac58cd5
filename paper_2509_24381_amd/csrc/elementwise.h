// HBM-bound helper kernels: RMSNorm row factors and input repack, K / V append (V transposing), weight packing, cache
// export/import.
#pragma once
#include "attention.h"
#include "common.h"

// ---------------------------------------------------------------- layer input: RMSNorm row factor + fragment-major copy
// One pass over x: inv_rms[row] = rsqrt(mean(x[row]^2) + eps) (fp32 sums; the factor is applied inside the next GEMM's
// epilogue), and dst receives x in the GEMMs' token-operand layout: blocks of 32 tokens x 16 features, the two 8-feature
// halves 512 bytes apart, tokens 16 bytes apart (rows of the last block past `rows` are left untouched: they are never
// used).  The first workgroups of the grid copy the call's descriptors (requests, attention work items, cache blocks, row
// positions) from the pinned host buffer the library filled, which the device reads in place, into the workspace: the
// later kernels of the call then find them in device memory, and no copy command sits between two calls (a runtime copy
// of a few tens of KB costs a blit kernel of 13 us plus the gaps around it).
// With PLANES it is the same pass with the row taken not from x but from the split-K partial planes of the previous
// layer's down projection (the layers of one rs_prefill_model_batch call): the row is
// bf16(resid[m, :] + sum_s partial[s][m][:]), summed and rounded exactly as splitk_reduce_residual_kernel does, stored
// row-major to y (the previous layer's output, this layer's residual input) and fragment-major to dst, and its 1/rms is
// taken from the rounded values in the same order as from x - so a stack of layers run this way leaves the same bits
// as the layers called one by one, without the previous layer's reduction kernel and this layer's pass over its output.
//
// The order of a row's sum is one for all forms and sizes (K and V of a token must not depend on the call, to the bit): 16-byte chunk
// c of the row belongs to place c % 256; a place adds its chunks in ascending order, each 64 places add up in a butterfly, the four sums
// in ascending order.  LANES = 256 spreads the places over the four wavefronts of a workgroup, a row each: with few rows the kernel is a
// chain of memory latencies, and this way every load of a row is in flight at once.  LANES = 32 gives a row half a wavefront, whose lanes
// hold eight places each, and a workgroup eight rows: their 16-byte chunks of one half k-step are one cache line (with a wavefront per
// row, 64 lines touched by a store, 2048 rows of 8192 took 33 us instead of 25).
// Before, 32 lanes shared a row in 14 steps, whatever the call.  us per step between events, 7B shape in a stack (sums of 4 planes): 1 row
// 14.0 -> 7.1, 64: 19.0 -> 7.9, 250: 19.7 -> 11.1, 512: 19.2 -> 15.4, 1000: 20.9 -> 19.2, 2048: 23.2 -> 22.1 (14.7 -> 13.4 without a sum);
// 72B, 64 rows 30.9 -> 8.7, 720 rows 32.1 -> 26.6, 2048 rows without a sum 24.2 -> 23.0.
// In calls whose QKV projection stores k and v straight into the caches (EPI_QKV_APPEND), the first kernel also copies the rows' places
// there (KVRow), and zeroes what their last 64-token blocks of V^T hold behind the call's last token: `tails`, one per request, read from
// the host buffer.
struct KVTail {
    uint64_t v;            // the request's last V^T tile [d][64] of KV head 0
    uint64_t head_bytes;   // from one KV head's tile to the next one's
    int first, pad_;       // the first place behind the last token: 1..64
};
struct AppendPrep {
    uint4* dst;            // where the chunks behind the descriptors go (first the tails, then the KVRows)
    int chunks;
    int tails, hkv, d;     // requests, KV heads, features of a head; tails = 0: nothing to do
    KVTail only;           // tails = 1: that one, so that nothing waits for the host link
};
struct ReduceSource {
    const float* partial;   // [splits][rows][H] fp32
    int splits;             // 2..PLANES
    const bf16* resid;      // [rows, H] fragment-major
    bf16* y;                // [rows, H] row-major
};
// PLANES = 0 takes the rows from x; else the most planes that are summed.
constexpr int RMS_ROWS = 8;   // rows per workgroup with LANES = 32
template <int PLANES, int LANES>
__global__ __launch_bounds__(256) void rms_and_fragment_major_kernel(const bf16* __restrict__ x, bf16* __restrict__ dst,
                                                                     float* __restrict__ inv_rms, int rows, int H, float eps,
                                                                     const uint4* __restrict__ desc_src,
                                                                     uint4* __restrict__ desc_dst, int desc_chunks,
                                                                     ReduceSource red, AppendPrep app) {
    static_assert(LANES == 256 || LANES == 32, "lanes per row");
    constexpr bool REDUCE = PLANES > 0, FEW = LANES == 256;
    // (the copying workgroups come first in the grid: their reads cross the host link, several microseconds each, and
    // should be under way while the row blocks stream; launched last they were the tail of the kernel)
    const int desc_blocks = (desc_chunks + app.chunks + (int)blockDim.x - 1) / (int)blockDim.x;
    if ((int)blockIdx.x < desc_blocks) {
        const int i = (int)blockIdx.x * (int)blockDim.x + (int)threadIdx.x;
        if (i < desc_chunks) desc_dst[i] = desc_src[i];
        else if (i < desc_chunks + app.chunks) app.dst[i - desc_chunks] = desc_src[i];
        return;
    }
    const int row_blocks = FEW ? rows : (rows + RMS_ROWS - 1) / RMS_ROWS;
    if ((int)blockIdx.x >= desc_blocks + row_blocks) {   // a request's tail of one KV head
        const int z = (int)blockIdx.x - desc_blocks - row_blocks;
        const KVTail tail = app.tails == 1 ? app.only : reinterpret_cast<const KVTail*>(desc_src + desc_chunks)[z / app.hkv];
        char* const tile = reinterpret_cast<char*>(tail.v) + (size_t)(z % app.hkv) * tail.head_bytes;
        for (int i = threadIdx.x; i < app.d * 8; i += (int)blockDim.x) {   // feature i / 8, tokens 8 (i % 8) ..
            const int t0 = (i & 7) * 8;
            if (t0 >= tail.first) st_global_16(tile + (size_t)i * 16, make_uint4(0u, 0u, 0u, 0u));
            else
                for (int t = max(t0, tail.first); t < t0 + 8; ++t) *reinterpret_cast<bf16*>(tile + (size_t)(i >> 3) * 128 + t * 2) = f32_to_bf16(0.0f);
        }
        return;
    }
    const int c = (int)threadIdx.x % LANES;
    const int m = FEW ? (int)blockIdx.x - desc_blocks : ((int)blockIdx.x - desc_blocks) * RMS_ROWS + (int)threadIdx.x / LANES;
    if (m >= rows) return;   // (whole rows: nobody waits for them)
    constexpr int HELD = 256 / LANES;                        // places per lane: c + LANES h
    constexpr int U = FEW ? 2 : REDUCE ? 4 : 8;              // chunks in flight per lane
    constexpr int PASS = FEW ? 2 * 256 : 256;                // chunks per turn of the loop: U at a time
    const size_t frag_row = (size_t)(m >> 5) * (H >> 4) * 1024 + (size_t)(m & 31) * 16;   // row m in a fragment-major matrix; chunks are 512 bytes apart
    const char* src = REDUCE ? reinterpret_cast<const char*>(red.resid) + frag_row : reinterpret_cast<const char*>(x + (size_t)m * H);
    constexpr size_t SRC_STEP = REDUCE ? 512 : 16;   // bytes from one 16-byte chunk of the row to the next in the source
    char* out = reinterpret_cast<char*>(dst) + frag_row;
    float ss[HELD] = {};
    const int chunks = H >> 3;  // 16-byte chunks per row
    for (int c0 = c; c0 < chunks; c0 += PASS)
        static_for<0, PASS / LANES / U>([&](auto gc) RS_INLINE {
            constexpr int g = decltype(gc)::value;
            uint4 v[U];
            f32x4 part[REDUCE ? U : 1][REDUCE ? PLANES : 1][2];   // [chunk in flight][plane][half of the 8 features]
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int ch = c0 + (g * U + u) * LANES;
                if (ch < chunks) {
                    v[u] = ld_global_16(src + (size_t)ch * SRC_STEP);
                    if constexpr (REDUCE) {
#pragma unroll
                        for (int sp = 0; sp < PLANES; ++sp)
                            if (sp < red.splits) {
                                const float* pp = red.partial + ((size_t)sp * rows + m) * H + (size_t)ch * 8;
                                part[u][sp][0] = *reinterpret_cast<const f32x4*>(pp);
                                part[u][sp][1] = *reinterpret_cast<const f32x4*>(pp + 4);
                            }
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int ch = c0 + (g * U + u) * LANES;
                if (ch < chunks) {
                    bf16x8 h = as_bf16x8(v[u]);
                    if constexpr (REDUCE) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            float f = bf16_to_f32(h[e]);
#pragma unroll
                            for (int sp = 0; sp < PLANES; ++sp)
                                if (sp < red.splits) f += part[u][sp][e >> 2][e & 3];
                            h[e] = f32_to_bf16(f);
                        }
                        st_global_16(reinterpret_cast<char*>(red.y + (size_t)m * H) + (size_t)ch * 16, as_uint4(h));
                    }
                    float& s = ss[(g * U + u) % HELD];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float f = bf16_to_f32(h[e]);
                        s = __builtin_fmaf(f, f, s);
                    }
                    st_global_16(out + (size_t)ch * 512, as_uint4(h));
                }
            }
        });
    if constexpr (FEW) {
        __shared__ float part_sum[4];
        const float t = wave_sum(ss[0]);
        if ((threadIdx.x & 63) == 0) part_sum[threadIdx.x >> 6] = t;
        __syncthreads();
        if (threadIdx.x == 0) inv_rms[m] = rsqrtf((((part_sum[0] + part_sum[1]) + part_sum[2]) + part_sum[3]) / (float)H + eps);
    } else {
        float total = 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {   // places 64 j .. 64 j + 63: the butterfly's first step is between two places of a lane
            float t = ss[(2 * j) % HELD] + ss[(2 * j + 1) % HELD];
#pragma unroll
            for (int off = 16; off > 0; off >>= 1) t += __shfl_xor(t, off, WAVE);
            total = j == 0 ? t : total + t;
        }
        if (c == 0) inv_rms[m] = rsqrtf(total / (float)H + eps);
    }
}

// ---------------------------------------------------------------- first-token head: final RMSNorm + vocabulary projection
// h[r][k] = x[r][k] * g[k] * rsqrt(mean(x[r]^2) + eps), kept in fp32.  One wavefront per row.
__global__ __launch_bounds__(256) void final_norm_kernel(const bf16* __restrict__ x, const bf16* __restrict__ gain,
                                                         float* __restrict__ h, int rows, int H, float eps) {
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const bf16* xr = x + (size_t)row * H;
    float ss = 0.0f;
    for (int c = lane; c < H / 8; c += WAVE) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(xr + c * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) ss += bf16_to_f32(v[e]) * bf16_to_f32(v[e]);
    }
    ss = wave_sum(ss);
    const float inv = rsqrtf(ss / (float)H + eps);
    for (int c = lane; c < H / 8; c += WAVE) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(xr + c * 8);
        const bf16x8 g = *reinterpret_cast<const bf16x8*>(gain + c * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) h[(size_t)row * H + c * 8 + e] = bf16_to_f32(v[e]) * inv * bf16_to_f32(g[e]);
    }
}

// logits[r][v] = sum_k h[r][k] * w[v][k] for R <= LM_ROWS rows at a time.  HBM-bound on the vocabulary matrix (read once):
// the normalised rows sit in LDS (fp32); each wavefront walks the vocabulary four rows at a time, its 64 lanes covering
// K in contiguous 16-byte chunks (1 KB per load instruction and row), so that one LDS read of the activations serves
// four weight rows; lanes are reduced at the end of the group.
constexpr int LM_ROWS = 4;
constexpr int LM_VGROUP = 4;
// ONCE: the vocabulary is beyond the 256 MB Infinity Cache (LM_STREAM_BYTES) and loaded with the streaming hint, with which HBM streams
// faster: 152064 x 3584, 1 row 189 -> 171 us, 8 rows (the kernel below) 210 -> 186; 152064 x 8192, 1 row 450 -> 418.  A smaller one can
// still be there from the head before, and the hint then loses: 32000 x 3584, 3 rows 42.0 -> 43.9.  Head after head, the line lies at 270
// to 290 MB (152064 x 896, 272 MB, 8 rows 52 -> 54; 100000 x 1536, 307 MB, 1.05x to 1.13x faster); behind a
// fill of 1 GB every size from 57 MB on gains, 1.1x to 2x.
constexpr size_t LM_STREAM_BYTES = (size_t)256 << 20;
constexpr int LM_ONCE = 2;   // cache policy (nt)
template <bool ONCE>
__global__ __launch_bounds__(256) void lm_head_kernel(const bf16* __restrict__ w, const float* __restrict__ h,
                                                      float* __restrict__ logits, int R, int vocab, int H) {
    extern __shared__ __attribute__((aligned(16))) float h_lds[];  // [R][H]
    for (int i = threadIdx.x; i < R * H / 4; i += blockDim.x)
        reinterpret_cast<f32x4*>(h_lds)[i] = reinterpret_cast<const f32x4*>(h)[i];
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    for (int v0 = (blockIdx.x * 4 + wave) * LM_VGROUP; v0 < vocab; v0 += gridDim.x * 4 * LM_VGROUP) {
        const bf16* wr[LM_VGROUP];
#pragma unroll
        for (int j = 0; j < LM_VGROUP; ++j) wr[j] = w + (size_t)min(v0 + j, vocab - 1) * H;  // rows past the end repeat the last one
        float acc[LM_VGROUP][LM_ROWS];
#pragma unroll
        for (int j = 0; j < LM_VGROUP; ++j)
#pragma unroll
            for (int r = 0; r < LM_ROWS; ++r) acc[j][r] = 0.0f;
        for (int c = lane; c < H / 8; c += WAVE) {
            bf16x8 wv[LM_VGROUP];
#pragma unroll
            for (int j = 0; j < LM_VGROUP; ++j) {
                const bf16x8* const p = reinterpret_cast<const bf16x8*>(wr[j] + c * 8);
                wv[j] = ONCE ? __builtin_nontemporal_load(p) : *p;
            }
#pragma unroll
            for (int r = 0; r < LM_ROWS; ++r)
                if (r < R) {
                    const f32x4 h0 = *reinterpret_cast<const f32x4*>(h_lds + (size_t)r * H + c * 8);
                    const f32x4 h1 = *reinterpret_cast<const f32x4*>(h_lds + (size_t)r * H + c * 8 + 4);
#pragma unroll
                    for (int j = 0; j < LM_VGROUP; ++j)
                        acc[j][r] += bf16_to_f32(wv[j][0]) * h0[0] + bf16_to_f32(wv[j][1]) * h0[1] + bf16_to_f32(wv[j][2]) * h0[2] +
                                     bf16_to_f32(wv[j][3]) * h0[3] + bf16_to_f32(wv[j][4]) * h1[0] + bf16_to_f32(wv[j][5]) * h1[1] +
                                     bf16_to_f32(wv[j][6]) * h1[2] + bf16_to_f32(wv[j][7]) * h1[3];
                }
        }
#pragma unroll
        for (int j = 0; j < LM_VGROUP; ++j)
#pragma unroll
            for (int r = 0; r < LM_ROWS; ++r)
                if (r < R) {
                    const float t = wave_sum(acc[j][r]);
                    if (lane == 0 && v0 + j < vocab) logits[(size_t)r * vocab + v0 + j] = t;
                }
    }
}

// The same for 3 rows and more, on the matrix pipe.  A value of the normalised row is the product of u = x / rms
// (fp32) and the gain; it is cut into three bfloat16 pieces, hi = bf16(u g), mid = bf16(u g - hi), lo = bf16(u g - hi - mid),
// whose sum is within 2^-26 of it (fp32: 2^-24; below 2^-110 lo runs out of exponents); products of a piece with a bfloat16
// weight are exact in fp32.  The pieces of up to 10 rows are the columns of ONE 32-column B
// operand (column 10 s + r = piece s of row r), so the kernel streams the vocabulary once per 10 NG rows and spends one
// 32x32x16 MFMA per 32 vocabulary rows, 16 k and 10 rows, far below the stream's time.
//   operand layout: [group of 10 rows][k-step of 16][half][column 32][8 bfloat16]: a wavefront's load is one contiguous KB.
// One workgroup per compute unit owns an even share of the vocabulary and walks it 64 rows at a time; each of its 4
// wavefronts takes a quarter of K and streams its part of the rows global -> LDS by DMA (a row's 128 bytes are then 8
// neighbouring lanes: whole cache lines; loaded straight into the MFMA layout, where neighbouring lanes are different rows,
// the stream reached 3.5 TB/s) through a ring of its own, three steps of 8 KB ahead and on across the tiles, without a
// barrier; they meet in LDS at the end of a tile.  The accumulators are emptied after every 64 k, and those sums after every
// 256: short chains keep the error against 64 bits below that of the fp32 kernel above (3584: 1.0e-7 against 1.2e-7;
// 8192: 1.2e-7 against 1.4e-7).
// Measured on 152064 x 3584, us (LDS kernel, which streams the vocabulary once per 4 rows -> this one; without the streaming hint on both
// sides): 1 row 189 -> 206, 2: 205 -> 206, 3: 271 -> 209, 8: 584 -> 207, 10: 805 -> 217, 11: 860 -> 250 (a second group's operand comes
// from L2 beside the stream); now 3 rows 182, 8: 186 (5.9 TB/s), 11: 230, 22: 415, and 1 and 2 rows in the LDS kernel 170 and 177.
constexpr int LM_MFMA_ROWS = 3;   // from this many rows on
constexpr int LM_GROUP = 10;      // rows per B operand
constexpr int LM_MAX_GROUPS = 2;  // B operands per launch (three spill: 525 us for 30 rows, two passes take 470)
constexpr int LM_VROWS = 64;      // vocabulary rows per workgroup
__global__ __launch_bounds__(256) void final_norm_split_kernel(const bf16* __restrict__ x, const bf16* __restrict__ gain,
                                                               bf16* __restrict__ hb, int rows, int H, float eps) {
    // one workgroup per place of a group of rows (grid x: LM_GROUP, + 1 for the two columns that hold no row; grid y: groups)
    const int rg = blockIdx.x;
    const int row = blockIdx.y * LM_GROUP + rg;
    const size_t base = (size_t)blockIdx.y * (size_t)(H / 16) * 512;   // elements
    const auto place = [&](int col, int c) {   // chunk c (8 features) of a column: k-step c / 2, half c % 2
        return hb + base + (size_t)(c >> 1) * 512 + (size_t)(c & 1) * 256 + (size_t)col * 8;
    };
    const bf16x8 zero = {};
    if (rg == LM_GROUP || row >= rows) {
        for (int c = threadIdx.x; c < H / 8; c += blockDim.x) {
            if (rg == LM_GROUP) {
                for (int col = 3 * LM_GROUP; col < 32; ++col) *reinterpret_cast<bf16x8*>(place(col, c)) = zero;
            } else {
                for (int s = 0; s < 3; ++s) *reinterpret_cast<bf16x8*>(place(s * LM_GROUP + rg, c)) = zero;
            }
        }
        return;
    }
    // (every wavefront sums the whole row in the order of final_norm_kernel: the same factor, no exchange)
    const int lane = threadIdx.x & 63;
    const bf16* xr = x + (size_t)row * H;
    float ss = 0.0f;
    for (int c = lane; c < H / 8; c += WAVE) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(xr + c * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) ss += bf16_to_f32(v[e]) * bf16_to_f32(v[e]);
    }
    ss = wave_sum(ss);
    const float inv = rsqrtf(ss / (float)H + eps);
    for (int c = threadIdx.x; c < H / 8; c += blockDim.x) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(xr + c * 8);
        const bf16x8 g = *reinterpret_cast<const bf16x8*>(gain + c * 8);
        bf16x8 hi, mid, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            constexpr float BF16_MAX = 3.38953139e38f;
            const float u = bf16_to_f32(v[e]) * inv, gain_e = bf16_to_f32(g[e]), h = u * gain_e;
            // (the largest finite values would round to an infinite bfloat16)
            hi[e] = f32_to_bf16(fabsf(h) <= 3.402823466e38f ? fminf(fmaxf(h, -BF16_MAX), BF16_MAX) : h);
            const float r1 = __builtin_fmaf(u, gain_e, -bf16_to_f32(hi[e]));   // (of the product, not of its fp32 rounding)
            mid[e] = f32_to_bf16(r1);
            lo[e] = f32_to_bf16(r1 - bf16_to_f32(mid[e]));
        }
        *reinterpret_cast<bf16x8*>(place(rg, c)) = hi;
        *reinterpret_cast<bf16x8*>(place(LM_GROUP + rg, c)) = mid;
        *reinterpret_cast<bf16x8*>(place(2 * LM_GROUP + rg, c)) = lo;
    }
}

constexpr int LM_SLOTS = 4;
template <int NG, bool ONCE>
__global__ __launch_bounds__(256, 1) void lm_head_mfma_kernel(const bf16* __restrict__ w, const bf16* __restrict__ hb,
                                                              float* __restrict__ logits, int R, int vocab, int H) {
    constexpr int PAD = 33;   // a column's 32 sums, padded: neighbouring columns start in different banks
    constexpr int SLOT = LM_VROWS * 128;   // one wavefront's step: 64 rows x 64 k
    static_assert(3 * (8 + 4 * NG) <= 63, "the wait for a step must fit the vmcnt field");
    typedef __attribute__((address_space(3))) void* lds_ptr;
    // (separate objects, so that the compiler can tell the slot being read from those being filled)
    __shared__ __attribute__((aligned(16))) char ring0[4 * SLOT];
    __shared__ __attribute__((aligned(16))) char ring1[4 * SLOT];
    __shared__ __attribute__((aligned(16))) char ring2[4 * SLOT];
    __shared__ __attribute__((aligned(16))) char ring3[4 * SLOT];
    __shared__ float red[4][32 * PAD];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    // this workgroup's vocabulary rows [row0, row0 + n_rows)
    const int share = vocab / gridDim.x, extra = vocab % gridDim.x;
    const int row0 = (int)blockIdx.x * share + min((int)blockIdx.x, extra);
    const int n_rows = share + ((int)blockIdx.x < extra ? 1 : 0);
    const int tiles = (n_rows + LM_VROWS - 1) / LM_VROWS;
    // this wavefront's groups of 64 k
    const int nk = H >> 6, kg0 = wave * nk / 4, ns = (wave + 1) * nk / 4 - kg0;
    const int ns4 = (ns + LM_SLOTS - 1) / LM_SLOTS * LM_SLOTS;   // steps per tile, whole rounds of the ring
    // (rows past the share, and steps past the last one, fall outside the buffer: they read as zeros and move no data)
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc((void*)(w + (size_t)row0 * H), 0, (int)((uint32_t)n_rows * (uint32_t)H * 2u), 0x00020000);
    const uint32_t group_bytes = (uint32_t)(H >> 4) * 1024u;
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void*)hb, 0, (int)(NG * group_bytes), 0x00020000);
    constexpr uint32_t DEAD = 0x80000000u;
    // load instruction i fills rows [8 i, 8 i + 8) of the slot; 16-byte chunk c of row r sits at place c ^ ((r >> 1) & 7)
    const uint32_t row_bytes = (uint32_t)H * 2u;
    uint32_t src[2];   // rows 8 i + lane / 8 for even and odd i: the swizzle repeats every 16 rows
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        const uint32_t r = (uint32_t)(o * 8 + (lane >> 3));
        src[o] = r * row_bytes + (((uint32_t)(lane & 7) ^ ((r >> 1) & 7u)) * 16u);
    }
    const uint32_t frag0 = (uint32_t)l32 * 128u;
    const uint32_t swz = (uint32_t)(l32 >> 1) & 7u;
    int l_tile = 0, l_s = 0;   // the step the load stream is at
    bf16x8 b[LM_SLOTS][NG][4];
    const auto load_step = [&](auto slotc, char* ring) RS_INLINE {
        constexpr int slot = decltype(slotc)::value;
        const bool live = l_tile < tiles && l_s < ns;
        const int kg = kg0 + (l_s < ns ? l_s : 0);
        // (steps past the last one read zeros here too: an infinite value times a zero weight would be NaN)
        const uint32_t boff = l_s < ns ? (uint32_t)lane * 16u + (uint32_t)kg * 4096u : DEAD;
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                b[slot][g][j] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rb, boff + (uint32_t)j * 1024u, (int)((uint32_t)g * group_bytes), 0));
        const uint32_t off = live ? (uint32_t)(l_tile * LM_VROWS) * row_bytes + (uint32_t)kg * 128u : DEAD;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr)(uintptr_t)(uint32_t)(uintptr_t)(ring + wave * SLOT + i * 1024), 16,
                                                     src[i & 1] + off + (uint32_t)(i >> 1) * 16u * row_bytes, 0, 0, ONCE ? LM_ONCE : 0);
        if (++l_s == ns4) {
            l_s = 0;
            ++l_tile;
        }
    };
    f32x16 round[NG][2], sum[NG][2];   // sums over the steps of one round of the ring, and over the rounds
    const auto each = [&](auto&& f) RS_INLINE {
        static_for<0, NG>([&](auto gc) RS_INLINE {
            static_for<0, 2>([&](auto tc) RS_INLINE {
                static_for<0, 16>([&](auto rc) RS_INLINE { f(gc, tc, rc); });
            });
        });
    };
    const auto multiply = [&](auto slotc, const char* ring) RS_INLINE {
        constexpr int slot = decltype(slotc)::value;
        f32x16 acc[NG][2];
        bf16x8 a[2][4];
        // loads retire in order: this step's have landed when at most those of the three steps behind it are in flight (the
        // compiler does not see LDS written by DMA; nor may it move the refill of a slot above the reads of it)
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * (8 + 4 * NG)) : "memory");
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                a[t][j] = *reinterpret_cast<const bf16x8*>(ring + wave * SLOT + t * 4096 + frag0 + (((uint32_t)(j * 2 + half) ^ swz) * 16u));
        const f32x16 zero = {};
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int g = 0; g < NG; ++g)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[g][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t][j], b[slot][g][j], j == 0 ? zero : acc[g][t], 0, 0, 0);
        each([&](auto gc, auto tc, auto rc) RS_INLINE {
            constexpr int g = decltype(gc)::value, t = decltype(tc)::value, r = decltype(rc)::value;
            round[g][t][r] = slot == 0 ? acc[g][t][r] : round[g][t][r] + acc[g][t][r];
        });
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
    };
    if (ns > 0) {
        load_step(std::integral_constant<int, 0>{}, ring0);
        load_step(std::integral_constant<int, 1>{}, ring1);
        load_step(std::integral_constant<int, 2>{}, ring2);
    }
    for (int tile = 0; tile < tiles; ++tile) {
        each([&](auto gc, auto tc, auto rc) RS_INLINE { sum[decltype(gc)::value][decltype(tc)::value][decltype(rc)::value] = 0.0f; });
        for (int s = 0; s < ns4; s += LM_SLOTS) {
            // (a slot is refilled behind the step that read it: its fragments are in registers by then)
            load_step(std::integral_constant<int, 3>{}, ring3);
            multiply(std::integral_constant<int, 0>{}, ring0);
            load_step(std::integral_constant<int, 0>{}, ring0);
            multiply(std::integral_constant<int, 1>{}, ring1);
            load_step(std::integral_constant<int, 1>{}, ring1);
            multiply(std::integral_constant<int, 2>{}, ring2);
            load_step(std::integral_constant<int, 2>{}, ring2);
            multiply(std::integral_constant<int, 3>{}, ring3);
            each([&](auto gc, auto tc, auto rc) RS_INLINE {
                constexpr int g = decltype(gc)::value, t = decltype(tc)::value, r = decltype(rc)::value;
                sum[g][t][r] += round[g][t][r];
            });
        }
        // the four quarters of K, and the three pieces of every row, meet: 32 vocabulary rows and one group at a time
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // (the last reader of red is done; the DMA stays in flight)
#pragma unroll
                for (int r = 0; r < 16; ++r) red[wave][l32 * PAD + 8 * (r >> 2) + 4 * half + (r & 3)] = sum[g][t][r];
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                const int rows = min(R - g * LM_GROUP, LM_GROUP);
                for (int i = threadIdx.x; i < rows * 32; i += 256) {
                    const int r = i >> 5, v = tile * LM_VROWS + t * 32 + (i & 31);   // v: inside the share
                    float piece[3];
#pragma unroll
                    for (int s = 0; s < 3; ++s) {
                        const int at = (s * LM_GROUP + r) * PAD + (i & 31);
                        piece[s] = (red[0][at] + red[1][at]) + (red[2][at] + red[3][at]);
                    }
                    if (v < n_rows) {
                        // An infinite or NaN weight or value makes the sum of the first pieces infinite or NaN as it makes the
                        // row's own (they carry the values' signs, and a value of the row is zero where they are); of the other
                        // two it makes anything (0 * inf, inf - inf), so then they do not count
                        const float out = fabsf(piece[0]) <= 3.402823466e38f ? piece[0] + (piece[1] + piece[2]) : piece[0];
                        logits[(size_t)(g * LM_GROUP + r) * vocab + row0 + v] = out;
                    }
                }
            }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the stream's last (empty) loads still target this workgroup's LDS
}

// ---------------------------------------------------------------- K / V append
struct KVBlockItem {
    int req;
    int block;  // absolute 64-token block index in the request's cache
};

// One workgroup per (touched 64-token block, KV head).  The rotated k rows are copied from the qkv buffer to the
// request's K cache (256-byte rows, 16-byte vector copies).  The v rows are transposed through LDS and written as
// [d][64] with the token index innermost, 16 bytes (8 tokens) per store.  Tokens before P keep their content; V
// positions at or beyond P+T inside the block are zero-filled.
template <int D>
__global__ __launch_bounds__(256) void append_kv_kernel(const bf16* __restrict__ qkv, int ld_qkv,
                                                        const ReqDesc* __restrict__ reqs,
                                                        const KVBlockItem* __restrict__ blocks, int Hq, int Hkv) {
    __shared__ __attribute__((aligned(16))) bf16 tile[64][D + 8];  // row stride D*2 + 16 bytes: 16-byte aligned, odd in 16-byte units
    const KVBlockItem it = blocks[blockIdx.x];
    const ReqDesc rq = reqs[it.req];
    const int c = blockIdx.y;
    const int tok0 = it.block * 64;
    const int k_col = (Hq + c) * D;
    const int v_col = (Hq + Hkv + c) * D;
    constexpr int CPR = D / 8;  // 16-byte chunks per row
    const KVHeadTiles tiles = kv_head_tiles<D>(rq, c);
    const int tile_index = tiles.index_of(it.block);
    bf16* const k_tile = reinterpret_cast<bf16*>(tiles.k_tile(tile_index));
    for (int idx = threadIdx.x; idx < 64 * CPR; idx += blockDim.x) {
        const int kk = idx / CPR, ch = idx - kk * CPR;
        const int pos = tok0 + kk;
        const bool live = pos >= rq.P && pos < rq.P + rq.T;
        uint4 k = make_uint4(0u, 0u, 0u, 0u), v = make_uint4(0u, 0u, 0u, 0u);
        if (live) {
            const bf16* row = qkv + (size_t)(rq.row0 + pos - rq.P) * ld_qkv + ch * 8;
            k = ld_global_16(row + k_col);
            v = ld_global_16(row + v_col);
            st_global_16(k_tile + (size_t)kk * D + ch * 8, k);
        }
        *reinterpret_cast<uint4*>(&tile[kk][ch * 8]) = v;  // zeros for positions outside [P, P+T)
    }
    __syncthreads();
    bf16* dst = reinterpret_cast<bf16*>(tiles.v_tile(tile_index));
    // thread -> (feature dd, group of 8 tokens): gathers the 8 tokens' values of feature dd and stores them as one chunk
    for (int idx = threadIdx.x; idx < D * 8; idx += blockDim.x) {
        const int dd = idx >> 3, g8 = idx & 7;
        const int t0 = g8 * 8;
        if (tok0 + t0 + 7 < rq.P) continue;  // all 8 tokens are older than this call: keep them
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = tile[t0 + e][dd];
        if (tok0 + t0 >= rq.P) {
            *reinterpret_cast<bf16x8*>(dst + dd * 64 + t0) = o;
        } else {  // the group straddles P: element-wise, older tokens untouched
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (tok0 + t0 + e >= rq.P) dst[dd * 64 + t0 + e] = o[e];
        }
    }
}

// ---------------------------------------------------------------- weight packing (one-time)
// packed[prow][k] = bf16(src[srow][k] * gain[k]), stored fragment-major (units of 32 rows, see frag_offset_bytes in
// gemm_strip.h): the RMSNorm gain is folded into the weight columns of the GEMM that follows the norm (gain null: copied
// as they are), and rows are reordered so that what an epilogue combines sits in one 32-row unit (one MFMA tile), in rows
// t and t + 16, which one lane holds:
//   PACK_GATE_UP (p0 = I):  unit u = 16 gate rows 16u..16u+15, then the up rows I + 16u..
//   PACK_QKV_ROPE (p0 = head_dim, p1 = number of q and k rows): unit u of a head = features 16u..16u+15 of the head's
//                 first half, then their rotate-half partners head_dim/2 + 16u..; v rows keep their order
// Bound by HBM.  One workgroup per unit and PACK_K features, neighbours along the features: 512 contiguous bytes of each of the 32
// source rows are read by 32 neighbouring lanes, all loads of a thread in flight together, and turned through LDS into the unit's
// chunks, of which a wavefront stores a contiguous kilobyte, past the caches.  7B layer (466 MB each way) 167 us, 5.6 TB/s; with the
// units as neighbours 193, with ordinary stores 176, with a lane per row (32 bytes of it at a time, no LDS) 207.
// `wide`: the source can be read 16 bytes at a time.
constexpr int PACK_K = 256;
enum PackMode { PACK_IDENTITY = 0, PACK_GATE_UP = 1, PACK_QKV_ROPE = 2 };
__global__ __launch_bounds__(256) void pack_rows_kernel(const bf16* __restrict__ src, const bf16* __restrict__ gain,
                                                        bf16* __restrict__ dst, int K, int mode, int p0, int p1, int wide) {
    constexpr int CH = PACK_K / 8;   // 16-byte chunks of a row
    __shared__ uint4 tile[32][CH + 1];   // (rows one chunk further: 16 rows' reads of one chunk cover all banks)
    const int slices = (K + PACK_K - 1) / PACK_K;
    const int u = (int)blockIdx.x / slices, c0 = ((int)blockIdx.x % slices) * CH;
    const int c = threadIdx.x % CH, r0 = threadIdx.x / CH;
    const bool live = c0 + c < K / 8;
    constexpr int N = 32 * CH / 256;   // rows r0, r0 + 256 / CH, ...
    uint4 in[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int t = r0 + i * (256 / CH);
        const int prow = u * 32 + t;
        int srow = prow;
        if (mode == PACK_GATE_UP) {
            srow = (t < 16) ? (u * 16 + t) : (p0 + u * 16 + (t - 16));
        } else if (mode == PACK_QKV_ROPE && prow < p1) {
            const int head = prow / p0, uh = (prow % p0) >> 5;
            srow = head * p0 + ((t < 16) ? (uh * 16 + t) : (p0 / 2 + uh * 16 + (t - 16)));
        }
        if (live) in[i] = load8(src + (size_t)srow * K + (c0 + c) * 8, wide != 0);
    }
    if (live) {
        bf16x8 g = {};
        if (gain != nullptr) g = *reinterpret_cast<const bf16x8*>(gain + (c0 + c) * 8);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            uint4 v = in[i];
            if (gain != nullptr) {
                const bf16x8 h = as_bf16x8(v);
                bf16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = f32_to_bf16(bf16_to_f32(h[e]) * bf16_to_f32(g[e]));
                v = as_uint4(o);
            }
            tile[r0 + i * (256 / CH)][c] = v;
        }
    }
    __syncthreads();
    const int t = threadIdx.x & 31;
    bf16* d = dst + (size_t)u * 32 * K + t * 8;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int co = (int)(threadIdx.x >> 5) + i * 8;
        if (c0 + co < K / 8) st_global_16_stream(d + (size_t)(c0 + co) * 256, tile[t][co]);
    }
}

// ---------------------------------------------------------------- tiles of a cache in export / import (kv_transfer.h)
// The cache is described like a request (ReqDesc: contiguous planes, or the pool base for a paged cache).  The page
// numbers of a paged cache travel in the kernel arguments, a window of KV_PAGE_WINDOW blocks per launch starting at
// block `block0`; tokens [t0, t0 + n) are handled, t0 a multiple of 64 inside the window.
constexpr int KV_PAGE_WINDOW = 256;
struct KVPageWindow {
    int page[KV_PAGE_WINDOW];
};

template <int D>
RS_DEVICE bf16* kv_window_tile(const ReqDesc& rq, const KVPageWindow& win, int block0, bool v, int c, int block) {
    constexpr size_t TILE = (size_t)64 * D;  // elements
    if (rq.pages == nullptr)   // (any non-null value marks a paged cache here; the numbers come from the window)
        return (v ? rq.vtcache : rq.kcache) + ((size_t)c * (size_t)(rq.cap >> 6) + (size_t)block) * TILE;
    return rq.kcache + ((size_t)win.page[block - block0] * 2 * rq.hkv + (size_t)(v ? rq.hkv : 0) + (size_t)c) * TILE;
}

// bf16 MFMA GEMM for calls of few rows (at most 32 TB TW tokens):  out[M,N] = epilogue( X[M,K] * W[N,K]^T ), the same operand
// layouts, epilogues and, along K, the same order of accumulation as gemm_strip.h.
//
// With so few rows the weights' stream is all there is (64 rows: 64 flop per weight byte, a twentieth of what the matrix pipe
// needs), and what bounds it is bytes in flight: the strip kernel's ring holds 28 KB per compute unit and its loop costs 480
// clocks per step of 64 k with every load removed, against 128 to 256 of MFMA.  Here nothing is shared and nothing waits for
// another wavefront: both operands are stored in the MFMA's register order, so a wavefront loads each fragment as one
// contiguous kilobyte straight into the registers the MFMA reads, DEPTH k-steps ahead.  One workgroup owns one unit of 32
// weight rows.
//   KW > 1: its wavefronts split K between them and add up through LDS at the end, so that a residual projection needs no
//           partial planes in memory and no second kernel unless its K is long (then the grid's y cuts it, see gemm_residual).
//   KW = 1: TW wavefronts take 32 tokens each and walk the whole K: the QKV projection, whose K may not be split (the bits of
//           K and V must not depend on the call), and the gate/up projection of narrow layers.
// (Reading a word of every line of the unit's weights ahead of time, from one more wavefront, made it slower: QKV at 20 rows
// 14.4 -> 16.9 us.)
// Measured, us per step between events (3 to 4 us of them the events'), strip kernel (with its reduction) -> this one:
//   7B, 1 row:   QKV 22.0 -> 14.2, O 18.8 -> 14.8, down 36.4 -> 35.6;  64 rows: QKV 22.1 -> 18.7
//   tiny, 40 rows: QKV 9.9 -> 7.2, O 9.1 -> 7.5, down 11.7 -> 8.7
#pragma once
#include "common.h"
#include "gemm_strip.h"

template <int EPI, int TB, int TW, int KW, int DEPTH>
__global__ __launch_bounds__(64 * TW * KW, (TW * KW + 3) / 4) void gemm_skinny_kernel(GemmArgs a) {
    static_assert(KW == 1 ? TB == 1 : (TW == 1 && KW >= TB), "wavefronts split K or the tokens");
    static_assert(DEPTH * (1 + TB) <= 60, "the loads in flight must fit the vmcnt field");
    extern __shared__ __attribute__((aligned(16))) float skinny_red[];   // KW > 1: [KW][TB][16][64]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int unit = blockIdx.x, split = blockIdx.y;
    const uint32_t unit_bytes = 32u * (uint32_t)a.K * 2u;
    const int kk0 = split * a.steps_per_split * 4, kk_end = min(kk0 + a.steps_per_split * 4, a.K >> 4);   // k-steps of 16
    const int tw = wave % TW, kw = wave / TW;
    const int n_kk = kk_end - kk0;
    const int kb = kk0 + n_kk * kw / KW, ke = kk0 + n_kk * (kw + 1) / KW;
    const uint32_t x_block_bytes = (uint32_t)(a.K >> 4) * 1024u;
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc((void*)a.X, 0, ((a.M + 31) >> 5) * (int)x_block_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc((void*)(reinterpret_cast<const char*>(a.W) + (size_t)unit * unit_bytes), 0, (int)unit_bytes, 0x00020000);
    const uint32_t vl = (uint32_t)lane * 16u;
    uint32_t xv[TB];   // token blocks past the end of the call fall outside the buffer and read as zeros
#pragma unroll
    for (int j = 0; j < TB; ++j) xv[j] = (uint32_t)(tw * TB + j) * x_block_bytes + vl;
    bf16x8 wf[DEPTH], xf[DEPTH][TB];
    const auto load = [&](auto uc, int kk) RS_INLINE {   // (past the range: the last k-step again, never used)
        constexpr int u = decltype(uc)::value;
        const uint32_t so = (uint32_t)min(kk, ke - 1) * 1024u;
        wf[u] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rw, vl, so, 0));
        static_for<0, TB>([&](auto jc) RS_INLINE {
            constexpr int j = decltype(jc)::value;
            xf[u][j] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rx, xv[j], so, 0));
        });
    };
    f32x16 acc[1][TB];
#pragma unroll
    for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][j][r] = 0.0f;
    const auto multiply = [&](auto uc) RS_INLINE {
        constexpr int u = decltype(uc)::value;
        static_for<0, TB>([&](auto jc) RS_INLINE {
            constexpr int j = decltype(jc)::value;
            acc[0][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[u], xf[u][j], acc[0][j], 0, 0, 0);
        });
    };
    float row_val[1] = {0.0f};
    if constexpr (EPI == EPI_SWIGLU) {   // (behind nothing here: few rows and parts)
        const int mj[1] = {min(tw * 32 + l32, a.M - 1)};
        load_row_factors<1>(a, mj, half, row_val);
        close_row_factors<1>(a, row_val);
    }
    if (ke > kb) {
        static_for<0, DEPTH>([&](auto uc) RS_INLINE { load(uc, kb + decltype(uc)::value); });
        int kk = kb;
        for (; kk + DEPTH <= ke; kk += DEPTH)
            static_for<0, DEPTH>([&](auto uc) RS_INLINE {
                multiply(uc);
                __builtin_amdgcn_sched_barrier(0);
                load(uc, kk + DEPTH + decltype(uc)::value);
                __builtin_amdgcn_sched_barrier(0);
            });
        static_for<0, DEPTH>([&](auto uc) RS_INLINE {
            if (kk + decltype(uc)::value < ke) multiply(uc);
        });
    }
    if constexpr (KW == 1) {
        gemm_epilogue<EPI, 1, 1>(a, acc, tw * 32, unit, half, l32, split, row_val);
    } else {
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) skinny_red[(size_t)((wave * TB + j) * 16 + r) * 64 + lane] = acc[0][j][r];
        __syncthreads();
        if (wave >= TB) return;
        f32x16 sum[1][1];   // wavefront j closes token block j: the parts in ascending order of K
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float v = 0.0f;
#pragma unroll
            for (int k = 0; k < KW; ++k) v += skinny_red[(size_t)((k * TB + wave) * 16 + r) * 64 + lane];
            sum[0][0][r] = v;
        }
        gemm_epilogue<EPI, 1, 1>(a, sum, wave * 32, unit, half, l32, split, row_val);
        if constexpr (EPI == EPI_RESIDUAL) {
            if (a.rowss != nullptr) {   // (as in gemm_strip_kernel: one part per unit here)
                const float ss = row_val[0] + __shfl_xor(row_val[0], 32, WAVE);
                const int m = wave * 32 + l32;
                if (half == 0 && m < a.M) a.rowss[(size_t)unit * a.M + m] = ss;
            }
        }
    }
}

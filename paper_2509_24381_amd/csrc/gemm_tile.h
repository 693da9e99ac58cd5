// bf16 MFMA GEMM for calls of some dozens to about a thousand rows:  out[M,N] = epilogue( X[M,K] * W[N,K]^T ), the operand layouts,
// the epilogues and, along K, the order of accumulation of gemm_strip.h (the same bits, whichever runs).
//
// What bounds these calls is what a compute unit can fetch.  All workgroups walk K in step, so every line a workgroup asks for is
// still on its way from memory for all of them, and a compute unit sustains 50 to 60 bytes per ns however many loads it keeps in
// flight beyond 32 KB and whichever way they go (LDS or registers, with the MFMAs or without, measured on 36 to 224 compute units;
// L2-resident lines 126).  A projection's time is then the bytes of ONE workgroup, K (rows + features) 2, over that rate, plus 4 to
// 5 us, and the shape of the tile is what matters: a block of 256 rows by one or two units of 32 features (what strips of a short
// call are) moves two to three times the bytes that a squarer tile of the same area does.  Hence tiles of 64 or 128 rows by 2 to 5
// units, chosen per call from that sum (tile_ns in rserve_prefill.hip).  Both operands go global -> LDS by DMA, each byte once per
// workgroup, through a ring of SLOTS steps of 64 k; a wavefront reads the fragments of a whole step into registers while it multiplies
// those of the step before, so that neither the LDS latency nor the one barrier of a step shows.
// Measured beside the strips they replace, us per step between events (7B shape in a stack, weights from HBM): QKV 250 rows 33.9 -> 31.0,
// 512 rows 45.1 -> 34.9, 1000 rows 51.4 -> 47.4; O 64 rows 20.3 -> 15.7, 250 rows 27.8 -> 21.7, 512 rows 34.5 -> 29.6; down 64 rows 37.4 ->
// 32.5, 250 rows 62.5 -> 56.7.
#pragma once
#include "common.h"
#include "gemm_strip.h"

// Tiles of BMB token blocks by BU units: 4 wavefronts, WM along the tokens, each TM token blocks by TN units.
template <int BMB, int BU> struct TileShape;
template <> struct TileShape<2, 2> { static constexpr int WM = 2, TM = 1, TN = 1, SLOTS = 6; };
template <> struct TileShape<2, 4> { static constexpr int WM = 2, TM = 1, TN = 2, SLOTS = 5; };
template <> struct TileShape<4, 2> { static constexpr int WM = 4, TM = 1, TN = 2, SLOTS = 5; };
template <> struct TileShape<4, 3> { static constexpr int WM = 4, TM = 1, TN = 3, SLOTS = 5; };
template <> struct TileShape<4, 4> { static constexpr int WM = 2, TM = 2, TN = 2, SLOTS = 4; };
template <> struct TileShape<4, 5> { static constexpr int WM = 4, TM = 1, TN = 5, SLOTS = 4; };
template <int BMB, int BU> constexpr int tile_lds_bytes() { return TileShape<BMB, BU>::SLOTS * (BMB + BU) * 4096; }

// ONCE: the call has one block of rows, every weight is read by one workgroup: the loads say so (nt), and HBM streams faster.
template <int EPI, int BMB, int BU, bool ONCE>
__global__ __launch_bounds__(256, 1) void gemm_tile_kernel(GemmArgs a) {
    using S = TileShape<BMB, BU>;
    constexpr int WM = S::WM, WN = 4 / WM, TM = S::TM, TN = S::TN, SLOTS = S::SLOTS;
    static_assert(WM * TM == BMB && WN * TN == BU, "the wavefronts cover the tile");
    constexpr int L = BMB + BU;                    // DMA instructions per wavefront and step of 64 k: its k-step of every block
    constexpr uint32_t SLOT_BYTES = L * 4096u;
    static_assert(SLOTS * L <= 63, "the loads in flight must fit the vmcnt field");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    typedef __attribute__((address_space(3))) void* lds_ptr;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int wm = wave % WM, wn = wave / WM;

    // ---- which tile: workgroup ids go round-robin over the 8 XCDs; each XCD owns a contiguous range of tiles, the row blocks of one
    //      range of weights first, then the ranges of weights, then the K ranges
    const int nwg = gridDim.x, pid = blockIdx.x;
    const int xcd = pid & 7, loc = pid >> 3;
    const int wbase = nwg >> 3, wrem = nwg & 7;
    const int logical = (xcd < wrem ? xcd * (wbase + 1) : wrem * (wbase + 1) + (xcd - wrem) * wbase) + loc;
    const int tm = logical % a.tiles_m;
    const int strip = (logical / a.tiles_m) % a.strips;
    const int split = logical / (a.tiles_m * a.strips);
    const int m0 = tm * BMB * 32, u0 = strip * BU;
    const int st0 = split * a.steps_per_split;
    const int ns = min(a.steps_per_split, a.K / GS_BK - st0);

    // ---- the load stream (row blocks and units past the end of the operands fall outside the buffers and read as zeros)
    const uint32_t x_block_bytes = (uint32_t)(a.K >> 4) * 1024u;   // one block of 32 tokens, or one unit of weights, all of K
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc((void*)a.X, 0, ((a.M + 31) >> 5) * (int)x_block_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)a.W, 0, a.N * a.K * 2, 0x00020000);
    constexpr uint32_t DEAD = 0x80000000u;   // beyond any buffer: reads as zeros, moves no data
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    const uint32_t vx = (uint32_t)(m0 >> 5) * x_block_bytes + (uint32_t)(wave * 1024 + lane * 16);
    const uint32_t vw = (uint32_t)u0 * x_block_bytes + (uint32_t)(wave * 1024 + lane * 16);
    uint32_t f_slot = 0;                        // byte offset of the slot being filled
    uint32_t f_koff = (uint32_t)st0 * 4096u;    // byte offset of the step being loaded inside a block
    uint32_t f_dead = 0;                        // DEAD behind the last step
    int f_s = 0;
    const auto load = [&](auto kc) RS_INLINE {
        constexpr int k = decltype(kc)::value;
        const uint32_t dst = __builtin_amdgcn_readfirstlane(lds0 + f_slot + k * 4096 + wave * 1024);
        if constexpr (k < BMB)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr)(uintptr_t)dst, 16, vx + (f_dead + k * x_block_bytes), f_koff, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr)(uintptr_t)dst, 16, vw + (f_dead + (k - BMB) * x_block_bytes), f_koff, 0,
                                                     ONCE ? GS_ONCE : 0);
    };
    const auto advance = [&]() RS_INLINE {
        f_slot = f_slot + SLOT_BYTES == SLOTS * SLOT_BYTES ? 0u : f_slot + SLOT_BYTES;
        f_koff += 4096u;
        f_dead = ++f_s >= ns ? DEAD : 0u;
    };

    f32x16 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    float row_val[TM];
#pragma unroll
    for (int j = 0; j < TM; ++j) row_val[j] = 0.0f;

    static_for<0, SLOTS>([&](auto) RS_INLINE {
        static_for<0, L>([&](auto kc) RS_INLINE { load(kc); });
        advance();
    });
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((SLOTS - 1) * L) : "memory");
    asm volatile("s_barrier" ::: "memory");
    const int mw = m0 + wm * TM * 32, uw = u0 + wn * TN;   // this wavefront's rows and units
    if (mw < a.M) {
        const uint32_t rx0 = lds0 + (uint32_t)(wm * TM) * 4096u + (uint32_t)lane * 16u;
        const uint32_t rw0 = lds0 + (uint32_t)(BMB + wn * TN) * 4096u + (uint32_t)lane * 16u;
        uint32_t c_slot = 0;
        bf16x8 fa[4][TM + TN], fb[4][TM + TN];   // fragments of two steps: per k-step the token blocks, then the units
        const auto read_frag = [](auto offc, bf16x8& dst, const uint32_t addr) RS_INLINE { RS_DS_READ_B128(dst, addr, decltype(offc)::value); };
        const auto read = [&](auto oc, bf16x8 (&f)[4][TM + TN], const uint32_t slot) RS_INLINE {   // read number o of a step
            constexpr int kk = decltype(oc)::value / (TM + TN), o = decltype(oc)::value % (TM + TN);
            if constexpr (o < TM) read_frag(std::integral_constant<int, o * 4096 + kk * 1024>{}, f[kk][o], rx0 + slot);
            else read_frag(std::integral_constant<int, (o - TM) * 4096 + kk * 1024>{}, f[kk][o], rw0 + slot);
        };
        const auto wait_frags = [&](bf16x8 (&f)[4][TM + TN]) RS_INLINE {   // "s_waitcnt lgkmcnt(0)" tied to the fragments it guards
            tie_wait_lgkm0<TM + TN>(f[0]);
#pragma unroll
            for (int kk = 1; kk < 4; ++kk)
#pragma unroll
                for (int o = 0; o < TM + TN; ++o) asm volatile("" : "+v"(f[kk][o]));
        };
        // a step on the fragments f, read during the step before; the next step's are read into fn and the slot that f came from is
        // filled again behind its MFMAs
        const auto step = [&](bf16x8 (&f)[4][TM + TN], bf16x8 (&fn)[4][TM + TN]) RS_INLINE {
            const uint32_t n_slot = c_slot + SLOT_BYTES == SLOTS * SLOT_BYTES ? 0u : c_slot + SLOT_BYTES;
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((SLOTS - 2) * L) : "memory");   // this wavefront's share of the next step has landed
            asm volatile("s_barrier" ::: "memory");
            RS_FENCE();
            constexpr int READS = 4 * (TM + TN), OPS = READS + L, MF = 4 * TM * TN;
            static_for<0, MF>([&](auto qc) RS_INLINE {
                constexpr int q = decltype(qc)::value, kk = q / (TM * TN), i = q / TM % TN, j = q % TM;
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[kk][TM + i], f[kk][j], acc[i][j], 0, 0, 0);
                static_for<q * OPS / MF, (q + 1) * OPS / MF>([&](auto oc) RS_INLINE {
                    constexpr int o = decltype(oc)::value;
                    if constexpr (o < READS) read(oc, fn, n_slot);
                    else load(std::integral_constant<int, o - READS>{});
                });
                RS_FENCE();
            });
            advance();
            c_slot = n_slot;
            wait_frags(fn);
        };
        static_for<0, 4 * (TM + TN)>([&](auto oc) RS_INLINE { read(oc, fa, 0u); });
        wait_frags(fa);
        int s = 0;
        for (; s + 2 <= ns; s += 2) {
            step(fa, fb);
            step(fb, fa);
        }
        if (s < ns) step(fa, fb);
    } else {   // no rows: this wavefront's share of the loads, and the barriers
        for (int s = 0; s < ns; ++s) {
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((SLOTS - 2) * L) : "memory");
            asm volatile("s_barrier" ::: "memory");
            static_for<0, L>([&](auto kc) RS_INLINE { load(kc); });
            advance();
        }
    }
    if (mw < a.M) gemm_epilogue<EPI, TN, TM>(a, acc, mw, uw, half, l32, split, row_val, (a.N >> 5) - uw);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the stream's last (empty) loads still target this workgroup's LDS
    if constexpr (EPI == EPI_RESIDUAL) {
        if (a.rowss != nullptr && uw < (a.N >> 5)) {   // (a wavefront past the last unit has no part)
#pragma unroll
            for (int j = 0; j < TM; ++j) {
                const float ss = row_val[j] + __shfl_xor(row_val[j], 32, WAVE);
                const int m = mw + j * 32 + l32;
                if (half == 0 && m < a.M) a.rowss[(size_t)(strip * WN + wn) * a.M + m] = ss;
            }
        }
    }
}

// Chunk-vs-cache causal GQA attention for gfx950 (flash-style, one pass over the keys, online softmax).
//
// Work item = (request, KV head, block of 256 query rows).  The g = Hq/Hkv query heads that share a KV head are
// stacked into the row dimension: row r of a request's chunk means (token r / g, head r % g), so each K / V tile
// is fetched once per KV head rather than once per query head.  A 512-thread workgroup (8 wavefronts x 32 query
// rows, one workgroup per compute unit; or 256 threads and 128 rows, two per unit, see attention_plan.h) walks the request's cache in
// tiles of 64 keys.
//
// The kernel computes transposed products so that every per-query quantity lives in one lane:
//   S^T[key, query] = K[key, :] . Q[query, :]      MFMA "A" = K rows from LDS, "B" = Q rows held in registers
//   O^T[d,   query] = sum_key V^T[d, key] P^T[key, query]    "A" = V^T rows from LDS, "B" = P^T from the S^T registers
// With v_mfma_f32_32x32x16_bf16 a lane's accumulator column is one query (lane & 31); the two half-waves hold
// different keys (or different d) of that query, so the online softmax is lane-local but for the reference maximum,
// which rarely moves.  The MFMA row -> key assignment swaps two index
// bits so that the 8 probabilities a lane must feed to one k-step of the second product are 8 consecutive keys
// sitting in 8 consecutive accumulator registers (no data movement between the two products).
//
// Cache layout (private to the library): K is [Hkv][capacity][d]; V is stored transposed in blocks of 64 tokens,
// [Hkv][capacity/64][d][64], so that a V^T tile is one contiguous 64*d*2-byte run with the key index innermost,
// which is what the MFMA A operand needs.  A paged cache keeps the same 64-token tiles, gathered per page instead of per
// plane (see KVHeadTiles).  Positions >= len inside the last V block hold zeros (the append and import kernels, and
// the first kernel of calls whose QKV projection fills the caches, maintain this), so masked probabilities (exact zeros) never meet NaN bit patterns.
#pragma once
#include <type_traits>

#include "attention_plan.h"
#include "common.h"

struct ReqDesc {
    int row0;       // first row of this request in the packed [sum T, ...] activations
    int T;          // rows this call
    int P;          // tokens already cached before this call
    int cap;        // capacity (tokens, multiple of 64) of this request's cache (contiguous caches)
    bf16* kcache;   // contiguous: this layer's K [Hkv][cap][d];  paged: the pool's first page
    bf16* vtcache;  // contiguous: this layer's V^T [Hkv][cap/64][d][64];  paged: unused
    const int* pages;  // paged: pages[b] = pool page that holds this layer's 64-token block b;  contiguous: null
    int hkv;           // KV heads (a page is [Hkv] K tiles followed by [Hkv] V^T tiles)
    int pad_;
};

// Where the 64-token tiles of one KV head live.  A tile is K rows [64][d] or V^T [d][64], either one contiguous run of
// 64*D*2 bytes, at  base + index * stride:  in a contiguous cache both planes are arrays of tiles [kvh][block], so the
// index is the block and the stride one tile; in a paged cache the index is the block's page (looked up in the request's
// table, a uniform load) and the stride one page, which holds the K tiles of all heads followed by their V^T tiles.
// Set up once per workgroup, so that a tile's address costs one multiply-add in the loop whatever the kind of cache.
struct KVHeadTiles {
    char* k_base;
    char* v_base;
    uint32_t stride;
    const int* pages;
    // MAY_PAGE = false is for kernels launched only when every cache of the call is contiguous: no lookup, and nothing
    // in the loop that the compiler cannot see to be uniform (the software-pipelined attention kernel is about 3 % slower
    // with the lookup in its loop).
    // The index of a block: may be called long before the address is needed (the lookup's latency then passes unseen).
    template <bool MAY_PAGE = true>
    __device__ __forceinline__ int index_of(int block) const {
        if constexpr (!MAY_PAGE) return block;
        // (a load through the global address space: a generic pointer gives a flat load, which counts on the LDS counter
        //  as well, and every wait for an LDS fragment while it is in flight then becomes a wait for all of them)
        typedef const __attribute__((address_space(1))) int* global_ints;
        return pages == nullptr ? block : ((global_ints)pages)[block];
    }
    // (the index is the same for the whole wavefront; saying so here, where the value is used and not where it was
    // loaded, keeps the address in scalar registers, which the buffer resource of an LDS-DMA load needs)
    template <bool MAY_PAGE = true>
    __device__ __forceinline__ char* k_tile(int index) const {
        if constexpr (!MAY_PAGE) return k_base + (size_t)(uint32_t)index * stride;
        return k_base + (size_t)(uint32_t)__builtin_amdgcn_readfirstlane(index) * stride;
    }
    template <bool MAY_PAGE = true>
    __device__ __forceinline__ char* v_tile(int index) const {
        if constexpr (!MAY_PAGE) return v_base + (size_t)(uint32_t)index * stride;
        return v_base + (size_t)(uint32_t)__builtin_amdgcn_readfirstlane(index) * stride;
    }
};
template <int D>
RS_DEVICE KVHeadTiles kv_head_tiles(const ReqDesc& rq, int kvh) {
    constexpr uint32_t TILE = 64u * D * 2u;
    KVHeadTiles t;
    t.pages = rq.pages;
    if (rq.pages == nullptr) {
        const size_t head = (size_t)kvh * (size_t)(rq.cap >> 6) * TILE;
        t.k_base = reinterpret_cast<char*>(rq.kcache) + head;
        t.v_base = reinterpret_cast<char*>(rq.vtcache) + head;
        t.stride = TILE;
    } else {
        t.k_base = reinterpret_cast<char*>(rq.kcache) + (size_t)kvh * TILE;
        t.v_base = reinterpret_cast<char*>(rq.kcache) + (size_t)(rq.hkv + kvh) * TILE;
        t.stride = 2u * (uint32_t)rq.hkv * TILE;
    }
    return t;
}

// Split key ranges.  With few query rows and a long cache there are fewer blocks than compute units (a 256-token chunk
// at the 7B shape gives 28), each walking the whole cache, and requests of one call may have caches of very different
// lengths.  The host then cuts blocks' tiles into up to ATT_MAX_PARTS consecutive parts (attention_plan.h), one workgroup
// each; a part leaves  O~ = sum_k 2^((s_k - m) c) v_k  (fp32, unnormalised), its reference maximum m
// and its row sums l in a slot of the split buffer, and attn_merge_kernel combines the parts of a block:
//   M = max_p m_p,  w_p = 2^((m_p - M) c),  out = sum_p w_p O~_p / sum_p w_p l_p.
// A slot holds the block's rows: O~ as [D/4 chunks of 4 floats][rows] (the 32 lanes of a store cover 512 contiguous bytes),
// then m, then l.
template <int D>
struct AttnPartial {
    static constexpr int CHUNKS = D / 4;
    static constexpr size_t SLOT_FLOATS = (size_t)32 * ATT_WAVES * (D + 2);
};

// ------------------------------------------------------------------------------------------------------------------
// The kernel is software-pipelined over half tiles of 32 keys.  In the step of half h a wavefront issues the score
// products of half h + 2, the P.V products of half h and, one score per MFMA, the exponentials of half h + 1: the vector
// work (per score one fma, one exponential, one add and half a conversion: about 18 issue clocks) then sits evenly behind
// the MFMAs (32 clocks each), whatever phase the other wavefront of the SIMD is in.  With whole tiles - all exponentials
// behind the score products, the running maximum behind P.V - the first phase is bound by the vector ALU and the second by
// the matrix pipe.  Measured against that form (128 rows and four wavefronts per workgroup, two workgroups per compute
// unit): 4096 rows on 28672 cached tokens, 64 / 8 heads: 3855 -> 3555 us (1.07 -> 1.16 PFLOP/s) with the same four
// wavefronts, 3400 us with eight that share each K / V tile (half the DMA traffic into LDS), 3300 us (1.25 PFLOP/s) with
// one score behind each MFMA instead of two behind every second one; 2048 rows on 6144, 28 / 4 heads: 220 -> 200 us.  The
// board's power limit is near: a fifth fewer tiles on the fullest compute unit shortens the latter by 7 % only.  64 queries
// per wavefront (half the fragment reads, one wavefront per SIMD) is slower: 4450 us, the vector latencies then show.
// K runs one tile ahead of V: iteration kb reads K(kb+1) and V(kb) from LDS while K(kb+2) and V(kb+1) travel
// global -> LDS by DMA (buffer_load ... lds: no staging registers).  Fragments are read FRAG_AHEAD MFMAs before their
// use; the iteration's one barrier sits where its last fragment has been read, so the next tile's first fragments are read
// behind the MFMAs that are left.  The four buffers are separate LDS objects so that the compiler can tell that the
// fragment reads do not touch the buffers being filled.
//
// There is no running maximum in the loop.  A query's reference starts 2^ATT_HEADROOM_LOG2 above the exact maximum of its first 64
// keys (at the lowest finite number if they all score minus infinity) and stays until the probabilities of a half tile sum to more
// than ATT_RESCALE_SUM in one of the query's two lanes - the row sum is needed anyway -; then the reference moves as far above that
// half's maximum, the accumulated output and row sum are rescaled and the half's probabilities are taken again from its raw scores,
// which are still in registers.  Probabilities thus stay below ATT_RESCALE_SUM, which fp32 sums and bf16's relative rounding do not
// mind, the final division by the row sum cancels the reference, and what the headroom costs is range at the far end: weights
// below 2^-120 of the largest flush to zero.  A move stops all wavefronts of the workgroup at the next barrier, so it has to be
// rare: without headroom, and with the first 32 keys alone, scores of a standard deviation of 3 (hidden 8192, weights N(0, 0.02))
// moved some query of a wavefront in each of a request's first tiles.  72B shape, us: 4096 rows on 0 tokens 331 -> 276 (the exact
// running maximum of the whole-tile kernel: 313), 1200 on 0: 45.7 -> 39.7, 2048 on 2000: 217 -> 206; 7B, 2048 on 0: 47.7 -> 46.0.
constexpr float ATT_RESCALE_SUM = 256.0f, ATT_HEADROOM_LOG2 = 6.0f;

template <int D, bool MAY_PAGE, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 2) void attn_prefill_pipelined_kernel(const ReqDesc* __restrict__ reqs,
                                                                                const AttnItem* __restrict__ items,
                                                                                const bf16* __restrict__ qkv, int ld_qkv,
                                                                                bf16* __restrict__ out, int ld_out,
                                                                                int g, float scale_log2e,
                                                                                float* __restrict__ split_buf) {
    constexpr int ROWS = 32 * WAVES, THREADS = 64 * WAVES;
    constexpr int KSTEPS = D / 16;
    constexpr int DT = D / 32;
    constexpr int K_ROW_BYTES = D * 2;
    constexpr int K_CPR = K_ROW_BYTES / 16;
    constexpr int TILE_BYTES = ATT_KEYS * D * 2;
    constexpr int LOADS = TILE_BYTES / (THREADS * 16);
    constexpr int HS = 4 * DT;             // MFMAs of a half step: KSTEPS = 2 DT score products and 2 DT of P.V, alternating
    constexpr int FRAG_AHEAD = 3;          // a fragment is read this many MFMAs before its use
    constexpr int FRAGS = FRAG_AHEAD + 1;  // (divides the MFMAs of an iteration)
    static_assert(KSTEPS == 2 * DT && (2 * HS) % FRAGS == 0, "one iteration is a whole number of fragment rings");
    typedef __attribute__((address_space(3))) void* lds_ptr;
    __shared__ __attribute__((aligned(16))) char k_buf0[TILE_BYTES];
    __shared__ __attribute__((aligned(16))) char k_buf1[TILE_BYTES];
    __shared__ __attribute__((aligned(16))) char v_buf0[TILE_BYTES];
    __shared__ __attribute__((aligned(16))) char v_buf1[TILE_BYTES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;

    const AttnItem item = items[blockIdx.x];
    const ReqDesc rq = reqs[item.req];
    const int rows_total = rq.T * g;
    const int wrow0 = item.qblock * ROWS + wave * 32;
    const int row = wrow0 + l32;
    const int row_c = min(row, rows_total - 1);
    const int tok = row_c / g;
    const int head = item.kvh * g + (row_c - tok * g);
    const int qpos = rq.P + tok;
    const int wpos_lo = rq.P + min(wrow0, rows_total - 1) / g;  // every query of this wavefront sees all keys <= wpos_lo

    // ---- tile loader: a tile is a contiguous TILE_BYTES run of this KV head's cache; load instruction i of a wavefront
    //      fills LDS bytes [(i*THREADS + wave*64)*16, +1 KB) linearly by lane, each lane fetching the 16-byte chunk that
    //      belongs in its (swizzled) place.  Tiles past the item's last one are not fetched.
    const int nkb = item.nkb;
    uint32_t k_src_off[4], v_src_off[4];  // (fixed bound: LOADS <= 4; a template-dependent bound breaks the host-side stub)
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int q = i * THREADS + tid;
        {
            const int r = q / K_CPR, p = q % K_CPR;
            const int c = (K_CPR == 16) ? (p ^ (r & 15)) : (p ^ ((r >> 1) & 7));
            k_src_off[i] = (uint32_t)(r * K_ROW_BYTES + c * 16);
        }
        {
            const int r = q >> 3, p = q & 7;
            const int c = p ^ ((r >> 1) & 7);
            v_src_off[i] = (uint32_t)(r * 128 + c * 16);
        }
    }
    // (the page of a tile is looked up one iteration before the tile is fetched: see the iteration)
    const KVHeadTiles tiles = kv_head_tiles<D>(rq, item.kvh);
    auto page_of = [&](int kb) RS_INLINE { return kb < nkb ? tiles.template index_of<MAY_PAGE>(kb) : 0; };
    auto fetch_k = [&](char* buf, int kb, int page) RS_INLINE {
        if (kb < nkb) {
            const __amdgpu_buffer_rsrc_t rk =
                __builtin_amdgcn_make_buffer_rsrc((void*)tiles.template k_tile<MAY_PAGE>(page), 0, TILE_BYTES, 0x00020000);
#pragma unroll
            for (int i = 0; i < LOADS; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (lds_ptr)(uintptr_t)(uint32_t)(uintptr_t)(buf + (i * THREADS + wave * 64) * 16), 16, k_src_off[i],
                                                         0, 0, 0);
        }
    };
    auto fetch_v = [&](char* buf, int kb, int page) RS_INLINE {
        if (kb < nkb) {
            const __amdgpu_buffer_rsrc_t rv =
                __builtin_amdgcn_make_buffer_rsrc((void*)tiles.template v_tile<MAY_PAGE>(page), 0, TILE_BYTES, 0x00020000);
#pragma unroll
            for (int i = 0; i < LOADS; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (lds_ptr)(uintptr_t)(uint32_t)(uintptr_t)(buf + (i * THREADS + wave * 64) * 16), 16, v_src_off[i],
                                                         0, 0, 0);
        }
    };
    const int kb0 = item.kb0;       // this workgroup's tiles are [kb0, nkb)
    int pg_v = page_of(kb0 + 2);    // pages of the next V and K tiles to be fetched inside the loop
    int pg_k = page_of(kb0 + 3);
    {
        const int pg0 = page_of(kb0), pg1 = page_of(kb0 + 1);
        fetch_k(k_buf0, kb0, pg0);
        fetch_v(v_buf0, kb0, pg0);
        fetch_k(k_buf1, kb0 + 1, pg1);
        fetch_v(v_buf1, kb0 + 1, pg1);
    }
    // the buffers iteration kb has finished with (K(kb+1)'s and V(kb)'s) receive K(kb+3) and V(kb+2)
    auto refill = [&](int kb, char* k_done, char* v_done) RS_INLINE {
        fetch_k(k_done, kb + 3, pg_k);
        fetch_v(v_done, kb + 2, pg_v);
        pg_v = pg_k;
        pg_k = page_of(kb + 4);  // needed in the next iteration: the lookup's latency passes behind this one
    };
    // A wavefront without rows (the ragged end of a request, or a chunk of few rows) only does its share of the DMA and
    // meets the others at their barriers.
    if (wrow0 >= rows_total) {
        __syncthreads();
        __syncthreads();
        fetch_k(k_buf0, kb0 + 2, pg_v);
        int kb = kb0;
        for (; kb + 2 < nkb; kb += 2) {
            __syncthreads();
            refill(kb, k_buf1, v_buf0);
            __syncthreads();
            refill(kb + 1, k_buf0, v_buf1);
        }
        if (kb + 1 < nkb) __syncthreads();
        return;
    }

    bf16x8 qf[KSTEPS];
    {
        const bf16* qp = qkv + (size_t)(rq.row0 + tok) * ld_qkv + head * D + half * 8;
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qp + kk * 16);
    }
    const int pi = (l32 & 0x13) | ((l32 & 4) << 1) | ((l32 & 8) >> 1);
    // byte offset of K fragment (half tile 0, k-step kk) and V^T fragment (16-key group ks, features 0..31) in a tile
    uint32_t k_off[KSTEPS], v_off[4];
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) {
        const uint32_t swz = (K_CPR == 16) ? (uint32_t)(pi & 15) : (uint32_t)((pi >> 1) & 7);   // (the same for row pi + 32)
        k_off[kk] = (uint32_t)(pi * K_ROW_BYTES) + (((uint32_t)(kk * 2 + half) ^ swz) * 16u);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) v_off[ks] = (uint32_t)l32 * 128u + (((uint32_t)(ks * 2 + half) ^ (uint32_t)((l32 >> 1) & 7)) * 16u);
    auto k_frag = [&](const char* buf, int hh, int kk) RS_INLINE {
        return *reinterpret_cast<const bf16x8*>(buf + k_off[kk] + hh * 32 * K_ROW_BYTES);
    };
    auto v_frag = [&](const char* buf, int ks, int t) RS_INLINE { return *reinterpret_cast<const bf16x8*>(buf + v_off[ks] + t * 32 * 128); };

    f32x16 acc_o[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_o[t][r] = 0.0f;
    f32x16 s0, s1;            // raw scores of the two halves of a tile: register r of half hh holds key
                              // key0 + hh*32 + 16*(r>>3) + 8*half + (r&7)
    bf16x8 pf0[2], pf1[2];    // probabilities of the two halves, as the P.V product wants them
    const float headroom = ATT_HEADROOM_LOG2 / scale_log2e;   // (raw scores)
    float m_ref;        // reference of this lane's query, raw scores (shared by both half-waves)
    float l_run = 0.0f; // running sum over THIS half-wave's keys
    const f32x16 zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};

    auto mask = [&](f32x16& sc, int key0) RS_INLINE {   // sc: the half that starts at key0
        if (key0 + 31 > wpos_lo) {  // some query of this wavefront does not see all of it
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = key0 + 16 * (r >> 3) + 8 * half + (r & 7);
                sc[r] = (key <= qpos) ? sc[r] : -INFINITY;
            }
        }
    };
    auto half_max = [&](const f32x16& sc) RS_INLINE {
        float m = sc[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) m = fmaxf(m, sc[r]);
        return fmaxf(m, __shfl_xor(m, 32, WAVE));
    };
    auto exp_score = [&](float sc, float mb) RS_INLINE { return __builtin_amdgcn_exp2f(__builtin_fmaf(sc, scale_log2e, -mb)); };
    auto all_exps = [&](const f32x16& sc, bf16x8 (&p)[2]) RS_INLINE {
        const float mb = m_ref * scale_log2e;
        float sum = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float e = exp_score(sc[r], mb);
            sum += e;
            p[r >> 3][r & 7] = f32_to_bf16(e);
        }
        return sum;
    };
    // after the exponentials of a half: take its row sum, or move the reference first (see above)
    auto settle = [&](const f32x16& sc, bf16x8 (&p)[2], float psum) RS_INLINE {
        const unsigned long long over = __builtin_amdgcn_ballot_w64(!(psum <= ATT_RESCALE_SUM));
        if (__builtin_expect(over != 0, 0)) {
            const bool mine = ((((uint32_t)over | (uint32_t)(over >> 32)) >> l32) & 1u) != 0;   // either half-wave's sum
            const float m_half = half_max(sc);
            const float m_new = mine ? fmaxf(m_ref, m_half + headroom) : m_ref;
            const float alpha = __builtin_amdgcn_exp2f((m_ref - m_new) * scale_log2e);
            m_ref = m_new;
            l_run *= alpha;
#pragma unroll
            for (int t = 0; t < DT; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc_o[t][r] *= alpha;
            psum = all_exps(sc, p);
        }
        l_run += psum;
    };

    // ---- prologue: scores of tile kb0, the reference, the probabilities of its first half
    __syncthreads();
    bf16x8 frag[FRAGS];
    auto first_scores = [&](auto hhc, f32x16& sc) RS_INLINE {
        static_for<0, KSTEPS>([&](auto kc) RS_INLINE {
            constexpr int kk = decltype(kc)::value, hh = decltype(hhc)::value;
            sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_frag(k_buf0, hh, kk), qf[kk], kk == 0 ? zero : sc, 0, 0, 0);
        });
        mask(sc, kb0 * ATT_KEYS + decltype(hhc)::value * 32);
    };
    first_scores(std::integral_constant<int, 0>{}, s0);
    first_scores(std::integral_constant<int, 1>{}, s1);
    // The first key of a part is visible to every query of the block, but its score, and those of the other 63, may be minus
    // infinity (an infinite key element, an overflow): from the lowest finite reference such keys weigh nothing, and the first
    // finite score moves it.
    m_ref = fmaxf(fmaxf(half_max(s0), half_max(s1)) + headroom, -3.402823466e38f);
    l_run = all_exps(s0, pf0);
    __syncthreads();  // every wavefront is done with the first K tile: it may be overwritten
    fetch_k(k_buf0, kb0 + 2, pg_v);

    // fragment of MFMA number q of an iteration: even q a K fragment, odd q a V^T fragment
    auto read_frag = [&](auto qc, const char* k_next, const char* v_cur) RS_INLINE {
        constexpr int q = decltype(qc)::value, hh = q / HS, i = (q % HS) >> 1;
        if constexpr (q & 1) return v_frag(v_cur, hh * 2 + i / DT, i % DT);
        else return k_frag(k_next, hh, i);
    };
    static_for<0, FRAG_AHEAD>([&](auto qc) RS_INLINE { frag[decltype(qc)::value] = read_frag(qc, k_buf1, v_buf0); });

    // Half step hh of iteration kb: scores of that half of tile kb+1 (K from k_next) into sc_new, P.V of that half of tile kb
    // (V from v_cur, probabilities p_use), exponentials of sc_old - the second half of tile kb (hh 0) or the first of tile
    // kb+1 (hh 1) - into p_new.  k_after / v_after are the next iteration's buffers.  LAST: there is no tile kb+1.
    auto half_step = [&](auto last_c, auto hhc, int kb, f32x16& sc_new, const f32x16& sc_old, const bf16x8 (&p_use)[2], bf16x8 (&p_new)[2],
                         char* k_next, char* v_cur, char* k_after, char* v_after) {
        constexpr bool LAST = decltype(last_c)::value;
        constexpr int hh = decltype(hhc)::value;
        constexpr bool EXPS = !LAST || hh == 0;
        constexpr int PER = 16 / HS;   // scores behind each MFMA (1 for d = 128, 2 for d = 64)
        const float mb = m_ref * scale_log2e;
        float psum = 0.0f, e[2];
        // sum and conversion of the pair of probabilities that ends in score r
        auto close_pair = [&](auto rc) RS_INLINE {
            constexpr int r = decltype(rc)::value;
            // plain adds: a v_dot2 here would be one instruction instead of two, but the dot instructions do not run
            // beside an MFMA (measured: each one stalls the matrix pipe for its own duration and more)
            psum += e[0] + e[1];
            bf16x2 pp = {f32_to_bf16(e[0]), f32_to_bf16(e[1])};
            asm volatile("" : "+v"(pp), "+v"(psum));   // (here: left alone, all conversions sink in front of the P.V products)
            p_new[r >> 3][(r & 7) - 1] = pp[0];
            p_new[r >> 3][r & 7] = pp[1];
        };
        static_for<0, HS>([&](auto ic) RS_INLINE {
            constexpr int i = decltype(ic)::value, q = hh * HS + i, qn = q + FRAG_AHEAD;
            if constexpr (!LAST && q == 2 * HS - FRAG_AHEAD) {
                // every fragment of this iteration has been read: its buffers may be refilled, and the next tiles have landed
                __syncthreads();
                refill(kb, k_next, v_cur);
            }
            if constexpr (qn < 2 * HS) {
                if constexpr (!LAST || (qn & 1)) frag[qn % FRAGS] = read_frag(std::integral_constant<int, qn>{}, k_next, v_cur);
            } else if constexpr (!LAST) {
                frag[qn % FRAGS] = read_frag(std::integral_constant<int, qn - 2 * HS>{}, k_after, v_after);
            }
            __builtin_amdgcn_sched_barrier(0);  // the read goes out first
            if constexpr (i & 1) {
                constexpr int j = i >> 1;
                acc_o[j % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[q % FRAGS], p_use[j / DT], acc_o[j % DT], 0, 0, 0);
            } else if constexpr (!LAST) {
                sc_new = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[q % FRAGS], qf[i >> 1], i == 0 ? zero : sc_new, 0, 0, 0);
            }
            if constexpr (EXPS) {
                static_for<0, PER>([&](auto ec) RS_INLINE {
                    constexpr int r = i * PER + decltype(ec)::value;
                    if constexpr ((r & 1) == 0 && r > 0) close_pair(std::integral_constant<int, r - 1>{});   // (one MFMA behind: its latency has passed)
                    // raw v_exp_f32: results below the normal range may flush to zero
                    e[r & 1] = exp_score(sc_old[r], mb);
                    asm volatile("" : "+v"(e[r & 1]));   // pins the vector work here
                });
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (EXPS) close_pair(std::integral_constant<int, 15>{});
        if constexpr (!LAST) mask(sc_new, (kb + 1) * ATT_KEYS + hh * 32);
        if constexpr (EXPS) settle(sc_old, p_new, psum);
    };
    auto iteration = [&](auto last_c, int kb, char* k_next, char* v_cur, char* k_after, char* v_after) RS_INLINE {
        half_step(last_c, std::integral_constant<int, 0>{}, kb, s0, s1, pf0, pf1, k_next, v_cur, k_after, v_after);
        half_step(last_c, std::integral_constant<int, 1>{}, kb, s1, s0, pf1, pf0, k_next, v_cur, k_after, v_after);
    };

    int kb = kb0;
    for (; kb + 2 < nkb; kb += 2) {
        iteration(std::false_type{}, kb, k_buf1, v_buf0, k_buf0, v_buf1);
        iteration(std::false_type{}, kb + 1, k_buf0, v_buf1, k_buf1, v_buf0);
    }
    if (kb + 1 < nkb) {
        iteration(std::false_type{}, kb, k_buf1, v_buf0, k_buf0, v_buf1);
        iteration(std::true_type{}, kb + 1, k_buf0, v_buf1, k_buf1, v_buf0);
    } else {
        iteration(std::true_type{}, kb, k_buf1, v_buf0, k_buf0, v_buf1);
    }

    const float l_tot = l_run + __shfl_xor(l_run, 32, WAVE);
    if (item.slot >= 0) {
        // a part of a split block: unnormalised output, reference maximum and row sum go to the slot (all 32 rows of
        // the wavefront, clamped duplicates included: the merge kernel decides what is stored; wavefronts without rows left above)
        float* const slot = split_buf + (size_t)item.slot * AttnPartial<D>::SLOT_FLOATS;
        const int rs = wave * 32 + l32;  // row inside the block
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 o = {acc_o[t][4 * q], acc_o[t][4 * q + 1], acc_o[t][4 * q + 2], acc_o[t][4 * q + 3]};
                // chunk (features 32t + 8q + 4half .. +3) of row rs
                *reinterpret_cast<f32x4*>(slot + ((size_t)(t * 8 + q * 2 + half) * ROWS + rs) * 4) = o;
            }
        if (half == 0) {
            slot[(size_t)D * ROWS + rs] = m_ref;
            slot[(size_t)(D + 1) * ROWS + rs] = l_tot;
        }
        return;
    }
    if (row < rows_total) {
        const float inv = 1.0f / l_tot;
        const uint32_t m = (uint32_t)(rq.row0 + tok);
        char* op = reinterpret_cast<char*>(out) + (size_t)(m >> 5) * (size_t)(ld_out >> 4) * 1024 + (m & 31u) * 16u + half * 8;
        const int ks0 = (head * D) >> 4;
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = f32_to_bf16(acc_o[t][4 * q + e] * inv);
                *reinterpret_cast<bf16x4*>(op + (size_t)(((ks0 + 2 * t + (q >> 1)) * 2 + (q & 1)) * 512)) = o;
            }
    }
}

// Combines the parts of split blocks (see AttnPartial).  ATT_MERGE_Y workgroups per block (grid y): the threads of
// workgroup y handle the block's rows and the chunks y, y + ATT_MERGE_Y, ... of their D/4 chunks of 4 features - one or two
// chunks, so all of a thread's loads are in flight together (one workgroup per block walking all its chunks one after the
// other took 13 us, more than a short key range saves).  Every workgroup computes the rows' weights.
// MAXP: no block has more parts.  EARLY: the outputs are loaded with the references and row sums, ahead of the weights; it takes 10
// registers per part, so with many parts only launches that are resident at once anyway gain by it.  us, late with room for 16 -> now:
// 64 rows on 2048 (256 workgroups) 6.1 -> 3.9, 250 on 8192 (448) 10.4 -> 8.4; up to 4 parts, 512 on 1536 (1792) 7.1 -> 6.0, 1000 on 12000
// 10.3 -> 10.4 (early with room for 16: 8.7 and 13.0).
constexpr int ATT_MERGE_Y = 16;
constexpr int ATT_FEW_PARTS = 4;
constexpr int ATT_MERGE_EARLY_WAVES = 12;   // wavefronts per compute unit that the early form's registers leave room for
template <int D, int WAVES, int MAXP, bool EARLY>
__global__ __launch_bounds__(32 * WAVES) void attn_merge_kernel(const ReqDesc* __restrict__ reqs, const AttnMergeItem* __restrict__ items,
                                                         const float* __restrict__ split_buf, bf16* __restrict__ out, int ld_out,
                                                         int g, float scale_log2e) {
    constexpr int ROWS = 32 * WAVES;
    const AttnMergeItem item = items[blockIdx.x];
    const ReqDesc rq = reqs[item.req];
    const int rs = threadIdx.x;
    const int row = item.qblock * ROWS + rs;
    if (row >= rq.T * g) return;
    const int tok = row / g;
    const int head = item.kvh * g + (row - tok * g);
    const float* const base = split_buf + (size_t)item.slot0 * AttnPartial<D>::SLOT_FLOATS;
    // (all loads of a round are issued together: absent parts read as m = -inf, l = 0 and get weight 0)
    static_assert(AttnPartial<D>::CHUNKS % ATT_MERGE_Y == 0, "chunks divide among the merge workgroups");
    constexpr int MY = AttnPartial<D>::CHUNKS / ATT_MERGE_Y;   // chunks of a thread
    float mp[MAXP], lp[MAXP];
    f32x4 o[EARLY ? MY : 1][EARLY ? MAXP : 1];
#pragma unroll
    for (int p = 0; p < MAXP; ++p) {
        mp[p] = -INFINITY;
        lp[p] = 0.0f;
        if (p < item.n_parts) {
            const float* sp = base + p * AttnPartial<D>::SLOT_FLOATS;
            mp[p] = sp[(size_t)D * ROWS + rs];
            lp[p] = sp[(size_t)(D + 1) * ROWS + rs];
            if constexpr (EARLY)
#pragma unroll
                for (int k = 0; k < MY; ++k) o[k][p] = *reinterpret_cast<const f32x4*>(sp + ((size_t)(blockIdx.y + k * ATT_MERGE_Y) * ROWS + rs) * 4);
        }
    }
    float m_all = -INFINITY;
#pragma unroll
    for (int p = 0; p < MAXP; ++p) m_all = fmaxf(m_all, mp[p]);
    float l_all = 0.0f;
    float w[MAXP];
#pragma unroll
    for (int p = 0; p < MAXP; ++p) {
        w[p] = 0.0f;
        if (p < item.n_parts) {
            w[p] = __builtin_amdgcn_exp2f((mp[p] - m_all) * scale_log2e);
            l_all += w[p] * lp[p];
        }
    }
    const float inv = 1.0f / l_all;
    const uint32_t m = (uint32_t)(rq.row0 + tok);
    char* const op = reinterpret_cast<char*>(out) + (size_t)(m >> 5) * (size_t)(ld_out >> 4) * 1024 + (m & 31u) * 16u;
    const int ks0 = (head * D) >> 4;
#pragma unroll
    for (int k = 0; k < MY; ++k) {
        const int c = blockIdx.y + k * ATT_MERGE_Y;
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int p = 0; p < MAXP; ++p)
            if (p < item.n_parts) {
                const f32x4 part = EARLY ? o[EARLY ? k : 0][EARLY ? p : 0]
                                        : *reinterpret_cast<const f32x4*>(base + p * AttnPartial<D>::SLOT_FLOATS + ((size_t)c * ROWS + rs) * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] += w[p] * part[e];
            }
        bf16x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = f32_to_bf16(acc[e] * inv);
        // chunk c = 8t + 2q + half holds features 32t + 8q + 4half .. +3: the same place the unsplit kernel writes
        const int t = c >> 3, q = (c >> 1) & 3, hf = c & 1;
        *reinterpret_cast<bf16x4*>(op + hf * 8 + (size_t)(((ks0 + 2 * t + (q >> 1)) * 2 + (q & 1)) * 512)) = o4;
    }
}

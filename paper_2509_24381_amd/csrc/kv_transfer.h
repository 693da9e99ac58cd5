// Cache export and import (canonical [tokens][Hkv][d] arrays on one side, the cache's 64-token tiles on the other), for
// bfloat16 and 8-bit caches, contiguous and paged.
//
// Bound by HBM: every element is read and written once.  One workgroup moves one 64-token block of one KV head, 8 elements
// (one 16-byte chunk of bfloat16) per access; K rows are contiguous on both sides, V^T tiles are turned through LDS.  The
// element-by-element form before it (one thread per element, V^T read or written with a stride of 128 bytes) took
// 67 us for export, import and export of 8192 tokens at the 7B shape (100 MB moved); this one takes 31 (3.2 TB/s with the three
// launches in it; a thread has one access in flight, and a workgroup of few tiles waits for four or five in a row).  Behind a layer call, 8442 paged tokens: the call and its export 296 -> 273 us; 13000 tokens of 8-bit pages,
// with the attention kernel's gain: 706 -> 644.
//
// The canonical arrays come from the caller and need only their element's alignment: `wide` says that both can be accessed
// 8 elements at a time.
//
// The cache is described as for the other kernels, `pages` being only a marker here (non-null: paged): the page numbers of
// blocks [block0, block0 + KV_PAGE_WINDOW) ride in the kernel arguments.  Tokens [t0, t0 + n) are handled, t0 a multiple of
// 64; block t0/64 + blockIdx.x, KV head blockIdx.y.
#pragma once
#include "attention.h"
#include "common.h"
#include "elementwise.h"
#include "kv_fp8.h"

// 8 stored elements <-> 8 canonical ones
RS_DEVICE uint4 convert8(uint4 v, float, bf16*) { return v; }
RS_DEVICE uint2 convert8(uint2 v, float, uint8_t*) { return v; }
RS_DEVICE uint4 convert8(uint2 codes, float scale, bf16*) {   // read an 8-bit cache
    const bf16x4 lo = bf16x4_from_e4m3(codes.x, scale), hi = bf16x4_from_e4m3(codes.y, scale);
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        o[e] = lo[e];
        o[4 + e] = hi[e];
    }
    return as_uint4(o);
}
RS_DEVICE uint2 convert8(uint4 v, float inv, uint8_t*) { return e4m3_from_bf16x8(as_bf16x8(v), inv); }   // store to one

// Eight elements of an LDS tile, element(0) .. element(7), as one value.  (Put together word by word: out of a union of eight bf16 the
// compiler makes four stores.)
template <class T, class F>
RS_DEVICE typename Pack8<T>::type gather8(F&& element) {
    typename Pack8<T>::type v;
    uint32_t* w = reinterpret_cast<uint32_t*>(&v);
    constexpr int PER = 4 / (int)sizeof(T);
#pragma unroll
    for (int j = 0; j < 8 / PER; ++j) {
        w[j] = 0u;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const T x = element(j * PER + e);
            if constexpr (sizeof(T) == 2) w[j] |= (uint32_t)__builtin_bit_cast(uint16_t, x) << (16 * e);
            else w[j] |= (uint32_t)x << (8 * e);
        }
    }
    return v;
}

// T: the cache's element (bf16, or uint8_t for E4M3 codes), C: the canonical one (bf16, or uint8_t for codes).
// The K or V^T tile of one KV head and block:
template <int D, class T>
RS_DEVICE T* transfer_tile(const ReqDesc& rq, const Fp8CacheDesc& fc, const KVPageWindow& win, int block0, bool v, int c, int block) {
    if constexpr (sizeof(T) == 2) return kv_window_tile<D>(rq, win, block0, v, c, block);
    else return fp8_window_tile<D>(fc, win, block0, v, c, block);
}

// (rows of the LDS tiles are padded by 3 words: 8 rows further, the step between the elements one thread gathers and its
//  neighbour's, is then 24 banks)
template <int D, class T, class C>
__global__ __launch_bounds__(256) void kv_export_kernel(ReqDesc rq, Fp8CacheDesc fc, KVPageWindow win, int block0, C* __restrict__ k_out,
                                                        C* __restrict__ v_out, int t0, int n, int wide) {
    typedef typename Pack8<T>::type P;
    constexpr int ROW = 64 + 12 / (int)sizeof(T);
    __shared__ __attribute__((aligned(16))) T vt[D][ROW];
    const int hkv = sizeof(T) == 2 ? rq.hkv : fc.hkv, c = blockIdx.y;
    const int tok0 = t0 + (int)blockIdx.x * 64, left = min(64, t0 + n - tok0);   // tokens of this block
    const T* kt = transfer_tile<D, T>(rq, fc, win, block0, false, c, tok0 >> 6);
    const T* vtile = transfer_tile<D, T>(rq, fc, win, block0, true, c, tok0 >> 6);
    for (int i = threadIdx.x; i < D * 8; i += 256) {   // feature i / 8, tokens 8 (i % 8) ..
        const P v = load8(vtile + (size_t)i * 8, true);
        uint32_t* dst = reinterpret_cast<uint32_t*>(&vt[i >> 3][(i & 7) * 8]);
        const uint32_t* w = reinterpret_cast<const uint32_t*>(&v);
#pragma unroll
        for (int j = 0; j < (int)(sizeof(P) / 4); ++j) dst[j] = w[j];
    }
    constexpr int CPR = D / 8;
    C* const k0 = k_out + ((size_t)tok0 * hkv + c) * D;
    C* const v0 = v_out + ((size_t)tok0 * hkv + c) * D;
    for (int i = threadIdx.x; i < left * CPR; i += 256) {
        const int t = i / CPR, ch = i % CPR;
        store8(k0 + (size_t)t * hkv * D + ch * 8, convert8(load8(kt + (size_t)i * 8, true), fc.k_scale, (C*)nullptr), wide);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < left * CPR; i += 256) {
        const int t = i / CPR, ch = i % CPR;
        const P v = gather8<T>([&](int e) { return vt[ch * 8 + e][t]; });
        store8(v0 + (size_t)t * hkv * D + ch * 8, convert8(v, fc.v_scale, (C*)nullptr), wide);
    }
}

// V^T positions of the last touched block at and beyond t0 + n become zero; K rows there keep what they hold.
template <int D, class T, class C>
__global__ __launch_bounds__(256) void kv_import_kernel(ReqDesc rq, Fp8CacheDesc fc, KVPageWindow win, int block0, const C* __restrict__ k_in,
                                                        const C* __restrict__ v_in, int t0, int n, int wide) {
    typedef typename Pack8<T>::type P;
    constexpr int ROW = D + 12 / (int)sizeof(T);
    __shared__ __attribute__((aligned(16))) T rows[64][ROW];
    const int hkv = sizeof(T) == 2 ? rq.hkv : fc.hkv, c = blockIdx.y;
    const int tok0 = t0 + (int)blockIdx.x * 64, left = min(64, t0 + n - tok0);
    T* kt = transfer_tile<D, T>(rq, fc, win, block0, false, c, tok0 >> 6);
    T* vtile = transfer_tile<D, T>(rq, fc, win, block0, true, c, tok0 >> 6);
    constexpr int CPR = D / 8;
    const C* const k0 = k_in + ((size_t)tok0 * hkv + c) * D;
    const C* const v0 = v_in + ((size_t)tok0 * hkv + c) * D;
    for (int i = threadIdx.x; i < 64 * CPR; i += 256) {
        const int t = i / CPR, ch = i % CPR;
        P v = {};
        if (t < left) {
            v = convert8(load8(v0 + (size_t)t * hkv * D + ch * 8, wide), fc.v_inv, (T*)nullptr);
            store8(kt + (size_t)i * 8, convert8(load8(k0 + (size_t)t * hkv * D + ch * 8, wide), fc.k_inv, (T*)nullptr), true);
        }
        uint32_t* dst = reinterpret_cast<uint32_t*>(&rows[t][ch * 8]);
        const uint32_t* w = reinterpret_cast<const uint32_t*>(&v);
#pragma unroll
        for (int j = 0; j < (int)(sizeof(P) / 4); ++j) dst[j] = w[j];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < D * 8; i += 256) {   // feature i / 8, tokens 8 (i % 8) ..
        store8(vtile + (size_t)i * 8, gather8<T>([&](int e) { return rows[(i & 7) * 8 + e][i >> 3]; }), true);
    }
}

// bf16 MFMA attention for gfx950 against the paged cache: causal prefill and
// split-KV decode.  Both kernels compute the TRANSPOSED products
//     S^T = K * Q^T        (rows = cached tokens, columns = queries)
//     O^T = V^T * P^T      (rows = head dimension, columns = queries)
// so that the accumulator of the first product is already in the register
// layout the second product wants for its B operand (each lane owns one query
// column and a run of tokens): P never travels through LDS or across lanes.
// K pages are [head][16][D] and V pages are stored transposed, [head][D][16] (token order 0-3, 8-11, 4-7, 12-15),
// so both MFMA A operands are plain vector loads straight from the pages.
//
// The contraction order inside one MFMA is free as long as both operands agree:
// the token <-> k-slot assignment below is chosen to match what the S^T
// accumulator holds, and the V^T operand is gathered with the same assignment.
#include <type_traits>

#include "ss_device.h"
#include "ss_kernels.h"

namespace SS_NS {
using namespace ssk;

// 2^x on the hardware's exponential unit (v_exp_f32, about 1 ulp for normal results; results below the
// normal range flush to zero, which a softmax weight may).  The library exp2f wraps the same instruction
// in range scaling for denormal results: four more VALU operations per element in the innermost loop.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// max of a value with the one held by the lane 32 positions away (v_permlane32_swap: no LDS round trip)
__device__ __forceinline__ float max_with_other_half(float x) {
    const unsigned u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

typedef half8_t bf16x8_t;       // MFMA operand: 8 elements of the 16-bit type
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef int i32x8_t __attribute__((ext_vector_type(8)));

struct __attribute__((aligned(8))) vec8 { uint32_t w[2]; };

union Frag {
    bf16x8_t v;
    vec16 q;
    vec8 h[2];
    uint32_t w[4];
};

// ======================================================================
// Prefill.  Block = 4 waves = 256 consecutive queries of one (sequence, q head);
// each wave owns QT = 2 tiles of 32 queries and walks the pages its queries can
// see, two pages (32 tokens) per step, with v_mfma_f32_32x32x16_bf16:
//   accumulator register v of lane l <-> token 8*(v/4) + 4*(l/32) + v%4, query l%32.
// Every K and V^T fragment loaded from the pages feeds both query tiles.
// ======================================================================
template <int D, int QT>
__global__ __launch_bounds__(256) void attn_prefill_mfma_kernel(const bf16_t* __restrict__ qkv,
                                                                bf16_t* __restrict__ out, int n_q, int n_kv,
                                                                BatchMeta bm, const bf16_t* __restrict__ k_pool,
                                                                const bf16_t* __restrict__ v_pool,
                                                                float scale_log2e) {
    constexpr int KS = D / 16;      // k-steps of the score product
    constexpr int DT = D / 32;      // 32-row tiles of O^T
    const int sq = blockIdx.z, a = blockIdx.y;
    const int q_begin = bm.cu_q[sq], q_len = bm.cu_q[sq + 1] - q_begin;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int q0 = blockIdx.x * (128 * QT) + wave * (32 * QT);
    if (q0 >= q_len) return;
    const int before = bm.kv_before[sq];
    const int g = a / (n_q / n_kv);
    const int lq = lane & 31, g2 = lane >> 5;
    const int last_q = (q0 + 32 * QT - 1 < q_len) ? q0 + 32 * QT - 1 : q_len - 1;
    const int n_pages = (before + last_q) / 16 + 1;
    const size_t row_stride = (size_t)(n_q + 2 * n_kv) * D;

    Frag qf[QT][KS];
    int p[QT];
    bool valid[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
        const int qi = q0 + t * 32 + lq;
        valid[t] = qi < q_len;
        p[t] = before + (valid[t] ? qi : 0);
        const bf16_t* qp = qkv + (size_t)(q_begin + (valid[t] ? qi : 0)) * row_stride + (size_t)a * D + g2 * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[t][ks].q = *reinterpret_cast<const vec16*>(qp + ks * 16);
    }
    f32x16_t o[QT][DT];
    float m[QT], l[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
        m[t] = -INFINITY;
        l[t] = 0.f;
#pragma unroll
        for (int u = 0; u < DT; ++u)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[t][u][v] = 0.f;
    }

    const int32_t* pt = bm.page_tables + (size_t)sq * bm.pt_stride;
    const size_t page_elems = (size_t)n_kv * 16 * D;
    const size_t head_off = (size_t)g * 16 * D;
    const int tok = lq;                       // token row this lane loads of the 32-token step
    for (int pi = 0; pi < n_pages; pi += 2) {
        const int pA = pt[pi];
        const int pB = pt[(pi + 1 < n_pages) ? pi + 1 : pi];
        // ---- S^T = K Q^T for both query tiles
        const bf16_t* kp = k_pool + (size_t)(tok < 16 ? pA : pB) * page_elems + head_off + (size_t)(tok & 15) * D + g2 * 8;
        f32x16_t s[QT];
#pragma unroll
        for (int t = 0; t < QT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) s[t][v] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            Frag kf;
            kf.q = *reinterpret_cast<const vec16*>(kp + ks * 16);
#pragma unroll
            for (int t = 0; t < QT; ++t) s[t] = SS_MFMA_32x32x16(kf.v, qf[t][ks].v, s[t], 0, 0, 0);
        }
        // ---- mask + streaming softmax (per query column = per lane pair l, l^32)
        const int t0 = pi * 16;
        Frag pfA[QT], pfB[QT];
#pragma unroll
        for (int t = 0; t < QT; ++t) {
            float mx = m[t];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int tpos = t0 + 8 * (v >> 2) + 4 * g2 + (v & 3);
                s[t][v] = (tpos <= p[t]) ? s[t][v] * scale_log2e : -INFINITY;
                mx = fmaxf(mx, s[t][v]);
            }
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float alpha = fast_exp2(m[t] - mx);
            m[t] = mx;
            float rs = 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) { s[t][v] = fast_exp2(s[t][v] - mx); rs += s[t][v]; }
            l[t] = l[t] * alpha + rs;
#pragma unroll
            for (int u = 0; u < DT; ++u)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[t][u][v] *= alpha;
            // k-slots of step A: tokens {4*g2 + i, 8 + 4*g2 + i} of page A; step B: the same of page B
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                pfA[t].w[i] = pack_bf16x2(s[t][2 * i], s[t][2 * i + 1]);
                pfB[t].w[i] = pack_bf16x2(s[t][8 + 2 * i], s[t][8 + 2 * i + 1]);
            }
        }
        // ---- O^T += V^T P^T
        // the page keeps each row as [0-3, 8-11, 4-7, 12-15] (halves swapped in rows with bit 3 of the row index set,
        // see vpos): lane group g2's eight tokens are 16 contiguous bytes
        const int vhalf = g2 ^ ((lq >> 3) & 1);
        const bf16_t* vA = v_pool + (size_t)pA * page_elems + head_off + (size_t)lq * 16 + 8 * vhalf;
        const bf16_t* vB = v_pool + (size_t)pB * page_elems + head_off + (size_t)lq * 16 + 8 * vhalf;
        Frag va[DT], vb[DT];
#pragma unroll
        for (int u = 0; u < DT; ++u) {
            va[u].q = *reinterpret_cast<const vec16*>(vA + u * 32 * 16);
            vb[u].q = *reinterpret_cast<const vec16*>(vB + u * 32 * 16);
        }
        // tokens behind the last one that the wave sees: what the page's last user left, or a page that is only repeated
        if (t0 + 31 > before + last_q) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int at = t0 + 4 * g2 + 2 * (w & 1) + 8 * (w >> 1), seen = before + last_q;
                const uint32_t ka = (at <= seen ? 0xffffu : 0u) | (at + 1 <= seen ? 0xffff0000u : 0u);
                const uint32_t kb = (at + 16 <= seen ? 0xffffu : 0u) | (at + 17 <= seen ? 0xffff0000u : 0u);
#pragma unroll
                for (int u = 0; u < DT; ++u) {
                    va[u].w[w] &= ka;
                    vb[u].w[w] &= kb;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < DT; ++u)
#pragma unroll
            for (int t = 0; t < QT; ++t) {
                o[t][u] = SS_MFMA_32x32x16(va[u].v, pfA[t].v, o[t][u], 0, 0, 0);
                o[t][u] = SS_MFMA_32x32x16(vb[u].v, pfB[t].v, o[t][u], 0, 0, 0);
            }
    }
#pragma unroll
    for (int t = 0; t < QT; ++t) {
        l[t] += __shfl_xor(l[t], 32, 64);
        if (valid[t]) {
            const float inv = 1.0f / l[t];
            bf16_t* op = out + (size_t)(q_begin + q0 + t * 32 + lq) * ((size_t)n_q * D) + (size_t)a * D;
#pragma unroll
            for (int u = 0; u < DT; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    vec8 w;
                    w.w[0] = pack_bf16x2(o[t][u][4 * j] * inv, o[t][u][4 * j + 1] * inv);
                    w.w[1] = pack_bf16x2(o[t][u][4 * j + 2] * inv, o[t][u][4 * j + 3] * inv);
                    *reinterpret_cast<vec8*>(op + u * 32 + 8 * j + 4 * g2) = w;
                }
        }
    }
}

// ----------------------------------------------------------------------
// Prefill, LDS-staged.  A block of 8 waves works on one item at a time: 256 consecutive queries of one (sequence, q head).  The K
// and V^T chunks of 64 tokens (4 pages, 32 KB) are brought into a three-stage LDS ring (two tiles in flight) with direct
// global->LDS loads and shared by all eight waves, which cuts the L2 traffic of the attention by 8
// against every wave fetching its own operands.  K rows (256 bytes) are stored with the 16-byte
// chunk index XOR-ed with the row number, so the 16 rows one pass of a fragment read touches fall
// on different banks; V^T chunks are stored exactly as in the page (a fragment read is 1 KB
// contiguous).  A wave skips the MFMAs of tiles none of its queries can see, but takes part in every
// load and barrier.
// ----------------------------------------------------------------------
__device__ __forceinline__ void dma16a(const void* gptr, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gptr), "s"(lds_addr) : "memory");
}

template <int D>
__global__ __launch_bounds__(512) void attn_prefill_lds_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ out,
                                                               int n_q, int n_kv, BatchMeta bm,
                                                               const bf16_t* __restrict__ k_pool,
                                                               const bf16_t* __restrict__ v_pool, float scale_log2e) {
    static_assert(D == 128, "layout below assumes 256-byte K rows");
    constexpr int KS = D / 16, DT = D / 32, NS = 3;
    constexpr int KBYTES = 64 * D * 2, STAGE = 2 * KBYTES;     // 16 KB of K + 16 KB of V^T
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    // Persistent blocks, one per compute unit: block b walks its list of items (sequence, q head, block of
    // 256 queries) that the host has laid out (see BatchMeta::pf_items): launching a block of this size per
    // item costs 3-4 us of dispatch each, a sixth of the kernel's time on prompts of one or two thousand tokens.
    const int G = n_q / n_kv;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lq = lane & 31, g2 = lane >> 5;
    const size_t row_stride = (size_t)(n_q + 2 * n_kv) * D;
    const size_t page_elems = (size_t)n_kv * 16 * D;
    const uint32_t lds_base = (uint32_t)(uintptr_t)smem;
    for (int pj = 0;; ++pj) {
    // the item's record through the scalar cache: one load, a few hundred nanoseconds (as ordinary loads the
    // six values would be as many dependent round trips, the loop's memory clobbers keep them from being merged)
    const int32_t* item = bm.pf_items + ((size_t)blockIdx.x * bm.pf_stride + pj) * 8;
    i32x8_t rec;
    asm volatile("s_load_dwordx8 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(rec) : "s"(item) : "memory");
    const int sq = rec[0];
    if (sq < 0) break;                                         // end of the list: the whole block leaves
    const int a = rec[1], qb0 = rec[2], q_begin = rec[3], q_len = rec[4];
    const int g = a / G;
    // every wave is done with the LDS stages of the previous item before the first requests of this one
    __builtin_amdgcn_s_barrier();
    const int before = rec[5];
    const int q0 = qb0 + wave * 32;
    const int qi = q0 + lq;
    const bool valid = qi < q_len;
    const int p = before + (valid ? qi : 0);
    // last position any query of this wave / of the block can see
    const int wave_last = before + ((q0 + 31 < q_len) ? q0 + 31 : q_len - 1);
    const bool wave_active = q0 < q_len;
    const int blk_last = before + ((qb0 + 255 < q_len) ? qb0 + 255 : q_len - 1);
    const int n_pages = blk_last / 16 + 1;
    const int n_tiles = (n_pages + 3) / 4;
    const int32_t* pt = bm.page_tables + (size_t)sq * bm.pt_stride;
    const size_t head_off = (size_t)g * 16 * D;

    f32x16_t o[DT];
#pragma unroll
    for (int u = 0; u < DT; ++u)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[u][v] = 0.f;
    float m = -INFINITY, l = 0.f;

    // DMA assignment per stage: wave w brings K rows [8w, 8w+8) (two loads of 4 rows) and V^T pieces 2w, 2w+1
    // (piece i = page i/4 of the tile, d rows [32*(i%4), +32): 1 KB contiguous in the page).  All of a wave's
    // rows and pieces lie in page w/2 of the tile, so one page-table entry per wave and tile is needed.  Lane i
    // holds the entry for tile pages_base + i (refilled every 64 tiles) and the loop picks it with a lane
    // read: no memory access, and so no wait for one, sits between the barrier and the requests.
    int pages_vec;
    auto load_pages = [&](int base) {
        int pg = (base + lane) * 4 + (wave >> 1);
        pg = pg < n_pages ? pg : n_pages - 1;
        pages_vec = pt[pg];
    };
    load_pages(0);
    auto issue = [&](int tile) {
        const uint32_t st = lds_base + (uint32_t)(tile % NS) * STAGE;
        const int page = __builtin_amdgcn_readlane(pages_vec, tile & 63);
        const size_t page_off = (size_t)page * page_elems + head_off;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = wave * 8 + i * 4 + (lane >> 4);     // token row of the tile
            const int chunk = (lane & 15) ^ (row & 15);
            const bf16_t* src = k_pool + page_off + (size_t)(row & 15) * D + chunk * 8;
            dma16a(src, st + (wave * 8 + i * 4) * 256);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int piece = wave * 2 + i;
            const bf16_t* src = v_pool + page_off + (size_t)(piece & 3) * 512 + lane * 8;
            dma16a(src, st + KBYTES + piece * 1024);
        }
    };

    // One step of the streaming softmax (base 2, scale folded into the exponent) on the 32 tokens of a
    // score accumulator: updates m and l, leaves the weights packed as the B operands of the two P V
    // products and returns the factor the accumulated output has to be multiplied by.  The reference
    // maximum m follows the true running maximum only when that has grown by more than 8 (in the exponent's
    // units): until then weights may reach 2^8 instead of 1, which fp32 sums and the 16-bit weights hold
    // without loss, the result o / l is the same, and the 64 multiplications of the output accumulator
    // are skipped in all but the first steps of a row.
    auto softmax_step = [&](f32x16_t& sc, Frag& pfA, Frag& pfB) {
        float mr = fmaxf(fmaxf(sc[0], sc[1]), sc[2]);
#pragma unroll
        for (int v = 3; v < 15; v += 2) mr = fmaxf(fmaxf(mr, sc[v]), sc[v + 1]);
        mr = fmaxf(mr, sc[15]);
        mr = max_with_other_half(mr);
        const float mx = fmaxf(m, mr * scale_log2e);
        const bool moved = mx - m > 8.0f;               // also true for the first step (m = -inf)
        const float alpha = moved ? fast_exp2(m - mx) : 1.0f;
        m = moved ? mx : m;
        float rs = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) { sc[v] = fast_exp2(fmaf(sc[v], scale_log2e, -m)); rs += sc[v]; }
        l = l * alpha + rs;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pfA.w[i] = pack_bf16x2(sc[2 * i], sc[2 * i + 1]);
            pfB.w[i] = pack_bf16x2(sc[8 + 2 * i], sc[8 + 2 * i + 1]);
        }
        // the weights are complete here, not wherever their first use is moved to
        asm volatile("" : "+v"(pfA.w[0]), "+v"(pfA.w[1]), "+v"(pfA.w[2]), "+v"(pfA.w[3]), "+v"(pfB.w[0]), "+v"(pfB.w[1]),
                          "+v"(pfB.w[2]), "+v"(pfB.w[3]));
        return alpha;
    };
    // causal mask of a score accumulator whose first token is t0
    auto mask_step = [&](f32x16_t& sc, int t0) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int tpos = t0 + 8 * (v >> 2) + 4 * g2 + (v & 3);
            sc[v] = (tpos <= p) ? sc[v] : -INFINITY;
        }
    };
    auto rescale = [&](float alpha) {
        if (__ballot(alpha != 1.0f) != 0ull) {          // the reference maximum moved for some query of the wave
#pragma unroll
            for (int u = 0; u < DT; ++u)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[u][v] *= alpha;
        }
    };

    // Start of a block: the page-table entries first (the tile requests need them), then the requests for
    // the first two tiles, then the query fragments, whose load latency the tile requests overlap.  The query
    // fragments are loads into registers, the tiles loads into LDS; the two kinds do not complete in issue
    // order with respect to each other, so the counter arithmetic of the loop (vmcnt <= 4: everything but
    // the newest tile has landed) holds only while nothing but tile loads is in flight: the loop is entered
    // with everything landed.  (The empty statements make the loaded registers inputs of something that
    // precedes, in program order, what must follow the load.)
    asm volatile("" : "+v"(pages_vec));
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __builtin_amdgcn_sched_barrier(0);
    issue(0);
    if (n_tiles > 1) issue(1);
    Frag qf[KS];
    {
        const bf16_t* qp = qkv + (size_t)(q_begin + (valid ? qi : 0)) * row_stride + (size_t)a * D + g2 * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks].q = *reinterpret_cast<const vec16*>(qp + ks * 16);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[ks].w[0]), "+v"(qf[ks].w[1]), "+v"(qf[ks].w[2]), "+v"(qf[ks].w[3]));
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __builtin_amdgcn_sched_barrier(0);
    // No tile is requested past the last one (the block would only have to wait for it at the end), so the
    // last iteration waits for everything and the others for all but the newest tile.
    for (int it = 0; it < n_tiles; ++it) {
        if (it + 1 < n_tiles) {
            __builtin_amdgcn_s_waitcnt(0x0F74);        // vmcnt <= 4: this wave's part of tile `it` has landed
        } else {
            __builtin_amdgcn_s_waitcnt(0x0F70);
            // Values behind the block's last token (left there by the page's last user, or of a page that is only repeated)
            // become zeros in this wave's part of the tile: weight 0 would not keep one that is not finite out of the sums.
            const int past = it * 64 + (wave >> 1) * 16 + 15 - blk_last;
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("" ::: "memory");
            if (past > 0) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int piece = wave * 2 + i, row = (piece & 3) * 32 + (lane >> 1);
                    vec16* at = reinterpret_cast<vec16*>(smem + (it % NS) * STAGE + KBYTES + piece * 1024 + lane * 16);
                    vec16 v = *at;
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const int t = vtok(8 * (lane & 1) + 2 * w, row);      // and the token behind it
                        v.w[w] &= (t <= 15 - past ? 0xffffu : 0u) | (t + 1 <= 15 - past ? 0xffff0000u : 0u);
                    }
                    *at = v;
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // written before the others are let on
            }
        }
        __builtin_amdgcn_s_barrier();                  // everyone's part landed; stage (it-1)%NS is free
        __builtin_amdgcn_sched_barrier(0);
        if (it + 2 < n_tiles) {
            if (((it + 2) & 63) == 0) {                // every 64 tiles; waited for here, so that no wait
                load_pages(it + 2);                    // is due where the entries are picked
                __builtin_amdgcn_s_waitcnt(0x0F70);
            }
            issue(it + 2);
        }
        if (!wave_active || it * 64 > wave_last) continue;     // nothing visible to this wave in the tile
        const uint8_t* st = smem + (it % NS) * STAGE;
        // The two halves of 32 tokens are software-pipelined so that the MFMA pipe and the vector ALU work at
        // the same time: the score product of the second half is issued next to the softmax of the first,
        // the P V product of the first half next to the softmax of the second, and every LDS fragment read
        // is issued a phase ahead of its use.  Only the last tile or two of a wave hold tokens that some of
        // its queries must not see (wave-uniform test); a half that is hidden altogether is computed and
        // masked like the rest (weights 0).
        const bool diag = it * 64 + 63 > before + q0;
        const uint8_t* kp = st + lq * 256;
        const int sw = lq & 15;                         // rows lq and 32 + lq share the swizzle
        Frag ka[KS], kb[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) ka[ks].v = *reinterpret_cast<const bf16x8_t*>(kp + (((ks * 2 + g2) ^ sw) << 4));
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kb[ks].v = *reinterpret_cast<const bf16x8_t*>(kp + 32 * 256 + (((ks * 2 + g2) ^ sw) << 4));
        f32x16_t s0, s1;
#pragma unroll
        for (int v = 0; v < 16; ++v) { s0[v] = 0.f; s1[v] = 0.f; }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) s0 = SS_MFMA_32x32x16(ka[ks].v, qf[ks].v, s0, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        const uint8_t* vp = st + KBYTES + lq * 32 + (g2 ^ ((lq >> 3) & 1)) * 16;      // halves swapped in rows 8-15 of 16 (vpos)
        Frag va[DT], vb[DT];
#pragma unroll
        for (int u = 0; u < DT; ++u) {
            va[u].v = *reinterpret_cast<const bf16x8_t*>(vp + u * 1024);
            vb[u].v = *reinterpret_cast<const bf16x8_t*>(vp + 4096 + u * 1024);
        }
        if (diag) mask_step(s0, it * 64);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) s1 = SS_MFMA_32x32x16(kb[ks].v, qf[ks].v, s1, 0, 0, 0);
        Frag pA, pB;
        float alpha = softmax_step(s0, pA, pB);
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // one MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);      // vector ALU work of the softmax
            __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);      // two exponentials
        }
        __builtin_amdgcn_sched_barrier(0);
        if (diag) mask_step(s1, it * 64 + 32);
        rescale(alpha);
        Frag vc[DT], vd[DT];
#pragma unroll
        for (int u = 0; u < DT; ++u) {
            vc[u].v = *reinterpret_cast<const bf16x8_t*>(vp + 8192 + u * 1024);
            vd[u].v = *reinterpret_cast<const bf16x8_t*>(vp + 12288 + u * 1024);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < DT; ++u) {
            o[u] = SS_MFMA_32x32x16(va[u].v, pA.v, o[u], 0, 0, 0);
            o[u] = SS_MFMA_32x32x16(vb[u].v, pB.v, o[u], 0, 0, 0);
        }
        Frag pC, pD;
        alpha = softmax_step(s1, pC, pD);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);          // the row maximum has to be there before
        __builtin_amdgcn_sched_group_barrier(0x002, 16, 0);         // the first exponential
#pragma unroll
        for (int i = 1; i < 2 * DT; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
            __builtin_amdgcn_sched_group_barrier(0x400, 3, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        rescale(alpha);
#pragma unroll
        for (int u = 0; u < DT; ++u) {
            o[u] = SS_MFMA_32x32x16(vc[u].v, pC.v, o[u], 0, 0, 0);
            o[u] = SS_MFMA_32x32x16(vd[u].v, pD.v, o[u], 0, 0, 0);
        }
    }
    l += __shfl_xor(l, 32, 64);
    if (valid) {
        const float inv = 1.0f / l;
        bf16_t* op = out + (size_t)(q_begin + qi) * ((size_t)n_q * D) + (size_t)a * D;
#pragma unroll
        for (int u = 0; u < DT; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                vec8 w;
                w.w[0] = pack_bf16x2(o[u][4 * j] * inv, o[u][4 * j + 1] * inv);
                w.w[1] = pack_bf16x2(o[u][4 * j + 2] * inv, o[u][4 * j + 3] * inv);
                *reinterpret_cast<vec8*>(op + u * 32 + 8 * j + 4 * g2) = w;
            }
    }
    }   // items
}

hipError_t attn_generic(int dt, const void* qkv, void* out, int n_q, int n_kv, const BatchMeta& bm,
                        const KvLayer& kv, const float* rope_table, hipStream_t s);

hipError_t attn_prefill(int dt, const void* qkv, void* out, int n_q, int n_kv, const BatchMeta& bm,
                        const KvLayer& kv, bool force_generic, hipStream_t s) {
    if (bm.T <= 0 || bm.n_seqs <= 0) return hipSuccess;
    if (dt != BF16 || force_generic || kv.d != 128) return attn_generic(dt, qkv, out, n_q, n_kv, bm, kv, nullptr, s);
    if (kv.page_size != 16 || n_kv <= 0 || n_q % n_kv != 0 || kv.n_heads != n_kv) return hipErrorInvalidValue;
    if (bm.n_seqs > 65535 || n_q > 65535) return hipErrorInvalidValue;
    const float sl2 = 1.4426950408889634f / sqrtf((float)kv.d);
    if (bm.max_q_len <= 64 || !bm.pf_items || bm.pf_blocks <= 0) {       // short prompts (or no work lists): per-wave operand loads, no ring to fill
        dim3 grid((bm.max_q_len + 127) / 128, n_q, bm.n_seqs);
        attn_prefill_mfma_kernel<128, 1><<<grid, 256, 0, s>>>((const bf16_t*)qkv, (bf16_t*)out, n_q, n_kv, bm,
                                                               (const bf16_t*)kv.k_pool, (const bf16_t*)kv.v_pool, sl2);
        return hipGetLastError();
    }
    constexpr int LDS = 3 * 32768;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)attn_prefill_lds_kernel<128>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    attn_prefill_lds_kernel<128><<<(unsigned)bm.pf_blocks, 512, LDS, s>>>((const bf16_t*)qkv, (bf16_t*)out, n_q, n_kv, bm,
                                                        (const bf16_t*)kv.k_pool, (const bf16_t*)kv.v_pool, sl2);
    return hipGetLastError();
}

// ======================================================================
// Decode.  One wave per (work item, kv head).  A work item is a run of pages of
// one sequence.  All G = n_q / n_kv (<= 16) query heads that share the kv head
// form the 16 query columns of v_mfma_f32_16x16x32_bf16 (unused columns are
// zero), so K and V are read from HBM once per group.  Each step covers two pages, A and B.  The rows of the two score
// products are tokens 0-7 of A and of B, and tokens 8-15 of A and of B, so that lane group g4 = l/16 holds tokens
// 4*(g4%2) + v and 8 + 4*(g4%2) + v (v = 0..3) of page A (g4 < 2) or B: the eight tokens that are one 16-byte piece of
// a row of V^T, and the eight k-slots of the group in the second product.  One 16-byte load in place of two of 8 bytes (four
// tokens of each page per group): no more than 0.2 % either way (six steps of 1024 sequences on one kv head 3175 -> 3169 us, of
// 256 sequences of the 7B shape 8075 -> 8093).  Bound by the page reads: 5.5 TB/s with 32 kv heads, 5 with one.  A third wave
// per SIMD (146 registers) changes neither.
// The new token's q, k and v come unrotated from the products.  Every wave rotates its q fragments in registers (k-step
// ks holds the partners of ks + 2 in the same lane); the one whose item has the new token's page starts its sums with the
// new token, out of registers.  The merge kernel writes its key and value into the page: that takes a launch out of the
// chain (eight chat users of the 7B shape, eight tokens through two layers 1995 -> 1932 us; six steps of 1024 sequences on one
// kv head 3161 -> 3114, of 512 on ten heads 7306 -> 7279, of 256 on 32 heads 8081 -> 8034).  Written by this kernel the value
// alone, in stores of two bytes or as whole 4 KB pieces of the page, cost 50 us a step of 256 sequences on 32 heads: writes
// between the page reads of the other waves.  It wins the launch and its gap, not kernel time (256 sequences on 32 heads, us a
// step: rotation 17.4 gone, merge 5.0 -> 20.5, this kernel 1153.9 -> 1154.0; 1024 on one head 7.1 gone, 5.0 -> 6.9, 237.8 ->
// 241.3), so it is left out where the waves are short (attn_decode_rotates).
// Partial (max, sum, O) of every item go to scratch and are merged per sequence.
// scratch layout: float [n_items][n_q][D + 4]  (O[D], running max, running sum)
// ======================================================================
// ROPE false: the new tokens are rotated and in their pages (attn_decode_rotates).
template <int D, bool ROPE>
__global__ __launch_bounds__(64) void attn_decode_mfma_kernel(const bf16_t* __restrict__ qkv, int n_q, int n_kv,
                                                              BatchMeta bm, DecodeWork wk, const float* __restrict__ rope,
                                                              const bf16_t* __restrict__ k_pool,
                                                              const bf16_t* __restrict__ v_pool,
                                                              float* __restrict__ scratch, float scale_log2e) {
    constexpr int KS = D / 32;
    constexpr int DT = D / 16;
    static_assert(D == 128, "the rotation pairs k-step ks with ks + 2");
    const int item = wk.item_order[blockIdx.x / n_kv], g = blockIdx.x % n_kv;     // the heads of an item side by side
    const int G = n_q / n_kv;
    const int sq = wk.item_seq[item];
    // an item is pages page0, page0 + stride, ... (npg of them) of its sequence: the items of a sequence interleave
    const int page0 = wk.item_page0[item], npg = wk.item_npages[item] & 0xffff;
    const int stride = (wk.item_npages[item] >> 16) > 0 ? (wk.item_npages[item] >> 16) : 1;
    const int n_old = bm.kv_before[sq];                  // cached tokens; the new one has this position
    const int n_page = ROPE ? n_old : n_old + 1;         // tokens to take from the pages
    const int lane = threadIdx.x;
    const int lq = lane & 15, g4 = lane >> 4;
    const size_t row_stride = (size_t)(n_q + 2 * n_kv) * D;

    Frag qf[KS];
    const bf16_t* tok = qkv + (size_t)bm.cu_q[sq] * row_stride;
    if (lq < G) {
        const bf16_t* qp = tok + (size_t)(g * G + lq) * D + g4 * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks].q = *reinterpret_cast<const vec16*>(qp + ks * 32);
    } else {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks].w[0] = qf[ks].w[1] = qf[ks].w[2] = qf[ks].w[3] = 0u;
    }
    // cos / sin of this lane's element pairs: k-steps ks and ks + 2 hold the two halves
    float cs[KS / 2][16];
    if constexpr (ROPE) {
        const float* rp = rope + (size_t)n_old * D + 16 * g4;             // [D / 2][2] = cos, sin of the new token's position
#pragma unroll
        for (int h = 0; h < KS / 2; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4_t v = *reinterpret_cast<const f32x4_t*>(rp + 64 * h + 4 * j);
#pragma unroll
                for (int e = 0; e < 4; ++e) cs[h][4 * j + e] = v[e];
            }
    }
    // the wave whose item has the new token's page: its key and value
    const int past0 = n_old / 16 - page0;
    const bool fresh = ROPE && past0 >= 0 && past0 % stride == 0 && past0 / stride < npg;
    Frag kf[KS];
    vec8 vn[DT];
    if (fresh) {
        const bf16_t* kn = tok + (size_t)(n_q + g) * D;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kf[ks].q = *reinterpret_cast<const vec16*>(kn + ks * 32 + g4 * 8);
#pragma unroll
        for (int t = 0; t < DT; ++t) vn[t] = *reinterpret_cast<const vec8*>(kn + (size_t)n_kv * D + t * 16 + 4 * g4);
    }
    f32x4_t o[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t) o[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;

    const int32_t* pt = bm.page_tables + (size_t)sq * bm.pt_stride + page0;
    const size_t page_elems = (size_t)n_kv * 16 * D;
    const size_t head_off = (size_t)g * 16 * D;
    // the group's tokens are half g4 & 1 of a V^T row, in rows with bit 3 of the row index set the other half (see vpos)
    const int vhalf = (g4 & 1) ^ ((lq >> 3) & 1);
    const size_t k_lane = head_off + (size_t)(lq & 7) * D + g4 * 8, v_lane = head_off + (size_t)lq * 16 + 8 * vhalf;
    // The loop is software-pipelined over page pairs: the K fragments of the next pair (8 KB per wave) are
    // requested right after the score product of this pair has consumed its own, and the V^T fragments of
    // this pair before that product, so that a wave always has 8 to 16 KB on their way instead of the 2 KB
    // the plain order (load two fragments, multiply, load the next two) keeps in flight.  Past the last
    // pair the prefetch repeats the last page (a cache hit), which keeps the loop free of a branch that
    // would make the load counter's bookkeeping conservative.
    auto pair_pages = [&](int pi, int& pgA, int& pgB) {
        const int ia = pi < npg ? pi : npg - 1, ib = pi + 1 < npg ? pi + 1 : npg - 1;
        pgA = pt[ia * stride];
        pgB = pt[ib * stride];
    };
    auto load_k = [&](int pgA, int pgB, Frag* fa, Frag* fb) {
        const bf16_t* kp = k_pool + (size_t)(lq < 8 ? pgA : pgB) * page_elems + k_lane;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            fa[ks].q = *reinterpret_cast<const vec16*>(kp + ks * 32);
            fb[ks].q = *reinterpret_cast<const vec16*>(kp + 8 * D + ks * 32);
        }
    };
    // one pair of pages: fragments ka / kb hold its K, na / nb receive the K of the next pair
    auto step = [&](auto prefetch, int pi, int pA, int pB, const Frag* ka, const Frag* kb, int nA, int nB, Frag* na, Frag* nb) {
        const bool hasB = pi + 1 < npg;
        const bf16_t* vp = v_pool + (size_t)(g4 < 2 ? pA : pB) * page_elems + v_lane;
        Frag vf[DT];
#pragma unroll
        for (int t = 0; t < DT; ++t) vf[t].q = *reinterpret_cast<const vec16*>(vp + t * 16 * 16);
        __builtin_amdgcn_sched_barrier(0);
        f32x4_t sA = {0.f, 0.f, 0.f, 0.f}, sB = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            sA = SS_MFMA_16x16x32(ka[ks].v, qf[ks].v, sA, 0, 0, 0);
            sB = SS_MFMA_16x16x32(kb[ks].v, qf[ks].v, sB, 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(prefetch)::value) load_k(nA, nB, na, nb);
        __builtin_amdgcn_sched_barrier(0);
        const int pos0 = (page0 + (pi + (g4 >> 1)) * stride) * 16 + 4 * (g4 & 1);
        const bool there = g4 < 2 || hasB;
        float mx = m;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            sA[v] = (there && pos0 + v < n_page) ? sA[v] * scale_log2e : -INFINITY;
            sB[v] = (there && pos0 + 8 + v < n_page) ? sB[v] * scale_log2e : -INFINITY;
            mx = fmaxf(mx, fmaxf(sA[v], sB[v]));
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        // the item's first page holds a visible token, or the new one came first: mx is finite
        const float alpha = fast_exp2(m - mx);
        m = mx;
        float rs = 0.f;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            sA[v] = fast_exp2(sA[v] - mx);
            sB[v] = fast_exp2(sB[v] - mx);
            rs += sA[v] + sB[v];
        }
        l = l * alpha + rs;
        // The page of the new token: its own slot and those behind it hold what the page's last user left.  Weight 0 would
        // not keep a value that is not finite out of the sums; nor one of a page that is only repeated.
        if ((page0 + (pi + 1) * stride) * 16 + 16 > n_page || !hasB) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int p = pos0 + 2 * (w & 1) + 8 * (w >> 1);
                const uint32_t keep = there ? (p < n_page ? 0xffffu : 0u) | (p + 1 < n_page ? 0xffff0000u : 0u) : 0u;
#pragma unroll
                for (int t = 0; t < DT; ++t) vf[t].w[w] &= keep;
            }
        }
        Frag pf;
        pf.w[0] = pack_bf16x2(sA[0], sA[1]);
        pf.w[1] = pack_bf16x2(sA[2], sA[3]);
        pf.w[2] = pack_bf16x2(sB[0], sB[1]);
        pf.w[3] = pack_bf16x2(sB[2], sB[3]);
#pragma unroll
        for (int t = 0; t < DT; ++t) {
#pragma unroll
            for (int v = 0; v < 4; ++v) o[t][v] *= alpha;
            o[t] = SS_MFMA_16x16x32(vf[t].v, pf.v, o[t], 0, 0, 0);
        }
    };
    // two steps per trip, the two fragment sets changing roles, so that no set is ever copied; a last
    // single pair runs without a prefetch
    int pA, pB;
    pair_pages(0, pA, pB);
    Frag k0a[KS], k0b[KS], k1a[KS], k1b[KS];
    load_k(pA, pB, k0a, k0b);
    auto rotate = [&](Frag* f) {
#pragma unroll
        for (int h = 0; h < KS / 2; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float x[4], r[4];
                unpack_bf16x2(f[h].w[j], x[0], x[1]);
                unpack_bf16x2(f[h + 2].w[j], x[2], x[3]);
#pragma unroll
                for (int e = 0; e < 2; ++e) rope_rotate(x[e], x[2 + e], cs[h][4 * j + 2 * e], cs[h][4 * j + 2 * e + 1], r[e], r[2 + e]);
                f[h].w[j] = pack_rotated(r[0], r[1]);
                f[h + 2].w[j] = pack_rotated(r[2], r[3]);
            }
    };
    if constexpr (ROPE) rotate(qf);
    // The new token is the first term of the wave that has its page, taken from registers: weight 1 at its own score.
    if (fresh) {
#pragma unroll
        for (int t = 0; t < DT; ++t) {
            float x[4];
            unpack_bf16x2(vn[t].w[0], x[0], x[1]);
            unpack_bf16x2(vn[t].w[1], x[2], x[3]);
            o[t] = f32x4_t{x[0], x[1], x[2], x[3]};
        }
        rotate(kf);
        f32x4_t sn = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) sn = SS_MFMA_16x16x32(kf[ks].v, qf[ks].v, sn, 0, 0, 0);      // every row is the new token
        m = sn[0] * scale_log2e;
        l = g4 == 0 ? 1.f : 0.f;
    }
    int pi = 0;
    for (; pi + 2 < npg; pi += 4) {
        int nA, nB;
        pair_pages(pi + 2, nA, nB);
        step(std::true_type{}, pi, pA, pB, k0a, k0b, nA, nB, k1a, k1b);
        pair_pages(pi + 4, pA, pB);
        step(std::true_type{}, pi + 2, nA, nB, k1a, k1b, pA, pB, k0a, k0b);
    }
    if (pi < npg) step(std::false_type{}, pi, pA, pB, k0a, k0b, pA, pB, k1a, k1b);
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (lq < G) {
        float* sp = scratch + ((size_t)item * n_q + (size_t)(g * G + lq)) * (D + 4);
#pragma unroll
        for (int t = 0; t < DT; ++t)
            *reinterpret_cast<f32x4_t*>(sp + t * 16 + 4 * g4) = o[t];
        if (g4 == 0) { sp[D] = m; sp[D + 1] = l; }
    }
}

// Merge of the per-item partials: D / 4 threads per (q head, sequence), HB heads per block.  Bound by latency: a
// sequence has one to a few items, so the maxima, sums and outputs of four of them are requested together.  Against two
// dependent passes over them, one item at a time: eight sequences of the 7B shape, two layers and the LM head 251.8 -> 248.4 us
// a token, 1024 sequences on one kv head 536 -> 528 us a step.
// Blocks behind the merging ones write the new tokens' keys (rotated again, the same operations as in the attention kernel)
// and values into their pages, HB kv heads each.  Blocks of their own: in front of the merge in the same blocks 1 % of a
// chat user's token slower.
template <int D, int HB>
__global__ __launch_bounds__(D / 4 * HB) void attn_decode_merge_kernel(const float* __restrict__ scratch,
                                                                       bf16_t* __restrict__ out, int n_q, int n_kv, BatchMeta bm,
                                                                       DecodeWork wk, const bf16_t* __restrict__ qkv,
                                                                       const float* __restrict__ rope, bf16_t* __restrict__ k_pool,
                                                                       bf16_t* __restrict__ v_pool) {
    const int sq = blockIdx.y, e = threadIdx.x % (D / 4) * 4;
    const int merge_blocks = (n_q + HB - 1) / HB;
    if ((int)blockIdx.x >= merge_blocks) {
        const int g = ((int)blockIdx.x - merge_blocks) * HB + threadIdx.x / (D / 4), pos = bm.kv_before[sq], slot = pos & 15;
        if (g >= n_kv) return;
        const bf16_t* kn = qkv + (size_t)bm.cu_q[sq] * ((size_t)(n_q + 2 * n_kv) * D) + (size_t)(n_q + g) * D;
        const bf16_t* vn = kn + (size_t)n_kv * D;
        const size_t page = ((size_t)bm.page_tables[(size_t)sq * bm.pt_stride + pos / 16] * n_kv + g) * 16 * D;
        const int i0 = e % (D / 2);
        const f32x4_t c0 = *reinterpret_cast<const f32x4_t*>(rope + (size_t)pos * D + 2 * i0);
        const f32x4_t c1 = *reinterpret_cast<const f32x4_t*>(rope + (size_t)pos * D + 2 * i0 + 4);
        const bool first = e < D / 2;
        const vec8 own = *reinterpret_cast<const vec8*>(kn + e), other = *reinterpret_cast<const vec8*>(kn + (first ? e + D / 2 : i0));
        const vec8 v = *reinterpret_cast<const vec8*>(vn + e);
        vec8 k;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float x[2], o[2];
            unpack_bf16x2(own.w[j], x[0], x[1]);
            unpack_bf16x2(other.w[j], o[0], o[1]);
            const f32x4_t c = j ? c1 : c0;
            k.w[j] = pack_rotated(rope_half(x[0], first ? -o[0] : o[0], c[0], c[1]), rope_half(x[1], first ? -o[1] : o[1], c[2], c[3]));
        }
        *reinterpret_cast<vec8*>(k_pool + page + slot * D + e) = k;
#pragma unroll
        for (int j = 0; j < 4; ++j) v_pool[page + (size_t)(e + j) * 16 + vpos(slot, e + j)] = (bf16_t)(v.w[j >> 1] >> (16 * (j & 1)));
        return;
    }
    const int a = blockIdx.x * HB + threadIdx.x / (D / 4);
    if (a >= n_q) return;
    const int i0 = wk.seq_item0[sq], i1 = wk.seq_item0[sq + 1];
    float M = -INFINITY, den = 0.f;
    f32x4_t num = {0.f, 0.f, 0.f, 0.f};
    for (int i = i0; i < i1; i += 4) {
        float m[4], l[4];
        f32x4_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float* sp = scratch + ((size_t)(i + u < i1 ? i + u : i1 - 1) * n_q + a) * (D + 4);
            m[u] = sp[D];
            l[u] = sp[D + 1];
            v[u] = *reinterpret_cast<const f32x4_t*>(sp + e);
        }
        float mx = M;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (i + u >= i1) {                  // repeated: weight 0, and 0 times an infinite result must not count either
                m[u] = -INFINITY;
                v[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
            mx = fmaxf(mx, m[u]);
        }
        const float ref = mx == -INFINITY ? 0.f : mx;
        const float alpha = fast_exp2(M - ref);
        M = mx;
        num *= alpha;
        den *= alpha;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float w = fast_exp2(m[u] - ref);
            num += w * v[u];
            den += w * l[u];
        }
    }
    vec8 w;
    w.w[0] = pack_bf16x2(num[0] / den, num[1] / den);
    w.w[1] = pack_bf16x2(num[2] / den, num[3] / den);
    *reinterpret_cast<vec8*>(out + (size_t)bm.cu_q[sq] * ((size_t)n_q * D) + (size_t)a * D + e) = w;
}

static bool decode_mfma(int dt, int n_q, int n_kv, int d, bool force_generic) {
    return dt == BF16 && !force_generic && d == 128 && n_kv > 0 && n_q / n_kv <= 16;
}

// The plain kernel rotates where the launch saved is worth the registers that the rotation takes (fp32 148 in place of 94 or 128):
// heads of 64 and few blocks, that is n_q * n_seqs.  Layer call with / without, 16 heads: fp32, 32 sequences of 40 tokens 27.2
// / 28.4 us, 64 37.3 / 35.1, 256 of 8 tokens 80 / 65; 16-bit, 64 of 40 25.2 / 26.8, 128 37.3 / 34.5, 512 72 / 54; the tiny fp32
// model's run of four prompts and eight tokens 494 / 522.  Heads of 128 need 256 registers and more with it: 32 heads over one, 256
// sequences of 40 tokens 165 / 64, and at 1 to 8 sequences no gain either.
// The matrix-core kernel rotates but for batches of one query head per kv head and 256 sequences and more (from where the kernel of
// its own takes several heads a block) with 4096 waves and more and about three pages a sequence, or with more than 16384 waves and
// one page: there its waves are so short that the loads of cos / sin, of the new key and value show.  Layer call with /
// without: 256 sequences of 8 / 40 / 100 tokens on 32 heads 112 / 107 us, 130.6 / 128.5, 172.5 / 178.6; 512 of 40 on 10 heads 109 /
// 106; 1024 of 24 on 40 heads 402 / 418; 64 of 40 on 32 heads 65.4 / 67.7, 128 of one page on 40 111.2 / 115.6; 512 of 40 with
// four query heads each on 8 113 either way.
bool attn_decode_rotates(int dt, int n_q, int n_kv, int d, int n_seqs, long long pages, bool force_generic) {
    if (decode_mfma(dt, n_q, n_kv, d, force_generic)) {
        const long long waves = (long long)n_seqs * n_kv;
        return n_q != n_kv || n_seqs < 256 || waves < 4096 || 2 * pages > (waves <= 16384 ? 7 : 2) * (long long)n_seqs;
    }
    return d == 64 && (long long)n_q * n_seqs <= (dt == F32 ? 512 : 1024);
}

size_t attn_decode_scratch_floats(int n_items, int n_q, int d) { return (size_t)n_items * n_q * (d + 4); }

hipError_t attn_decode(int dt, const void* qkv, void* out, int n_q, int n_kv, const BatchMeta& bm,
                       const KvLayer& kv, const DecodeWork& wk, const float* rope_table, float* scratch, bool force_generic,
                       hipStream_t s) {
    if (bm.n_seqs <= 0) return hipSuccess;
    if (n_kv <= 0 || n_q % n_kv != 0) return hipErrorInvalidValue;
    if (!decode_mfma(dt, n_q, n_kv, kv.d, force_generic)) return attn_generic(dt, qkv, out, n_q, n_kv, bm, kv, rope_table, s);
    if (kv.page_size != 16 || kv.n_heads != n_kv || !scratch || wk.n_items <= 0) return hipErrorInvalidValue;
    if (n_kv > 65535 || bm.n_seqs > 65535) return hipErrorInvalidValue;
    const float sl2 = 1.4426950408889634f / sqrtf((float)kv.d);
    if ((long long)wk.n_items * n_kv > 0x7fffffffll) return hipErrorInvalidValue;
    dim3 grid((unsigned)(wk.n_items * n_kv));
    const auto kernel = rope_table ? attn_decode_mfma_kernel<128, true> : attn_decode_mfma_kernel<128, false>;
    kernel<<<grid, 64, 0, s>>>((const bf16_t*)qkv, n_q, n_kv, bm, wk, rope_table, (const bf16_t*)kv.k_pool, (const bf16_t*)kv.v_pool,
                               scratch, sl2);
    dim3 mgrid((n_q + 7) / 8 + (rope_table ? (n_kv + 7) / 8 : 0), bm.n_seqs);
    attn_decode_merge_kernel<128, 8><<<mgrid, 256, 0, s>>>(scratch, (bf16_t*)out, n_q, n_kv, bm, wk, (const bf16_t*)qkv, rope_table,
                                                         (bf16_t*)kv.k_pool, (bf16_t*)kv.v_pool);
    return hipGetLastError();
}

}  // namespace SS_NS

// for the tests of the dispatch
#ifndef SS_HALF_F16
extern "C" bool ssk_decode_rotates(int dt, int n_q, int n_kv, int d, int n_seqs, long long pages) {
    return ssk::attn_decode_rotates(dt, n_q, n_kv, d, n_seqs, pages, false);
}
#endif

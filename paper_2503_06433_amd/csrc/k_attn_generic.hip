// Plain (non-MFMA) paged causal attention, any dtype, head_dim 64 or 128.
// Serves the fp32 configuration, and prefill and decode alike: a decode batch
// is a batch whose sequences each bring one query.
//
// One 256-thread block per (64-query tile, q head, sequence).  Four threads
// share a query row, each owning a quarter of the head dimension.  The block
// walks the sequence's pages in order; a page's K [16][D] and V^T [D][16]
// chunks are staged through LDS as floats; softmax is the streaming
// (running max / running sum) form in fp32.
//
// Slots of the last page behind the last visible token hold what an earlier owner of the page left, which may not be finite:
// their values count as zeros (weight 0 alone would not keep them out of the sums), here and in the matrix-core kernels.
#include "ss_device.h"
#include "ss_kernels.h"

namespace SS_NS {
using namespace ssk;

template <typename T, int D>
__global__ __launch_bounds__(256) void attn_generic_kernel(const T* __restrict__ qkv, T* __restrict__ out, int n_q,
                                                           int n_kv, BatchMeta bm, const T* __restrict__ k_pool,
                                                           const T* __restrict__ v_pool, float scale) {
    constexpr int PS = 16;
    constexpr int DS = D / 4;
    __shared__ float Ks[PS][D];
    __shared__ float Vs[D][PS + 1];
    const int sq = blockIdx.z, a = blockIdx.y, tile = blockIdx.x;
    const int q_begin = bm.cu_q[sq], q_len = bm.cu_q[sq + 1] - q_begin;
    if (tile * 64 >= q_len) return;
    const int before = bm.kv_before[sq];
    const int g = a / (n_q / n_kv);
    const int r = threadIdx.x >> 2, sub = threadIdx.x & 3;
    const int qi = tile * 64 + r;
    const bool valid = qi < q_len;
    const int p = before + (valid ? qi : 0);              // absolute position of this row's query
    const int last_q = (tile * 64 + 63 < q_len ? tile * 64 + 63 : q_len - 1);
    const int n_pages = (before + last_q) / PS + 1;
    const size_t row_stride = (size_t)(n_q + 2 * n_kv) * D;
    const T* qp = qkv + (size_t)(q_begin + (valid ? qi : 0)) * row_stride + (size_t)a * D + sub * DS;
    float q[DS], acc[DS];
#pragma unroll
    for (int e = 0; e < DS; ++e) { q[e] = ldf(qp + e) * scale; acc[e] = 0.f; }
    float m = -INFINITY, l = 0.f;
    const int32_t* pt = bm.page_tables + (size_t)sq * bm.pt_stride;
    const size_t page_elems = (size_t)n_kv * PS * D;
    for (int j = 0; j < n_pages; ++j) {
        const T* kp = k_pool + (size_t)pt[j] * page_elems + (size_t)g * PS * D;
        const T* vp = v_pool + (size_t)pt[j] * page_elems + (size_t)g * PS * D;
        for (int i = threadIdx.x; i < PS * D; i += 256) {
            (&Ks[0][0])[i] = ldf(kp + i);
            Vs[i / PS][i % PS] = j * PS + vtok(i % PS, i / PS) <= before + last_q ? ldf(vp + i) : 0.f;
        }
        __syncthreads();
        float s[PS];
        float mx = m;
#pragma unroll
        for (int jj = 0; jj < PS; ++jj) {
            float d = 0.f;
#pragma unroll
            for (int e = 0; e < DS; ++e) d = fmaf(q[e], Ks[jj][sub * DS + e], d);
            d += __shfl_xor(d, 1, 64);
            d += __shfl_xor(d, 2, 64);
            s[jj] = (j * PS + jj <= p) ? d : -INFINITY;
            mx = fmaxf(mx, s[jj]);
        }
        // page 0 always holds position 0, which every query sees: mx is finite
        const float alpha = __expf(m - mx);
        l *= alpha;
#pragma unroll
        for (int e = 0; e < DS; ++e) acc[e] *= alpha;
#pragma unroll
        for (int jj = 0; jj < PS; ++jj) {
            const float pj = __expf(s[jj] - mx);
            l += pj;
#pragma unroll
            for (int e = 0; e < DS; ++e) acc[e] = fmaf(pj, Vs[sub * DS + e][vpos(jj, sub * DS + e)], acc[e]);
        }
        m = mx;
        __syncthreads();
    }
    if (valid) {
        T* op = out + (size_t)(q_begin + qi) * ((size_t)n_q * D) + (size_t)a * D + sub * DS;
        const float inv = 1.0f / l;
#pragma unroll
        for (int e = 0; e < DS; ++e) stf(op + e, acc[e] * inv);
    }
}

// One query per sequence.  A block per (q head, sequence) whose four waves take every fourth page each and merge their
// partial results in LDS: the tiled kernel above puts its one query on four of 256 lanes and walks the pages one after
// the other, two barriers each.  Bound by the latency of the page loads, so a wave requests K and V of a page together.
// K: four lanes per token, a quarter of the head dimension each.  V^T: a lane owns whole rows of 16 tokens and fetches
// their weights from the lanes that hold them.  Four sequences of 32 to 40 tokens, fp32, 4 heads of 64: a run of
// eight tokens through two layers in 612 us with this kernel and 750 us with the tiled one.
//
// AHEAD: a wave's first page is requested in front of everything else and the next ones as soon as the registers are free (layer
// call, fp32, 16 heads of 64, 256 sequences of 800 tokens 449 -> 369 us; 8 heads of 128, 128 of 1600 501 -> 387).  It takes registers
// (110 in place of 94, heads of 128 159 and 127), so not where no wave has a second page (8 heads of 128, 512 sequences of 8
// tokens 113 us without and 128 with it), nor for many blocks of a 16-bit type, which wait for the vector ALU (32 heads
// over one of 128, 256 sequences of 800 tokens 248 and 325; 16 sequences of 1600 70 and 63).
// ROPE: the new tokens come as the products leave them; the kernel rotates q and k and writes the page (attn_decode_rotates).
template <typename T, int D, bool ROPE, bool AHEAD>
__global__ __launch_bounds__(256) void attn_generic_decode_kernel(const T* __restrict__ qkv, T* __restrict__ out, int n_q,
                                                                  int n_kv, BatchMeta bm, const float* __restrict__ rope,
                                                                  T* k_pool, T* v_pool, float scale) {
    constexpr int PS = 16, DS = D / 4, DR = D / 64;
    constexpr int EV = 16 / (int)sizeof(T);             // elements of a 16-byte load
    __shared__ float sm[4], sl[4], so[4][D];
    const int a = blockIdx.x, sq = blockIdx.y;
    const int q_begin = bm.cu_q[sq];
    if (bm.cu_q[sq + 1] - q_begin != 1) return;
    const int p = bm.kv_before[sq], n_pages = p / PS + 1, slot = p % PS;
    const int g = a / (n_q / n_kv);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int tok = lane >> 2, sub = lane & 3;
    float q[DS], acc[DR];
    const T* row = qkv + (size_t)q_begin * ((size_t)(n_q + 2 * n_kv) * D);
    const int32_t* pt = bm.page_tables + (size_t)sq * bm.pt_stride;
    const size_t page_elems = (size_t)n_kv * PS * D;
    vec16 kr[DS / EV], vr[DR][PS / EV];
    auto load_page = [&](int j) {
        const size_t page = (size_t)pt[j] * page_elems + (size_t)g * PS * D;
#pragma unroll
        for (int i = 0; i < DS / EV; ++i) kr[i] = *reinterpret_cast<const vec16*>(k_pool + page + tok * D + sub * DS + i * EV);
#pragma unroll
        for (int r = 0; r < DR; ++r)
#pragma unroll
            for (int i = 0; i < PS / EV; ++i) vr[r][i] = *reinterpret_cast<const vec16*>(v_pool + page + (r * 64 + lane) * PS + i * EV);
    };
    // Everything that does not depend on something loaded is requested together: a lane's quarter of the new token's q and (the
    // wave that has the new token's page) k, the quarters they are rotated with, cos / sin, the new value, the first page.
    const bool last_here = ROPE && (n_pages - 1) % 4 == wave;
    const T *qh = row + (size_t)a * D, *kh = row + (size_t)(n_q + g) * D, *vh = kh + (size_t)n_kv * D;
    vec16 q_own[DS / EV], q_other[ROPE ? DS / EV : 1], k_own[ROPE ? DS / EV : 1], k_other[ROPE ? DS / EV : 1];
    T v_new[DR];
    float cs[ROPE ? 2 * DS : 1];
#pragma unroll
    for (int i = 0; i < DS / EV; ++i) q_own[i] = *reinterpret_cast<const vec16*>(qh + sub * DS + i * EV);
    if constexpr (ROPE) {
#pragma unroll
        for (int i = 0; i < DS / EV; ++i) q_other[i] = *reinterpret_cast<const vec16*>(qh + (sub ^ 2) * DS + i * EV);
#pragma unroll
        for (int i = 0; i < DS / 2; ++i)
            unpack16<float>(*reinterpret_cast<const vec16*>(rope + (size_t)p * D + 2 * (sub & 1) * DS + 4 * i), cs + 4 * i);
        if (last_here) {
#pragma unroll
            for (int i = 0; i < DS / EV; ++i) {
                k_own[i] = *reinterpret_cast<const vec16*>(kh + sub * DS + i * EV);
                k_other[i] = *reinterpret_cast<const vec16*>(kh + (sub ^ 2) * DS + i * EV);
            }
#pragma unroll
            for (int r = 0; r < DR; ++r) v_new[r] = vh[r * 64 + lane];
        }
    }
    if (AHEAD && wave < n_pages) load_page(wave);
    if constexpr (ROPE) {
        // rotated, rounded as stored
        auto rotate = [&](const vec16* own, const vec16* other, float* f) {
#pragma unroll
            for (int i = 0; i < DS / EV; ++i) {
                float o[EV];
                unpack16<T>(own[i], f + i * EV);
                unpack16<T>(other[i], o);
#pragma unroll
                for (int e = 0; e < EV; ++e) {
                    T st;
                    stf(&st, rope_half(f[i * EV + e], sub < 2 ? -o[e] : o[e], cs[2 * (i * EV + e)], cs[2 * (i * EV + e) + 1]));
                    f[i * EV + e] = ldf(&st);
                }
            }
        };
        rotate(q_own, q_other, q);
        if (last_here) {
            float kn[DS];
            rotate(k_own, k_other, kn);
#pragma unroll
            for (int i = 0; i < DS / EV; ++i) k_own[i] = pack16<T>(kn + i * EV);
        }
    } else {
#pragma unroll
        for (int i = 0; i < DS / EV; ++i) unpack16<T>(q_own[i], q + i * EV);
    }
#pragma unroll
    for (int e = 0; e < DS; ++e) q[e] *= scale;
#pragma unroll
    for (int r = 0; r < DR; ++r) acc[r] = 0.f;
    float m = -INFINITY, l = 0.f;
    for (int j = wave; j < n_pages; j += 4) {
        if (!AHEAD) load_page(j);
        // The new token's key and value come from the products, for every head of the group; the first head's block writes
        // them into the page.
        const bool fresh = last_here && j == n_pages - 1;
        if constexpr (ROPE)
            if (fresh && tok == slot) {
#pragma unroll
                for (int i = 0; i < DS / EV; ++i) {
                    kr[i] = k_own[i];
                    if (a % (n_q / n_kv) == 0)
                        *reinterpret_cast<vec16*>(k_pool + (size_t)pt[j] * page_elems + (size_t)g * PS * D + tok * D + sub * DS + i * EV) = kr[i];
                }
            }
        float d = 0.f;
#pragma unroll
        for (int i = 0; i < DS / EV; ++i) {
            float k[EV];
            unpack16<T>(kr[i], k);
#pragma unroll
            for (int e = 0; e < EV; ++e) d = fmaf(q[i * EV + e], k[e], d);
        }
        d += __shfl_xor(d, 1, 64);
        d += __shfl_xor(d, 2, 64);
        d = (j * PS + tok <= p) ? d : -INFINITY;
        float mx = d;
#pragma unroll
        for (int o = 4; o < 64; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        mx = fmaxf(mx, m);
        const float ref = mx == -INFINITY ? 0.f : mx;     // scores of -infinity only: weights 0, not NaN, in this share
        const float alpha = __expf(m - ref), w = __expf(d - ref);
        m = mx;
        l = l * alpha + w;
#pragma unroll
        for (int r = 0; r < DR; ++r) {
            float v[PS], sum = acc[r] * alpha;
#pragma unroll
            for (int i = 0; i < PS / EV; ++i) unpack16<T>(vr[r][i], v + i * EV);
            if constexpr (ROPE)
                if (fresh) {
                    const int e = r * 64 + lane, at = vpos(slot, e);
#pragma unroll
                    for (int t = 0; t < PS; ++t) v[t] = t == at ? ldf(&v_new[r]) : v[t];
                    if (a % (n_q / n_kv) == 0) v_pool[(size_t)pt[j] * page_elems + (size_t)g * PS * D + e * PS + at] = v_new[r];
                }
            // rows lane, lane + 64: one order.  Slots of the last page that nobody may see count as zeros: fp32 ahead in a loop of its own
            // (heads of 128 159 registers, 208 with the values chosen in front of one loop: layer call of 16 sequences of 3200 tokens
            // 214 and 237 us), otherwise in front (16 heads of 64 in 16 bits, 4 sequences of 3200 70 and 84 us the other way).
            constexpr bool OWN = AHEAD && sizeof(T) == 4;
            const bool tail = j == n_pages - 1;
            if (!OWN && tail) {
#pragma unroll
                for (int t = 0; t < PS; ++t) v[t] = vtok(t, lane) <= slot ? v[t] : 0.f;
            }
            if (OWN && tail) {
#pragma unroll
                for (int t = 0; t < PS; ++t) sum = fmaf(__shfl(w, 4 * vtok(t, lane), 64), vtok(t, lane) <= slot ? v[t] : 0.f, sum);
            } else {
#pragma unroll
                for (int t = 0; t < PS; ++t) sum = fmaf(__shfl(w, 4 * vtok(t, lane), 64), v[t], sum);
            }
            acc[r] = sum;
        }
        if (AHEAD && j + 4 < n_pages) load_page(j + 4);
    }
#pragma unroll
    for (int o = 4; o < 64; o <<= 1) l += __shfl_xor(l, o, 64);
    if (lane == 0) { sm[wave] = m; sl[wave] = l; }
#pragma unroll
    for (int r = 0; r < DR; ++r) so[wave][r * 64 + lane] = acc[r];
    __syncthreads();
    if ((int)threadIdx.x < D) {
        const float M = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float w = __expf(sm[i] - M);
            num = fmaf(w, so[i][threadIdx.x], num);
            den = fmaf(w, sl[i], den);
        }
        stf(out + (size_t)q_begin * ((size_t)n_q * D) + (size_t)a * D + threadIdx.x, num / den);
    }
}

// With a rope table the new tokens come unrotated and their pages are written here: one query per sequence, heads of 64.
hipError_t attn_generic(int dt, const void* qkv, void* out, int n_q, int n_kv, const BatchMeta& bm,
                        const KvLayer& kv, const float* rope_table, hipStream_t s) {
    if (bm.T <= 0 || bm.n_seqs <= 0) return hipSuccess;
    if (kv.page_size != 16 || (kv.d != 64 && kv.d != 128) || n_kv <= 0 || n_q % n_kv != 0 || kv.n_heads != n_kv)
        return hipErrorInvalidValue;
    if (bm.n_seqs > 65535 || n_q > 65535) return hipErrorInvalidValue;
    // every sequence brings one query: the kernel made for that, whatever the number of cached tokens
    const bool one = bm.max_q_len == 1;
    if (rope_table && (!one || kv.d != 64)) return hipErrorInvalidValue;
    dim3 grid((bm.max_q_len + 63) / 64, n_q, bm.n_seqs);
    // the longest sequence has a second page for some wave; two blocks per compute unit or fewer
    const bool ahead = bm.pt_stride > 4 && (dt == F32 || (long long)n_q * bm.n_seqs <= 512);
    const float scale = 1.0f / sqrtf((float)kv.d);
#define SS_ONE(TT, DD, ROPE, AHEAD)                                                                         \
    attn_generic_decode_kernel<TT, DD, ROPE, AHEAD><<<dim3(n_q, bm.n_seqs), 256, 0, s>>>(                          \
        (const TT*)qkv, (TT*)out, n_q, n_kv, bm, rope_table, (TT*)kv.k_pool, (TT*)kv.v_pool, scale)
#define SS_GO(TT, DD)                                                                                       \
    if (one && rope_table)                                                                                  \
        SS_ONE(TT, 64, true, true);                                                                         \
    else if (one && ahead)                                                                                  \
        SS_ONE(TT, DD, false, true);                                                                        \
    else if (one)                                                                                           \
        SS_ONE(TT, DD, false, false);                                                                            \
    else                                                                                                    \
        attn_generic_kernel<TT, DD><<<grid, 256, 0, s>>>((const TT*)qkv, (TT*)out, n_q, n_kv, bm,           \
                                                         (const TT*)kv.k_pool, (const TT*)kv.v_pool, scale)
    if (dt == F32) {
        if (kv.d == 64) { SS_GO(float, 64); } else { SS_GO(float, 128); }
    } else {
        if (kv.d == 64) { SS_GO(bf16_t, 64); } else { SS_GO(bf16_t, 128); }
    }
#undef SS_GO
#undef SS_ONE
    return hipGetLastError();
}

}  // namespace SS_NS

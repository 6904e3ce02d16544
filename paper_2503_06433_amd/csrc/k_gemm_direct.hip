// GEMM for few token rows: C[M,N] = A[M,K] * Wt[N,K]^T without a block-wide LDS tile.  Serves the 16-bit types up to
// DIRECT_MAX_M16 token rows (chat-sized decode batches) and fp32.
//
// What bounds it: the weight stream (every weight is used by at most four matrix instructions), and at these
// sizes the number of launches.  So there is no LDS staging and no barrier in the K loop: a block owns NT tiles of
// 16 weight rows and all the token rows (MT tiles of 16), its W waves take the 128-byte K chunks of those rows
// in turn, each wave with DEPTH chunks on their way, and the W partial tiles meet in LDS once, at the end.
// K is therefore never cut over blocks: no partial sums in memory and no second kernel, and the epilogue
// (RMSNorm factor, SwiGLU, residual) runs on the finished sums.
//
// Operand order needs neighbouring lanes on different rows, and a load in that order takes the vector L1 64 clocks per
// kilobyte instead of 16 (four lanes of a quad on four lines): at 64 token rows that alone held the kernel to 1.4
// times its present time.  So the loads cover whole lines with neighbouring lanes, into registers (that is what
// is in flight), and every chunk passes through 2 KB of LDS that belong to the wave alone, once written and once read.
//
// The RMSNorm factor of a token row needs sum(x^2) over the whole row, and the block has the whole row passing
// through its registers anyway: one more matrix instruction per token tile multiplies the token fragment with
// itself, the diagonal of that 16 x 16 product is the 16 sums of squares (products exact, sums in fp32 like the
// statistics kernel's).  That takes the statistics kernel out of the chain.
//
// The product is formed transposed (weights as the row operand): accumulator register v of lane l is
// column 4 * (l / 16) + v of token l % 16, four consecutive output columns per lane.
#include <algorithm>

#include "ss_device.h"
#include "ss_kernels.h"

namespace SS_NS {
using namespace ssk;

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

namespace {

// the two k-steps of a 32-byte piece of both operands
template <typename T> struct DirectOp;
template <> struct DirectOp<bf16_t> {
    static constexpr int CH = 64;                            // elements of a 128-byte chunk
    static __device__ __forceinline__ f32x4_t mul(const u32x4_t* a, const u32x4_t* b, f32x4_t c) {
#pragma unroll
        for (int h = 0; h < 2; ++h) c = SS_MFMA_16x16x32(__builtin_bit_cast(half8_t, a[h]), __builtin_bit_cast(half8_t, b[h]), c, 0, 0, 0);
        return c;
    }
};
template <> struct DirectOp<float> {
    static constexpr int CH = 32;
    static __device__ __forceinline__ f32x4_t mul(const u32x4_t* a, const u32x4_t* b, f32x4_t c) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[h][e]), __uint_as_float(b[h][e]), c, 0, 0, 0);
        return c;
    }
};

// silu(g) * u.  Gate and up rows in turns (the layers that the tile kernels take as well): on the hardware's exponential
// and reciprocal, as there.  fp32, and 16-bit layers with the gate rows first: by the library's exponential and an IEEE
// division like the kernel that serves those layers beyond 64 rows, so that the gate's left tail (reciprocals below
// 2^-126, which the hardware flushes) is not lost at some row counts.
__device__ __forceinline__ float direct_swiglu(float g, float u, bool divide) {
    if (divide) return g / (1.0f + expf(-g)) * u;
    return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(g * -1.4426950408889634f)) * u;
}

template <typename T> __device__ __forceinline__ void store4(T* p, const float* o);
template <> __device__ __forceinline__ void store4<float>(float* p, const float* o) {
    *reinterpret_cast<f32x4_t*>(p) = f32x4_t{o[0], o[1], o[2], o[3]};
}
template <> __device__ __forceinline__ void store4<bf16_t>(bf16_t* p, const float* o) {
    uint2 w;
    w.x = pack_bf16x2(o[0], o[1]);
    w.y = pack_bf16x2(o[2], o[3]);
    *reinterpret_cast<uint2*>(p) = w;
}

// 16 bytes of scaled activations, rounded to nearest (pack16 tests every value for NaN: 4 us more in the head below)
template <typename T> __device__ __forceinline__ u32x4_t pack_row(const float* x);
template <> __device__ __forceinline__ u32x4_t pack_row<float>(const float* x) { return __builtin_bit_cast(u32x4_t, pack16<float>(x)); }
template <> __device__ __forceinline__ u32x4_t pack_row<bf16_t>(const float* x) {
    return u32x4_t{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7])};
}

}  // namespace

// internal kinds
constexpr int EPI_HEAD = 100;      // EPI_STORE_F32 of rows that are scaled by `gain`, column by column, on their way in
constexpr int EPI_UPLOAD = 101;    // EPI_STORE that takes a batch's metadata along

// EPI_HEAD: final norm and LM head in one launch.  The rows meet their gains in registers, in the order they are loaded in, and
// are rounded once to the storage type like the separate norm's result, but before the row's factor instead of behind it; the
// sums of squares come from the unscaled values there (a row's 128-byte chunk lies in eight neighbouring lanes).  Eight
// rows, 2048 x 4096: norm kernel and product apart 12.7 us, together 7.6.
// 32-bit rows: the factor meets the finished sum, one rounding more that a whole row shares, so it is worked out in 64 bits:
// error against 64 bits (256 columns, 64 rows) 1.299e-7 apart, 1.304e-7 together with a 32-bit factor, 1.275e-7 with this one.
//
// SwiGLU: a tile is 8 gate rows and the 8 up rows that belong to them, so a block of NT tiles has 8 NT output columns.
// Gate rows come in blocks of gate_blk, each followed by its up rows (gate_blk = N / 2: all gate rows first).
template <typename T, int MT, int NT, int W, int DEPTH, int EPI>
__global__ __launch_bounds__(64 * W) void gemm_direct_kernel(const T* __restrict__ A, int lda, const T* __restrict__ Wt,
                                                             void* __restrict__ Cv, int ldc, const T* __restrict__ R,
                                                             int M, int N, int K, int gate_blk, int divide,
                                                             float norm_eps, const T* __restrict__ gain, int vec_ok, int up_blocks,
                                                             const vec16* __restrict__ up_src, vec16* __restrict__ up_dst, int64_t up_n) {
    constexpr int CH = DirectOp<T>::CH;
    constexpr int EV = VecOf<T>::N;
    constexpr bool SWI = EPI == EPI_SWIGLU, HEAD = EPI == EPI_HEAD;
    constexpr int TO = SWI ? 8 : 16;                                         // output columns of a tile
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    f32x4_t* red = reinterpret_cast<f32x4_t*>(smem);                         // [W][NT * MT][64]
    float* sq = reinterpret_cast<float*>(smem + (size_t)W * NT * MT * 1024);     // [W][MT * 16]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    // The QKV projection of a new batch: the first blocks of the first row of blocks take its metadata along (UploadJob).  A
    // kernel of its own: the test alone, in front of the first loads, costs every launch 0.2 to 0.5 us.
    int bx = blockIdx.x;
    if constexpr (EPI == EPI_UPLOAD) {
        if (bx < up_blocks) {
            if (blockIdx.y == 0) upload_pieces(up_src, up_dst, up_n, (int64_t)bx * (64 * W) + threadIdx.x, (int64_t)up_blocks * (64 * W));
            return;
        }
        bx -= up_blocks;
    }
    const int m0 = blockIdx.y * (16 * MT);
    const int n_out = SWI ? N / 2 : N;
    const int o0 = bx * (TO * NT);                                           // first output column of the block
    const bool norm = norm_eps >= 0.f;

    // Loads cover whole 128-byte lines with neighbouring lanes: load h of a tile brings rows 8h .. 8h + 7, lane l row
    // 8h + l / 8, piece l % 8 (rows beyond the matrix: the last one, never stored).
    const int sr = lane >> 3, sp = lane & 7;
    const T* wp[NT][2];
    const T* xp[MT][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int r16 = 8 * h + sr;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            int row;
            if (SWI) {
                int col = o0 + 8 * j + (r16 & 7);
                col = col < n_out ? col : n_out - 1;
                row = (col / gate_blk) * (2 * gate_blk) + col % gate_blk + (r16 >> 3) * gate_blk;
            } else {
                row = o0 + 16 * j + r16;
                row = row < N ? row : N - 1;
            }
            wp[j][h] = Wt + (size_t)row * K;
        }
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            int row = m0 + 16 * i + r16;
            row = row < M ? row : M - 1;
            xp[i][h] = A + (size_t)row * lda;
        }
    }
    // this wave's transposer: one 2 KB image of a 16-row chunk per tile, 16-byte pieces XOR-swizzled with the row
    uint8_t* tr = smem + (size_t)wave * ((NT + MT) * 2048);
    int st_off[2], ld_off[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int r = 8 * h + sr;
        st_off[h] = r * 128 + ((sp ^ ((r >> 1) & 7)) << 4);
        ld_off[h] = lr * 128 + (((4 * h + lg) ^ ((lr >> 1) & 7)) << 4);
    }
    f32x4_t acc[NT][MT], gram[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        gram[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[j][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }

    // The residual's values are requested in front of the weights where a thread has at most one piece of the output: behind the
    // sums they would be one more memory latency (8 rows 4096 x 11008 21.5 -> 21.0 us, 5120 x 1280 5.6 -> 5.2, 32 rows 27.4 -> 26.7 and
    // 6.1 -> 5.8; 48 and 64 rows 0 to 2 % slower, so not there).
    constexpr int LO = SWI ? 32 : 64;                                        // four-column pieces of an output tile
    constexpr bool EARLY = EPI == EPI_RESIDUAL && MT <= 2 && NT * MT * LO <= 64 * W;
    float early[4] = {0.f, 0.f, 0.f, 0.f};
    if constexpr (EARLY) {
        const int l = threadIdx.x % LO, t = threadIdx.x / LO, tok = m0 + 16 * (t % MT) + (l & 15), col = o0 + TO * (t / MT) + 4 * (l >> 4);
        if (t < NT * MT && tok < M)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < n_out) early[e] = ldf(R + (size_t)tok * ldc + col + e);
    }
    // chunks of this wave: wave, wave + W, ...; the pieces of the last one that lie beyond K count as zeros
    const int nch = (K + CH - 1) / CH;
    struct Buf { u32x4_t w[NT][2], x[MT][2], g[HEAD ? 1 : 0]; } buf[DEPTH];
    float xx[HEAD ? MT : 1][2];
    if constexpr (HEAD)
#pragma unroll
        for (int i = 0; i < MT; ++i) xx[i][0] = xx[i][1] = 0.f;
    auto load_full = [&](int d, int c) {
        const size_t k0 = (size_t)c * CH + sp * EV;
        if constexpr (HEAD) buf[d].g[0] = *reinterpret_cast<const u32x4_t*>(gain + k0);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int j = 0; j < NT; ++j) buf[d].w[j][h] = *reinterpret_cast<const u32x4_t*>(wp[j][h] + k0);
#pragma unroll
            for (int i = 0; i < MT; ++i) buf[d].x[i][h] = *reinterpret_cast<const u32x4_t*>(xp[i][h] + k0);
        }
    };
    auto load = [&](int d, int c) {
        const u32x4_t z = {0u, 0u, 0u, 0u};
        const bool in = (long long)c * CH + sp * EV < K;
        const size_t k0 = in ? (size_t)c * CH + sp * EV : 0;                 // some piece of the row, dropped below
        if constexpr (HEAD) {
            const u32x4_t v = *reinterpret_cast<const u32x4_t*>(gain + k0);
            buf[d].g[0] = in ? v : z;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const u32x4_t v = *reinterpret_cast<const u32x4_t*>(wp[j][h] + k0);
                buf[d].w[j][h] = in ? v : z;
            }
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const u32x4_t v = *reinterpret_cast<const u32x4_t*>(xp[i][h] + k0);
                buf[d].x[i][h] = in ? v : z;
            }
        }
    };
    // through the transposer into operand order (a wave's LDS operations execute in order: no barrier)
    auto multiply = [&](int d) {
        if constexpr (HEAD) {
            float g[EV];
            unpack16<T>(__builtin_bit_cast(vec16, buf[d].g[0]), g);
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (m0 + 16 * i + 8 * h >= M) continue;                  // repeated rows
                    float x[EV];
                    unpack16<T>(__builtin_bit_cast(vec16, buf[d].x[i][h]), x);
#pragma unroll
                    for (int e = 0; e < EV; ++e) {
                        xx[i][h] = fmaf(x[e], x[e], xx[i][h]);
                        x[e] *= g[e];
                    }
                    buf[d].x[i][h] = pack_row<T>(x);
                }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int j = 0; j < NT; ++j) *reinterpret_cast<u32x4_t*>(tr + j * 2048 + st_off[h]) = buf[d].w[j][h];
#pragma unroll
            for (int i = 0; i < MT; ++i) *reinterpret_cast<u32x4_t*>(tr + (NT + i) * 2048 + st_off[h]) = buf[d].x[i][h];
        }
        u32x4_t wf[NT][2], xf[MT][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int j = 0; j < NT; ++j) wf[j][h] = *reinterpret_cast<const u32x4_t*>(tr + j * 2048 + ld_off[h]);
#pragma unroll
            for (int i = 0; i < MT; ++i) xf[i][h] = *reinterpret_cast<const u32x4_t*>(tr + (NT + i) * 2048 + ld_off[h]);
        }
#pragma unroll
        for (int i = 0; i < MT; ++i) {
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[j][i] = DirectOp<T>::mul(wf[j], xf[i], acc[j][i]);
            if (!HEAD && norm) gram[i] = DirectOp<T>::mul(xf[i], xf[i], gram[i]);
        }
    };
    // whole rounds of DEPTH chunks that lie inside K run a round ahead without a test; what is left (fewer than DEPTH
    // whole chunks, and the one that K cuts) is loaded behind the last of them
    const int whole = K / CH;
    const int full = (whole > wave ? (whole - wave + W - 1) / W : 0) / DEPTH;
    int c = wave;
    // (the zeros of a cut chunk are chosen behind its loads, that is by waiting for them: only where a chunk is cut.  fp32 of
    // more than 16 rows, whose many waves fill that wait, is faster without the second kind of load: the MLP of a 1024-wide
    // layer at 2048 rows 507.1 -> 503.6 us, 32 to 128 rows the same)
    auto load_rest = [&](int d, int at) {
        if (!(sizeof(T) == 4 && MT == 2) && at < whole) load_full(d, at);
        else if (at < nch) load(d, at);
    };
    if (full > 0) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) load_full(d, c + d * W);
        for (int r = 1; r < full; ++r) {
            c += DEPTH * W;
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                multiply(d);
                load_full(d, c + d * W);
            }
        }
        c += DEPTH * W;
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            multiply(d);
            load_rest(d, c + d * W);
        }
    } else {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) load_rest(d, c + d * W);
    }
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        if (c + d * W < nch) multiply(d);
    // ---- the W partial tiles meet (in the LDS of the transposers)
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < MT; ++i) red[(wave * (NT * MT) + j * MT + i) * 64 + lane] = acc[j][i];
    if constexpr (HEAD) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float v = xx[i][h];
#pragma unroll
                for (int o = 1; o < 8; o <<= 1) v += __shfl_xor(v, o, 64);
                if (sp == 0) sq[wave * (MT * 16) + i * 16 + 8 * h + sr] = v;
            }
    } else if (norm) {
        const int v = lr - 4 * lg;                                           // register that holds the diagonal
#pragma unroll
        for (int i = 0; i < MT; ++i)
            if (v >= 0 && v < 4) sq[wave * (MT * 16) + i * 16 + lr] = v == 0 ? gram[i][0] : v == 1 ? gram[i][1] : v == 2 ? gram[i][2] : gram[i][3];
    }
    __syncthreads();
    for (int p = threadIdx.x; p < NT * MT * LO; p += 64 * W) {
        const int l = p % LO, t = p / LO, i = t % MT, j = t / MT;
        const int tok = m0 + 16 * i + (l & 15), col = o0 + TO * j + 4 * (l >> 4);
        if (tok >= M || col >= n_out) continue;
        // Sixteen waves have 128 registers: not all the partial sums of gate and up at once, which would spill (2752 rows of weights x 4096
        // at 8 token rows 7.8 -> 7.3 us, 3456 x 5120 at 12 10.0 -> 9.3, 5504 x 4096 at 16 12.1 -> 11.8).
        constexpr int AT_ONCE = SWI && W > 8 ? 5 : W;
        auto sum = [&](int ll) {
            f32x4_t s = red[(j * MT + i) * 64 + ll];
#pragma unroll AT_ONCE
            for (int w = 1; w < W; ++w) s += red[(w * (NT * MT) + j * MT + i) * 64 + ll];
            return s;
        };
        float rs = 1.0f;
        if (norm) {
            float ss = 0.f;
#pragma unroll
            for (int w = 0; w < W; ++w) ss += sq[w * (MT * 16) + i * 16 + (l & 15)];
            if constexpr (HEAD && sizeof(T) == 4) rs = (float)(1.0 / sqrt((double)ss / K + norm_eps));
            else rs = 1.0f / sqrtf(ss / (float)K + norm_eps);
        }
        float o[4];
        const f32x4_t s = sum(l);
        if (SWI) {
            const f32x4_t u = sum(l + 32);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = direct_swiglu(s[e] * rs, u[e] * rs, sizeof(T) == 4 || divide);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = s[e] * rs;
        }
        const size_t off = (size_t)tok * ldc + col;
        const int cols = n_out - col < 4 ? n_out - col : 4;
        if constexpr (EARLY) {
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] += early[e];
        } else if (EPI == EPI_RESIDUAL) {
            for (int e = 0; e < cols; ++e) o[e] += ldf(R + off + e);
        }
        if (EPI == EPI_STORE_F32 || HEAD) {
            float* C = reinterpret_cast<float*>(Cv);
            if (vec_ok && cols == 4) store4<float>(C + off, o);
            else for (int e = 0; e < cols; ++e) C[off + e] = o[e];
        } else {
            T* C = reinterpret_cast<T*>(Cv);
            if (vec_ok && cols == 4) store4<T>(C + off, o);
            else for (int e = 0; e < cols; ++e) stf(C + off + e, o[e]);
        }
    }
}

template <typename T, int MT, int NT, int W, int DEPTH>
static hipError_t launch_direct(const void* A, int lda, const void* Wt, void* C, int ldc, const void* R, int M, int N, int K,
                                int epi, int gate_blk, int divide, float norm_eps, const void* gain, const UploadJob& job, hipStream_t s) {
    const int n_out = epi == EPI_SWIGLU ? N / 2 : N, per = (epi == EPI_SWIGLU ? 8 : 16) * NT;
    // four pieces a thread: the batches of few rows bring a few kilobytes, at most some hundred
    const int up = (int)std::min<int64_t>((job.n16 + 256 * W - 1) / (256 * W), 64);
    const dim3 grid((unsigned)((n_out + per - 1) / per + up), (unsigned)((M + 16 * MT - 1) / (16 * MT)));
    if (grid.y > 65535) return hipErrorInvalidValue;
    constexpr size_t LDS_TR = (size_t)W * (NT + MT) * 2048, LDS_RED = (size_t)W * NT * MT * 1024 + (size_t)W * MT * 64;
    constexpr size_t LDS = LDS_TR > LDS_RED ? LDS_TR : LDS_RED;
    const size_t out_es = epi == EPI_STORE_F32 ? 4 : sizeof(T);
    const int vec_ok = ldc % 4 == 0 && ((uintptr_t)C & (4 * out_es - 1)) == 0;
    const T* a = (const T*)A;
    const T* w = (const T*)Wt;
    const T* r = (const T*)R;
#define SS_GO(E)                                                                                                 \
    {                                                                                                           \
        auto kfn = gemm_direct_kernel<T, MT, NT, W, DEPTH, E>;                                                  \
        if constexpr (LDS > 65536) {                                                                            \
            static bool attr_set = false;                                                                       \
            if (!attr_set) {                                                                                    \
                hipError_t e = hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS); \
                if (e != hipSuccess) return e;                                                                  \
                attr_set = true;                                                                                \
            }                                                                                                   \
        }                                                                                                       \
        kfn<<<grid, 64 * W, LDS, s>>>(a, lda, w, C, ldc, r, M, N, K, gate_blk, divide, norm_eps, (const T*)gain, vec_ok, up, (const vec16*)job.src, \
                                      (vec16*)job.dst, job.n16);                                               \
    }
    if constexpr (NT == 2 && W == 16) {                                      // pick_direct: SwiGLU only
        if (epi != EPI_SWIGLU) return hipErrorInvalidValue;
        SS_GO(EPI_SWIGLU)
    } else {
        switch (epi) {
            case EPI_STORE:
                if (up) SS_GO(EPI_UPLOAD) else SS_GO(EPI_STORE)
                break;
            case EPI_RESIDUAL:
                if (!R) return hipErrorInvalidValue;
                SS_GO(EPI_RESIDUAL) break;
            case EPI_STORE_F32:
                if (!gain) {
                    SS_GO(EPI_STORE_F32)
                } else {
#ifdef SS_HALF_F16
                    return hipErrorInvalidValue;                             // head_norms_itself: half keeps the norm apart
#else
                    SS_GO(EPI_HEAD)
#endif
                }
                break;
            case EPI_SWIGLU: SS_GO(EPI_SWIGLU) break;
            default: return hipErrorInvalidValue;
        }
    }
#undef SS_GO
    return hipGetLastError();
}

// Which products come here.  16-bit types: up to 64 token rows.  Measured against the 128 x 128 tile kernel with its
// statistics, split-K and reduce launches, on the projections of the 7B layer and of the 13B / 70B shards: 1 row
// 1.5-2.9 times, 32 rows 1.3-2.5 times, 64 rows up to 2.3 times as fast (QKV 12288 x 4096: 31.7 -> 18.9 us at 1 row =
// 5.3 TB/s of weights, 33.1 -> 21.5 at 32, 37.1 -> 24.9 at 64; down 4096 x 11008: 41.5 -> 21.8, 43.7 -> 28.8,
// 45.1 -> 37.2).  Not where the tile kernel or that one is faster:
//  - more than 16 rows of an output wider than 12288, that is of more blocks of three tiles than compute units: the second
//    round of blocks reads all token rows again (here / tile kernel with its statistics, 64 rows: 13824 x 5120 54 / 39 us,
//    27648 x 5120 84 / 59, 57344 x 8192 203 / 168; 17 rows: 37.8 / 31.2, 59.9 / 53.5, 174 / 169; up to 16 rows 22016 x 4096
//    35.1 / 36.1);
//  - more than 48 rows of a contraction of 12800 and more, more than 32 where the blocks do not fill the chip either: the
//    chunks of a wave, one behind the other, outweigh the second launch of split K (here / split K: 8192 x 28672
//    at 48 rows 107 / 112, at 64 122 / 113; 5120 x 13824 in 160 blocks at 32 rows 40.6 / 42.3, at 48 47.6 / 43, at 64 55 / 45;
//    4096 x 11008 at 64 rows 38 / 45).
// Both only where those kernels take the product (rows of whole 16-byte pieces, K in whole slices).  An output of other rows
// (an odd vocabulary) has the register-staged kernel beside it, which is faster than three rounds of blocks and more:
// here / there, 64 rows 20001 x 4096 45 / 59 us, 32001 x 1024 25 / 20, 32001 x 4096 67 / 66, 50257 x 4096 112 / 94; 48 rows 32001 x 1024
// 22 / 20, 32001 x 4096 61 / 65; 24 rows 32001 x 1024 18 / 19, 50257 x 768 24 / 20; 16 rows 50257 x 768 18 / 20.
// fp32: every aligned shape.  Against the 64 x 64 FMA kernel, 256-wide layer of 4 rows: QKV 28.1 ->
// 3.8 us, down (K = 688) 60.4 -> 4.0; 4096 x 4096 at 64 rows 469 -> 42 us, at 2048 rows 1803 -> 911 us.
constexpr int DIRECT_MAX_M16 = 64;

bool gemm_direct_takes(int dt, const void* A, const void* Wt, int M, int N, int K, int lda, int epi) {
    const int ev = dt == F32 ? 4 : 8;
    if (M <= 0 || N <= 0 || K <= 0 || K % ev != 0 || lda % ev != 0) return false;
    if (((uintptr_t)A & 15) != 0 || ((uintptr_t)Wt & 15) != 0) return false;
    if ((epi == EPI_SWIGLU && N % 64 != 0) || (epi == EPI_SWIGLU_HALVES && N % 2 != 0)) return false;
    if (dt == F32) return M <= 65535 * 16;
    if (M > DIRECT_MAX_M16) return false;
    if (K % 64 == 0 && N % 8 == 0 && epi != EPI_SWIGLU_HALVES) {
        if (M > 16 && N > 48 * 256) return false;
        const int blocks = N <= 4096 ? N / 16 : N <= 8192 ? N / 32 : N / 48;
        if (M > (blocks >= 224 ? 48 : 32) && K >= 12800 && epi != EPI_STORE_F32) return false;
    } else if (K % 64 == 0 && epi != EPI_SWIGLU_HALVES) {
        if (M > (N > 48 * 1024 ? 16 : N > 48 * 512 ? (K <= 2048 ? 32 : 48) : DIRECT_MAX_M16)) return false;
    }
    return true;
}

// NT (tiles of weight rows per block): more tiles mean fewer times that the token rows are read (every block reads
// them all), fewer tiles more blocks.  The line is where the blocks still fill the 256 compute units: up to 256 tiles
// one per block, up to 512 two, beyond that three (gate/up 22016 x 4096 at 16 rows, blocks of 1 / 2 / 3 / 6 tiles:
// 36.0 / 44 / 34.6 / 36.0 us; QKV 12288 x 4096 at 64 rows: 53 / 37 / 24.9 us).  A chunk is 2 (NT + MT) KB, so with DEPTH 2 a wave
// has 8 to 24 KB on their way (eight waves a block); the widest blocks keep one chunk, 8 to 14 KB, as two would spill.
// Up to 16 rows (16-bit) and K of 2048 and more:
//  - 129 to 256 tiles, a block for each: sixteen waves (4096 x 4096 at 8 / 16 rows 9.0 / 9.5 -> 8.5 / 8.9 us, 4096 x 11008 22.6 / 23.4
//    -> 21.4 / 22.5; 80 tiles, 1280 x 8192 10.5 -> 10.8, stay with eight);
//  - up to 8 rows one tile and four chunks on their way per wave, whatever the width (22016 x 4096 33.0 us, 34.8 by the rule
//    above, 12288 x 4096 19.4 and 21.4), but two tiles for 257 to 384 of them with K of 8192 and more, where some units would
//    have a second long block (5120 x 13824 36.1 -> 30.6; whole MLPs of 8 rows with one / two: 4112 x 11008 71.3 / 66.7, 4160 x 13824
//    73.5 / 68.9, 4608 x 11008 69.9 / 66.3, 4864 x 20480 118.7 / 115.6, 5888 x 13824 97.0 / 92.1, 6144 x 8192 62.7 / 62.0; not 5504 x
//    4096, 12.4 and 13.8, nor 7168 x 8192, 25.6 and 28.4);
//  - 9 to 16 rows, SwiGLU over 257 to 512 tiles: sixteen waves (7168 x 8192 28.4 -> 25.4, 5504 x 4096 13.8 -> 12.7; without SwiGLU 5120 x
//    13824 33.3 -> 33.8, 8192 x 3584 12.9 -> 13.1);
//  - 9 to 16 rows, wider: four tiles where their rounds of blocks are fuller than with three (14336 x 8192 59.5 -> 47.2, 27648 x
//    5120 58.1 -> 53.4; 22016 x 4096 stays at three, 35.2, 12288 x 4096 as well, 21.3 and 21.5).  Over 62 such outputs of K 2048
//    to 8192 3 to 23 % less at 12800 to 64000 columns (4096 x 32000, 2 to 3 % more, and 8192 x 64000 but for); a thirtieth
//    fuller is not enough (128256 x 4096 188.0 and 194.6).
// Shorter: 50257 x 768 one tile 27 us, by the rule above 18; 32001 x 1024 21 and 14.
template <typename T, int MT>
static hipError_t pick_direct(const void* A, int lda, const void* Wt, void* C, int ldc, const void* R, int M, int N, int K,
                              int epi, int gate_blk, int divide, float norm_eps, const void* gain, const UploadJob& job, hipStream_t s) {
    const long long tiles = (long long)((N + 15) / 16) * ((M + 16 * MT - 1) / (16 * MT));
#define SS_GO(NT, W, D) return launch_direct<T, MT, NT, W, D>(A, lda, Wt, C, ldc, R, M, N, K, epi, gate_blk, divide, norm_eps, gain, job, s)
    if constexpr (MT == 1 && sizeof(T) == 2) {
        if (K >= 2048) {
            if (tiles > 128 && tiles <= 256) SS_GO(1, 16, 2);
            if (M <= 8 && tiles > 256 && tiles <= 384 && K >= 8192) SS_GO(2, 8, 2);
            if (M <= 8) SS_GO(1, 8, 4);
            if (tiles > 256 && tiles <= 512 && epi == EPI_SWIGLU) SS_GO(2, 16, 2);
            if (tiles > 512) {      // three or four tiles a block: four if their rounds of blocks are a twentieth fuller
                const long long b3 = (tiles + 2) / 3, b4 = (tiles + 3) / 4;
                if (20 * b4 * ((b3 + 255) / 256) > 21 * b3 * ((b4 + 255) / 256)) SS_GO(4, 8, 2);
            }
        }
    }
    if (tiles <= 256) SS_GO(1, 8, 2);
    if (tiles <= 512) SS_GO(2, 8, 2);
    SS_GO(3, 8, 1);
#undef SS_GO
}

hipError_t gemm_direct(int dt, const void* A, int lda, const void* Wt, void* C, int ldc, const void* R, int M, int N, int K,
                       int epi, float norm_eps, const void* gain, const UploadJob& job, hipStream_t s) {
    if (!gemm_direct_takes(dt, A, Wt, M, N, K, lda, epi)) return hipErrorInvalidValue;
    if (job.n16 < 0 || (job.n16 > 0 && epi != EPI_STORE) || (((uintptr_t)job.src | (uintptr_t)job.dst) & 15) != 0) return hipErrorInvalidValue;
    if (gain && (epi != EPI_STORE_F32 || norm_eps < 0.f || ((uintptr_t)gain & 15) != 0)) return hipErrorInvalidValue;
    const int gate_blk = epi == EPI_SWIGLU ? 32 : N / 2;
    const int divide = epi == EPI_SWIGLU_HALVES;
    if (divide) epi = EPI_SWIGLU;
#define SS_GO(TT, MT) return pick_direct<TT, MT>(A, lda, Wt, C, ldc, R, M, N, K, epi, gate_blk, divide, norm_eps, gain, job, s)
#ifndef SS_HALF_F16          // fp32 is the same code in both builds of this file: only the first has it
    if (dt == F32) {
        if (M <= 16) SS_GO(float, 1);
        SS_GO(float, 2);
    }
#else
    if (dt == F32) return hipErrorInvalidValue;
#endif
    if (M <= 16) SS_GO(bf16_t, 1);
    if (M <= 32) SS_GO(bf16_t, 2);
    if (M <= 48) SS_GO(bf16_t, 3);
    SS_GO(bf16_t, 4);
#undef SS_GO
}

}  // namespace SS_NS

// GEMM for outputs of too few 256 x 256 tiles for the persistent kernel (decode batches, short prompts, chunks):
// C[M,N] = A[M,K] * Wt[N,K]^T, 16-bit types.
//
// At these sizes neither the weight stream nor the matrix pipes bound the launch by themselves; a tile for every compute
// unit does.  So the tile is chosen per shape, such that one round of tiles just covers the chip, K is cut over
// blocks only for long contractions of narrow outputs (gemm_tile_split_estimate), and inside a block the waves are made as large as registers
// allow and doubled by splitting the k-steps of every stage between two or four groups of waves: the fragment reads from
// LDS depend on the wave tile, the latencies are covered by the number of waves.  The groups' sums meet in LDS once.
//
// Operands go global -> LDS by direct loads into a ring of up to nine stages, counted by hand; one barrier per stage.  The
// fragments of the next k-step are read while the matrix instructions of the current one run.
//
// What bounds it (parts of the loop switched off, 128 x 96 tiles, 256 x 12288 x 4096): whole 40.5 us, loads and
// barriers alone 38.5, the same with all weights found in the L2 21.9, matrix instructions and fragment reads alone 29.6.
// It waits for lines: a compute unit takes in about 26 bytes of weights per nanosecond next to the token lines, at 3 as at 5
// stages; the two streams add up, and no layout, stride or K phase of the weights changes that by more than some per cent.  Touching weight lines ahead (one dword per line, by turns of the blocks that share
// them, singly or in bursts, 6 to 24 stages ahead) made it 5-30 % slower.
//
// Measured against the 128 x 128 register-staged kernel or the persistent kernel with split K and their reduce launch:
// 256 rows: 12288 x 4096 54 -> 39 us, gate/up 22016 x 4096 74 -> 57, 4096 x 11008 54 with its reduce -> 41 (four ranges), 4096 x 4096
// 27 -> 22; 333 rows: 73 -> 47, 132 -> 72, 79 -> 45, 34 -> 27; 864 rows: 12288 x 4096 160 -> 97, 4096 x 4096 61 -> 42.
#include <type_traits>

#include "ss_device.h"
#include "ss_kernels.h"

namespace SS_NS {
using namespace ssk;

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

// silu(g) * u on the hardware's exponential and reciprocal (the result is rounded to 16 bits)
__device__ __forceinline__ float tile_swiglu(float g, float u) {
    return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(g * -1.4426950408889634f)) * u;
}

__device__ __forceinline__ void tile_dma16(uint32_t off, const void* base, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds_addr) : "memory");
}

// own loads but the newest V have landed, own LDS reads are done, and so have and are everyone else's
template <int V> __device__ __forceinline__ void tile_wait_barrier() {
    static_assert(V >= 0 && V <= 63, "vmcnt");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(V) : "memory");
}

// Geometry of one instance: BM x BN output tile, WM x WN waves over it, KG groups of such waves that split every stage's
// k-steps among themselves, stages of SL slices of 64 elements, NS stages in the ring.
template <int BM_, int BN_, int WM_, int WN_, int KG_, int SL_, int NS_> struct TileCfg {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, KG = KG_, SL = SL_, NS = NS_;
    static constexpr int NW = WM * WN * KG, TM = BM / WM / 16, TN = BN / WN / 16;
    static constexpr int SUB = (BM + BN) * 128, STAGE = SL * SUB, P = 2 * SL / KG;
    static constexpr int NL = (BM + BN) / 8 * SL, L = NL / NW, REM = NL % NW, LMAX = L + (REM ? 1 : 0);
    static constexpr int PITCH = BN + 4;
    static constexpr int LDS_MAX = 160 * 1024;
    static constexpr int passes() {
        int p = 1;
        while (TM % p != 0 || (long long)KG * (BM / p) * PITCH * 4 > LDS_MAX) ++p;
        return p;
    }
    static constexpr int PASSES = passes(), RP = BM / PASSES;
    static constexpr int LDS = NS * STAGE > KG * RP * PITCH * 4 ? NS * STAGE : KG * RP * PITCH * 4;
    static_assert(BM % (16 * WM) == 0 && BN % (16 * WN) == 0 && BN % 32 == 0 && (2 * SL) % KG == 0 && NS >= 2, "geometry");
    static_assert(LDS <= LDS_MAX && (NS - 1) * LMAX <= 63, "ring");
};

}  // namespace

template <class G>
__global__ __launch_bounds__(64 * G::NW) void gemm_tile_kernel(const bf16_t* __restrict__ A, int lda,
                                                               const bf16_t* __restrict__ Wt, void* __restrict__ Cv, int ldc,
                                                               const bf16_t* __restrict__ R, int M, int N, int K, int epi,
                                                               int tiles_m, int n_tiles, int ksplit, int per_xcd,
                                                               const float* __restrict__ RS) {
    constexpr int BM = G::BM, BN = G::BN, TM = G::TM, TN = G::TN, P = G::P, NS = G::NS;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    // K in ranges: the tiles of one range after those of another, so that an XCD has one or two ranges of many tiles and not
    // all ranges of a few; a range's fp32 sums go to its plane of C, [ksplit][M][N]
    int logical = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || logical >= n_tiles * ksplit) return;
    const int range = logical / n_tiles;
    logical -= range * n_tiles;
    const int tile_m = logical % tiles_m, tile_n = logical / tiles_m;
    const bool swi = epi == EPI_SWIGLU;
    const int m0 = tile_m * BM, n0 = tile_n * BN, oc0 = tile_n * (BN / 2);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wg = wave / (G::WM * G::WN), wi = wave % (G::WM * G::WN), wm = wi / G::WN, wn = wi % G::WN;
    const int l16 = lane & 15, l4 = lane >> 4;
    const uint32_t lds_base = (uint32_t)(uintptr_t)smem;

    // ---- loads
    const int nst = K / 64 / G::SL / ksplit;
    // The XCDs start at eight different places of K and wrap around: rows of a power-of-two length put one K slice of
    // all rows into few memory channels, and the whole chip walking K in step would ask for one slice at a time (7B
    // shapes of 256 rows: 3-5 % less time).  Blocks of one XCD stay in step, what they share they find in its L2.
    const int rot = (int)(blockIdx.x & 7) * nst / 8;
    const int wrow0 = swi ? (oc0 >> 5) * 64 : n0;
    const size_t k0 = (size_t)range * nst * (64 * G::SL);
    const uint8_t* abase = reinterpret_cast<const uint8_t*>(A + (size_t)m0 * lda + k0);
    const uint8_t* wbase = reinterpret_cast<const uint8_t*>(Wt + (size_t)wrow0 * K + k0);
    // byte offset of token row / weight row r of the tile from its base; rows beyond the matrix are clamped (their
    // products are never stored)
    auto a_row = [&](int r) -> uint32_t { return (uint32_t)(m0 + r < M ? r : M - 1 - m0) * (uint32_t)lda * 2u; };
    auto w_row = [&](int r) -> uint32_t {
        int gr;
        if (swi) {
            int oc = oc0 + (r >> 5) * 16 + (r & 15);
            oc = oc < N / 2 ? oc : N / 2 - 1;
            gr = (oc >> 5) * 64 + ((r >> 4) & 1) * 32 + (oc & 31);
        } else {
            gr = n0 + r < N ? n0 + r : N - 1;
        }
        return (uint32_t)(gr - wrow0) * (uint32_t)K * 2u;
    };
    uint32_t off[G::LMAX];
#pragma unroll
    for (int i = 0; i < G::LMAX; ++i) {
        const int q = wave + i * G::NW, sub = q / ((BM + BN) / 8), row = (q % ((BM + BN) / 8)) * 8 + (lane >> 3);
        off[i] = (row < BM ? a_row(row) : w_row(row - BM)) + (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) * 16 + sub * 128);
    }
    auto issue = [&](int t, int slot) {
        const int tr = t + rot < nst ? t + rot : t + rot - nst;
        const size_t koff = (size_t)tr * (128 * G::SL);
        const uint8_t* a = abase + koff;
        const uint8_t* w = wbase + koff;
        const uint32_t st = lds_base + (uint32_t)slot * G::STAGE;
#pragma unroll
        for (int i = 0; i < G::LMAX; ++i) {
            const int q = wave + i * G::NW;
            if (i < G::L || wave < G::REM)
                tile_dma16(off[i], (q % ((BM + BN) / 8)) < BM / 8 ? a : w, st + (uint32_t)q * 1024u);
        }
    };
    // wait until at most `stages` of the newest requested stages are still on their way
    auto wait_stages = [&](auto stages) {
        constexpr int S = decltype(stages)::value;
        if (G::REM != 0 && wave < G::REM) tile_wait_barrier<S * G::LMAX>();
        else tile_wait_barrier<S * G::L>();
    };

    f32x4_t acc[TN][TM];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[j][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // ---- fragments: group wg owns k-steps wg * P .. wg * P + P - 1 of a stage
    const int sw = (l16 >> 1) & 7;
    auto read = [&](int slot, int p, half8_t* wf, half8_t* tf) {
        const int ks = wg * P + p;
        const uint8_t* s = smem + slot * G::STAGE + (ks >> 1) * G::SUB + l16 * 128 + ((((ks & 1) * 4 + l4) ^ sw) << 4);
        const uint8_t* sa = s + wm * (BM / G::WM) * 128;
        const uint8_t* sb = s + (BM + wn * (BN / G::WN)) * 128;
#pragma unroll
        for (int j = 0; j < TN; ++j) wf[j] = *reinterpret_cast<const half8_t*>(sb + j * 2048);
#pragma unroll
        for (int i = 0; i < TM; ++i) tf[i] = *reinterpret_cast<const half8_t*>(sa + i * 2048);
    };
    auto multiply = [&](const half8_t* wf, const half8_t* tf) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i) acc[j][i] = SS_MFMA_16x16x32(wf[j], tf[i], acc[j][i], 0, 0, 0);
    };
    auto interleave = [&]() {
        constexpr int NF = TM + TN, NM = TM * TN, EACH = NM / NF > 0 ? NM / NF : 1;
#pragma unroll
        for (int r = 0; r < NF; ++r) {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, EACH, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, NM, 0);
    };

    half8_t wf[2][TN], tf[2][TM];
    const int first = nst < NS ? nst : NS;
    for (int t = 0; t < first; ++t) issue(t, t);
    if (nst >= NS) wait_stages(std::integral_constant<int, NS - 1>{});
    else wait_stages(std::integral_constant<int, 0>{});
    read(0, 0, wf[0], tf[0]);
    int slot = 0;
    // a stage's k-steps but the last, then the last one next to the hand-over to the next stage
    auto step = [&](int t, auto set0) {
        constexpr int S0 = decltype(set0)::value;
#pragma unroll
        for (int p = 0; p + 1 < P; ++p) {
            read(slot, p + 1, wf[(S0 + p + 1) & 1], tf[(S0 + p + 1) & 1]);
            multiply(wf[(S0 + p) & 1], tf[(S0 + p) & 1]);
            interleave();
            __builtin_amdgcn_sched_barrier(0);
        }
        if (t + 1 < nst) {
            if (t + NS <= nst) wait_stages(std::integral_constant<int, NS - 2>{});
            else wait_stages(std::integral_constant<int, 0>{});
            if (t + NS < nst) issue(t + NS, slot);
            slot = slot + 1 == NS ? 0 : slot + 1;
            read(slot, 0, wf[(S0 + P) & 1], tf[(S0 + P) & 1]);
        }
        multiply(wf[(S0 + P - 1) & 1], tf[(S0 + P - 1) & 1]);
        interleave();
        __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (P % 2 == 0) {
        for (int t = 0; t < nst; ++t) step(t, std::integral_constant<int, 0>{});
    } else {
        int t = 0;
        for (; t + 1 < nst; t += 2) {
            step(t, std::integral_constant<int, 0>{});
            step(t + 1, std::integral_constant<int, 1>{});
        }
        if (t < nst) step(t, std::integral_constant<int, 0>{});
    }

    // ---- the groups' sums meet in LDS; rows leave as 16-byte stores
    float* st = reinterpret_cast<float*>(smem);
    constexpr int TP = TM / G::PASSES, RP = G::RP, PITCH = G::PITCH;
    const int cpr = swi ? BN / 16 : BN / 8;
    const int n_out = swi ? N / 2 : N;
#pragma unroll
    for (int ps = 0; ps < G::PASSES; ++ps) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < TP; ++i)
                *reinterpret_cast<f32x4_t*>(st + (wg * RP + (wm * TP + i) * 16 + l16) * PITCH + wn * (BN / G::WN) + j * 16 + 4 * l4) =
                    acc[j][ps * TP + i];
        __syncthreads();
        for (int x = tid; x < RP * cpr; x += 64 * G::NW) {
            const int row = x / cpr, cc = (x - row * cpr) * 8;
            const int m = m0 + (row / (TP * 16)) * (BM / G::WM) + ps * TP * 16 + row % (TP * 16);
            const int c = (swi ? oc0 : n0) + cc;
            if (m >= M || c >= n_out) continue;
            const float* s = st + row * PITCH + (swi ? (cc >> 4) * 32 + (cc & 15) : cc);
            auto sum4 = [&](int at) {
                f32x4_t v = *reinterpret_cast<const f32x4_t*>(s + at);
#pragma unroll
                for (int g = 1; g < G::KG; ++g) v += *reinterpret_cast<const f32x4_t*>(s + g * RP * PITCH + at);
                return v;
            };
            f32x4_t o[2] = {sum4(0), sum4(4)};
            if (epi == EPI_STORE_F32) {
                float* cp = reinterpret_cast<float*>(Cv) + ((size_t)range * M + m) * ldc + c;
                *reinterpret_cast<f32x4_t*>(cp) = o[0];
                *reinterpret_cast<f32x4_t*>(cp + 4) = o[1];
                continue;
            }
            if (RS) {
                const float rs = RS[m];
                o[0] *= rs;
                o[1] *= rs;
            }
            if (swi) {
                f32x4_t u[2] = {sum4(16), sum4(20)};
                const float rs = RS ? RS[m] : 1.0f;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e >> 2][e & 3] = tile_swiglu(o[e >> 2][e & 3], u[e >> 2][e & 3] * rs);
            }
            if (epi == EPI_RESIDUAL) {
                float r[8];
                unpack16<bf16_t>(*reinterpret_cast<const vec16*>(R + (size_t)m * ldc + c), r);
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e >> 2][e & 3] += r[e];
            }
            vec16 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w.w[e] = pack_bf16x2(o[e >> 1][(e & 1) * 2], o[e >> 1][(e & 1) * 2 + 1]);
            *reinterpret_cast<vec16*>(reinterpret_cast<bf16_t*>(Cv) + (size_t)m * ldc + c) = w;
        }
    }
}

template <class G>
static hipError_t launch_tile(const bf16_t* A, int lda, const bf16_t* Wt, void* C, int ldc, const bf16_t* R, int M, int N, int K,
                              int epi, int ksplit, const float* rs, hipStream_t s) {
    if (epi == EPI_RESIDUAL && !R) return hipErrorInvalidValue;
    if (ksplit < 1 || (ksplit > 1 && epi != EPI_STORE_F32)) return hipErrorInvalidValue;
    const int tiles_m = (M + G::BM - 1) / G::BM, tiles_n = (N + G::BN - 1) / G::BN;
    const long long n_tiles = (long long)tiles_m * tiles_n;
    if (n_tiles * ksplit > (1ll << 27) || K % (64 * G::SL * ksplit) != 0) return hipErrorInvalidValue;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)gemm_tile_kernel<G>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int per_xcd = (int)((n_tiles * ksplit + 7) / 8);
    gemm_tile_kernel<G><<<8 * per_xcd, 64 * G::NW, G::LDS, s>>>(A, lda, Wt, C, ldc, R, M, N, K, epi, tiles_m, (int)n_tiles, ksplit,
                                                                per_xcd, rs);
    return hipGetLastError();
}

bool gemm_tile_supported(const void* A, const void* Wt, const void* C, const void* R, int ldc, int M, int N, int K, int lda, int epi) {
    if (M <= 0 || N <= 0 || K < 64 || K % 64 != 0 || lda % 8 != 0 || ldc % 8 != 0 || N % 8 != 0) return false;
    if (epi == EPI_SWIGLU && N % 64 != 0) return false;
    if (epi != EPI_STORE && epi != EPI_RESIDUAL && epi != EPI_SWIGLU && epi != EPI_STORE_F32) return false;
    if ((((uintptr_t)A | (uintptr_t)Wt | (uintptr_t)C) & 15) != 0 || (epi == EPI_RESIDUAL && ((uintptr_t)R & 15) != 0)) return false;
    // 32-bit byte offsets inside one tile of an operand (a SwiGLU tile spans up to 64 rows more than it has)
    return (long long)256 * lda * 2 < (1ll << 32) && (long long)320 * K * 2 < (1ll << 32);
}

// The tiles.  Small ones take stages of two slices (a barrier per slice would outweigh their few matrix instructions).
#define SS_TILES(X)                                                                                                         \
    X(64, 32, 2, 1, 4, 2, 6) X(64, 64, 2, 1, 4, 2, 4) X(64, 64, 2, 2, 2, 1, 9) X(64, 96, 2, 2, 2, 1, 7)                     \
    X(96, 32, 2, 1, 4, 2, 4) X(96, 64, 2, 2, 2, 1, 7) X(96, 128, 2, 2, 2, 1, 5) X(128, 64, 2, 2, 2, 1, 6)                   \
    X(128, 96, 2, 2, 2, 1, 5) X(128, 128, 2, 2, 2, 1, 5) X(128, 192, 2, 2, 2, 1, 4) X(192, 64, 2, 2, 2, 1, 5)               \
    X(192, 96, 2, 2, 2, 1, 4) X(192, 128, 2, 2, 2, 1, 4) X(192, 192, 2, 2, 2, 1, 3) X(256, 128, 2, 2, 2, 1, 3)              \
    X(256, 160, 4, 2, 1, 1, 3) X(256, 192, 4, 2, 1, 1, 2)

// Which tile: the one with the least estimated time (returned in microseconds, *pick = its place in the list).  A block
// spends on a K slice the larger of what its lines take (1.8 ns per token line, which the L2 mostly has, 3.3 ns per weight
// line, which it mostly has not) and what its products take (0.024 ns per output element, 15 % more where one group of
// waves does all k-steps); 7 us go to launch, first loads and epilogue, 8 more to every further round of tiles.  The four
// numbers were fitted to 31 shapes of 100 to 2000 rows, every tile timed on each.  Over 44 shapes of 65 to 1280 rows the choice,
// split kernels included, is within 1.2 % of the fastest on average, 7 % in 95 of 100, 16 % at worst; the estimate is 15 to 25 %
// above the measured time nearly everywhere, which leaves the order as it is, but right for the 96 x 32 tile with one row of tiles,
// whose weight lines no second block of the XCD shares: its token lines count 2.4 ns there (64 x 64 tiles instead, 96 rows:
// 5120 x 13824 65 -> 56 us, 8192 x 14336 72 -> 63, 5120 x 8192 37 -> 33, 6912 x 5120 28.5 -> 26.7; 5120 x 1280 at 80 rows
// loses 0.3 us of 7).
float gemm_tile_estimate(int M, int N, int K, int n_cus, int* pick) {
    float best = 0.f;
    *pick = -1;
    int at = 0;
#define X(BM, BN, WM, WN, KG, SL, NS)                                                                                       \
    if (K % (64 * SL) == 0) {                                                                                               \
        const long long tiles = (long long)((M + BM - 1) / BM) * ((N + BN - 1) / BN);                                       \
        const float rounds = (float)((tiles + n_cus - 1) / n_cus);                                                          \
        const float lines = (BN == 32 && BM == 96 && M <= BM ? 2.4f : 1.8f) * BM + 3.3f * BN, mul = (KG == 1 ? 0.0276f : 0.024f) * BM * BN;                            \
        const float us = 7.f + 8.f * (rounds - 1.f) + rounds * (K / 64) * (lines > mul ? lines : mul) * 1e-3f;              \
        if (*pick < 0 || us < best) { best = us; *pick = at; }                                                              \
    }                                                                                                                       \
    ++at;
    SS_TILES(X)
#undef X
    return best;
}

// Tile and ranges of K for a product whose ranges meet in memory: a compute unit loads token and weight lines at one rate
// whatever they are for (1.07 ns a line out of the L2, and the XCD another 0.13 ns for each that the L2 has not), and four ranges
// of tiles of twice the height and width have half the lines of one range.  Worth it for long contractions of narrow outputs:
// 4.4 us + 1.54 / 2.49 ns a token / weight line and slice (or the products, as above) + 2.4 us and 2.2 TB/s for the partial
// sums on their way out and in; fitted to 782 launches of 17 products at 80 to 1536 rows, 7 % off (12 % over unsplit ones).  One
// round of tiles, eight slices a range or more.  `*now` is the same estimate for tile `pick_now` unsplit.
float gemm_tile_split_estimate(int M, int N, int K, int n_cus, size_t ws_bytes, int pick_now, float* now, int* pick, int* split) {
    float best = 0.f;
    *pick = -1;
    *split = 1;
    *now = 0.f;
    int at = 0;
#define X(BM, BN, WM, WN, KG, SL, NS)                                                                                       \
    {                                                                                                                       \
        const long long tiles = (long long)((M + BM - 1) / BM) * ((N + BN - 1) / BN);                                       \
        const float lines = (BN == 32 && BM == 96 && M <= BM ? 2.4f : 1.54f) * BM + 2.49f * BN, mul = 0.95f * (KG == 1 ? 0.0276f : 0.024f) * BM * BN; \
        const float slice = (lines > mul ? lines : mul) * 1e-3f;                                                            \
        const float rounds = (float)((tiles + n_cus - 1) / n_cus);                                                          \
        if (at == pick_now) *now = 4.4f + 8.f * (rounds - 1.f) + rounds * (K / 64) * slice;                                 \
        for (int s = 2; s <= 8; s *= 2) {                                                                                   \
            const size_t bytes = (size_t)s * M * N * sizeof(float);                                                         \
            if (K % (64 * SL * s) != 0 || K / 64 / s < 8 || tiles * s > n_cus || bytes > ws_bytes) continue;                \
            const float us = 6.8f + (K / 64 / s) * slice + (float)bytes / 2.2e6f;                                           \
            if (*pick < 0 || us < best) { best = us; *pick = at; *split = s; }                                              \
        }                                                                                                                   \
        ++at;                                                                                                               \
    }
    SS_TILES(X)
#undef X
    return best;
}

hipError_t gemm_tile(int pick, const bf16_t* A, int lda, const bf16_t* Wt, void* C, int ldc, const bf16_t* R, int M, int N, int K,
                     int epi, int ksplit, const float* rs, hipStream_t s) {
    int at = 0;
#define X(BM, BN, WM, WN, KG, SL, NS) \
    if (pick == at++) return launch_tile<TileCfg<BM, BN, WM, WN, KG, SL, NS>>(A, lda, Wt, C, ldc, R, M, N, K, epi, ksplit, rs, s);
    SS_TILES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace SS_NS

// Plain LDS-tiled FMA GEMM: C[M,N] = A[M,K] * Wt[N,K]^T with fp32 accumulation.
// Serves the shapes that the MFMA kernels do not take (16-bit types with K not a
// multiple of 64, fp32 with rows that are not 16-byte aligned) and is the reference
// path of SS_FORCE_GENERIC.  64x64 output tile per 256-thread block, 16-deep
// K slices staged through LDS as floats, 4x4 outputs per thread.  Any M, N, K.
#include "ss_device.h"
#include "ss_kernels.h"

namespace SS_NS {
using namespace ssk;

template <typename T, int EPI>
__global__ __launch_bounds__(256) void gemm_generic_kernel(const T* __restrict__ A, int lda,
                                                           const T* __restrict__ Wt, void* __restrict__ Cv,
                                                           int ldc, const T* __restrict__ R, int M, int N, int K,
                                                           const float* __restrict__ RS) {
    constexpr int BM = 64, BN = 64, BK = 16;
    __shared__ float As[BK][BM + 4];
    __shared__ float Bs[BK][BN + 4];
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    float acc[4][4] = {};
    // loader mapping: thread -> (row = tid / 4, k = (tid % 4) * 4 .. +3)
    const int lr = threadIdx.x >> 2, lk = (threadIdx.x & 3) * 4;
    for (int k0 = 0; k0 < K; k0 += BK) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = k0 + lk + j;
            const int am = m0 + lr, bn = n0 + lr;
            As[lk + j][lr] = (am < M && k < K) ? ldf(A + (size_t)am * lda + k) : 0.f;
            Bs[lk + j][lr] = (bn < N && k < K) ? ldf(Wt + (size_t)bn * K + k) : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < BK; ++k) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { a[i] = As[k][ty * 4 + i]; b[i] = Bs[k][tx * 4 + i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + ty * 4 + i;
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = n0 + tx * 4 + j;
            if (n >= N) continue;
            float v = acc[i][j];
            if (RS) v *= RS[m];
            if (EPI == EPI_RESIDUAL) v += ldf(R + (size_t)m * ldc + n);
            if (EPI == EPI_STORE_F32)
                reinterpret_cast<float*>(Cv)[(size_t)m * ldc + n] = v;
            else
                stf(reinterpret_cast<T*>(Cv) + (size_t)m * ldc + n, v);
        }
    }
}

template <typename T>
static hipError_t launch_generic(const void* A, int lda, const void* Wt, void* C, int ldc, const void* R, int M,
                                 int N, int K, int epi, hipStream_t s, const float* rs) {
    dim3 grid((N + 63) / 64, (M + 63) / 64);
    if (grid.y > 65535) return hipErrorInvalidValue;
    const T* a = (const T*)A;
    const T* w = (const T*)Wt;
    const T* r = (const T*)R;
    switch (epi) {
        case EPI_STORE: gemm_generic_kernel<T, EPI_STORE><<<grid, 256, 0, s>>>(a, lda, w, C, ldc, r, M, N, K, rs); break;
        case EPI_RESIDUAL:
            if (!R) return hipErrorInvalidValue;
            gemm_generic_kernel<T, EPI_RESIDUAL><<<grid, 256, 0, s>>>(a, lda, w, C, ldc, r, M, N, K, rs);
            break;
        case EPI_STORE_F32: gemm_generic_kernel<T, EPI_STORE_F32><<<grid, 256, 0, s>>>(a, lda, w, C, ldc, r, M, N, K, rs); break;
        default: return hipErrorInvalidValue;   // the fused SwiGLU layout exists only for the MFMA kernel
    }
    return hipGetLastError();
}

hipError_t gemm_mfma_bf16(const void* A, int lda, const void* Wt, void* C, int ldc, const void* R, int M, int N,
                          int K, int epi, hipStream_t s, float* ws, size_t ws_bytes, int max_rounds, const float* rs);
bool gemm_mfma_supported(int M, int N, int K, int lda, int ldc, int epi);
bool gemm_mfma_stream_supported(const void* C, const void* R, int ldc, int M, int N, int K, int lda, int epi);
bool gemm_tile_supported(const void* A, const void* Wt, const void* C, const void* R, int ldc, int M, int N, int K, int lda, int epi);
int gemm_stream_columns(int M, int N, int K, int n_cus, int* pick);
GemmPlan gemm_mfma_plan(bool stream_ok, bool tile_ok, int M, int N, int K, int epi, size_t ws_bytes, int n_cus);
bool gemm_direct_takes(int dt, const void* A, const void* Wt, int M, int N, int K, int lda, int epi);
hipError_t gemm_direct(int dt, const void* A, int lda, const void* Wt, void* C, int ldc, const void* R, int M, int N, int K,
                       int epi, float norm_eps, const void* gain, const UploadJob& job, hipStream_t s);

bool gemm_norms_itself(int dt, const void* A, int lda, const void* Wt, int M, int N, int K, int epi, bool force_generic) {
    return !force_generic && gemm_direct_takes(dt, A, Wt, M, N, K, lda, epi);
}

hipError_t norm_nt(int dt, const void* A, int lda, const void* Wt, void* C, int ldc, int M, int N, int K, int epi, float norm_eps,
                   const UploadJob& job, hipStream_t s) {
    if (M <= 0 || N <= 0) return job.n16 ? hipErrorInvalidValue : hipSuccess;
    if (K <= 0 || lda < K || !A || !Wt || !C || norm_eps < 0.f || !gemm_norms_itself(dt, A, lda, Wt, M, N, K, epi, false)) return hipErrorInvalidValue;
    return gemm_direct(dt, A, lda, Wt, C, ldc, nullptr, M, N, K, epi, norm_eps, nullptr, job, s);
}

// Few rows: every column block scales the rows again, which has to cost less than the launch that it saves (2.5 to 4 us).  With the
// norm apart / inside, us:
//  - 16-bit, up to 8 rows (blocks of one column tile): contractions of 2048 and more up to 8192 columns (8 rows 4096 x 8192
//    16.0 / 15.3, 2048 x 16000 15.0 / 16.9, 4096 x 64000 91 / 109; 1024 x 64000 23.5 / 21.5);
//  - 9 to 16 rows (up to four): all but wide outputs of contractions beyond 4096 (4096 x 32000 44.8 / 43.2, 8192 x 16000 47.4 / 44.4,
//    8192 x 32000 103.3 / 106.1);
//  - 17 to 32 rows all that come here (4096 x 8192 18.7 / 16.6); more rows up to 48 rows of 2048 or so (48 rows 2048 x 4096 9.8
//    / 8.8, 8192 x 512 17.5 / 19.1; 64 rows 1024 x 2048 7.8 / 7.2, 4096 x 2048 13.8 / 15.2);
//  - fp32: up to 16 rows all (1024 x 64000 47.6 / 44.3), up to 32 rows 16384 columns (4096 x 16000 74.6 / 74.1, 1024 x 32000
//    36.2 / 37.3), beyond that 8192 (64 rows 1024 x 8192 25.5 / 24.8, x 16000 35.9 / 36.4).
// IEEE half keeps the norm apart: a row times its gains has to fit the type before the row's factor brings it to size.
bool head_norms_itself(int dt, const void* A, int lda, const void* Wt, const void* gain, int M, int N, int K, bool force_generic) {
#ifdef SS_HALF_F16
    if (dt != F32) return false;
#endif
    if (M > 64 || ((uintptr_t)gain & 15) != 0 || !gemm_norms_itself(dt, A, lda, Wt, M, N, K, EPI_STORE_F32, force_generic)) return false;
    if (dt == F32) return M <= 16 || N <= (M <= 32 ? 16384 : 8192);
    if (M <= 8) return K < 2048 || N <= 8192;
    if (M <= 16) return K <= 4096 || N <= 16384;
    return M <= 32 || M * K <= 48 * 2048;
}

hipError_t head_nt(int dt, const void* A, int lda, const void* Wt, float* C, int ldc, int M, int N, int K, float norm_eps,
                   const void* gain, hipStream_t s) {
    if (M <= 0 || N <= 0) return hipSuccess;
    if (K <= 0 || lda < K || !A || !Wt || !C || !gain || !head_norms_itself(dt, A, lda, Wt, gain, M, N, K, false)) return hipErrorInvalidValue;
    return gemm_direct(dt, A, lda, Wt, C, ldc, nullptr, M, N, K, EPI_STORE_F32, norm_eps, gain, UploadJob(), s);
}

hipError_t gemm_nt(int dt, const void* A, int lda, const void* Wt, void* C, int ldc, const void* R, int M, int N,
                   int K, int epi, bool force_generic, hipStream_t s, float* ws, size_t ws_bytes, int max_rounds,
                   const float* row_scale) {
    if (M <= 0 || N <= 0) return hipSuccess;
    if (K <= 0 || lda < K || !A || !Wt || !C) return hipErrorInvalidValue;
    if (!row_scale && gemm_norms_itself(dt, A, lda, Wt, M, N, K, epi, force_generic))
        return gemm_direct(dt, A, lda, Wt, C, ldc, R, M, N, K, epi, -1.0f, nullptr, UploadJob(), s);
    if (epi == EPI_SWIGLU_HALVES) return hipErrorInvalidValue;     // only the kernel above does it
    if (dt == BF16 && !force_generic && gemm_mfma_supported(M, N, K, lda, ldc, epi))
        return gemm_mfma_bf16(A, lda, Wt, C, ldc, R, M, N, K, epi, s, ws, ws_bytes, max_rounds, row_scale);
    if (epi == EPI_SWIGLU) return hipErrorInvalidValue;
    if (dt == F32) return launch_generic<float>(A, lda, Wt, C, ldc, R, M, N, K, epi, s, row_scale);
    return launch_generic<bf16_t>(A, lda, Wt, C, ldc, R, M, N, K, epi, s, row_scale);
}

}  // namespace SS_NS

#ifndef SS_HALF_F16
// The choice of gemm_nt for dense operands on 16-byte boundaries, without a GPU (for tests of the rules).
extern "C" int ssk_gemm_plan(int dt, int M, int N, int K, int epi, long long ws_bytes, int n_cus, int* pick, int* split) {
    const void* p = (const void*)(uintptr_t)4096;
    const int ldc = epi == ssk::EPI_SWIGLU || epi == ssk::EPI_SWIGLU_HALVES ? N / 2 : N;
    ssk::GemmPlan plan{ssk::GEMM_GENERIC, 0, 1};
    if (ssk::gemm_direct_takes(dt, p, p, M, N, K, K, epi)) plan.kernel = ssk::GEMM_DIRECT;
    else if (dt == ssk::BF16 && ssk::gemm_mfma_supported(M, N, K, K, ldc, epi))
        plan = ssk::gemm_mfma_plan(ssk::gemm_mfma_stream_supported(p, p, ldc, M, N, K, K, epi),
                                   ssk::gemm_tile_supported(p, p, p, p, ldc, M, N, K, K, epi), M, N, K, epi, (size_t)ws_bytes, n_cus);
    *pick = plan.pick;
    *split = plan.split;
    return plan.kernel;
}
extern "C" int ssk_gemm_stream_columns(int M, int N, int K, int n_cus, int* pick) { return ssk::gemm_stream_columns(M, N, K, n_cus, pick); }
extern "C" bool ssk_head_norms_itself(int dt, int M, int N, int K) {
    const void* p = (const void*)(uintptr_t)4096;
    return ssk::head_norms_itself(dt, p, K, p, p, M, N, K, false);
}
#endif

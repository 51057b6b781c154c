// fp32 projection on the fp32 matrix instructions:  c[M,N] = a[M,K] * w[N,K]^T, or (SWIGLU) silu(a wg^T) * (a wu^T) with
// w = [gate; up].  (Projections of the layer: paper Section 2.2.)  Requires K % 4 == 0 and 16-byte aligned operands.
//
// Both operands are K-contiguous, so a lane fetches four consecutive k of its row with one 16-byte load and feeds element j
// to the j-th of four matrix instructions; which k an instruction's slots hold does not matter as long as both operands
// agree.  Operands come straight from the caches: the shards that run in fp32 are small (a few MB), and what such a call
// takes is not bandwidth but one trip to memory after the other.
//   * MR = 16 (v_mfma_f32_16x16x4_f32), one 16 x 16 tile per workgroup, the k range split over its four waves: a wave of the
//     128-token layer (K = 256) makes ONE round trip.  Measured at 128 x 768 x 256: 4.9 us against 61 us of the SIMT tile
//     kernel, whose twelve to 24 workgroups walked 16 k at a time between barriers.
//   * MR = 32 (v_mfma_f32_32x32x2_f32), 2 x 2 tiles per workgroup, for products with at least 256 tiles of 64 x 64.
#include "iso_internal.h"

namespace {

template <int MR> struct F32Mfma;
template <> struct F32Mfma<16> {
    typedef f32x4_t acc_t;
    static constexpr int NACC = 4;
    static __device__ __forceinline__ acc_t mfma(float a, float b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int r, int grp) { return 4 * grp + r; }
};
template <> struct F32Mfma<32> {
    typedef f32x16_t acc_t;
    static constexpr int NACC = 16;
    static __device__ __forceinline__ acc_t mfma(float a, float b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int r, int grp) { return 8 * (r / 4) + 4 * grp + (r % 4); }
};

// KW waves share the k range of a tile, WM x WN tiles per workgroup; KW * WM * WN = 4.
template <int MR, int WM, int WN, int KW, bool SWIGLU>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float *__restrict__ A, const float *__restrict__ W,
                                                       float *__restrict__ C, int M, int N, int K) {
    using Op = F32Mfma<MR>;
    constexpr int NB = SWIGLU ? 2 : 1;              // W row blocks per tile: gate and up
    constexpr int GRP = 64 / MR, STEP = 4 * GRP;    // k per step (four matrix instructions)
    constexpr int UNROLL = MR == 16 ? 4 : 4;
    __shared__ float part[KW > 1 ? KW * NB * MR * (MR + 1) : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kw = wave % KW, wm = (wave / KW) % WM, wn = wave / (KW * WM);
    const int lrow = lane % MR, grp = lane / MR;
    const int m0 = (blockIdx.y * WM + wm) * MR, n0 = (blockIdx.x * WN + wn) * MR;
    const int n_out = SWIGLU ? N / 2 : N;
    const float *ap = A + (size_t)min(m0 + lrow, M - 1) * K;
    const float *wp[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) wp[b] = W + (size_t)(b * n_out + min(n0 + lrow, n_out - 1)) * K;
    typename Op::acc_t acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < Op::NACC; ++r) acc[b][r] = 0.f;
    const int steps = (K + STEP - 1) / STEP;
    const int s0 = steps * kw / KW, s1 = steps * (kw + 1) / KW;
    for (int s = s0; s < s1; s += UNROLL) {
        f32x4_t av[UNROLL], wv[NB][UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {          // all loads of the group before its first matrix instruction
            const int k = (s + u) * STEP + 4 * grp;
            const bool in = s + u < s1 && k < K;    // K % 4 == 0: a piece is entirely inside or outside
            av[u] = in ? *reinterpret_cast<const f32x4_t *>(ap + k) : f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int b = 0; b < NB; ++b)
                wv[b][u] = in ? *reinterpret_cast<const f32x4_t *>(wp[b] + k) : f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b] = Op::mfma(av[u][j], wv[b][u][j], acc[b]);
    }
    // accumulator register r of lane l: row Op::row(r, l / MR), column l % MR
    if constexpr (KW == 1) {
#pragma unroll
        for (int r = 0; r < Op::NACC; ++r) {
            const int m = m0 + Op::row(r, grp), n = n0 + lrow;
            if (m >= M || n >= n_out) continue;
            float v = acc[0][r];
            if constexpr (SWIGLU) v = v / (1.0f + expf(-v)) * acc[1][r];
            C[(size_t)m * n_out + n] = v;
        }
    } else {
        static_assert(WM == 1 && WN == 1, "one tile per workgroup");
        constexpr int P = MR + 1;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < Op::NACC; ++r) part[((kw * NB + b) * MR + Op::row(r, grp)) * P + lrow] = acc[b][r];
        __syncthreads();
        for (int e = tid; e < MR * MR; e += 256) {
            const int row = e / MR, col = e % MR, m = m0 + row, n = n0 + col;
            if (m >= M || n >= n_out) continue;
            float v[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                v[b] = part[(b * MR + row) * P + col];
#pragma unroll
                for (int k = 1; k < KW; ++k) v[b] += part[((k * NB + b) * MR + row) * P + col];
            }
            if constexpr (SWIGLU) v[0] = v[0] / (1.0f + expf(-v[0])) * v[1];
            C[(size_t)m * n_out + n] = v[0];
        }
    }
}

template <bool SWIGLU> hipError_t launch_f32(const void *a, const void *w, void *c, int M, int N, int K, hipStream_t s) {
    const int n_out = SWIGLU ? N / 2 : N;
    const long long big = (long long)((M + 63) / 64) * ((n_out + 63) / 64);
    if (big >= 256)
        hipLaunchKernelGGL((gemm_f32_kernel<32, 2, 2, 1, SWIGLU>), dim3((n_out + 63) / 64, (M + 63) / 64), dim3(256), 0, s,
                           (const float *)a, (const float *)w, (float *)c, M, N, K);
    else
        hipLaunchKernelGGL((gemm_f32_kernel<16, 1, 1, 4, SWIGLU>), dim3((n_out + 15) / 16, (M + 15) / 16), dim3(256), 0, s,
                           (const float *)a, (const float *)w, (float *)c, M, N, K);
    return hipGetLastError();
}

}  // namespace

bool iso_gemm_f32_supported(const void *a, const void *w, int M, int N, int K) {
    return (K % 4) == 0 && ((uintptr_t)a | (uintptr_t)w) % 16 == 0 && (M + 15) / 16 <= 65535;
}

hipError_t iso_launch_gemm_f32(const void *a, const void *w, void *c, int M, int N, int K, hipStream_t s) {
    return launch_f32<false>(a, w, c, M, N, K, s);
}

hipError_t iso_launch_gemm_swiglu_f32(const void *a, const void *w, void *act, int M, int F, int K, hipStream_t s) {
    return launch_f32<true>(a, w, act, M, 2 * F, K, s);
}

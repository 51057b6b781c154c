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

// What follows the sums: nothing, SwiGLU, or (the QKV projection) rotary embedding and KV-cache write.  The last two tie two
// rows of W to one output column index, gate and up or the two halves of a head, and a tile computes both.
enum { EPI_NONE = 0, EPI_SWIGLU = 1, EPI_ROPE = 2 };
struct RopeF32 {
    const float *cos_t, *sin_t;      // [max_seq, d / 2]
    float *k_cache, *v_cache;
    int q_offset, nq, nkv, d;
};

// What stands before the product: A as it is, or A = rmsnorm(x) * g / rmsnorm(x + delta) * g, computed by every workgroup for
// its own sixteen rows.  A wave then holds its whole part of the rows in registers (K <= 16 * KW * UNROLL), the squares meet in LDS,
// and the two launches before the projections of a short call are gone (128 tokens of 256: a pass is set by how fast the host
// enqueues: 11 launches 42.3 us; 7, with this and the copies to the host below, 35.5, of which the kernels take 34).  Where that
// pays: iso_gemm_f32_norm_supported.
enum { NORM_NONE = 0, NORM_X = 1, NORM_X_DELTA = 2 };
struct NormF32 {
    const float *delta, *g;
    float eps;
};

// KW waves share the k range of a tile, WM x WN tiles per workgroup; KW * WM * WN = 4.  UNROLL steps of k are requested at a
// time: twelve where a wave has more than four of them, so that the down projection (K = 688) is one trip to memory as well
// (128 x 256 x 688: 5.2 -> 4.1 us).
// `sink` (small tiles, EPI_NONE): pinned host memory that receives C as well; null: none.
template <int MR, int WM, int WN, int KW, int UNROLL, int EPI, int NORM = NORM_NONE>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float *__restrict__ A, const float *__restrict__ W,
                                                       float *__restrict__ C, float *__restrict__ sink, int M, int N, int K,
                                                       RopeF32 rope, NormF32 norm) {
    using Op = F32Mfma<MR>;
    constexpr bool SWIGLU = EPI == EPI_SWIGLU, ROPE = EPI == EPI_ROPE;
    constexpr int NB = EPI == EPI_NONE ? 1 : 2;     // W row blocks per tile
    constexpr int GRP = 64 / MR, STEP = 4 * GRP;    // k per step (four matrix instructions)
    static_assert(!ROPE || KW > 1, "the rotary step works on the tile in LDS");
    static_assert(NORM == NORM_NONE || (MR == 16 && WM == 1 && WN == 1), "one tile per workgroup");
    __shared__ float part[KW > 1 ? KW * NB * MR * (MR + 1) : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kw = wave % KW, wm = (wave / KW) % WM, wn = wave / (KW * WM);
    const int lrow = lane % MR, grp = lane / MR;
    const int m0 = (blockIdx.y * WM + wm) * MR, n0 = (blockIdx.x * WN + wn) * MR;
    const int n_out = NB == 2 ? N / 2 : N;
    const float *ap = A + (size_t)min(m0 + lrow, M - 1) * K;
    const float *wp[NB];
    const int half = ROPE ? rope.d / 2 : 1, head = ROPE ? n0 / half : 0;     // half % 16 == 0: a tile lies in one head
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int n = min(n0 + lrow, n_out - 1);
        wp[b] = W + (size_t)(ROPE ? n + (head + b) * half : b * n_out + n) * K;
    }
    typename Op::acc_t acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < Op::NACC; ++r) acc[b][r] = 0.f;
    const int steps = (K + STEP - 1) / STEP;
    const int s0 = steps * kw / KW, s1 = steps * (kw + 1) / KW;
    for (int s = s0; s < (NORM == NORM_NONE ? s1 : s0 + 1); s += UNROLL) {   // NORM: one round, waves without a step included
        f32x4_t av[UNROLL], wv[NB][UNROLL], gv[NORM == NORM_NONE ? 1 : UNROLL], dv[NORM == NORM_X_DELTA ? UNROLL : 1];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {          // all loads of the group before its first matrix instruction
            const int k = (s + u) * STEP + 4 * grp;
            const bool in = s + u < s1 && k < K;    // K % 4 == 0: a piece is entirely inside or outside
            av[u] = in ? *reinterpret_cast<const f32x4_t *>(ap + k) : f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int b = 0; b < NB; ++b)
                wv[b][u] = in ? *reinterpret_cast<const f32x4_t *>(wp[b] + k) : f32x4_t{0.f, 0.f, 0.f, 0.f};
            if constexpr (NORM != NORM_NONE)
                gv[u] = in ? *reinterpret_cast<const f32x4_t *>(norm.g + k) : f32x4_t{0.f, 0.f, 0.f, 0.f};
            if constexpr (NORM == NORM_X_DELTA)
                dv[u] = in ? *reinterpret_cast<const f32x4_t *>(norm.delta + (ap - A) + k) : f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
        if constexpr (NORM != NORM_NONE) {
            // the squares are added in the norm kernel's order (16-byte pieces of a row over 64 lanes, lane bits from the highest
            // down, then the waves), so that it makes no difference which of the two computes a row
            constexpr int PIECES = 4 * KW * UNROLL;
            __shared__ float sums[MR][PIECES + 1];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                if constexpr (NORM == NORM_X_DELTA) av[u] += dv[u];
                float ss = 0.f;
#pragma unroll
                for (int j = 0; j < 4; ++j) ss += av[u][j] * av[u][j];
                if (s + u < s1) sums[lrow][4 * (s + u) + grp] = ss;
            }
            __syncthreads();
            float total = 0.f;
#pragma unroll
            for (int w = 0; w < PIECES / 64; ++w) {
                float v[16];
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int at = 64 * w + 4 * q + grp;
                    v[q] = at < 4 * steps ? sums[lrow][at] : 0.f;
                }
#pragma unroll
                for (int o = 8; o > 0; o >>= 1)
#pragma unroll
                    for (int q = 0; q < o; ++q) v[q] += v[q + o];
                v[0] += __shfl_xor(v[0], 32, 64);
                v[0] += __shfl_xor(v[0], 16, 64);
                total = w ? total + v[0] : v[0];
            }
            const float scale = 1.0f / sqrtf(total / (float)K + norm.eps);
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) av[u] = av[u] * scale * gv[u];
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
            if constexpr (ROPE) {
                const int i = n - head * half, pos = rope.q_offset + m;
                float *lo = C + (size_t)m * N + (size_t)head * rope.d + i;
                if (head >= rope.nq) {              // k and v heads go to their caches only
                    const bool is_k = head < rope.nq + rope.nkv;
                    lo = (is_k ? rope.k_cache : rope.v_cache) +
                         ((size_t)pos * rope.nkv + head - rope.nq - (is_k ? 0 : rope.nkv)) * rope.d + i;
                }
                float a = v[0], b = v[1];
                if (head < rope.nq + rope.nkv) {
                    const float c = rope.cos_t[(size_t)pos * half + i], sn = rope.sin_t[(size_t)pos * half + i];
                    a = fmaf(v[0], c, -(v[1] * sn));
                    b = fmaf(v[1], c, v[0] * sn);
                }
                lo[0] = a;
                lo[half] = b;
            } else {
                C[(size_t)m * n_out + n] = v[0];
                if (EPI == EPI_NONE && sink) sink[(size_t)m * n_out + n] = v[0];
            }
        }
    }
}

// Small tiles until there are 256 of the large ones.
bool small_tiles(int M, int n_out) { return (long long)((M + 63) / 64) * ((n_out + 63) / 64) < 256; }

// A row in the registers of four waves, with the rounds of loads that a norm is built for (see iso_gemm_f32_norm_supported).
constexpr int norm_max_k(int norm) { return 16 * 4 * (norm == NORM_X_DELTA ? 4 : 12); }

template <int EPI, int NORM = NORM_NONE>
hipError_t launch_f32(const void *a, const void *w, void *c, void *sink, int M, int N, int K, const RopeF32 &rope,
                      const NormF32 &norm, hipStream_t s) {
    const int n_out = EPI == EPI_NONE ? N : N / 2;
    const float *af = (const float *)a, *wf = (const float *)w;
    const dim3 grid16((n_out + 15) / 16, (M + 15) / 16);
    if constexpr (EPI != EPI_ROPE && NORM == NORM_NONE) {
        if (!small_tiles(M, n_out)) {
            if (sink) return hipErrorInvalidValue;
            hipLaunchKernelGGL((gemm_f32_kernel<32, 2, 2, 1, 4, EPI>), dim3((n_out + 63) / 64, (M + 63) / 64), dim3(256), 0, s, af, wf,
                               (float *)c, (float *)nullptr, M, N, K, rope, norm);
            return hipGetLastError();
        }
    }
    if (NORM != NORM_NONE && K > norm_max_k(NORM)) return hipErrorInvalidValue;
    if constexpr (NORM != NORM_X_DELTA) {
        if (K > 4 * 4 * 16) {
            hipLaunchKernelGGL((gemm_f32_kernel<16, 1, 1, 4, 12, EPI, NORM>), grid16, dim3(256), 0, s, af, wf, (float *)c,
                               (float *)sink, M, N, K, rope, norm);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((gemm_f32_kernel<16, 1, 1, 4, 4, EPI, NORM>), grid16, dim3(256), 0, s, af, wf, (float *)c, (float *)sink, M, N,
                       K, rope, norm);
    return hipGetLastError();
}

}  // namespace

bool iso_gemm_f32_supported(const void *a, const void *w, int M, int N, int K) {
    return (K % 4) == 0 && ((uintptr_t)a | (uintptr_t)w) % 16 == 0 && (M + 15) / 16 <= 65535;
}

bool iso_gemm_f32_sink_supported(int M, int N) { return small_tiles(M, N); }

hipError_t iso_launch_gemm_f32(const void *a, const void *w, void *c, void *sink, int M, int N, int K, hipStream_t s) {
    return launch_f32<EPI_NONE>(a, w, c, sink, M, N, K, RopeF32{}, NormF32{}, s);
}

// The projections behind a norm take the norm's inputs instead of its output where that is not behind the norm kernel: every column
// tile computes the norm again, against one launch and one trip to memory saved.  Layers of seven shapes, 1 to 2048 tokens, us a
// layer with the norm kernel / in the projection:
//   * Gate/up, whose norm adds two rows and whose tiles hold two blocks of W: K <= 256 and two tiles for every unit.  K = 256: 128
//     tokens (344 tiles) 29.2 / 28.8, 160 (430) 31.0 / 30.4, 192 (516) 34.0 / 34.4, 777 (2107) 66.6 / 69.8; K = 128: 333 tokens
//     (462) 31.6 / 30.6.  Beyond K = 256 a wave holds twelve rounds of everything and never gains: K = 512, 32 tokens 38.0 / 38.9, 64
//     42.6 / 47.1, 512 122 / 166; K = 768, 400 tokens 191 / 253.
//   * QKV: K <= 256 always, beyond it four tiles for every unit.  K = 256: 128 tokens 30.6 / 29.2, 777 69.1 / 66.6; K = 512: 333
//     tokens (1008 tiles) 94.8 / 93.1; K = 264: 640 tokens (640) 78.2 / 78.4, 1472 (1472) 135.0 / 137.8.
bool iso_gemm_f32_norm_supported(const iso_norm_args &norm, int M, int n_out, int K) {
    const long long tiles = (long long)((M + 15) / 16) * ((n_out + 15) / 16), units = iso_num_cu();
    if (norm.delta ? K > norm_max_k(NORM_X_DELTA) || tiles > 2 * units : K > 256 && (K > norm_max_k(NORM_X) || tiles > 4 * units))
        return false;
    return small_tiles(M, n_out) && ((uintptr_t)norm.x | (uintptr_t)norm.delta | (uintptr_t)norm.g) % 16 == 0;
}

hipError_t iso_launch_gemm_swiglu_f32(const void *a, const void *w, void *act, int M, int F, int K, const iso_norm_args *norm,
                                      hipStream_t s) {
    if (!norm) return launch_f32<EPI_SWIGLU>(a, w, act, nullptr, M, 2 * F, K, RopeF32{}, NormF32{}, s);
    const NormF32 nf{(const float *)norm->delta, (const float *)norm->g, norm->eps};
    return norm->delta ? launch_f32<EPI_SWIGLU, NORM_X_DELTA>(norm->x, w, act, nullptr, M, 2 * F, K, RopeF32{}, nf, s)
                       : launch_f32<EPI_SWIGLU, NORM_X>(norm->x, w, act, nullptr, M, 2 * F, K, RopeF32{}, nf, s);
}

// QKV projection with rotary embedding and KV-cache write in its epilogue (the k and v columns of qkv are not written): one
// launch less for the small tiles (128 tokens, 12 heads of 64: 4.6 + 2.5 -> 5.0 us and a gap); larger products keep the two
// kernels.
bool iso_gemm_rope_f32_supported(const void *a, const void *w, int M, int N, int K) {
    return iso_gemm_f32_supported(a, w, M, N, K) && small_tiles(M, N);
}

hipError_t iso_launch_gemm_rope_f32(const void *a, const void *w, void *qkv, int M, int K, const iso_norm_args *norm,
                                    const iso_rope_args &rp, hipStream_t s) {
    const RopeF32 rope{rp.cos_t, rp.sin_t, (float *)rp.k_cache, (float *)rp.v_cache, rp.q_offset, rp.nq, rp.nkv, rp.d};
    const int N = (rp.nq + 2 * rp.nkv) * rp.d;
    if (!norm) return launch_f32<EPI_ROPE>(a, w, qkv, nullptr, M, N, K, rope, NormF32{}, s);
    if (norm->delta) return hipErrorInvalidValue;
    return launch_f32<EPI_ROPE, NORM_X>(norm->x, w, qkv, nullptr, M, N, K, rope,
                                        NormF32{nullptr, (const float *)norm->g, norm->eps}, s);
}

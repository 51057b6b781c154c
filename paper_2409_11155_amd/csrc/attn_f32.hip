// Chunk attention over the KV cache in fp32 on the fp32 matrix instructions (v_mfma_f32_16x16x4_f32).  Local query row i is
// token q_offset + i and sees keys j <= q_offset + i, j < kv_len.  (Chunk over the cache written by the earlier chunk: paper
// Section 3.1.)
//
// One workgroup = 16 query rows of one head; its waves take the key tiles in turn and merge their online softmax states through
// LDS: heads of 64 four waves up to 128 keys and eight above, tiles of 32 keys; heads of 128 four waves, tiles of 64.  Scores are
// computed transposed, S^T = K Q^T: a lane then holds four keys of one query per 16-key block, the softmax statistics are per-lane
// scalars up to two lane exchanges, and its probabilities are already the B operand of O^T = V^T P^T (instruction r takes the keys
// 4 (lane / 16) + r), so nothing is rearranged.  K and Q rows are fetched four dims at a time (16 bytes per lane); V one dim per
// lane, 64 contiguous bytes per 16 lanes.
// Bound by the trips to memory of a few waves.  Measured on 128 tokens, 4 heads: heads of 64 5.8 us, heads of 128 10.1, against
// 18 and 22 us of the kernel that gives every query row a wave and every lane a whole key row (which is ahead over a handful of
// keys, see attention() in iso_api.hip).
#include "attn_row.h"

namespace {

constexpr int QB = 16;               // query rows per workgroup

template <int D, int KB, int NW>     // KB keys per tile, NW waves
__global__ __launch_bounds__(NW * 64) void attn_f32_kernel(const float *__restrict__ Q, const float *__restrict__ Kc,
                                                       const float *__restrict__ Vc, float *__restrict__ Out, int Tc,
                                                       int q_offset, int kv_len, int nq, int nkv, int q_stride) {
    constexpr int DS = D / 16;       // 16-dim steps of a score (four instructions each), 16-dim blocks of an output
    __shared__ float so[NW][QB][D + 4];
    __shared__ float sm[NW][QB], sl[NW][QB];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, grp = lane >> 4;
    const int i0 = ((int)gridDim.x - 1 - (int)blockIdx.x) * QB;      // longest rows first
    const int h = blockIdx.y, g = h / (nq / nkv);
    const float scale = 1.0f / sqrtf((float)D);
    const int q_abs = q_offset + i0 + col;
    f32x4_t qf[DS];
    {
        const float *qp = Q + (size_t)min(i0 + col, Tc - 1) * q_stride + (size_t)h * D + 4 * grp;
#pragma unroll
        for (int s = 0; s < DS; ++s) qf[s] = *reinterpret_cast<const f32x4_t *>(qp + 16 * s) * scale;
    }
    const size_t row = (size_t)nkv * D;
    const float *kp = Kc + (size_t)g * D + 4 * grp, *vp = Vc + (size_t)g * D + col;
    const int n_vis = min(kv_len, q_offset + min(i0 + QB, Tc));
    f32x4_t o[DS];
#pragma unroll
    for (int d = 0; d < DS; ++d) o[d] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;
    for (int j0 = wave * KB; j0 < n_vis; j0 += NW * KB) {
        f32x4_t sc[KB / 16];
        // V is requested along with K, so that a tile is one trip to memory (D = 128 has no registers for that).
        // Rows past the visible keys of every query here have probability zero, but must not bring a NaN: clamp.
        constexpr bool EARLY_V = D == 64;
        float vf[EARLY_V ? KB / 16 : 1][4][DS];
        auto load_v = [&](int b, float (&dst)[4][DS]) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float *vr = vp + (size_t)min(j0 + 16 * b + 4 * grp + r, n_vis - 1) * row;
#pragma unroll
                for (int d = 0; d < DS; ++d) dst[r][d] = vr[16 * d];
            }
        };
#pragma unroll
        for (int b = 0; b < KB / 16; ++b) {
            if (EARLY_V) load_v(b, vf[EARLY_V ? b : 0]);
            const float *kr = kp + (size_t)min(j0 + 16 * b + col, n_vis - 1) * row;
            f32x4_t kf[DS];
#pragma unroll
            for (int s = 0; s < DS; ++s) kf[s] = *reinterpret_cast<const f32x4_t *>(kr + 16 * s);
            sc[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < DS; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j) sc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[s][j], qf[s][j], sc[b], 0, 0, 0);
        }
        float mx = -INFINITY;
#pragma unroll
        for (int b = 0; b < KB / 16; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int key = j0 + 16 * b + 4 * grp + r;
                if (key > q_abs || key >= kv_len) sc[b][r] = -INFINITY;
                mx = fmaxf(mx, sc[b][r]);
            }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m, mx);
        const float base = m_new == -INFINITY ? 0.f : m_new;         // no visible key so far: all probabilities are zero
        const float alpha = expf(m - base);
        float psum = 0.f;
#pragma unroll
        for (int b = 0; b < KB / 16; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                sc[b][r] = expf(sc[b][r] - base);
                psum += sc[b][r];
            }
        l = l * alpha + psum;
        m = m_new;
#pragma unroll
        for (int d = 0; d < DS; ++d) o[d] *= alpha;
#pragma unroll
        for (int b = 0; b < KB / 16; ++b) {
            if (!EARLY_V) load_v(b, vf[0]);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int d = 0; d < DS; ++d)
                    o[d] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[EARLY_V ? b : 0][r][d], sc[b][r], o[d], 0, 0, 0);
        }
    }
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (grp == 0) {
        sm[wave][col] = m;
        sl[wave][col] = l;
    }
#pragma unroll
    for (int d = 0; d < DS; ++d) *reinterpret_cast<f32x4_t *>(&so[wave][col][16 * d + 4 * grp]) = o[d];
    __syncthreads();
    for (int q = wave; q < QB && i0 + q < Tc; q += NW) {             // a wave per row
        float mt = sm[0][q];
#pragma unroll
        for (int w = 1; w < NW; ++w) mt = fmaxf(mt, sm[w][q]);
        float num[D / 64] = {}, den = 0.f, probe = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float f = expf(sm[w][q] - mt);                     // a wave without keys has m = -inf and weight zero
#pragma unroll
            for (int r = 0; r < D / 64; ++r) num[r] += so[w][q][lane + 64 * r] * f;
            den += sl[w][q] * f;
        }
        float *op = Out + ((size_t)(i0 + q) * nq + h) * D;
#pragma unroll
        for (int r = 0; r < D / 64; ++r) {
            num[r] /= den;
            op[lane + 64 * r] = num[r];
            probe = fmaf(num[r], 0.f, probe);
        }
        // A key that a row does not see has probability zero there, but 0 x infinity and 0 x NaN in the second product are
        // NaN: a row with a result that is not finite, and such a key behind it, is computed again from the keys it sees --
        // unless the sum of its probabilities, which come from visible keys alone, is NaN as well.
        int at;
        if (__builtin_amdgcn_ballot_w64(probe != 0.f && den == den) != 0 &&
            attn_rows_not_finite<float, D>(Vc + (size_t)g * D, row, q_offset + i0 + q + 1, n_vis, lane, &at)) {
            __builtin_amdgcn_s_waitcnt(0);                           // the stores above come first
            const float *qp = Q + (size_t)(i0 + q) * q_stride + (size_t)h * D;
            attn_row<float, D>([&](int e) { return qp[e] * scale; }, Kc + (size_t)g * D, Vc + (size_t)g * D, row,
                               min(kv_len, q_offset + i0 + q + 1), op, lane);
        }
    }
}

}  // namespace

hipError_t iso_launch_attn_f32(const void *q, const void *k, const void *v, void *out, int Tc, int q_offset, int kv_len, int nq,
                               int nkv, int d, int q_stride, hipStream_t s) {
    const dim3 grid((Tc + QB - 1) / QB, nq);
    const float *qf = (const float *)q, *kf = (const float *)k, *vf = (const float *)v;
    if (d == 64 && kv_len <= 128)
        hipLaunchKernelGGL((attn_f32_kernel<64, 32, 4>), grid, dim3(256), 0, s, qf, kf, vf, (float *)out, Tc, q_offset, kv_len, nq,
                           nkv, q_stride);
    else if (d == 64)
        hipLaunchKernelGGL((attn_f32_kernel<64, 32, 8>), grid, dim3(512), 0, s, qf, kf, vf, (float *)out, Tc, q_offset, kv_len, nq,
                           nkv, q_stride);
    else if (d == 128)
        hipLaunchKernelGGL((attn_f32_kernel<128, 64, 4>), grid, dim3(256), 0, s, qf, kf, vf, (float *)out, Tc, q_offset, kv_len, nq,
                           nkv, q_stride);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

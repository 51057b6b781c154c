// One query row of one head by one wavefront, over the visible keys only: online softmax over 64-key slices, fp32
// throughout.  The kernel of attn_simple.hip is this for every row; the matrix-core kernels, whose tiles multiply the values
// of a key by the zero probability of a row that does not see it, come here for rows whose result is not finite.
#pragma once
#include "iso_internal.h"

template <typename T> __device__ __forceinline__ float attn_row_exp(float z);
template <> __device__ __forceinline__ float attn_row_exp<float>(float z) { return expf(z); }
template <> __device__ __forceinline__ float attn_row_exp<bf16_t>(float z) { return __expf(z); }

// q(e): element e of the scaled query; kc / vc: first row of the head's slice, `stride` elements between rows; keys
// [0, n_vis).  D = head_dim (64 or 128): lane l owns output dims l, l + 64 (D = 128) or l (D = 64).
template <typename T, int D, typename Q>
__device__ __forceinline__ void attn_row(Q &&q, const T *kc, const T *vc, size_t stride, int n_vis, T *out, int lane) {
    constexpr int PER = D / 64;
    float o[PER] = {};
    float m = -INFINITY, l = 0.f;
#pragma nounroll
    for (int j0 = 0; j0 < n_vis; j0 += 64) {
        const int j = j0 + lane;
        float sc = -INFINITY;
        if (j < n_vis) {
            const T *kr = kc + (size_t)j * stride;
            float acc = 0.f;
#pragma unroll 8
            for (int e = 0; e < D; ++e) acc = fmaf(q(e), iso_to_f32(kr[e]), acc);
            sc = acc;
        }
        const float m_new = fmaxf(m, iso_wave_max(sc));
        const float p = (j < n_vis) ? attn_row_exp<T>(sc - m_new) : 0.f;
        const float alpha = attn_row_exp<T>(m - m_new);     // m = -inf on the first slice gives 0
        l = l * alpha + iso_wave_sum(p);
#pragma unroll
        for (int r = 0; r < PER; ++r) o[r] *= alpha;
        const int cnt = min(64, n_vis - j0);
        for (int jj = 0; jj < cnt; ++jj) {
            const float pj = __shfl(p, jj, 64);
            const T *vr = vc + (size_t)(j0 + jj) * stride;
#pragma unroll
            for (int r = 0; r < PER; ++r) o[r] = fmaf(pj, iso_to_f32(vr[lane + 64 * r]), o[r]);
        }
        m = m_new;
    }
    const float inv = 1.0f / l;
#pragma unroll
    for (int r = 0; r < PER; ++r) out[lane + 64 * r] = iso_from_f32<T>(o[r] * inv);
}

// Whether one of the rows [lo, hi) of a head's V slice holds an infinity or a NaN; *last = the last such row.
template <typename T, int D>
__device__ __forceinline__ bool attn_rows_not_finite(const T *vc, size_t stride, int lo, int hi, int lane, int *last) {
    bool any = false;
    for (int j = lo; j < hi; ++j) {
        float probe = 0.f;
#pragma unroll
        for (int r = 0; r < D / 64; ++r) probe = fmaf(iso_to_f32(vc[(size_t)j * stride + lane + 64 * r]), 0.f, probe);
        if (__builtin_amdgcn_ballot_w64(probe != 0.f) == 0) continue;
        any = true;
        *last = j;
    }
    return any;
}

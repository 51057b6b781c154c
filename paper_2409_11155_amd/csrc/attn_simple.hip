// Chunk attention over the KV cache, one wavefront per (query row, query head): online softmax over
// 64-key slices, fp32 throughout.  It takes calls that see a handful of keys, caches too large for the
// 32-bit offsets of the tiles with heads of 64, and whatever ISO_FLAG_SIMPLE_ATTN forces here.  (Chunk over the cache written by the earlier chunk: paper
// Section 3.1; chunked prefill, Section 2.1.)
#include "attn_row.h"

namespace {

template <typename T, int D>
__global__ __launch_bounds__(256) void attn_simple_kernel(const T *__restrict__ q, const T *__restrict__ kc,
                                                          const T *__restrict__ vc, T *__restrict__ out, int Tc,
                                                          int q_offset, int kv_len, int nq, int nkv, int q_stride) {
    __shared__ float qs[4][D];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + wave;       // local query row
    const int h = blockIdx.y;
    const bool active = i < Tc;
    const int g = h / (nq / nkv);
    const float scale = 1.0f / sqrtf((float)D);
    if (active) {
        for (int e = lane; e < D; e += 64) qs[wave][e] = iso_to_f32(q[(size_t)i * q_stride + (size_t)h * D + e]) * scale;
    }
    __syncthreads();
    if (!active) return;
    int n_vis = q_offset + i + 1;
    if (n_vis > kv_len) n_vis = kv_len;
    const T *k0 = kc + (size_t)g * D, *v0 = vc + (size_t)g * D;
    attn_row<T, D>([&](int e) { return qs[wave][e]; }, k0, v0, (size_t)nkv * D, n_vis, out + ((size_t)i * nq + h) * D, lane);
}

}  // namespace

hipError_t iso_launch_attn_simple(int dtype, const void *q, const void *k, const void *v, void *out, int Tc,
                                  int q_offset, int kv_len, int nq, int nkv, int d, int q_stride, hipStream_t s) {
    dim3 grid((Tc + 3) / 4, nq), block(256);
#define ISO_ATTN_SIMPLE(TT, DD)                                                                              \
    hipLaunchKernelGGL((attn_simple_kernel<TT, DD>), grid, block, 0, s, (const TT *)q, (const TT *)k,        \
                       (const TT *)v, (TT *)out, Tc, q_offset, kv_len, nq, nkv, q_stride)
    if (dtype == ISO_F32 && d == 64) ISO_ATTN_SIMPLE(float, 64);
    else if (dtype == ISO_F32 && d == 128) ISO_ATTN_SIMPLE(float, 128);
    else if (dtype == ISO_BF16 && d == 64) ISO_ATTN_SIMPLE(bf16_t, 64);
    else if (dtype == ISO_BF16 && d == 128) ISO_ATTN_SIMPLE(bf16_t, 128);
    else return hipErrorInvalidValue;
#undef ISO_ATTN_SIMPLE
    return hipGetLastError();
}

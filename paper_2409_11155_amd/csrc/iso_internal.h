// Internal declarations shared by the HIP sources of libiso (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>
#include <mutex>

#include "iso.h"

typedef __bf16 bf16_t;
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

// Workspace of one stream-K GEMM in flight (flag words + one fp32 partial tile per workgroup).  Launches that
// share a workspace must be ordered (same stream); the context keeps one per stream of its own.  Host threads may enqueue
// products on the same stream: `lock` keeps a launch number with its launch, and the kernel that leaves partial sums next to
// the one that adds them.
struct iso_sk_ws {
    void *base;        // device; flag words zeroed once at creation, never reset (each launch uses a new epoch)
    unsigned *err;     // pinned host word the kernel sets if a bounded wait ran out
    unsigned epoch;    // launch counter
    int num_wg;        // grid size = compute units of the device
    std::mutex lock;
};

// Workspace of the attention launches that split the keys of a row block across workgroups: partial states and one
// arrival counter per (row block, head).  Counters are zero between launches (the last arriver resets its own).
// Launches that share a workspace must be ordered (same stream); the context keeps one per stream of its own.
struct iso_attn_ws {
    unsigned char *part;   // device, max_slots * iso_attn_part_bytes()
    unsigned *cnt;         // device, max_blocks words, zeroed at creation
    int max_slots;         // (row block, head, share) triples a launch may use
    int max_blocks;        // (row block, head) pairs a launch may use
};

struct iso_ctx {
    iso_cfg cfg;
    int device;
    int flags;
    hipStream_t stream[2];
    hipStream_t xstream[ISO_MAX_CHUNKS];   // own streams for chunks 2.. of ISO_SCHED_STREAM_PER_CHUNK, made on first use
    hipEvent_t ev_fork, ev_join[ISO_MAX_CHUNKS], ev_kv[ISO_MAX_CHUNKS];
    size_t elt;        // bytes per element
    // device workspace, each sized for max_seq tokens; chunks use disjoint row ranges
    void *ws;          // one allocation
    size_t ws_bytes;
    void *y;           // [max_seq, hidden]   normed activations (both norms)
    void *qkv;         // [max_seq, n_qkv]
    void *attn;        // [max_seq, nq*d]
    void *part;        // [max_seq, hidden]   row-parallel partial of the attention block (o_proj)
    void *part_m;      // [max_seq, hidden]   row-parallel partial of the MLP block (down); both live until the layer closes
    void *gu;          // [max_seq, 2*ffn]
    void *act;         // [max_seq, ffn]
    signed char *q8;   // [max_seq, hidden + 16] int8 codes + fp32 scale per row (ISO_COMM_D2H_INT8)
    unsigned char *a8; // [max_seq, max(hidden, nq*d, ffn)] FP8 copy of the current projection input (bf16 contexts)
    float *a8s;        // [max_seq] its row scales
    size_t a8_pitch;   // bytes per token of a8
    float *rope_cos;   // [max_seq, d/2]
    float *rope_sin;   // [max_seq, d/2]
    int gemm_segments; // launches per projection GEMM along M (0 or 1: one launch)
    int sk_hold;       // set while a pass enqueues work for which stream-K is not to be picked
    int side_by_side;  // set while a pass enqueues chunks whose kernels share the chip all the time
    // GEMM workspaces (bf16 contexts only; base == null otherwise): [0], [1] for the caller's streams, used by the stream-K
    // launch and by split products; [k] for xstream[k], split products only
    iso_sk_ws sk[ISO_MAX_CHUNKS];
    iso_sk_ws sk_rec[2];                // the same for layers recorded into a HIP graph on the caller's streams, split products only
    iso_attn_ws aws[ISO_MAX_CHUNKS];   // key-split attention workspaces: [0], [1] for the caller's streams, [k] for xstream[k]
    void *host_sink;   // pinned, 2 * max_seq * hidden elements
    // optional per-launch timing (iso_timing_*): event pairs recorded around every launch, in its stream
    int timing;
    int n_tev, n_tev_created;
    hipEvent_t *tev0, *tev1;
    int *tkind;
};
constexpr int ISO_MAX_TIMED = 65536;

// ---- launchers; each validates nothing (callers do) and returns the launch status -------------
// x_new = x (+ delta (+ delta2)); x_out (may be x) receives it when given; y = rmsnorm(x_new) * g when given
hipError_t iso_launch_rmsnorm(int dtype, const void *x, const void *delta_or_null, const void *delta2_or_null,
                              void *x_out_or_null, const void *g, void *y_or_null, int T, int H, float eps, hipStream_t s);
hipError_t iso_launch_rope_kv(int dtype, void *qkv, void *k_cache, void *v_cache, const float *cos_t,
                              const float *sin_t, int Tc, int q_offset, int nq, int nkv, int d, hipStream_t s);
hipError_t iso_launch_quant_rows(int dtype, void *part, void *q8, int T, int H, hipStream_t s);
hipError_t iso_launch_copy_out(void *dst_pinned, const void *src, size_t bytes, hipStream_t s);
hipError_t iso_launch_swiglu(int dtype, const void *gu, void *a, int T, int F, hipStream_t s);
hipError_t iso_launch_gemm_simple(int dtype, const void *a, const void *w, void *c, int M, int N, int K,
                                  hipStream_t s);
// fp32 matrix instructions; *_supported: K % 4 == 0, 16-byte aligned operands
bool iso_gemm_f32_supported(const void *a, const void *w, int M, int N, int K);
bool iso_gemm_f32_sink_supported(int M, int N);
// sink_or_null: pinned host memory that receives c as well
hipError_t iso_launch_gemm_f32(const void *a, const void *w, void *c, void *sink_or_null, int M, int N, int K, hipStream_t s);
// Where the rotary step and the KV-cache write of a QKV projection go (W = [q heads | k heads | v heads] x d rows).
struct iso_rope_args {
    const float *cos_t, *sin_t;      // [max_seq, d/2]
    void *k_cache, *v_cache;         // [max_seq, nkv, d]
    int q_offset, nq, nkv, d;
};
// A projection's operand rmsnorm(x (+ delta)) * g, computed by the projection (then its `a` is not looked at).
struct iso_norm_args {
    const void *x, *delta, *g;       // delta may be null
    float eps;
};
bool iso_gemm_f32_norm_supported(const iso_norm_args &norm, int M, int n_out, int K);
hipError_t iso_launch_gemm_swiglu_f32(const void *a, const void *w, void *act, int M, int F, int K, const iso_norm_args *norm_or_null,
                                      hipStream_t s);
bool iso_gemm_rope_f32_supported(const void *a, const void *w, int M, int N, int K);
hipError_t iso_launch_gemm_rope_f32(const void *a, const void *w, void *qkv, int M, int K, const iso_norm_args *norm_or_null,
                                    const iso_rope_args &rope, hipStream_t s);
hipError_t iso_launch_attn_f32(const void *q, const void *k, const void *v, void *out, int Tc, int q_offset, int kv_len, int nq,
                               int nkv, int d, int q_stride, hipStream_t s);
hipError_t iso_launch_gemm_bf16_mfma(const void *a, const void *w, void *c, int M, int N, int K, hipStream_t s);
bool iso_gemm_bf16_mfma_supported(int M, int N, int K);
hipError_t iso_launch_gemm_bf16_dtl(const void *a, const void *w, void *c, int M, int N, int K, int variant,
                                    iso_sk_ws *sk_or_null, hipStream_t s);
bool iso_gemm_bf16_dtl_supported(int M, int N, int K);
// which variant (1..6; -1: none; +8: plain main loop) a launch with `variant` resolves to
int iso_gemm_bf16_dtl_resolve(int M, int N, int K, int variant, const iso_sk_ws *sk_or_null);
// Residual added by the product whose result closes the layer: x += pa + bf16(result) (x, pa: [M,N]); x null: none, the result is
// stored.
struct iso_resid_args {
    void *x;
    const void *pa;
};
// Tiles of 256 columns (gemm_pp_kernel.h): bm = 256, 192 or 128 rows; bf16 operands, or FP8 ones with their row scales sa, sw.
enum { ISO_PP_PLAIN = 0, ISO_PP_SWIGLU = 1, ISO_PP_ROPE = 2, ISO_PP_SHARE = 3, ISO_PP_RESID = 4 };
struct iso_pp_args {
    const void *a, *w;
    const float *sa, *sw;            // null: bf16
    void *c;                         // [M,N] (ISO_PP_SWIGLU: [M,N/2]; ISO_PP_ROPE: the q columns of [M,N])
    float *p;                        // ISO_PP_SHARE: [shares][M][N] partial sums
    int M, N, K, shares;
    iso_rope_args rope;              // ISO_PP_ROPE, head_dim 64 or 128
    iso_resid_args resid;            // ISO_PP_RESID
};
hipError_t iso_launch_gemm_pp(int bm, int epi, const iso_pp_args &o, hipStream_t s);
// QKV projection with rotary embedding + KV-cache write in the epilogue: of the 128 x 128 tile (bf16, head_dim 64) and of the
// stream-K launch (bf16, head_dim 128)
hipError_t iso_launch_gemm_qkv_rope_bf16_128(const void *a, const void *w, void *qkv, int M, int N, int K, const iso_rope_args &rope,
                                             hipStream_t s);
hipError_t iso_launch_gemm_qkv_rope_bf16_sk(const void *a, const void *w, void *qkv, int M, int N, int K, iso_sk_ws *sk,
                                            const iso_rope_args &rope, hipStream_t s);
hipError_t iso_launch_gemm_swiglu_bf16(const void *a, const void *w, void *act, int M, int F, int K, int variant,
                                       iso_sk_ws *sk_or_null, hipStream_t s);
void iso_gemm_bf16_dtl_plan(int M, int N, int K, int num_wg, int *kind, int *team, int *grid);
size_t iso_gemm_sk_ws_bytes(int num_wg);   // device bytes a stream-K workspace for num_wg workgroups needs
size_t iso_gemm_sk_slot_bytes(void);       // of which behind the flag words, per workgroup
int iso_gemm_sk_max_wg(void);
bool iso_gemm_swiglu_bf16_supported(int M, int F, int K);
bool iso_gemm_fp8_supported(int M, int N, int K);
bool iso_rmsnorm_fp8_supported(int H);
hipError_t iso_launch_rmsnorm_fp8(const void *x, const void *delta_or_null, const void *delta2_or_null, void *x_out_or_null,
                                  const void *g, void *q8, float *q_scale, int T, int H, float eps, hipStream_t s);
hipError_t iso_launch_quant_rows_fp8(const void *x, void *q, float *scale, int rows, int cols, hipStream_t s);
hipError_t iso_launch_gemm_fp8(const void *a8, const float *sa, const void *w8, const float *sw, void *c, int M, int N,
                               int K, int variant, iso_sk_ws *sk_or_null, hipStream_t s);
hipError_t iso_launch_gemm_swiglu_fp8(const void *a8, const float *sa, const void *w8, const float *sw, void *act, int M,
                                      int F, int K, int variant, iso_sk_ws *sk_or_null, hipStream_t s);
// What a projection is launched as.  tile >= 0: a tile shape of gemm_split.hip with the k range in `shares` parts (more than
// one share, and the rotary form always, needs a workspace); tile < 0: variant `whole` of the whole-tile kernels.
struct iso_split_plan {
    int tile, shares, whole;
};
iso_split_plan iso_gemm_split_plan(bool fp8, int rope, int whole, int M, int N, int K, size_t ws_bytes, int ncu, bool shared,
                                   double *us_or_null = nullptr);
int iso_gemm_fp8_whole(int M, int N, int K, const iso_sk_ws *sk_or_null);   // the FP8 rule's variant (1, 3 or 6)
int iso_gemm_fp8_resolve(int M, int N, int K, int variant, const iso_sk_ws *sk_or_null);   // `variant`, or the rule's if it is none
bool iso_gemm_split_supported(bool fp8, int M, int N, int K);
// sa / sw null: bf16 operands, else FP8 operands and their row scales
hipError_t iso_launch_gemm_split(const iso_split_plan &plan, const void *a, const void *w, const float *sa, const float *sw,
                                 void *c, int M, int N, int K, iso_sk_ws *ws_or_null, const iso_resid_args &resid, hipStream_t s);
hipError_t iso_launch_gemm_split_swiglu(const iso_split_plan &plan, const void *a, const void *w, const float *sa,
                                        const float *sw, void *act, int M, int F, int K, iso_sk_ws *ws_or_null, hipStream_t s);
hipError_t iso_launch_gemm_split_rope(const iso_split_plan &plan, const void *a, const void *w, const float *sa, const float *sw,
                                      void *qkv, int M, int N, int K, iso_sk_ws *ws, const float *cos_t, const float *sin_t,
                                      void *k_cache, void *v_cache, int q_offset, int nq, int nkv, int d, hipStream_t s);
// stream-K with the workspace in a static device array (no allocation at call time)
hipError_t iso_gemm_static_setup(void);     // once per device, with that device current
size_t iso_gemm_static_scratch_bytes(void);
hipError_t iso_launch_gemm_bf16_sk_static(const void *a, const void *w, void *c, int M, int N, int K, unsigned *err_word,
                                          hipStream_t s);
// stream-K launch shape for nk k-slices (team size, grid, grouped mapping); returns the k-slices per team
long long iso_gemm_sk_plan(int M, int N, int nk, int num_wg, int *team, int *grid, int *grouped);
hipError_t iso_launch_attn_simple(int dtype, const void *q, const void *k, const void *v, void *out, int Tc,
                                  int q_offset, int kv_len, int nq, int nkv, int d, int q_stride, hipStream_t s);
hipError_t iso_launch_attn_bf16_mfma(const void *q, const void *k, const void *v, void *out, int Tc,
                                     int q_offset, int kv_len, int nq, int nkv, int d, int q_stride, hipStream_t s);
bool iso_attn_bf16_mfma_supported(int d);
hipError_t iso_launch_attn_bf16_dtl(const void *q, const void *k, const void *v, void *out, int Tc, int q_offset,
                                    int kv_len, int nq, int nkv, int d, int q_stride, int shape, int ksplit_req,
                                    const iso_attn_ws *ws_or_null, hipStream_t s);
// 32-row blocks, keys dealt to the waves of a workgroup; the cache as for the kernel above.  `keys`: the last row's
bool iso_attn_bf16_wave_wanted(int Tc, int nq, int d, long long keys);
hipError_t iso_launch_attn_bf16_wave(const void *q, const void *k, const void *v, void *out, int Tc, int q_offset, int kv_len,
                                     int nq, int nkv, int d, int q_stride, hipStream_t s);
size_t iso_attn_part_bytes(void);      // bytes of one partial state in an iso_attn_ws
bool iso_attn_bf16_dtl_supported(int d, int kv_len, int nkv);

// ---- small device helpers ----------------------------------------------------------------------
__device__ __forceinline__ float iso_to_f32(float v) { return v; }
__device__ __forceinline__ float iso_to_f32(bf16_t v) { return (float)v; }
template <typename T> __device__ __forceinline__ T iso_from_f32(float v);
template <> __device__ __forceinline__ float iso_from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t iso_from_f32<bf16_t>(float v) { return (bf16_t)v; }  // RNE

__device__ __forceinline__ float iso_wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
// Raises a kernel's dynamic-LDS limit once per device (the attribute belongs to the function on the device that is
// current when it is set).  `done` is the caller's static mask of devices already served; ids beyond 63 are set every
// time.  Called from launchers only; host threads may race here (setting the attribute twice is harmless, the mask is
// atomic).
typedef std::atomic<unsigned long long> iso_dev_mask;
inline hipError_t iso_allow_lds(const void *kernel, int bytes, iso_dev_mask *done) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64 && ((done->load(std::memory_order_acquire) >> dev) & 1ull)) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess && dev >= 0 && dev < 64) done->fetch_or(1ull << dev, std::memory_order_release);
    return e;
}
// Compute units of the current device (looked up once per device; 256 if the query fails).
inline int iso_num_cu(void) {
    static std::atomic<int> ncu_of[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
    int n = ncu_of[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
        ncu_of[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

__device__ __forceinline__ float iso_wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

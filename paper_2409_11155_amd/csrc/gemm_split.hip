// Projections that a tile per compute unit cannot fill the chip with: short prompts (bound by the bytes of the weights)
// and narrow matrices.   c[M,N] = a[M,K] * w[N,K]^T  for bf16 and FP8 operands.  (Projections of the layer: paper
// Sections 2.2 and 4.1.)
//
// Two remedies, chosen together by a cost model (iso_gemm_split_plan below):
//   * smaller tiles (32 / 64 / 128 rows x 64 columns), gemm_narrow_kernel;
//   * the k range of a tile dealt to S workgroups, each of which leaves its fp32 partial sums in a workspace [S][M][N];
//     a second kernel adds them in the order of the shares (the result does not depend on who ran when) and does the
//     step that follows the projection on the way: nothing, SwiGLU, or rotary embedding + KV-cache write.
#include <math.h>

#include <algorithm>

#include "gemm_dtl_kernel.h"

namespace {

enum { EPI_BF16 = 0, EPI_SWIGLU = 1, EPI_PARTIAL = 2 };

// Workgroup tile BM x BN, NS LDS stages of one 128-byte k slice each for A and W.  The waves split the K-STEPS of a slice
// (KW of them) and, where there are more waves than k-steps, the columns: a wave multiplies all BM rows of its k-step, so
// every byte of the tile is read from LDS once (a spatial split of 128 x 64 over four waves reads it twice), and the KW
// partial tiles are added through LDS at the end.  With NS - 1 slices requested ahead a compute unit keeps 64 .. 120 KB
// of loads in flight, which is what streaming weights from HBM at full rate takes (21 KB per microsecond and unit).
template <typename OP, int BM_, int BN_, int NS_, int OCC_> struct NarrowCfg {
    static constexpr int BM = BM_, BN = BN_, NS = NS_, OCC = OCC_;
    static constexpr int KW = 8 / OP::CPS, NW = 4, WN = NW / KW, NT = NW * 64;
    static constexpr int STAGE = (BM + BN) * ROW_BYTES;
    static constexpr int A_LOADS = BM / 8 / NW, W_LOADS = BN / 8 / NW, LOADS = A_LOADS + W_LOADS;
    static constexpr int FM = BM / 32, WCOLS = BN / WN, FN = WCOLS / 32;
    static constexpr int EP = BN + 8;                                  // fp32 pitch of the staged rows (two-way conflicts at most)
    static constexpr int EPI_BYTES = KW * 32 * EP * 4;
    static constexpr int LDS_BYTES = NS * STAGE > EPI_BYTES ? NS * STAGE : EPI_BYTES;
    static_assert(LDS_BYTES * OCC <= 160 * 1024 && NW % KW == 0 && A_LOADS >= 1 && W_LOADS >= 1 && FN >= 1, "shape");
    static_assert((NS - 1) * LOADS < 64, "outstanding loads are counted in six bits");
};

// Eight results of a row as bf16 to c + at; or, with a residual (the layer's last step), x = (x + pa) + that, in fp32 and in the
// order of the residual kernel.
__device__ __forceinline__ void store_row_piece(const float (&v)[8], bf16_t *__restrict__ c, size_t at, const iso_resid_args &resid) {
    bf16x8_t o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (bf16_t)v[e];
    if (resid.x) {
        bf16_t *x = (bf16_t *)resid.x + at;
        const bf16x8_t xv = *reinterpret_cast<const bf16x8_t *>(x), pv = *reinterpret_cast<const bf16x8_t *>((const bf16_t *)resid.pa + at);
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (bf16_t)((float)xv[e] + (float)pv[e] + (float)o[e]);
        *reinterpret_cast<bf16x8_t *>(x) = o;
    } else {
        *reinterpret_cast<bf16x8_t *>(c + at) = o;
    }
}

template <typename Cfg, typename OP, int EPI>
__global__ __launch_bounds__(Cfg::NT, Cfg::OCC) void gemm_narrow_kernel(const typename OP::elem *__restrict__ A,
                                                                        const typename OP::elem *__restrict__ W,
                                                                        const float *__restrict__ sa,
                                                                        const float *__restrict__ sw,
                                                                        bf16_t *__restrict__ C, float *__restrict__ P, int M,
                                                                        int N, int K, int tiles_m, int tiles_n, int S,
                                                                        iso_resid_args resid) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int BM = Cfg::BM, BN = Cfg::BN, NS = Cfg::NS, NW = Cfg::NW, KW = Cfg::KW, FM = Cfg::FM, FN = Cfg::FN;
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = wave % KW, wn = wave / KW;

    // workgroup -> (share, tile column, tile row): each XCD gets a contiguous range, tile rows fastest (neighbours read the
    // same weights), shares slowest (an XCD reads few k ranges of A)
    int pid = blockIdx.x;
    const int per_xcd = gridDim.x / 8;
    if (pid < per_xcd * 8) pid = (pid % 8) * per_xcd + pid / 8;
    const int tile_m = pid % tiles_m, tile_n = (pid / tiles_m) % tiles_n, share = pid / (tiles_m * tiles_n);
    const int nk = K / OP::KE;
    const int kb = (int)((long long)nk * share / S), n = (int)((long long)nk * (share + 1) / S) - kb;
    const int m0 = tile_m * BM, n0 = tile_n * BN;

    const int ld_row = lane >> 3, ld_slot = lane & 7;
    const int a_bytes = (int)((uint32_t)M * (uint32_t)K * (uint32_t)OP::EB);
    const int w_bytes = (int)((uint32_t)N * (uint32_t)K * (uint32_t)OP::EB);
    uint32_t a_off[Cfg::A_LOADS], w_off[Cfg::W_LOADS];
#pragma unroll
    for (int i = 0; i < Cfg::A_LOADS; ++i) {
        const int r = (wave + NW * i) * 8 + ld_row;
        a_off[i] = (uint32_t)min(m0 + r, M - 1) * (uint32_t)K * (uint32_t)OP::EB + (uint32_t)((ld_slot ^ swz(r)) << 4);
    }
#pragma unroll
    for (int i = 0; i < Cfg::W_LOADS; ++i) {
        const int r = (wave + NW * i) * 8 + ld_row;
        int grow;
        if (EPI == EPI_SWIGLU) {        // 32-column blocks alternate gate / up of the same 32 MLP columns
            const int F = N / 2, f = tile_n * (BN / 2) + (r / 64) * 32 + (r % 32);
            grow = ((r / 32) & 1) * F + min(f, F - 1);
        } else {
            grow = min(n0 + r, N - 1);
        }
        w_off[i] = (uint32_t)grow * (uint32_t)K * (uint32_t)OP::EB + (uint32_t)((ld_slot ^ swz(r)) << 4);
    }
    // a slice past the share's end is requested through an empty descriptor: nothing is fetched, the count of outstanding
    // loads stays the same to the end
    auto issue = [&](int i, int stage) {
        const bool real = i < n;
        const __amdgpu_buffer_rsrc_t rs_a = __builtin_amdgcn_make_buffer_rsrc((void *)A, 0, real ? a_bytes : 0, 0x00020000);
        const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)W, 0, real ? w_bytes : 0, 0x00020000);
        unsigned char *base = lds + stage * Cfg::STAGE;
        const int off = (kb + i) * ROW_BYTES;
#pragma unroll
        for (int j = 0; j < Cfg::W_LOADS; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs_w, (__attribute__((address_space(3))) void *)(base + BM * ROW_BYTES + (wave + NW * j) * 1024), 16, w_off[j],
                off, 0, 0);
#pragma unroll
        for (int j = 0; j < Cfg::A_LOADS; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs_a, (__attribute__((address_space(3))) void *)(base + (wave + NW * j) * 1024), 16, a_off[j], off, 0, 0);
    };

    f32x16_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    const int frow = lane & 31, fgrp = lane >> 5;
    const int f_sw = swz(frow), c0 = kw * OP::CPS + fgrp * OP::RPF;
    // The operands of slice i + 1 are read from LDS, and slice i + NS is requested into the stage that slice i has left,
    // while slice i is multiplied from registers: a wave alone on its SIMD has nobody else to fill its waits with.  (One after
    // the other, reading, requesting and multiplying took twice the 64 bytes a clock that a unit can take in: 128 x 64 at 40
    // workgroups 0.35 us a slice of 24 KB, now 0.25.)  400 x 2048 x 2048 10.9 -> 9.2 us, 200 x 1280 x 8192 17.5 -> 15.8; even
    // where two workgroups share the unit.
    typename OP::frag_t af[2][FM], wf[2][FN];
    auto read = [&](int stage, int buf) {
        const unsigned char *ab = lds + stage * Cfg::STAGE + frow * ROW_BYTES;
        const unsigned char *wb = ab + (BM + wn * Cfg::WCOLS) * ROW_BYTES;
#pragma unroll
        for (int j = 0; j < FN; ++j) wf[buf][j] = OP::load(wb + j * 32 * ROW_BYTES, c0, f_sw);
#pragma unroll
        for (int j = 0; j < FM; ++j) af[buf][j] = OP::load(ab + j * 32 * ROW_BYTES, c0, f_sw);
    };
    auto wait_for = [](auto pending_c) {            // vmcnt <= pending, lgkmcnt = 0
        constexpr int P = decltype(pending_c)::value;
        __builtin_amdgcn_s_waitcnt((P & 15) | ((P >> 4) << 14) | (7 << 4));
        asm volatile("s_barrier" ::: "memory");
    };
    for (int i = 0; i < NS; ++i) issue(i, i);
    wait_for(std::integral_constant<int, (NS - 1) * Cfg::LOADS>{});
    read(0, 0);
    int cur = 0;                                    // stage of slice i
    auto step = [&](int i, auto buf_c) {
        constexpr int B = decltype(buf_c)::value;
        // my part of slice i + 1 has landed and my reads of slice i are done, and everybody's
        wait_for(std::integral_constant<int, (NS - 2) * Cfg::LOADS>{});
        const int nx = cur + 1 == NS ? 0 : cur + 1;
        read(nx, B ^ 1);
        issue(i + NS, cur);
#pragma unroll
        for (int x = 0; x < FM; ++x)
#pragma unroll
            for (int y = 0; y < FN; ++y) acc[x][y] = OP::mfma32(af[B][x], wf[B][y], acc[x][y]);
        __builtin_amdgcn_sched_group_barrier(0x100, OP::RPF * (FM + FN), 0);       // the LDS reads, then the requests
        constexpr int PER = (Cfg::LOADS + FM * FN - 1) / (FM * FN);                // between the products
#pragma unroll
        for (int k = 0; k < FM * FN; ++k) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x020, PER, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        cur = nx;
    };
    int i = 0;
    for (; i + 1 < n; i += 2) {
        step(i, std::integral_constant<int, 0>{});
        step(i + 1, std::integral_constant<int, 1>{});
    }
    if (i < n) step(i, std::integral_constant<int, 0>{});
    __builtin_amdgcn_s_waitcnt(7 << 4);             // everything, so that the staging below may overwrite the stages

    // epilogue, 32 rows at a time: the KW partial blocks go to LDS, every thread adds the KW values of its outputs in
    // k-step order
    float *st = reinterpret_cast<float *>(lds);
    constexpr int EP = Cfg::EP;
#pragma unroll
    for (int x = 0; x < FM; ++x) {
        __syncthreads();
#pragma unroll
        for (int y = 0; y < FN; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                st[(kw * 32 + 8 * (r / 4) + 4 * fgrp + (r % 4)) * EP + wn * Cfg::WCOLS + y * 32 + frow] = acc[x][y][r];
        __syncthreads();
        if (EPI != EPI_SWIGLU) {
            constexpr int PPR = BN / 8;                               // pieces of eight columns per row
            for (int p = tid; p < 32 * PPR; p += Cfg::NT) {
                const int row = p / PPR, cc = (p % PPR) * 8;
                const int gm = m0 + x * 32 + row, gn = n0 + cc;
                if (gm >= M || gn >= N) continue;                     // N % 8 == 0
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = st[row * EP + cc + e];
#pragma unroll
                for (int k = 1; k < KW; ++k)
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] += st[(k * 32 + row) * EP + cc + e];
                if (EPI == EPI_PARTIAL) {
                    f32x4_t *o = reinterpret_cast<f32x4_t *>(P + ((size_t)share * M + gm) * N + gn);
                    o[0] = f32x4_t{v[0], v[1], v[2], v[3]};
                    o[1] = f32x4_t{v[4], v[5], v[6], v[7]};
                } else {
                    if constexpr (OP::SCALED) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] *= sa[gm] * sw[gn + e];
                    }
                    store_row_piece(v, C, (size_t)gm * N + gn, resid);
                }
            }
        } else {
            constexpr int PPR = BN / 2 / 4;                           // pieces of four MLP columns per row
            const int F = N / 2;
            for (int p = tid; p < 32 * PPR; p += Cfg::NT) {
                const int row = p / PPR, cc = (p % PPR) * 4;
                const int gm = m0 + x * 32 + row, gf = tile_n * (BN / 2) + cc;
                if (gm >= M || gf >= F) continue;                     // F % 8 == 0
                const int lc = (cc / 32) * 64 + (cc % 32);
                bf16x4_t o;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float g = 0.f, u = 0.f;
#pragma unroll
                    for (int k = 0; k < KW; ++k) {
                        g += st[(k * 32 + row) * EP + lc + e];
                        u += st[(k * 32 + row) * EP + lc + 32 + e];
                    }
                    if constexpr (OP::SCALED) {
                        g *= sa[gm] * sw[gf + e];
                        u *= sa[gm] * sw[F + gf + e];
                    }
                    o[e] = (bf16_t)(g / (1.0f + __expf(-g)) * u);
                }
                *reinterpret_cast<bf16x4_t *>(C + (size_t)gm * F + gf) = o;
            }
        }
    }
#endif
}

// The shares of the 128 x 128 tile of gemm_dtl_kernel.h (four waves, two workgroups per unit).
template <typename OP, int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(WM * WN * 64) void gemm_share_kernel(const typename OP::elem *__restrict__ A,
                                                                  const typename OP::elem *__restrict__ W,
                                                                  float *__restrict__ P, int M, int N, int K, int tiles_m,
                                                                  int tiles_n, int S) {
    gemm_dtl_body<OP, BM, BN, WM, WN, false, true, false, false, true>(A, W, nullptr, nullptr, nullptr, M, N, K, tiles_m,
                                                                       tiles_n, reinterpret_cast<unsigned char *>(P), 0u,
                                                                       nullptr, S, 0, RopeArgs{});
}

// ---- second kernels: sum of the shares, eight columns per thread --------------------------------------------------
struct Shares {
    const float *p;              // [S][M][N]
    size_t stride;               // M * N
    int S;
    const float *sa, *sw;        // FP8 row scales, or null
};
__device__ __forceinline__ void sum_shares(const Shares &sh, int row, int col, int N, float (&v)[8]) {
    const float *p = sh.p + (size_t)row * N + col;
    f32x4_t lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll 4
    for (int s = 0; s < sh.S; ++s) {
        lo += *reinterpret_cast<const f32x4_t *>(p + (size_t)s * sh.stride);
        hi += *reinterpret_cast<const f32x4_t *>(p + (size_t)s * sh.stride + 4);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) { v[e] = lo[e]; v[e + 4] = hi[e]; }
    if (sh.sa) {
        const float a = sh.sa[row];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] *= a * sh.sw[col + e];
    }
}

__global__ __launch_bounds__(256) void share_sum_kernel(Shares sh, bf16_t *__restrict__ C, int M, int N, iso_resid_args resid) {
    const int u = blockIdx.x * 256 + threadIdx.x, per_row = N / 8;
    const int row = u / per_row, col = (u % per_row) * 8;
    if (row >= M) return;
    float v[8];
    sum_shares(sh, row, col, N, v);
    store_row_piece(v, C, (size_t)row * N + col, resid);
}

__global__ __launch_bounds__(256) void share_sum_swiglu_kernel(Shares sh, bf16_t *__restrict__ act, int M, int F) {
    const int u = blockIdx.x * 256 + threadIdx.x, per_row = F / 8;
    const int row = u / per_row, col = (u % per_row) * 8;
    if (row >= M) return;
    float g[8], up[8];
    sum_shares(sh, row, col, 2 * F, g);
    sum_shares(sh, row, F + col, 2 * F, up);
    bf16x8_t o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (bf16_t)(g[e] / (1.0f + __expf(-g[e])) * up[e]);
    *reinterpret_cast<bf16x8_t *>(act + (size_t)row * F + col) = o;
}

// Rotary embedding and KV-cache write (same arithmetic and roundings as rope_kv_kernel: the projection output is rounded
// to bf16, rotated in fp32 and rounded again); the k and v columns of qkv are not written.
__global__ __launch_bounds__(256) void share_sum_rope_kernel(Shares sh, bf16_t *__restrict__ qkv, RopeArgs rope, int M, int d) {
    const int half = d / 2, N = (rope.nq + 2 * rope.nkv) * d;
    const int per_head = half / 8, per_row = (rope.nq + 2 * rope.nkv) * per_head;
    const int u = blockIdx.x * 256 + threadIdx.x;
    const int row = u / per_row;
    if (row >= M) return;
    const int head = (u % per_row) / per_head, i0 = (u % per_head) * 8, col = head * d + i0;
    float lo[8], hi[8];
    sum_shares(sh, row, col, N, lo);
    sum_shares(sh, row, col + half, N, hi);
    const size_t pos = (size_t)(rope.q_offset + row);
    bf16_t *dst = qkv + (size_t)row * N + col;
    if (head >= rope.nq + rope.nkv) dst = rope.v_cache + (pos * rope.nkv + (head - rope.nq - rope.nkv)) * d + i0;
    else if (head >= rope.nq) dst = rope.k_cache + (pos * rope.nkv + (head - rope.nq)) * d + i0;
    bf16x8_t olo, ohi;
    if (head >= rope.nq + rope.nkv) {
#pragma unroll
        for (int e = 0; e < 8; ++e) { olo[e] = (bf16_t)lo[e]; ohi[e] = (bf16_t)hi[e]; }
    } else {
        const float *cp = rope.cos_t + pos * half + i0, *sp = rope.sin_t + pos * half + i0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float l = (float)(bf16_t)lo[e], h = (float)(bf16_t)hi[e];
            olo[e] = (bf16_t)fmaf(l, cp[e], -(h * sp[e]));
            ohi[e] = (bf16_t)fmaf(h, cp[e], l * sp[e]);
        }
    }
    *reinterpret_cast<bf16x8_t *>(dst) = olo;
    *reinterpret_cast<bf16x8_t *>(dst + half) = ohi;
}

// ---- launchers ----------------------------------------------------------------------------------------------------
struct Operands {
    const void *a, *w;
    const float *sa, *sw;
    void *c;
    float *p;
    int M, N, K;
    iso_resid_args resid;
};

template <typename OP, typename Cfg, int EPI> hipError_t launch_narrow(const Operands &o, int S, hipStream_t s) {
    static iso_dev_mask lds_allowed{0};
    auto kern = gemm_narrow_kernel<Cfg, OP, EPI>;
    if (hipError_t e = iso_allow_lds(reinterpret_cast<const void *>(kern), Cfg::LDS_BYTES, &lds_allowed); e != hipSuccess)
        return e;
    const int tiles_m = (o.M + Cfg::BM - 1) / Cfg::BM, tiles_n = (o.N + Cfg::BN - 1) / Cfg::BN;
    typedef const typename OP::elem *ptr;
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n * S), dim3(Cfg::NT), Cfg::LDS_BYTES, s, (ptr)o.a, (ptr)o.w, o.sa, o.sw,
                       (bf16_t *)o.c, o.p, o.M, o.N, o.K, tiles_m, tiles_n, S, o.resid);
    return hipGetLastError();
}

template <typename OP, int BM, int BN, int WM, int WN> hipError_t launch_share(const Operands &o, int S, hipStream_t s) {
    using Cfg = DtlCfg<BM, BN, WM, WN>;
    constexpr int LDS_BYTES = Cfg::W3 ? Cfg::LDS_BYTES_W3 : Cfg::LDS_BYTES;
    static iso_dev_mask lds_allowed{0};
    auto kern = gemm_share_kernel<OP, BM, BN, WM, WN>;
    if (hipError_t e = iso_allow_lds(reinterpret_cast<const void *>(kern), LDS_BYTES, &lds_allowed); e != hipSuccess) return e;
    const int tiles_m = (o.M + BM - 1) / BM, tiles_n = (o.N + BN - 1) / BN;
    typedef const typename OP::elem *ptr;
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n * S), dim3(Cfg::NT), LDS_BYTES, s, (ptr)o.a, (ptr)o.w, o.p, o.M, o.N, o.K,
                       tiles_m, tiles_n, S);
    return hipGetLastError();
}

template <typename OP, int EPI> hipError_t launch_cfg(int cfg, const Operands &o, int S, hipStream_t s) {
    // A 128 x 64 tile that has its compute unit to itself takes six stages: 7 % at up to half the units busy, 2 % above.
    // (The two smaller tiles lose 4 % with all of the LDS: the launch before them has to leave a unit completely.)
    const bool alone = (long long)((o.M + 127) / 128) * ((o.N + 63) / 64) * S <= iso_num_cu();
    switch (cfg) {
        case 0: return launch_narrow<OP, NarrowCfg<OP, 32, 64, 6, 2>, EPI>(o, S, s);
        case 1: return launch_narrow<OP, NarrowCfg<OP, 64, 64, 5, 2>, EPI>(o, S, s);
        case 2: return alone ? launch_narrow<OP, NarrowCfg<OP, 128, 64, 6, 1>, EPI>(o, S, s)
                             : launch_narrow<OP, NarrowCfg<OP, 128, 64, 3, 2>, EPI>(o, S, s);
        default: break;
    }
    if constexpr (EPI == EPI_PARTIAL) {
        if (cfg == 3) return launch_share<OP, 128, 128, 2, 2>(o, S, s);
        if (cfg >= 4 && cfg <= 6)
            return iso_launch_gemm_pp(cfg == 4 ? 256 : cfg == 5 ? 192 : 128, ISO_PP_SHARE,
                                      iso_pp_args{o.a, o.w, o.sa, o.sw, nullptr, o.p, o.M, o.N, o.K, S, {}, {}}, s);
    }
    return hipErrorInvalidValue;
}

unsigned blocks_for(size_t units) { return (unsigned)((units + 255) / 256); }


// ---- which kernel ----------------------------------------------------------------------------------------------
// Microseconds of a launch, as fitted to 75 000 launches of 2434 products measured on MI355X (16 matrix shapes of the 30B / 70B shards
// and of a heads-of-64 layer with 58 row counts from 1 to 16384, 300 others with 8 to 16000 columns and k from 128 to 14336; narrow
// tiles whole up to four rounds of the chip, all tiles with 2 to 15 shares; every launch's weights from HBM, which takes a gigabyte of
// them in turn: 24 copies of a small matrix stay in the 256 MB cache):
//     start + rounds * round + slices * slice(load) + w_mb * MB of weights + [shares > 1] (sum0 + sum_mb * MB of partial sums)
// with rounds = times the launch fills the chip (`per_cu` workgroups on each unit), load = workgroups per unit in the last
// round: slice(load) = slice + crowd * min(load, 1), and + pair * (pair0 + (1 - pair0) (load - 1)) when some units hold two.
// A launch that shares the chip with the other chunk's (`shared`: two chunks computing side by side) leaves its last round's
// idle units to that one, so there 0.7 of the price is the part of the chip it uses (measured over 60 split layers: 0 and 1
// instead of 0.7 lose 5 and 2 %) and the switch has to promise 8 %.  (A blend, not a model of the other launch: the QKV products
// of a 4096-token 70B TP=8 prompt cut in half, 2048 x 1280 x 8192 each, are priced at 55 us and take 94 and 127 side by side.)
// Never below the time of the weights' bytes from HBM.  Root mean square error 3-7 % where a launch is within 1.3 of the best; the
// fastest by these numbers is 0.8 % (bf16) and 1.4 % (FP8) slower than the best measured launch on average.  (Fitted to launches of
// at most 600 workgroups and eight shares over weights half of which were in the cache it was 1.4 and 2.1 %, and narrow tiles were
// taken for twenty rounds of the chip: 5442 x 7992 x 192 83 us, now 33.)  251 layers of six shards, 1 to 16000 tokens, against that
// fit: 0.992 of the time.
// The 256-column tiles (kinds 4 to 6, -1, -4, -5) are those of gemm_pp_kernel.h; 192 and 128 rows are for row counts that 256 fit
// badly or that leave units idle: 1500 x 8192 x 3584 73.8 us with 256 rows, 65.5 with 192; 8192 x 2560 x 8192 300 / 250; 1024 x 8960
// x 6656 125 / 101; 777 x 7168 x 8192 123 / 105, with 128 rows 96.  Stream-K was the fastest of all launches in 5 of 1228
// bf16 products and in no FP8 one.
struct Tile {
    int bm, bn, per_cu, kind;    // kind: tile in shares (0 .. 6), or -v: variant v of the whole-tile kernels, one share
    double start, round, slice, crowd, pair, pair0, w_mb, sum0, sum_mb;
};
constexpr Tile TILES_BF16[] = {
    {32, 64, 2, 0, 2.19, 1.32, 0.131, 0.019, 0.145, 1.00, 0.081, 2.28, 0.481},
    {64, 64, 2, 1, 2.59, 1.37, 0.172, 0.033, 0.202, 1.00, 0.055, 2.19, 0.497},
    {128, 64, 2, 2, 4.08, 1.49, 0.260, 0.070, 0.314, 0.83, 0.023, 1.90, 0.433},
    {128, 128, 2, 3, 2.92, 1.29, 0.475, 0.000, 0.326, 0.91, 0.061, 2.73, 0.323},
    {128, 128, 2, -3, 1.12, 2.87, 0.470, 0.048, 0.385, 0.68, 0.055, 0.00, 0.000},
    {256, 256, 1, 4, 1.69, 6.60, 0.812, 0.247, 0.000, 0.00, 0.036, 1.78, 0.285},
    {192, 256, 1, 5, 3.46, 3.74, 0.712, 0.101, 0.000, 0.00, 0.043, 1.79, 0.313},
    {128, 256, 1, 6, 4.28, 3.07, 0.632, 0.038, 0.000, 0.00, 0.055, 0.14, 0.309},
    {256, 256, 1, -1, 0.00, 7.14, 0.811, 0.461, 0.000, 0.00, 0.011, 0.00, 0.000},
    {192, 256, 1, -5, 0.73, 5.52, 0.680, 0.322, 0.000, 0.00, 0.020, 0.00, 0.000},
    {128, 256, 1, -4, 1.60, 3.56, 0.574, 0.187, 0.000, 0.00, 0.080, 0.00, 0.000},
};
constexpr Tile TILES_FP8[] = {
    {32, 64, 2, 0, 2.24, 1.20, 0.131, 0.024, 0.154, 1.00, 0.078, 2.27, 0.501},
    {64, 64, 2, 1, 2.59, 1.27, 0.166, 0.049, 0.213, 1.00, 0.051, 2.14, 0.478},
    {128, 64, 2, 2, 3.61, 1.41, 0.250, 0.109, 0.316, 0.84, 0.012, 1.94, 0.412},
    {128, 128, 2, 3, 3.30, 1.21, 0.611, 0.000, 0.119, 1.00, 0.067, 2.18, 0.338},
    {128, 128, 2, -3, 1.32, 3.51, 0.572, 0.032, 0.228, 0.73, 0.095, 0.00, 0.000},
    {256, 256, 1, 4, 2.01, 6.36, 0.832, 0.077, 0.000, 0.00, 0.041, 1.85, 0.308},
    {192, 256, 1, 5, 4.50, 4.01, 0.692, 0.039, 0.000, 0.00, 0.050, 0.59, 0.324},
    {128, 256, 1, 6, 5.10, 2.48, 0.629, 0.000, 0.000, 0.00, 0.057, 0.15, 0.331},
    {256, 256, 1, -1, 0.31, 8.33, 0.772, 0.433, 0.000, 0.00, 0.012, 0.00, 0.000},
    {192, 256, 1, -5, 1.05, 6.26, 0.638, 0.294, 0.000, 0.00, 0.048, 0.00, 0.000},
    {128, 256, 1, -4, 2.05, 4.06, 0.540, 0.177, 0.000, 0.00, 0.095, 0.00, 0.000},
};
// Stream-K by team size 1, 2, 4, 8: start + slice * k-slices of a team + fetch * teams per tile column.
struct StreamK {
    double start, slice, fetch;
};
constexpr StreamK SK_BF16[] = {{20.4, 2.08, 2.9}, {25.7, 1.56, 2.6}, {24.4, 1.61, 1.3}, {11.7, 1.71, 4.0}};
constexpr StreamK SK_FP8[] = {{29.1, 2.14, 0.0}, {36.5, 1.39, 0.0}, {30.4, 1.59, 0.0}, {20.5, 1.77, 0.0}};
double stream_k_us(bool fp8, int M, int N, int nk, int ncu) {
    int team, grid, grouped;
    const double slices = (double)iso_gemm_sk_plan(M, N, nk, ncu, &team, &grid, &grouped);
    const double teams = grid / team, cols = (double)(((M + 255) / 256) / team) * ((N + 255) / 256);
    const StreamK &k = (fp8 ? SK_FP8 : SK_BF16)[team == 8 ? 3 : team / 2];
    return k.start + k.slice * slices + k.fetch * teams / cols;
}

// What the operands' bytes take at least.
double bytes_us(int M, int N, int nk) { return ((double)N * nk / 5.2e6 + (double)M * nk / 1e7) * ROW_BYTES; }

double tile_us(const Tile &t, int M, int N, int nk, int S, int ncu, bool shared) {
    const double wgs = (double)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) * S;
    const double slots = (double)ncu * t.per_cu, full = std::max(0.0, ceil(wgs / slots) - 1.0);
    const double load = (wgs - full * slots) / ncu, slices = (nk + S - 1) / S;
    auto slice = [&](double x) {
        return t.slice + t.crowd * std::min(x, 1.0) + (x > 1.0 ? t.pair * (t.pair0 + (1.0 - t.pair0) * (x - 1.0)) : 0.0);
    };
    double us = t.start + (full + 1.0) * t.round + slices * (full * slice(t.per_cu) + slice(load));
    if (shared) us = 0.3 * us + 0.7 * (t.start + wgs / slots * (t.round + slices * slice(t.per_cu)));
    us = std::max(us + t.w_mb * ((double)N * nk * ROW_BYTES * 1e-6), t.start + bytes_us(M, N, nk));
    if (S > 1) us += t.sum0 + t.sum_mb * ((double)S * M * N * 4e-6);
    if (S > 6) us *= S > 8 ? 1.10 : 1.02;      // eight shares take 1-2 % more than this, twelve 6 % (at 1.06 ties go to twelve, 2-4 % behind eight)
    return us;
}

}  // namespace

bool iso_gemm_split_supported(bool fp8, int M, int N, int K) {
    const int ke = fp8 ? Fp8Op::KE : Bf16Op::KE;
    return M >= 1 && N >= 8 && (N % 8) == 0 && K >= ke && (K % ke) == 0 && (long long)M * K < (1ll << 31) &&
           (long long)N * K < (1ll << 31) && (long long)M * (N / 8) < (1ll << 31) - 256;
}

// `whole` is the whole-tile rule's own choice (variant 1, 3, 4, 5 or 6 = stream-K).  It stays unless something else is estimated
// faster (by 8 % beside another chunk).  ws_bytes: room for partial sums (0: one share only).  `rope`: the QKV projection's head_dim
// (0: another product); tiles of 256 columns and shares (through their second kernel) finish with the rotary step, the others need
// a kernel more (5 us), bf16 128 x 128 tiles with heads of 64 rotate as well (2.2 us).
// *us_or_null: the estimate for the plan returned.
iso_split_plan iso_gemm_split_plan(bool fp8, int rope, int whole, int M, int N, int K, size_t ws_bytes, int ncu, bool shared,
                                   double *us_or_null) {
    const int nk = K / (fp8 ? Fp8Op::KE : Bf16Op::KE);
    const Tile *tiles = fp8 ? TILES_FP8 : TILES_BF16;
    const int n_tiles = fp8 ? (int)(sizeof(TILES_FP8) / sizeof(Tile)) : (int)(sizeof(TILES_BF16) / sizeof(Tile));
    auto whole_extra = [&](int v) {
        if (!rope || !(v == 2 || v == 3 || (v == 6 && fp8))) return 0.0;
        return v == 3 && rope == 64 && !fp8 ? 2.2 : 5.0;
    };
    double best = 1e30;
    if (whole == 6) best = stream_k_us(fp8, M, N, nk, ncu) + whole_extra(6);
    for (int i = 0; i < n_tiles; ++i)
        if (tiles[i].kind == -whole) best = tile_us(tiles[i], M, N, nk, 1, ncu, shared) + whole_extra(whole);
    double estimate = best;
    if (shared) best *= 0.92;
    iso_split_plan plan{-1, 1, whole};
    if (nk == 1) {       // a single slice is all start and epilogue, below what the fit resolves: it would pick the 128 x 256 tile
        if (us_or_null) *us_or_null = estimate;      // (K = 64: 3 x 32 3.6 / 3.1 us of the rule, 86 x 560 4.1 / 3.6, 202 x 136 3.9 / 3.6)
        return plan;
    }
    constexpr int SHARES[] = {1, 2, 3, 4, 5, 6, 8, 12};      // (small tiles with ten shares are 8 % over the estimate, with fifteen 16 %)
    const double floor_us = bytes_us(M, N, nk), mb = (double)M * N * 4e-6;
    for (int i = 0; i < n_tiles; ++i) {
        const Tile &t = tiles[i];
        for (int S : SHARES) {
            if (t.kind >= 3 && S == 1) continue;
            if (S > 1 && (t.kind < 0 || S * 2 > nk)) break;
            if ((S > 1 || (rope && t.kind >= 0)) && (size_t)S * M * N * 4 > ws_bytes) break;
            // this and every larger number of shares costs at least so much (host time: this runs at every launch)
            if (t.start + floor_us + (S > 1 ? t.sum0 + t.sum_mb * S * mb : 0.0) >= best) break;
            double us = tile_us(t, M, N, nk, S, ncu, shared);
            if (t.kind < 0) us += whole_extra(-t.kind);
            else if (rope && S == 1) us += t.sum0 + t.sum_mb * ((double)M * N * 4e-6);
            if (us < best) {
                best = estimate = us;
                plan = t.kind < 0 ? iso_split_plan{-1, 1, -t.kind} : iso_split_plan{t.kind, S, 0};
            }
        }
    }
    if (us_or_null) *us_or_null = estimate;
    return plan;
}

hipError_t iso_launch_gemm_split(const iso_split_plan &plan, const void *a, const void *w, const float *sa, const float *sw,
                                 void *c, int M, int N, int K, iso_sk_ws *ws, const iso_resid_args &resid, hipStream_t s) {
    const bool fp8 = sa != nullptr;
    float *p = plan.shares > 1 && ws && ws->base ? (float *)((char *)ws->base + SK_HDR) : nullptr;
    if (plan.shares > 1 && !p) return hipErrorInvalidValue;
    const Operands o{a, w, sa, sw, c, p, M, N, K, resid};
    if (plan.shares == 1)
        return fp8 ? launch_cfg<Fp8Op, EPI_BF16>(plan.tile, o, 1, s) : launch_cfg<Bf16Op, EPI_BF16>(plan.tile, o, 1, s);
    const std::lock_guard<std::mutex> hold(ws->lock);
    hipError_t e = fp8 ? launch_cfg<Fp8Op, EPI_PARTIAL>(plan.tile, o, plan.shares, s)
                       : launch_cfg<Bf16Op, EPI_PARTIAL>(plan.tile, o, plan.shares, s);
    if (e != hipSuccess) return e;
    const Shares sh{p, (size_t)M * N, plan.shares, sa, sw};
    hipLaunchKernelGGL(share_sum_kernel, dim3(blocks_for((size_t)M * (N / 8))), dim3(256), 0, s, sh, (bf16_t *)c, M, N,
                       resid);
    return hipGetLastError();
}

hipError_t iso_launch_gemm_split_swiglu(const iso_split_plan &plan, const void *a, const void *w, const float *sa,
                                        const float *sw, void *act, int M, int F, int K, iso_sk_ws *ws, hipStream_t s) {
    const bool fp8 = sa != nullptr;
    float *p = plan.shares > 1 && ws && ws->base ? (float *)((char *)ws->base + SK_HDR) : nullptr;
    if (plan.shares > 1 && !p) return hipErrorInvalidValue;
    const Operands o{a, w, sa, sw, act, p, M, 2 * F, K, {}};
    if (plan.shares == 1)
        return fp8 ? launch_cfg<Fp8Op, EPI_SWIGLU>(plan.tile, o, 1, s) : launch_cfg<Bf16Op, EPI_SWIGLU>(plan.tile, o, 1, s);
    const std::lock_guard<std::mutex> hold(ws->lock);
    hipError_t e = fp8 ? launch_cfg<Fp8Op, EPI_PARTIAL>(plan.tile, o, plan.shares, s)
                       : launch_cfg<Bf16Op, EPI_PARTIAL>(plan.tile, o, plan.shares, s);
    if (e != hipSuccess) return e;
    const Shares sh{p, (size_t)M * 2 * F, plan.shares, sa, sw};
    hipLaunchKernelGGL(share_sum_swiglu_kernel, dim3(blocks_for((size_t)M * (F / 8))), dim3(256), 0, s, sh, (bf16_t *)act, M, F);
    return hipGetLastError();
}

hipError_t iso_launch_gemm_split_rope(const iso_split_plan &plan, const void *a, const void *w, const float *sa, const float *sw,
                                      void *qkv, int M, int N, int K, iso_sk_ws *ws, const float *cos_t, const float *sin_t,
                                      void *k_cache, void *v_cache, int q_offset, int nq, int nkv, int d, hipStream_t s) {
    if (!ws || !ws->base) return hipErrorInvalidValue;
    float *p = (float *)((char *)ws->base + SK_HDR);
    const Operands o{a, w, sa, sw, nullptr, p, M, N, K, {}};
    const std::lock_guard<std::mutex> hold(ws->lock);
    hipError_t e = sa ? launch_cfg<Fp8Op, EPI_PARTIAL>(plan.tile, o, plan.shares, s)
                      : launch_cfg<Bf16Op, EPI_PARTIAL>(plan.tile, o, plan.shares, s);
    if (e != hipSuccess) return e;
    const Shares sh{p, (size_t)M * N, plan.shares, sa, sw};
    const RopeArgs rope{cos_t, sin_t, (bf16_t *)k_cache, (bf16_t *)v_cache, q_offset, nq, nkv};
    hipLaunchKernelGGL(share_sum_rope_kernel, dim3(blocks_for((size_t)M * (N / 16))), dim3(256), 0, s, sh, (bf16_t *)qkv, rope,
                       M, d);
    return hipGetLastError();
}

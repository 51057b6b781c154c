// Chunk attention over the KV cache for calls of few rows (bf16, head_dim 128 or 64): the keys of a row block are dealt to the
// waves of one workgroup.  Local query row i is token q_offset + i and sees keys j <= q_offset + i, j < kv_len.  (Chunk over the
// cache written by the earlier chunk: paper Section 3.1.)
//
// What such a call takes is a chain: launch, first tile, tile after tile, and, where attn_bf16_dtl.hip splits the keys of its
// 128-row blocks over workgroups, three more trips to memory for the partial states.  Here a workgroup has 32 rows of one head
// and eight waves, wave w takes the 32-key tiles w, w + 8, ... into LDS of its own, and nobody waits for anybody until the eight
// states (maximum, sum, output) meet in LDS at the end: four times as many workgroups, an eighth of the chain each, no memory
// between them.  A tile's K is requested as soon as the scores of the tile before are done with theirs, V likewise, so each
// travels under the other half of the step.  The price is that 32 rows share a fetched key instead of 128: a compute unit takes in
// 63 bytes a clock, about 7 us for 1800 keys of 128.
// Same mathematics and register layout as attn_bf16_dtl.hip (scores transposed, V read by transposing LDS reads).
#include "attn_row.h"
#include <type_traits>

namespace {

constexpr int RB = 32, KT = 32, NW = 8;      // rows and keys of a tile, waves
template <int D> struct Wv {
    static constexpr int ROW_B = D * 2, TILE_B = KT * ROW_B, CHUNKS = ROW_B / 16, RPL = 1024 / ROW_B, LOADS = TILE_B / 1024;
    static constexpr int PITCH = (D + 4) * 4;                       // merged output rows, fp32
    static constexpr int MERGE_B = NW * RB * PITCH;
    static constexpr int LDS_B = NW * 2 * TILE_B > MERGE_B ? NW * 2 * TILE_B : MERGE_B;
    // chunk swizzles, as in attn_bf16_dtl.hip
    static __device__ __forceinline__ int k_swz(int row) { return D == 128 ? (row & 15) : ((row >> 1) & 7); }
    static __device__ __forceinline__ int v_swz(int row) { return D == 128 ? ((row & 3) << 2) : (((row >> 1) & 1) << 2); }
};

typedef __bf16 bf16x4_v __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_v __attribute__((ext_vector_type(2)));

// Transposing LDS reads as an instruction, and their wait (see attn_bf16_dtl.hip)
template <int OFF> __device__ __forceinline__ bf16x4_v tr_read(uint32_t addr) {
    bf16x4_v r;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
    return r;
}
template <int N> __device__ __forceinline__ void tr_wait(bf16x8_t &a, bf16x8_t &b) {
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(a), "+v"(b) : "n"(N));
}
__device__ __forceinline__ float swap_max(float v) {                 // with the lane 32 places away
    const unsigned u = __float_as_uint(v);
    const u32x2_v r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

template <int D>
__global__ __launch_bounds__(NW * 64, 2) void attn_bf16_wave_kernel(const bf16_t *__restrict__ Q, const bf16_t *__restrict__ Kc,
                                                                    const bf16_t *__restrict__ Vc, bf16_t *__restrict__ Out,
                                                                    int Tc, int q_offset, int kv_len, int nq, int nkv,
                                                                    int q_stride) {
#if defined(__HIP_DEVICE_COMPILE__)
    using Cf = Wv<D>;
    constexpr int ROW_B = Cf::ROW_B, TILE_B = Cf::TILE_B, LOADS = Cf::LOADS;
    constexpr int NP = D == 64 ? 2 : 1;          // bf16 terms per probability (heads of 64: see attn_bf16_dtl.hip)
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    __shared__ float sm[NW][RB], sl[NW][RB];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lcol = lane & 31, lgrp = lane >> 5;

    // workgroup -> (head, row block): a contiguous range of heads per XCD (workgroup ids go round-robin over the 8 XCDs, each
    // with its own L2), longest row blocks of a head first
    const int nb = (Tc + RB - 1) / RB;
    int pid = blockIdx.x;
    const int per_xcd = (int)gridDim.x / 8;
    if (pid < per_xcd * 8) pid = (pid % 8) * per_xcd + pid / 8;
    const int h = pid / nb, m0 = (nb - 1 - pid % nb) * RB;
    const int g = h / (nq / nkv);

    const uint32_t row_stride = (uint32_t)nkv * D * 2u;
    const int kv_end = min(kv_len, q_offset + min(m0 + RB, Tc));     // keys that some row of the block sees; the rest read as zero
    const uint32_t n_rec = (uint32_t)(kv_end - 1) * row_stride + (uint32_t)ROW_B;
    const __amdgpu_buffer_rsrc_t rs_k = __builtin_amdgcn_make_buffer_rsrc((void *)(Kc + (size_t)g * D), 0, (int)n_rec, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_v = __builtin_amdgcn_make_buffer_rsrc((void *)(Vc + (size_t)g * D), 0, (int)n_rec, 0x00020000);
    uint32_t k_off[LOADS], v_off[LOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int r = i * Cf::RPL + lane / Cf::CHUNKS, slot = lane % Cf::CHUNKS;
        k_off[i] = (uint32_t)r * row_stride + (uint32_t)((slot ^ Cf::k_swz(r)) << 4);
        v_off[i] = (uint32_t)r * row_stride + (uint32_t)((slot ^ Cf::v_swz(r)) << 4);
    }
    unsigned char *const own = lds + wave * 2 * TILE_B;              // this wave's K tile, its V tile behind
    auto issue = [&](const __amdgpu_buffer_rsrc_t &rs, const uint32_t (&off)[LOADS], unsigned char *to, int tile) {
        const uint32_t at = (uint32_t)tile * KT * row_stride;
#pragma unroll
        for (int i = 0; i < LOADS; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(to + i * 1024), 16, off[i] + at, 0,
                                                     0, 0);
    };
    // 32 query rows as the B operand (requested first, so that the wait for a tile covers them)
    const int q_abs = q_offset + m0 + lcol;
    bf16x8_t qf[D / 16];
    {
        const bf16_t *qp = Q + (size_t)min(m0 + lcol, Tc - 1) * q_stride + (size_t)h * D + lgrp * 8;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) qf[ks] = *reinterpret_cast<const bf16x8_t *>(qp + ks * 16);
    }
    const int n_tiles = (kv_end + KT - 1) / KT;
    issue(rs_k, k_off, own, wave);                                   // a tile past the last visible key reads as zero
    issue(rs_v, v_off, own + TILE_B, wave);

    const uint32_t own_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)own;
    const int k_sw = Cf::k_swz(lcol);
    const int s16 = lane & 15, v_row = 4 * lgrp + (s16 >> 2), v_sw = Cf::v_swz(v_row);
    const int v_chunk = 2 * ((lane >> 4) & 1) + ((s16 & 3) >> 1);
    const uint32_t v_at = own_at + TILE_B + v_row * ROW_B + ((s16 & 1) << 3);

    f32x16_t o[D / 32];
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
    float m_run = -1e30f, l_run = 0.f;
    const float sc = 1.4426950408889634f / sqrtf((float)D);
    // the LOADS youngest requests may still be out
    auto landed = [&] {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(LOADS | (15 << 8));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int t = wave; t < n_tiles; t += NW) {
        const int j0 = t * KT;
        landed();                                                    // K of this tile; V is behind it
        f32x16_t s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
        bf16x8_t kf[D / 16];                                         // all at once: one LDS latency, not one per product
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
            kf[ks] = *reinterpret_cast<const bf16x8_t *>(own + lcol * ROW_B + (((2 * ks + lgrp) ^ k_sw) << 4));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], s, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);                           // every fragment is in registers
        issue(rs_k, k_off, own, t + NW);
        if (j0 + KT - 1 > q_offset + m0 || j0 + KT > kv_len) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = j0 + 8 * (r / 4) + 4 * lgrp + (r % 4);
                if (key > q_abs || key >= kv_len) s[r] = -INFINITY;
            }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[r]);
        mx = swap_max(mx);
        const float m_new = fmaxf(m_run, mx), neg_m = -m_new * sc;
        float psum = 0.f;
        bf16x8_t pb[NP][2];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float p = __builtin_amdgcn_exp2f(fmaf(s[r], sc, neg_m));
            psum += p;
            const bf16_t hi = (bf16_t)p;
            pb[0][r / 8][r % 8] = hi;
            if constexpr (NP == 2) pb[1][r / 8][r % 8] = (bf16_t)(p - (float)hi);
        }
        if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {
            const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * sc);
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
        }
        l_run += psum;
        landed();                                                    // V of this tile; the next K is behind it
        bf16x8_t vf[D / 32][2];
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt) {
            const uint32_t a = v_at + (uint32_t)(((4 * dt + v_chunk) ^ v_sw) << 4);
            vf[dt][0] = __builtin_shufflevector(tr_read<0 * ROW_B>(a), tr_read<8 * ROW_B>(a), 0, 1, 2, 3, 4, 5, 6, 7);
            vf[dt][1] = __builtin_shufflevector(tr_read<16 * ROW_B>(a), tr_read<24 * ROW_B>(a), 0, 1, 2, 3, 4, 5, 6, 7);
        }
        __builtin_amdgcn_sched_barrier(0);
        auto pv = [&](auto dt_c) {
            constexpr int DT = decltype(dt_c)::value;
            tr_wait<4 * (D / 32 - 1 - DT)>(vf[DT][0], vf[DT][1]);    // four reads a block
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
                for (int np = 0; np < NP; ++np)
                    o[DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[DT][st], pb[np][st], o[DT], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        pv(std::integral_constant<int, 0>{});
        pv(std::integral_constant<int, 1>{});
        if constexpr (D == 128) {
            pv(std::integral_constant<int, 2>{});
            pv(std::integral_constant<int, 3>{});
        }
        issue(rs_v, v_off, own + TILE_B, t + NW);
    }

    // ---- the eight states meet.  Lane: row lcol, dims 32 dt + 8 (r / 4) + 4 lgrp + r % 4; both halves of the wave hold the maximum
    const float l_wave = l_run + __shfl_xor(l_run, 32, 64);
    if (lgrp == 0) {
        sm[wave][lcol] = m_run;
        sl[wave][lcol] = l_wave;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                 // nothing is on its way to LDS any more
    __syncthreads();
    float m_tot = sm[0][lcol];
#pragma unroll
    for (int w = 1; w < NW; ++w) m_tot = fmaxf(m_tot, sm[w][lcol]);
    const float f = __builtin_amdgcn_exp2f((m_run - m_tot) * sc);
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
            *reinterpret_cast<f32x4_t *>(lds + (wave * RB + lcol) * Cf::PITCH + (32 * dt + 8 * r4 + 4 * lgrp) * 4) =
                f32x4_t{o[dt][4 * r4] * f, o[dt][4 * r4 + 1] * f, o[dt][4 * r4 + 2] * f, o[dt][4 * r4 + 3] * f};
    __syncthreads();
    constexpr int PPR = D / 8;                                       // 16-byte pieces of an output row
    const int row = tid / PPR, c = (tid % PPR) * 8;
    const bool mine = row < RB && m0 + row < Tc;                     // heads of 64: half of the threads
    float probe = 0.f, l_tot = 0.f;
    if (mine) {
        float mt = sm[0][row];
#pragma unroll
        for (int w = 1; w < NW; ++w) mt = fmaxf(mt, sm[w][row]);
#pragma unroll
        for (int w = 0; w < NW; ++w) l_tot += sl[w][row] * __builtin_amdgcn_exp2f((sm[w][row] - mt) * sc);
        f32x4_t lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const f32x4_t *src = reinterpret_cast<const f32x4_t *>(lds + (w * RB + row) * Cf::PITCH + c * 4);
            lo += src[0];
            hi += src[1];
        }
        const float inv = 1.0f / l_tot;
        bf16x8_t v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = (bf16_t)(lo[e] * inv);
            v[e + 4] = (bf16_t)(hi[e] * inv);
            probe = fmaf(lo[e], 0.f, probe);
            probe = fmaf(hi[e], 0.f, probe);
        }
        probe = fmaf(inv, 0.f, probe);
        *reinterpret_cast<bf16x8_t *>(Out + ((size_t)(m0 + row) * nq + h) * D + c) = v;
    }
    // Rows with a result that is not finite although their sum is a number are looked at again (see attn_bf16_dtl.hip): a key
    // that the row does not see may have met its zero probability with an infinity, or the sum is zero.
    uint64_t odd = __builtin_amdgcn_ballot_w64(mine && probe != 0.f && l_tot == l_tot);
    if (odd) {
        __builtin_amdgcn_s_waitcnt(0);                               // the stores above come first
        const uint64_t zero = __builtin_amdgcn_ballot_w64(l_tot == 0.f);
        const float scale = 1.0f / sqrtf((float)D);
        for (int r = 0; r < 64 / PPR; ++r) {
            const uint64_t lanes = ((1ull << PPR) - 1) << (r * PPR);
            if (!(odd & lanes)) continue;
            const int i = m0 + wave * (64 / PPR) + r;
            int last;
            if (NP == 1 && !(zero & lanes) &&
                !attn_rows_not_finite<bf16_t, D>(Vc + (size_t)g * D, (size_t)nkv * D, q_offset + i + 1, kv_end, lane, &last))
                continue;
            const bf16_t *qp = Q + (size_t)i * q_stride + (size_t)h * D;
            attn_row<bf16_t, D>([&](int e) { return (float)qp[e] * scale; }, Kc + (size_t)g * D, Vc + (size_t)g * D, (size_t)nkv * D,
                                min(kv_len, q_offset + i + 1), Out + ((size_t)i * nq + h) * D, lane);
        }
    }
#endif
}

template <int D>
hipError_t launch(const void *q, const void *k, const void *v, void *out, int Tc, int q_offset, int kv_len, int nq, int nkv,
                  int q_stride, hipStream_t s) {
    static iso_dev_mask lds_allowed{0};
    auto kern = attn_bf16_wave_kernel<D>;
    if (hipError_t e = iso_allow_lds(reinterpret_cast<const void *>(kern), Wv<D>::LDS_B, &lds_allowed); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((Tc + RB - 1) / RB * nq), dim3(NW * 64), Wv<D>::LDS_B, s, (const bf16_t *)q, (const bf16_t *)k,
                       (const bf16_t *)v, (bf16_t *)out, Tc, q_offset, kv_len, nq, nkv, q_stride);
    return hipGetLastError();
}

}  // namespace

// Where this kernel is ahead of the 128-row blocks.  It takes 5 us and 4 us for every 1000 keys of a round of the chip, the other
// one 7 to 12 us, less for every further key and row.  Measured, us, that one / this one (3700 sizes, 8 to 64 heads):
//   * One round: 13 heads of 128, 333 rows over 333 keys 12.1 / 7.8, over 1333 19.3 / 12.6, over 2333 22.7 / 18.1, over 4333 29.1 /
//     29.2; 16 rows over 2016 17.4 / 13.5, over 4016 20.7 / 25.5; 8 heads, 200 rows alone 10.2 / 6.8, 1024 rows alone 19.5 / 11.3.
//     Heads of 64 put two workgroups on a unit; where they do and the other kernel deals the keys to three workgroups, its line
//     is earlier: 12 heads, 859 rows alone 12.0 / 10.6, over 1609 keys 15.5 / 15.8, over 2459 18.6 / 20.8.
//   * Two rounds: no longer twice as good a start, so rows enough (more than 480) that the second round's blocks are short ones: 64
//     heads of 128, 197 rows alone 10.4 / 12.0; 28 heads, 384 rows over 1384 keys 20.4 / 22.3; 64 heads of 64, 453 rows 11.3 / 13.8.
//     Heads of 128: 13 heads, 777 rows over 1277 keys 22.3 / 21.8, over 1777 25.4 / 25.8; 16 heads, 1024 rows alone 22.5 / 18.6; where the
//     other kernel deals the keys to three workgroups, only while the block that runs second on a place ends before the longest
//     one: 8 heads, 1189 rows over 1439 18.2 / 16.6, but 20 heads, 507 rows over 1507 20.2 / 22.5.  Heads of 64 up to 1.6 rounds: 32
//     heads, 600 rows alone 13.5 / 12.0, 777 15.8 / 15.6, over 1777 30.6 / 27.8, but 965 over 1965 (1.94 rounds) 29.8 / 31.7, 40
//     heads, 667 alone (1.64) 13.5 / 14.6, 20 heads, 1600 alone (1.95) 23.5 / 24.2.
// At 2070 sizes that the lines were not drawn with (8 to 52 heads, a third of a round to two): 0.83 of the other kernel's time; 37 of
// them are more than 2 % behind it, 18 more than 4 %, the worst 12 % (36 heads of 64, 704 rows alone 13.3 / 14.9).
bool iso_attn_bf16_wave_wanted(int Tc, int nq, int d, long long keys) {
    const long long ncu = iso_num_cu(), wgs = (long long)((Tc + RB - 1) / RB) * nq, places = ncu * (d == 64 ? 2 : 1);
    const bool in_three = 3ll * ((Tc + 127) / 128) * nq <= ncu;      // the other kernel's 128-row blocks, keys in three shares
    if (wgs <= places) return keys <= (wgs > ncu && in_three ? 1536 : 2816);
    if (Tc <= 480) return false;
    if (d == 64) return 5 * wgs <= 8 * places && keys <= 2048;
    return wgs <= 2 * places && keys <= 1536 && !(in_three && keys * wgs > 2ll * Tc * places);
}

hipError_t iso_launch_attn_bf16_wave(const void *q, const void *k, const void *v, void *out, int Tc, int q_offset, int kv_len,
                                     int nq, int nkv, int d, int q_stride, hipStream_t s) {
    if (d == 128) return launch<128>(q, k, v, out, Tc, q_offset, kv_len, nq, nkv, q_stride, s);
    if (d == 64) return launch<64>(q, k, v, out, Tc, q_offset, kv_len, nq, nkv, q_stride, s);
    return hipErrorInvalidValue;
}

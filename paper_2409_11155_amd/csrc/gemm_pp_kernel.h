// The 256-column projection tile of libiso for gfx950: two groups of waves that take turns at the matrix cores (the published
// "ping-pong" schedule of two wave groups one barrier apart).
//   bf16:  c[M,N] = a[M,K] * w[N,K]^T, fp32 accumulate, bf16 output (RNE)            (projections: paper Section 2.2)
//   FP8:   c[M,N] = (a8[M,K] * w8[N,K]^T) * sa[M] * sw[N], E4M3 operands             (8-bit products: paper Section 4.1)
//
//   * BM x 256 tile (BM = 256, 192 or 128), eight waves, 2 x 4 of them; a wave owns BM/2 x 64 outputs as four quadrants:
//     its rows of the two halves of the A tile times its columns of the two halves of the W tile.
//   * Waves w and w + 4 share a SIMD.  Waves 4 .. 7 run one step behind waves 0 .. 3: while one group multiplies a quadrant
//     from registers (16 matrix instructions back to back), the other reads the operands of its next quadrant from LDS and
//     requests a half tile two slices ahead; a barrier, and they change places.  The matrix cores always have one wave that
//     does nothing but feed them, and one LDS read latency is hidden behind every 256 cycles of products.  (With both groups
//     running the same interleaved code they met at the slice's hand-over barrier and waited there together: bf16 8192^3 1460
//     TFLOP/s that way, 1600 this way; 8192 x 7168 x 8192 1380 / 1510, 2048 x 8192 x 3584 1330 / 1445, 1500 x 8192 x 3584 with
//     192 rows 1250 / 1325; FP8 8192^3 2620 / 2945, 1500 x 8192 x 3584 2080 / 2280.  Two longer steps a slice instead of four:
//     8192^3 1585.)
//   * The products are v_mfma_f32_16x16x32_bf16 / v_mfma_f32_16x16x128_f8f6f4 (more arithmetic per watt than the 32 x 32
//     shapes; the chip runs into its power limit).  W is the instruction's first operand, so that a lane's four results are
//     neighbouring columns of one row and leave as one 8-byte LDS write or one 16-byte store.
//   * Tiles travel global -> LDS directly; a half tile is requested as soon as both groups have read its predecessor of two
//     slices ago, seven steps before its first read, and up to 96 KB of requests are under way.  LDS rows are 128 bytes (64
//     bf16 or 128 FP8 elements); chunk c of row r lives in slot c ^ swz(r), applied on the global side, and 16-byte reads of 16
//     consecutive rows spread over all banks.
//   * Epilogue: the whole tile is staged in LDS as bf16 and leaves in full row segments.
// Requires K a multiple of the slice (64 bf16 / 128 FP8 elements), N % 8 == 0 and M*K, N*K < 2^31 elements.
#pragma once
#include "gemm_dtl_kernel.h"

namespace {

enum { PP_PLAIN = 0, PP_SWIGLU, PP_ROPE128, PP_ROPE64, PP_SHARE, PP_RESID };

template <int BM_> struct PpCfg {
    static constexpr int BM = BM_, BN = 256, NT = 512;
    static constexpr int A_BYTES = BM * ROW_BYTES, STAGE = A_BYTES + BN * ROW_BYTES;
    static constexpr int AL = BM / 64;                   // A requests per wave and slice, 8 rows each
    static constexpr int AE = BM / 2 / 64, AR = AL - AE; // early: rows of the first half only; the rest
    static constexpr int LPS = AL + 4;                   // requests per wave and slice
    static constexpr int WR = BM / 4, FM = WR / 16;      // rows of a wave per half, their 16-row blocks
    static constexpr bool SPLIT_HALF = (BM / 2) % 64 != 0;   // the first half needs one of the later requests
    static constexpr int PITCH = BN * 2 + 16;            // staged output rows
    static constexpr int SHARE_PITCH = BN * 4 + 16;      // staged partial sums, half a tile
    static constexpr int lds_bytes(bool share) {
        const int epi = share ? BM / 2 * SHARE_PITCH : BM * PITCH;
        return 2 * STAGE > epi ? 2 * STAGE : epi;
    }
    static_assert(BM % 64 == 0 && lds_bytes(true) <= 160 * 1024 && lds_bytes(false) <= 160 * 1024, "shape");
};

// c += a b^T, 16 x 16 x 128 E4M3.  In place: left to the builtin the compiler gives the result other registers than the sum it
// adds to, and the accumulators travel through the register file until some are spilled inside the loop.  The compiler does not
// see that this is a matrix instruction: nothing but another of the same may touch `c` within 18 wait states behind it, which the
// kernel sees to behind its loop and tests/test_isa_cpu.py in what is built.
__device__ __forceinline__ void pp_mac8(f32x4_t &c, const i32x8_t &a, const i32x8_t &b) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
#endif
}

template <bool F8, int BM, int EPI>
__global__ __launch_bounds__(512, 2) void gemm_pp_kernel(const unsigned char *__restrict__ A, const unsigned char *__restrict__ W,
                                                         const float *__restrict__ sa, const float *__restrict__ sw,
                                                         bf16_t *__restrict__ C, float *__restrict__ P, int M, int N, int K,
                                                         int tiles_m, int tiles_n, int S, RopeArgs rope, iso_resid_args resid) {
#if defined(__HIP_DEVICE_COMPILE__)
    using Cfg = PpCfg<BM>;
    constexpr int EB = F8 ? 1 : 2, KE = F8 ? 128 : 64;
    constexpr int A_BYTES = Cfg::A_BYTES, W_BYTES = 256 * ROW_BYTES, FM = Cfg::FM;
    constexpr int AE = Cfg::AE, AR = Cfg::AR, AL = Cfg::AL, LPS = Cfg::LPS;
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;

    // workgroup -> (share, tile): contiguous range per XCD (workgroup ids go round-robin over the 8 XCDs), groups of 8 tile
    // rows, tile row fastest inside a group (neighbours share the W tile)
    const int nt = tiles_m * tiles_n;
    int pid = blockIdx.x;
    const int per_xcd = (int)gridDim.x / 8;
    if (pid < per_xcd * 8) pid = (pid % 8) * per_xcd + pid / 8;
    const int share = EPI == PP_SHARE ? pid / nt : 0;
    if (EPI == PP_SHARE) pid %= nt;
    constexpr int GROUP = 8;
    const int width = GROUP * tiles_n;
    const int first_m = (pid / width) * GROUP;
    const int gsize = min(tiles_m - first_m, GROUP);
    const int tile_n = (pid % width) / gsize;
    const int m0 = (first_m + (pid % width) % gsize) * BM, n0 = tile_n * 256;
    const int nk_all = K / KE;
    const int kb = EPI == PP_SHARE ? (int)((long long)nk_all * share / S) : 0;
    const int nk = (EPI == PP_SHARE ? (int)((long long)nk_all * (share + 1) / S) : nk_all) - kb;

    // ---- requests.  Column of W half g that a wave-column w's row c (0 .. 31) of the half stands for: the two halves hold what
    // the epilogue combines in one lane (gate and up, the two halves of a head), else neighbouring blocks of 32.
    auto col_of = [&](int g, int w, int c) {
        if (EPI == PP_SWIGLU) return tile_n * 128 + w * 32 + c;                     // MLP column; g: gate / up row of W
        if (EPI == PP_ROPE128) return n0 + (w >> 1) * 128 + g * 64 + (w & 1) * 32 + c;
        return n0 + w * 64 + g * 32 + c;
    };
    const int ld_row = lane >> 3, ld_slot = lane & 7;
    const uint32_t row_bytes = (uint32_t)K * (uint32_t)EB;
    const int a_bytes = (int)((uint32_t)M * row_bytes), w_bytes = (int)((uint32_t)N * row_bytes);
    uint32_t a_off[AL], w_off[2][2];
#pragma unroll
    for (int i = 0; i < AL; ++i) {
        const int r = i * 64 + wave * 8 + ld_row;
        a_off[i] = (uint32_t)min(m0 + r, M - 1) * row_bytes + (uint32_t)((ld_slot ^ swz(r)) << 4);
    }
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = i * 64 + wave * 8 + ld_row;
            const int n = col_of(g, r >> 5, r & 31);
            const int grow = EPI == PP_SWIGLU ? g * (N / 2) + min(n, N / 2 - 1) : min(n, N - 1);
            w_off[g][i] = (uint32_t)grow * row_bytes + (uint32_t)((ld_slot ^ swz(r)) << 4);
        }
    // slice t of this workgroup's range into stage t & 1; past the end through an empty descriptor: nothing is fetched, the
    // count of outstanding requests stays the same
    auto issue_a = [&](int stage, int t, auto from_c, auto to_c) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)A, 0, t < nk ? a_bytes : 0, 0x00020000);
        unsigned char *base = lds + stage * A_BYTES + wave * 1024;
#pragma unroll
        for (int i = decltype(from_c)::value; i < decltype(to_c)::value; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(base + i * 8192), 16, a_off[i],
                                                     (kb + t) * ROW_BYTES, 0, 0);
    };
    auto issue_w = [&](int stage, int t, auto g_c) {
        constexpr int G = decltype(g_c)::value;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)W, 0, t < nk ? w_bytes : 0, 0x00020000);
        unsigned char *base = lds + 2 * A_BYTES + stage * W_BYTES + G * 16384 + wave * 1024;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(base + i * 8192), 16,
                                                     w_off[G][i], (kb + t) * ROW_BYTES, 0, 0);
    };

    // ---- operands: lane l holds row l % 16 of a block and 16-byte chunks l / 16 and l / 16 + 4 of its 128 bytes (bf16: two
    // k-steps of 32; FP8: the two halves of one k-step of 128, the same assignment of k to lanes for both operands)
    const int frow = lane & 15, fg = lane >> 4, fsw = swz(frow);
    i32x8_t af[FM], wf[2][2];
    // LDS addresses of this lane's two chunks in the first row block of each operand; everything else is a constant within the
    // reach of the instruction's offset (opaque, or the compiler keeps a register per stage and half)
    typedef const __attribute__((address_space(3))) unsigned char *lds_ptr;
    typedef const __attribute__((address_space(3))) i32x4_t *lds_vec;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr)lds;
    uint32_t a_at[2], w_at[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const uint32_t chunk = lds0 + (((fg + 4 * c) ^ fsw) << 4);
        a_at[c] = chunk + (wm * Cfg::WR + frow) * ROW_BYTES;
        w_at[c] = chunk + 2 * A_BYTES + (wn * 32 + frow) * ROW_BYTES;
        asm volatile("" : "+v"(a_at[c]), "+v"(w_at[c]));
    }
    auto load = [&](const uint32_t (&at)[2], uint32_t off) {
        return __builtin_shufflevector(*(lds_vec)(lds_ptr)(uintptr_t)(at[0] + off), *(lds_vec)(lds_ptr)(uintptr_t)(at[1] + off), 0,
                                       1, 2, 3, 4, 5, 6, 7);
    };
    auto read_a = [&](int stage, int h) {
#pragma unroll
        for (int i = 0; i < FM; ++i) af[i] = load(a_at, stage * A_BYTES + (h * (BM / 2) + i * 16) * ROW_BYTES);
    };
    auto read_w = [&](int stage, int g, auto set_c) {
#pragma unroll
        for (int j = 0; j < 2; ++j) wf[decltype(set_c)::value][j] = load(w_at, stage * W_BYTES + g * 16384 + j * 16 * ROW_BYTES);
    };
    f32x4_t acc[2][2][FM][2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[h][g][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto mul = [&](auto h_c, auto g_c, auto set_c) {
        constexpr int H = decltype(h_c)::value, G = decltype(g_c)::value, X = decltype(set_c)::value;
        if constexpr (F8) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    pp_mac8(acc[H][G][i][j], wf[X][j], af[i]);
        } else {
            auto half = [](i32x8_t v, int k) {
                return k ? __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(v, v, 4, 5, 6, 7))
                         : __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(v, v, 0, 1, 2, 3));
            };
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[H][G][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(half(wf[X][j], k), half(af[i], k), acc[H][G][i][j], 0, 0, 0);
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using IE = std::integral_constant<int, AE>;
    using IL = std::integral_constant<int, AL>;
    // at most n requests outstanding and every LDS read of this wave done
    auto wait = [](auto n_c) {
        constexpr int n = decltype(n_c)::value;
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | (7 << 4));
    };
    auto swap = [] {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
#define PP_WAIT(n) wait(std::integral_constant<int, (n)>{})
    issue_w(0, 0, I0{});
    issue_a(0, 0, I0{}, IE{});
    issue_w(0, 0, I1{});
    issue_a(0, 0, IE{}, IL{});
    issue_w(1, 1, I0{});
    issue_a(1, 1, I0{}, IE{});
    issue_w(1, 1, I1{});
    issue_a(1, 1, IE{}, IL{});
    PP_WAIT(AE + 2 + AR + LPS);
    swap();
    read_w(0, 0, I0{});
    PP_WAIT(Cfg::SPLIT_HALF ? AR - 1 + LPS : 2 + AR + LPS);
    swap();
    if (wm) swap();                      // waves 4 .. 7: one step behind from here on
    // One slice, four quadrants.  Reads: W0 of a slice in the last step of the slice before, then A0, W1, A1; a half tile's
    // successor of two slices on is requested in the step after its read (by then both groups have it in registers: each waits
    // for its LDS reads before the barrier).  The waits leave outstanding exactly what was requested after the half tile that
    // the next step reads.
    auto slice = [&](int t, auto stage_c, auto x0, auto x1) {
        constexpr int ST = decltype(stage_c)::value;
        read_a(ST, 0);
        issue_w(ST, t + 2, I0{});
        PP_WAIT(AR + LPS + 2);
        swap();
        mul(I0{}, I0{}, x0);
        swap();
        read_w(ST, 1, x1);
        issue_a(ST, t + 2, I0{}, IE{});
        PP_WAIT(LPS + 2 + AE);
        swap();
        mul(I0{}, I1{}, x1);
        swap();
        read_a(ST, 1);
        issue_w(ST, t + 2, I1{});
        PP_WAIT(AE + 2 + AR + 2 + AE + 2);
        swap();
        mul(I1{}, I1{}, x1);
        swap();
        read_w(ST ^ 1, 0, x1);
        issue_a(ST, t + 2, IE{}, IL{});
        PP_WAIT(Cfg::SPLIT_HALF ? AR - 1 + LPS : 2 + AR + LPS);
        swap();
        mul(I1{}, I0{}, x0);
        swap();
    };
    int t = 0;
    for (; t + 1 < nk; t += 2) {
        slice(t, I0{}, I0{}, I1{});
        slice(t + 1, I1{}, I1{}, I0{});
    }
    if (t < nk) slice(t, I0{}, I0{}, I1{});
    if (!wm) swap();
    if constexpr (F8) {                  // the last products, see pp_mac8: no use of a sum moves above the wait
        asm volatile("s_nop 15\n\ts_nop 15");
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) asm volatile("" : "+v"(acc[h][g][i][j]));
    }
    PP_WAIT(0);
    swap();                              // nothing is on its way to LDS any more, nobody reads operands
#undef PP_WAIT

    // ---- epilogue.  acc[h][g][i][j][r]: row m0 + h * BM/2 + wm * WR + i * 16 + erow, column col_of(g, wn, j * 16 + 4 fg + r)
    int etid = tid;                      // opaque: the epilogue's addresses are not kept through the loop
    asm volatile("" : "+v"(etid));
    const int erow = etid & 15, eg = (etid & 63) >> 4;
    if constexpr (EPI == PP_SHARE) {
        // through LDS, half a tile at a time, so that a store instruction covers one row's whole kilobyte (16 rows' 64 bytes
        // straight from the registers: 200 x 7168 x 8192 in six shares 45.2 us, this way 42.8; 512 rows and more 4-7 %)
        float *out = P + (size_t)share * M * N;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h) __syncthreads();
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int g = 0; g < 2; ++g)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        *reinterpret_cast<f32x4_t *>(lds + (wm * Cfg::WR + i * 16 + erow) * Cfg::SHARE_PITCH +
                                                     (col_of(g, wn, j * 16 + 4 * eg) - n0) * 4) = acc[h][g][i][j];
            __syncthreads();
            const int gn = n0 + (etid & 63) * 4;
#pragma unroll 4
            for (int row = etid >> 6; row < BM / 2; row += 8) {
                const int gm = m0 + h * (BM / 2) + row;
                if (gm < M && gn < N)
                    *reinterpret_cast<f32x4_t *>(out + (size_t)gm * N + gn) =
                        *reinterpret_cast<const f32x4_t *>(lds + row * Cfg::SHARE_PITCH + (etid & 63) * 16);
            }
        }
        return;
    }
    constexpr int OC = EPI == PP_SWIGLU ? 128 : 256;     // output columns of the tile
    constexpr int PITCH = OC * 2 + 16;
    // PP_RESID: x (+ pa) of this thread's pieces, in two batches: the first is requested here and travels under the staging.  (FP8,
    // 256 rows: in four, each requested one ahead of its use; two spill three registers.)
    constexpr int PIECES = BM * (OC / 8) / 512, BATCHES = F8 && BM == 256 ? 4 : 2, BATCH = PIECES / BATCHES, SETS = BATCHES / 2;
    bf16x8_t xv[SETS][EPI == PP_RESID ? BATCH : 1], pv[SETS][EPI == PP_RESID ? BATCH : 1];
    auto piece_at = [&](int it, size_t &at) {
        const int p = etid + it * 512, gm = m0 + p / (OC / 8), gn = n0 + (p % (OC / 8)) * 8;
        at = (size_t)gm * N + gn;
        return gm < M && gn < N;
    };
    auto fetch = [&](int b) {
        if constexpr (EPI == PP_RESID) {
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                size_t at;
                if (piece_at(b * BATCH + i, at)) {
                    xv[b % SETS][i] = *reinterpret_cast<const bf16x8_t *>((const bf16_t *)resid.x + at);
                    pv[b % SETS][i] = *reinterpret_cast<const bf16x8_t *>((const bf16_t *)resid.pa + at);
                }
            }
        }
    };
    fetch(0);
    f32x4_t scale_w[2][2];
    if constexpr (F8) {
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int n = col_of(g, wn, j * 16 + 4 * eg), cols = EPI == PP_SWIGLU ? N / 2 : N;
                scale_w[g][j] = *reinterpret_cast<const f32x4_t *>(sw + (EPI == PP_SWIGLU ? g * (N / 2) : 0) + min(n, cols - 4));
            }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int row = h * (BM / 2) + wm * Cfg::WR + i * 16 + erow;
            unsigned char *st = lds + row * PITCH;
            if constexpr (F8) {
                const float s = sa[min(m0 + row, M - 1)];
#pragma unroll
                for (int g = 0; g < 2; ++g)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[h][g][i][j][r] *= s * scale_w[g][j][r];
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const f32x4_t v0 = acc[h][0][i][j], v1 = acc[h][1][i][j];
                bf16x4_t o0, o1;
                if constexpr (EPI == PP_SWIGLU) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) o0[r] = (bf16_t)(v0[r] / (1.0f + __expf(-v0[r])) * v1[r]);
                    *reinterpret_cast<bf16x4_t *>(st + (wn * 32 + j * 16 + 4 * eg) * 2) = o0;
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) { o0[r] = (bf16_t)v0[r]; o1[r] = (bf16_t)v1[r]; }
                    *reinterpret_cast<bf16x4_t *>(st + (col_of(0, wn, j * 16 + 4 * eg) - n0) * 2) = o0;
                    *reinterpret_cast<bf16x4_t *>(st + (col_of(1, wn, j * 16 + 4 * eg) - n0) * 2) = o1;
                }
            }
        }
    __syncthreads();
    constexpr int PPR = OC / 8;                          // 16-byte pieces of a row
    if constexpr (EPI == PP_PLAIN || EPI == PP_SWIGLU) {
        const int cols = EPI == PP_SWIGLU ? N / 2 : N, base = EPI == PP_SWIGLU ? tile_n * 128 : n0;   // both multiples of 8
#pragma unroll 4
        for (int p = etid; p < BM * PPR; p += 512) {
            const int row = p / PPR, cc = (p % PPR) * 8, gm = m0 + row, gn = base + cc;
            if (gm < M && gn < cols)
                *reinterpret_cast<uint4 *>(C + (size_t)gm * cols + gn) = *reinterpret_cast<const uint4 *>(lds + row * PITCH + cc * 2);
        }
    }
    if constexpr (EPI == PP_RESID) {
        // x = (x + pa) + bf16(result), in fp32 and in the order of the residual kernel
#pragma unroll
        for (int b = 0; b < BATCHES; ++b) {
            if (SETS == 1 ? b > 0 : b + 1 < BATCHES) fetch(SETS == 1 ? b : b + 1);
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const int p = etid + (b * BATCH + i) * 512;
                size_t at;
                if (!piece_at(b * BATCH + i, at)) continue;
                const bf16x8_t v = *reinterpret_cast<const bf16x8_t *>(lds + p / PPR * PITCH + (p % PPR) * 16);
                bf16x8_t o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (bf16_t)((float)xv[b % SETS][i][e] + (float)pv[b % SETS][i][e] + (float)v[e]);
                *reinterpret_cast<bf16x8_t *>((bf16_t *)resid.x + at) = o;
            }
        }
    }
    if constexpr (EPI == PP_ROPE128 || EPI == PP_ROPE64) {
        // pieces of eight columns of a head's first half with their partners; q heads go to C, k and v heads to row
        // q_offset + m of the caches (rotary arithmetic and roundings as in rope_kv_kernel)
        constexpr int D = EPI == PP_ROPE128 ? 128 : 64, HP = D / 16, PAIRS = 256 / 16;
#pragma unroll 2
        for (int p = etid; p < BM * PAIRS; p += 512) {
            const int row = p / PAIRS, u = p % PAIRS, hd = u / HP, i0 = (u % HP) * 8;
            const int gm = m0 + row, head = n0 / D + hd;
            if (gm >= M || head >= rope.nq + 2 * rope.nkv) continue;
            const unsigned char *st = lds + row * PITCH + (hd * D + i0) * 2;
            bf16x8_t lo = *reinterpret_cast<const bf16x8_t *>(st), hi = *reinterpret_cast<const bf16x8_t *>(st + D);
            const size_t pos = (size_t)(rope.q_offset + gm);
            if (head < rope.nq + rope.nkv) {
                const f32x4_t *cp = reinterpret_cast<const f32x4_t *>(rope.cos_t + pos * (D / 2) + i0);
                const f32x4_t *sp = reinterpret_cast<const f32x4_t *>(rope.sin_t + pos * (D / 2) + i0);
                const f32x4_t cs[2] = {cp[0], cp[1]}, sn[2] = {sp[0], sp[1]};
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float l = (float)lo[e], h = (float)hi[e], c = cs[e / 4][e % 4], s = sn[e / 4][e % 4];
                    lo[e] = (bf16_t)fmaf(l, c, -(h * s));
                    hi[e] = (bf16_t)fmaf(h, c, l * s);
                }
            }
            bf16_t *dst;
            if (head < rope.nq) dst = C + (size_t)gm * N + head * D + i0;
            else if (head < rope.nq + rope.nkv) dst = rope.k_cache + (pos * rope.nkv + (head - rope.nq)) * D + i0;
            else dst = rope.v_cache + (pos * rope.nkv + (head - rope.nq - rope.nkv)) * D + i0;
            *reinterpret_cast<bf16x8_t *>(dst) = lo;
            *reinterpret_cast<bf16x8_t *>(dst + D / 2) = hi;
        }
    }
#endif
}

}  // namespace

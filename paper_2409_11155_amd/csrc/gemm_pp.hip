// Launcher of the 256-column projection tile (gemm_pp_kernel.h).
#include "gemm_pp_kernel.h"

namespace {

template <bool F8, int BM, int EPI> hipError_t launch(const iso_pp_args &o, hipStream_t s) {
    using Cfg = PpCfg<BM>;
    constexpr int LDS_BYTES = Cfg::lds_bytes(EPI == PP_SHARE);
    static iso_dev_mask lds_allowed{0};
    auto kern = gemm_pp_kernel<F8, BM, EPI>;
    if (hipError_t e = iso_allow_lds(reinterpret_cast<const void *>(kern), LDS_BYTES, &lds_allowed); e != hipSuccess)
        return e;
    const int tiles_m = (o.M + BM - 1) / BM, tiles_n = (o.N + 255) / 256;
    const RopeArgs rope{o.rope.cos_t, o.rope.sin_t, (bf16_t *)o.rope.k_cache, (bf16_t *)o.rope.v_cache, o.rope.q_offset,
                        o.rope.nq, o.rope.nkv};
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n * (EPI == PP_SHARE ? o.shares : 1)), dim3(Cfg::NT), LDS_BYTES, s,
                       (const unsigned char *)o.a, (const unsigned char *)o.w, o.sa, o.sw, (bf16_t *)o.c, o.p, o.M, o.N, o.K,
                       tiles_m, tiles_n, o.shares, rope, o.resid);
    return hipGetLastError();
}

template <bool F8, int BM> hipError_t launch_epi(int epi, const iso_pp_args &o, hipStream_t s) {
    switch (epi) {
        case ISO_PP_PLAIN: return launch<F8, BM, PP_PLAIN>(o, s);
        case ISO_PP_SWIGLU: return launch<F8, BM, PP_SWIGLU>(o, s);
        case ISO_PP_SHARE: return launch<F8, BM, PP_SHARE>(o, s);
        case ISO_PP_RESID: return launch<F8, BM, PP_RESID>(o, s);
        case ISO_PP_ROPE:
            if (o.N != (o.rope.nq + 2 * o.rope.nkv) * o.rope.d) return hipErrorInvalidValue;
            if (o.rope.d == 128) return launch<F8, BM, PP_ROPE128>(o, s);
            if (o.rope.d == 64) return launch<F8, BM, PP_ROPE64>(o, s);
    }
    return hipErrorInvalidValue;
}

template <bool F8> hipError_t launch_bm(int bm, int epi, const iso_pp_args &o, hipStream_t s) {
    if (bm == 256) return launch_epi<F8, 256>(epi, o, s);
    if (bm == 192) return launch_epi<F8, 192>(epi, o, s);
    return bm == 128 ? launch_epi<F8, 128>(epi, o, s) : hipErrorInvalidValue;
}

}  // namespace

hipError_t iso_launch_gemm_pp(int bm, int epi, const iso_pp_args &o, hipStream_t s) {
    return o.sa ? launch_bm<true>(bm, epi, o, s) : launch_bm<false>(bm, epi, o, s);
}

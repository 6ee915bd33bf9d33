// Launchers of the x passes of Eq. (2): forward real-to-complex (fused with
// the stage combination of Eq. 4) and inverse complex-to-real (fused with
// H_eff and the LLG right-hand side).
#include "fft_passes.hpp"

namespace llgx {

template <typename T, typename S>
hipError_t launch_xfwd(hipStream_t s, int LX, const Combo<T>& in, T* mk_out, int nin, long nrows, SpecPtr spec,
                       int SX, long blk_stride, const cx<T>* twL, const cx<T>* twP, T fscale, int variant) {
    using E = typename Spec<T, S>::elem;
    E* sp = (E*)spec;
    if (variant < 0 || variant >= NVAR_XFWD) return hipErrorInvalidValue;
    // mesh rows (nin <= LX) have a zero upper half; the tensor setup
    // transforms whole padded rows (nin = 2 LX)
    const bool half = nin <= LX;
    // blocked spectra (blk_stride > 0) are those of thin meshes' own rows
    if (blk_stride > 0 && !half) return hipErrorInvalidValue;
#define XF_B(L, R, H, B)                                                                                           \
    k_xfwd<T, S, L, R, H, B><<<(unsigned)((nrows + R - 1) / R), NT, 0, s>>>(in, mk_out, nin, nrows, sp, SX, blk_stride, \
                                                                            twL, twP, fscale)
#define XF_R(L, R)                       \
    do {                                 \
        if (!half)                       \
            XF_B(L, R, false, false);    \
        else if (blk_stride > 0)         \
            XF_B(L, R, true, (L > 0));   \
        else                             \
            XF_B(L, R, true, false);     \
    } while (0)
#define XF(L)                                      \
    case L: {                                      \
        if (variant == 0)                          \
            XF_R(L, (xfwd_rows<T>(L, 0)));         \
        else if (variant == 1)                     \
            XF_R(L, (xfwd_rows<T>(L, 1)));         \
        else                                       \
            XF_R(L, (xfwd_rows<T>(L, 2)));         \
        break;                                     \
    }
    switch (LX) {
        case 0:
            XF_R(0, 256);
            break;
        LLGX_FFT_LENGTHS(XF)
        default:
            return hipErrorInvalidValue;
    }
#undef XF
#undef XF_R
#undef XF_B
    return hipGetLastError();
}

template <typename T, typename S>
hipError_t launch_xinv(hipStream_t s, int LX, int mode, SpecPtr spec, int SX, long blk_stride, const T* M, const Phys<T>& ph,
                       const XinvOut& out, const cx<T>* twL, const cx<T>* twP, T hscale, int variant) {
    using E = typename Spec<T, S>::elem;
    const E* sp = (const E*)spec;
    const long nrow = (long)ph.ny * ph.nz;
    if (variant < 0 || variant >= NVAR_XINV) return hipErrorInvalidValue;
    if (blk_stride > 0 && LX == 0) return hipErrorInvalidValue;
#define XI_B(L, R, M_, B) \
    k_xinv<T, S, L, R, M_, B><<<nb, NT, 0, s>>>(sp, SX, blk_stride, M, ph, out, twL, twP, hscale)
#define XI_M(L, R, M_)                      \
    {                                       \
        if (blk_stride > 0)                 \
            XI_B(L, R, M_, (L > 0));        \
        else                                \
            XI_B(L, R, M_, false);          \
    }
#define XI_MODE(L, R)                                                      \
    {                                                                      \
        const dim3 nb((unsigned)((nrow + R - 1) / R), (unsigned)ph.nb, 1); \
        if (mode == XINV_DEMAG) XI_M(L, R, XINV_DEMAG)                     \
        else if (mode == XINV_HEFF) XI_M(L, R, XINV_HEFF)                  \
        else if (mode == XINV_UPDATE) XI_M(L, R, XINV_UPDATE)              \
        else XI_M(L, R, XINV_RHS)                                          \
    }
#define XI(L)                                          \
    case L: {                                          \
        if (variant == 0) {                            \
            constexpr int R = xinv_rows<T>(L, 0);      \
            XI_MODE(L, R)                              \
        } else if (variant == 1) {                     \
            constexpr int R = xinv_rows<T>(L, 1);      \
            XI_MODE(L, R)                              \
        } else {                                       \
            constexpr int R = xinv_rows<T>(L, 2);      \
            XI_MODE(L, R)                              \
        }                                              \
        break;                                         \
    }
    switch (LX) {
        case 0: {
            constexpr int R = 64;
            XI_MODE(0, R)
            break;
        }
        LLGX_FFT_LENGTHS(XI)
        default:
            return hipErrorInvalidValue;
    }
#undef XI
#undef XI_MODE
#undef XI_M
#undef XI_B
    return hipGetLastError();
}

#define INST_TS(T, S)                                                                                        \
    template hipError_t launch_xfwd<T, S>(hipStream_t, int, const Combo<T>&, T*, int, long, SpecPtr, int, long,   \
                                          const cx<T>*, const cx<T>*, T, int);                                   \
    template hipError_t launch_xinv<T, S>(hipStream_t, int, int, SpecPtr, int, long, const T*, const Phys<T>&,    \
                                          const XinvOut&, const cx<T>*, const cx<T>*, T, int);
// one object per working precision and storage (build_lib.py)
#if LLGX_INST == 0
INST_TS(float, float)
#elif LLGX_INST == 1
INST_TS(float, _Float16)
#elif LLGX_INST == 2
INST_TS(float, __bf16)
#else
INST_TS(double, double)
#endif
#undef INST_TS

}  // namespace llgx

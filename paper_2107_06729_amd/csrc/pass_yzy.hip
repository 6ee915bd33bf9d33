// Launcher of the fused y/z pass of thin meshes (Eq. (2)).
#include "pass_yzy.hpp"

namespace llgx {

// Threads of a tile.  Variant 0 gives every stage whole rounds: 3 nz LY/8
// radix-8 butterflies against LY product units.  Above 512 threads a second
// tile no longer fits beside the first (registers), and the last columns of
// an odd Kx run alone: 256x256x4 FP32 17.7 us with 768 threads, 14.3 with 512
// (13.5 with the rows' present padding).  Variants 1 and 2 (half of LY, LY) are the
// faster ones on some shapes
// (512x512x2 FP64 57.0 against 57.3, 1000x100x4 FP32 17.0 against 20.0).
constexpr int yzy_nth(int LY, int nz, int v) {
    const int n = v == 1 ? LY / 2 : v == 2 ? LY : nz == 1 ? LY / 2 : nz == 2 ? LY : LY * 3 * nz / 8;
    const int r = (n + 63) / 64 * 64;
    return r < 64 ? 64 : r > 512 ? 512 : r;
}

// The fused pass takes every thin mesh whose one-column tile fits a CU's LDS
// with room for the tile's launch beside it.  Microseconds of the y, z and y
// passes with their default tiles against this one, back to back:
//   60x60x1 FP32 10.1 / 3.9, 256x64x1 FP32 9.9 / 3.9, 32x32x2 FP64 8.7 / 3.9,
//   128x128x4 FP32 12.6 / 6.5, 256x256x4 FP32 23.1 / 13.5 and FP64 35.6 / 28.1,
//   512x512x1 FP32 28.5 / 12.0, 1000x1000x2 FP32 178 / 92, 7x1000x2 FP32 26 / 18,
//   300x512x4 FP32 69 / 59 at Px = 1024 (37 at the shorter Px it takes now).
// On the largest tiles (110 KB: one workgroup a CU) the separate passes come
// level once autotuned (300x512x4 at Px = 1024: 58), so larger ones are not taken.
// Meshes of 5 to 8 layers, FP32 spectra only (a thread's three z lines take about 200
// registers; FP64 ones do not fit, and 16-bit spectra keep the order of the separate
// passes): 21x13x5 10.2 / 5.9, 60x60x8 11.0 / 7.8, 160x80x8 15.6 / 9.0, 128x128x8
// 14.8 / 11.1, 200x120x6 18.4 / 13.0, 256x256x5 24.8 / 19.3, 300x200x7 31.6 / 27.8,
// 640x320x6 (95 KiB) level, and 256x256x8 (106 KiB) 30.6 / 32.9: the line is at 96.
template <typename T>
bool yzy_ok(int LY, int nz, bool native) {
    if (nz > 4 && !(native && sizeof(T) == 4)) return false;
    return LY >= 2 && LY <= MAX_LEN && nz >= 1 && nz <= YZY_MAX_NZ && yzy_lds<T>(LY, nz, 1) <= yzy_lds_max(nz);
}
#if LLGX_INST == 0
// Variant 0, but with 5 to 8 layers, more columns than CUs and two tiles in a CU's
// LDS fewer threads, so that two tiles fit its registers as well (us, 120 rows of 6
// layers: 257 columns 17.5 / 13.0, 321 18.3 / 13.9; 200 of 5: 257 22.1 / 18.5; one column
// a CU the other way, 193 columns 10.3 / 10.8, 128x128x8 11.2 / 11.6, and so tiles that are
// alone in the LDS, 300x200x7 28.7 / 39.1).
constexpr int CUS = 256;
int yzy_default(int LY, int nz, long columns) {
    if (nz <= 4 || columns <= CUS || yzy_lds<float>(LY, nz, 1) > 80 * 1024) return 0;
    return LY <= 256 ? 2 : 1;
}
template bool yzy_ok<float>(int, int, bool);
#elif LLGX_INST == 3
template bool yzy_ok<double>(int, int, bool);
#endif

template <typename T, typename S>
hipError_t launch_yzy(hipStream_t s, int LY, SpecPtr spec, long blk_stride, int Kx, int ny, int nz, int nb,
                      const T* kcol, int KYS, const cx<T>* tw, T yscale, int variant) {
    using E = typename Spec<T, S>::elem;
    E* sp = (E*)spec;
    if (variant < 0 || variant >= NVAR_ZMUL || 2 * ny > LY + 1 || KYS < LY / 2 + 1) return hipErrorInvalidValue;
    if ((long)3 * nz * ny * SpecBlock<E>::KB >= (1L << 31)) return hipErrorInvalidValue;
#define YZ_L(LL, NZ, V)                                                                                       \
    k_yzy<T, S, LL, NZ, 1, yzy_nth(LL, NZ, V)><<<dim3((unsigned)Kx, (unsigned)nb), yzy_nth(LL, NZ, V), 0, s>>>( \
        sp, blk_stride, Kx, ny, kcol, KYS, tw, yscale)
#define YZ_N(LL, NZ)                                          \
    case NZ:                                                  \
        if constexpr (yzy_lds<T>(LL, NZ, 1) <= yzy_lds_max(NZ)) { \
            if (variant == 0)                                 \
                YZ_L(LL, NZ, 0);                              \
            else if (variant == 1)                            \
                YZ_L(LL, NZ, 1);                              \
            else                                              \
                YZ_L(LL, NZ, 2);                              \
            return hipGetLastError();                         \
        }                                                     \
        return hipErrorInvalidValue;
#if LLGX_INST == 0
#define YZ_16(LL) YZ_N(LL, 5) YZ_N(LL, 6) YZ_N(LL, 7) YZ_N(LL, 8)
#else
#define YZ_16(LL)
#endif
#define YZ(LL)                                             \
    case LL:                                               \
        switch (nz) {                                      \
            YZ_N(LL, 1) YZ_N(LL, 2) YZ_N(LL, 3) YZ_N(LL, 4) YZ_16(LL) \
            default:                                       \
                return hipErrorInvalidValue;               \
        }
    switch (LY) {
        LLGX_FFT_LENGTHS(YZ) LLGX_FFT_LENGTHS_LONG(YZ)
        default:
            return hipErrorInvalidValue;
    }
#undef YZ
#undef YZ_N
#undef YZ_16
#undef YZ_L
}

#define INST_TS(T, S)                                                                                          \
    template hipError_t launch_yzy<T, S>(hipStream_t, int, SpecPtr, long, int, int, int, int, const T*, int, \
                                         const cx<T>*, T, int);
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

// The y and z work of Eq. (2) for thin meshes (nz <= 4, FP32 <= 8) in one kernel: y
// forward, z forward, k-space product, z inverse, y inverse of TK columns kx,
// every row and every component of them in LDS.
//
// Bound: on these meshes the three separate passes are short kernels that
// move spectrum B (twice the rows of A) out and in, with z tiles of a few KB;
// one kernel reads and writes A once and the folded kernel once.  What is
// left is the vector arithmetic (1.26 k instructions a wave at 256x256x4,
// 4.2 us of the 13.5 us at full issue), the LDS passes between the stages (3
// us) and the latency of the first loads, which one tile a CU cannot hide.  On
// small meshes it is the launches: three kernels an evaluation instead of
// five (figures at yzy_ok).
//
// Layouts.  Spectrum A is blocked by 32 bytes of kx (KB columns):
// [kx / KB][sample][component][z][y][kx % KB], so one column's rows are 32
// bytes apart (consecutive lanes take consecutive rows, 16 lines per wave
// load) and the x passes still write and read 32-byte pieces.  The folded
// kernel is held a second time as [kx][kz][component][ky] (ky fastest: lanes
// of the product take consecutive ky).
// In LDS each (component, z, column) is one padded row of the y transform
// (RowFFT's layout); the z transform of a (column, ky) is in one thread's
// registers, and its three components meet there for the product.
// The arithmetic is that of ColFFT and zmul_tile, operation for operation, with
// 16-bit spectra rounded where the separate passes store them: the same bits, but for
// FP32 at LY = 1024, where ColFFT starts with radix 16 (col_radix) and RowFFT with 2.
#pragma once
#include <hip/hip_runtime.h>

#include "fft_passes.hpp"
#include "fft_row.hpp"
#include "kernels.hpp"
#include "spec_store.hpp"
#include "tile_io.hpp"

namespace llgx {

constexpr int YZY_MAX_NZ = 8;

// z transform length of nz cells: 1, 4, 8, 8, then 16
constexpr int yzy_lz(int nz) { return nz == 1 ? 1 : nz == 2 ? 4 : nz <= 4 ? 8 : 16; }

// cos(z pi / 8) as the twiddle tables hold it; -sin is the value four places on
template <typename T>
__device__ __forceinline__ constexpr T cos16(int z) {
    constexpr double c[12] = {1.0, 0.92387953251128675613, 0.70710678118654752440, 0.38268343236508977173,
                              6.123233995736766e-17, -0.38268343236508977173, -0.70710678118654752440, -0.92387953251128675613,
                              -1.0, -0.92387953251128675613, -0.70710678118654752440, -0.38268343236508977173};
    return (T)c[z];
}

// z forward, product and z inverse of one (column, ky) with nz = 5 to 8 cells: 16
// outputs as two transforms of 8 over the cells, kz even and odd (the first stage of
// two, the other half of whose inputs is the padding, leaves the cells as they are)
template <typename T, int NZ>
__device__ __forceinline__ void yzy_z16(const T (&k)[9][6], bool yneg, cx<T> (&x)[3][8]) {
    using C = cx<T>;
    C out[3][8];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        C w[3][8];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
#pragma unroll
            for (int z = 0; z < 8; ++z)
                w[a][z] = j == 0 || z == 0 ? x[a][z] : cmul(x[a][z], C{cos16<T>(z), cos16<T>(z + 4)});
            dft_r<8, false>(w[a]);
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int kz = j + 2 * r;
            apply_kernel(k[kz <= 8 ? kz : 16 - kz], yneg, kz > 8, w[0][r], w[1][r], w[2][r]);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            dft_r<8, true>(w[a]);
#pragma unroll
            for (int z = 0; z < NZ; ++z) {
                if (j == 0)
                    out[a][z] = w[a][z];
                else
                    out[a][z] = cadd(out[a][z], z == 0 ? w[a][z] : cmulc(w[a][z], C{cos16<T>(z), cos16<T>(z + 4)}));
            }
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int z = 0; z < NZ; ++z) x[a][z] = out[a][z];
}

template <typename T, int LY, int NZ, int TK, int NTH>
struct YzyShared {
    static constexpr int NR = 3 * NZ * TK;
    using F = RowFFT<T, LY, false, NR, NTH, true, false>;
    alignas(16) cx<T> buf[F::LDS_ELEMS];
    alignas(16) cx<T> twl[LY];
};

// LDS bytes of a tile (for the host's choice of the path)
template <typename T>
constexpr long yzy_lds(int LY, int nz, int tk) {
    return (3L * nz * tk * (LY + ((LY & (LY - 1)) == 0 ? LY / (sizeof(T) == 4 ? 16 : 8) : 0) + 1) + LY) * 2 * (long)sizeof(T);
}
constexpr long yzy_lds_max(int nz) { return (nz <= 4 ? 128 : 96) * 1024; }

template <typename T, typename S, int LY, int NZ, int TK, int NTH>
__global__ __launch_bounds__(NTH) void k_yzy(typename Spec<T, S>::elem* __restrict__ spec, long blk_stride, int Kx,
                                             int ny, const T* __restrict__ kcol, int KYS, const cx<T>* __restrict__ tw,
                                             T yscale) {
    using C = cx<T>;
    using E = typename Spec<T, S>::elem;
    constexpr int LZ = yzy_lz(NZ), KZF = LZ > 1 ? LZ / 2 + 1 : 1;
    constexpr int KB = SpecBlock<E>::KB;
    using SH = YzyShared<T, LY, NZ, TK, NTH>;
    constexpr int NR = SH::NR;
    using Ff = RowFFT<T, LY, false, NR, NTH, true, false>;
    using Fi = RowFFT<T, LY, true, NR, NTH, false, true>;
    __shared__ SH sh;
    C* buf = sh.buf;
    C* twl = sh.twl;
    // the KB columns of one block share lines: consecutive tiles on one XCD
    const int pos = xcd_run(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
    const int smp = pos / gridDim.x, kx0 = (pos - smp * (int)gridDim.x) * TK;
    // row index of (component, z, y) within the sample: (component NZ + z) ny + y
    const long srow = (long)smp * (3 * NZ) * ny;
    auto column = [&](int c) -> E* {
        const int kx = kx0 + c;
        return spec + (long)(kx / KB) * blk_stride + srow * KB + kx % KB;
    };
    TwStage<T, LY, NTH> tws;
    tws.fetch(tw);
    // product units (column, ky) of this thread; with one unit a thread its
    // kernel values are loaded beside the columns, not after the y transform
    constexpr int NU = TK * LY, PER = (NU + NTH - 1) / NTH;
    T k[KZF][6];
    auto load_k = [&](int u0) {
        const int u = NU % NTH == 0 || u0 < NU ? u0 : NU - 1;
        const int c = u / LY, ky = u - c * LY;
        const int kx = kx0 + c < Kx ? kx0 + c : Kx - 1;
        const T* kp = kcol + (long)kx * (KZF * 6) * KYS + (2 * ky <= LY ? ky : LY - ky);
#pragma unroll
        for (int a = 0; a < KZF; ++a)
#pragma unroll
            for (int b = 0; b < 6; ++b) k[a][b] = kp[(a * 6 + b) * KYS];
    };
    {
        // y forward, first stage from global memory: every load from an
        // address clamped into the data, the padding zeroed after it arrives
        C v[Ff::U0][Ff::R0];
#pragma unroll
        for (int m = 0; m < Ff::U0; ++m) {
            const int u0 = threadIdx.x + m * NTH, u = Ff::live0(u0) ? u0 : Ff::NU0 - 1;
#pragma unroll
            for (int q = 0; q < Ff::R0; ++q) {
                if (2 * q >= Ff::R0) {
                    v[m][q] = C{T(0), T(0)};
                    continue;
                }
                int row, i;
                Ff::first_input(u, q, row, i);
                const int c = row % TK, g = row / TK;
                const int cc = kx0 + c < Kx ? c : 0;
                const E* p = column(cc) + (g * ny + (i < ny ? i : ny - 1)) * KB;
                const C w = Spec<T, S>::get(*p);
                v[m][q] = i < ny ? w : C{T(0), T(0)};
            }
        }
        if constexpr (PER == 1) load_k(threadIdx.x);
        tws.put(twl);
        Ff::first_to_lds(v, buf);
    }
    __syncthreads();
    Ff::rest(buf, twl);
    // z forward, product, z inverse of each (column, ky)
#pragma unroll 1
    for (int u = threadIdx.x; u < NU; u += NTH) {
        if constexpr (PER > 1) load_k(u);
        const int c = u / LY, ky = u - c * LY;
        const bool yneg = 2 * ky > LY;
        C* col = buf + c * Ff::RS + Ff::P(ky);
        if constexpr (LZ == 16) {
            C x[3][8];
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int z = 0; z < 8; ++z)
                    x[a][z] = z < NZ ? col[(a * NZ + z) * TK * Ff::RS] : C{T(0), T(0)};
            yzy_z16<T, NZ>(k, yneg, x);
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int z = 0; z < NZ; ++z) col[(a * NZ + z) * TK * Ff::RS] = x[a][z];
            continue;
        }
        C v[3][LZ];
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int z = 0; z < LZ; ++z) {
                if (z >= NZ) {
                    v[a][z] = C{T(0), T(0)};
                    continue;
                }
                v[a][z] = col[(a * NZ + z) * TK * Ff::RS];
                // 16-bit spectra: rounded where the separate passes store them
                if constexpr (!std::is_same<T, S>::value)
                    v[a][z] = Spec<T, S>::get(Spec<T, S>::put(C{v[a][z].x * yscale, v[a][z].y * yscale}));
            }
        if constexpr (LZ > 1) {
#pragma unroll
            for (int a = 0; a < 3; ++a) dft_r<LZ, false>(v[a]);
        }
#pragma unroll
        for (int kz = 0; kz < LZ; ++kz) {
            const int f = 2 * kz <= LZ ? kz : LZ - kz;
            const bool zneg = 2 * kz > LZ;
            const T nxx = k[f][0], nyy = k[f][1], nzz = k[f][2];
            const T nxy = yneg ? -k[f][3] : k[f][3];
            const T nxz = zneg ? -k[f][4] : k[f][4];
            const T yz = zneg ? -k[f][5] : k[f][5];
            const T nyz = yneg ? -yz : yz;
            const C mx = v[0][kz], my = v[1][kz], mz = v[2][kz];
            v[0][kz] = C{nxx * mx.x + nxy * my.x + nxz * mz.x, nxx * mx.y + nxy * my.y + nxz * mz.y};
            v[1][kz] = C{nxy * mx.x + nyy * my.x + nyz * mz.x, nxy * mx.y + nyy * my.y + nyz * mz.y};
            v[2][kz] = C{nxz * mx.x + nyz * my.x + nzz * mz.x, nxz * mx.y + nyz * my.y + nzz * mz.y};
        }
        if constexpr (LZ > 1) {
#pragma unroll
            for (int a = 0; a < 3; ++a) dft_r<LZ, true>(v[a]);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int z = 0; z < NZ; ++z)
                col[(a * NZ + z) * TK * Ff::RS] = Spec<T, S>::get(Spec<T, S>::put(v[a][z]));
    }
    __syncthreads();
    // y inverse, the last stage to global memory
    Fi::first_in_lds(buf);
    auto store = [&](int row, int y, const C& x) {
        const int c = row % TK, g = row / TK;
        if (y < ny && kx0 + c < Kx) column(c)[(g * ny + y) * KB] = Spec<T, S>::put(x);
    };
    if constexpr (Fi::NSTAGE > 1) {
        Fi::middle(buf, twl);
        Fi::last_each(buf, twl, store);
    } else {
        for (int e = threadIdx.x; e < NR * (LY / 2); e += NTH) {
            const int row = e / (LY / 2), y = e - row * (LY / 2);
            store(row, y, buf[row * Fi::RS + Fi::P(y)]);
        }
    }
}

}  // namespace llgx

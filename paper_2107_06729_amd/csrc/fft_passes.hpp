// Kernels of the FFT passes of Eq. (2) (zero-padded FFT convolution, Sec. II)
// for gfx950; instantiated by pass_x.hip, pass_col.hip and pass_z.hip.
//
// Data layout (complex elements, working precision T):
//   spectrum buffers are [comp][z][y][kx] with row stride SX >= Kx, where
//   Kx = Px/2 + 1 columns of the real-to-complex x transform (1 if Px = 1).
// Pass chain of one evaluation (5 kernels; fewer when an axis has length 1):
//   xfwd  : stage combination M_k = M0 + sum h b F (Eq. 4), real->complex x FFT
//   colfft: y forward (rows y >= ny are the zero padding, never loaded)
//   zmul  : z forward, H = -N^ M with the 6-component symmetric k-space
//           kernel, z inverse (only z < nz rows are loaded and stored)
//   colfft: y inverse (only y < ny rows stored)
//   xinv  : complex->real x FFT (x < nx kept) fused with H_eff and the LLG
//           right-hand side (Eq. 1), or writing H_d / H_eff alone.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "kernels.hpp"
#include "physics.hpp"
#include "fft_col.hpp"
#include "fft_row.hpp"
#include "spec_store.hpp"
#include "tile_io.hpp"

namespace llgx {

constexpr int NT = 256;

// ------------------------------------------------------------------------
// Tile choices (LDS budget per workgroup).  Every pass has launch variants
// (tile widths or rows per workgroup) that compute bit-identical results.  A
// handle starts with those of default_variants (llgx_api.hip); the autotuner
// picks among all of them by timing them on the problem's own shapes.
template <typename T>
constexpr int col_tile(int L, int v) {
    const int t = sizeof(T) == 4 ? (L <= 512 ? 16 : 8) : (L <= 512 ? 8 : 4);
    return v == 1 ? (t > 1 ? t / 2 : 1) : v == 2 ? (t > 3 ? t / 4 : 1) : t;
}
// Threads of a column tile: 512 where the tile's LDS leaves room for two
// workgroups a CU at most (FP32 300x300x20, 640 rows of 8 columns: y passes 27.0 and
// 25.6 us with 256 threads, 25.4 and 24.5 with 512; 1024 rows the same either way);
// smaller tiles have more workgroups (FP32 256x256x16 at 8 columns 14.9 and 13.9 us
// with 256 threads, 15.2 and 14.2 with 512)
constexpr int col_threads(int L, int TK) { return L * TK >= 5120 ? 512 : NT; }
template <typename T>
constexpr int zmul_tile(int L, int v) {
    const int t = sizeof(T) == 4 ? (L <= 64 ? 16 : L <= 128 ? 8 : L <= 256 ? 4 : 2)
                                 : (L <= 64 ? 8 : L <= 128 ? 4 : L <= 256 ? 2 : 1);
    // variant 2 doubles the tile while its spectrum stays within 48 KiB of LDS
    const bool fits = (long)(L > 1 ? L : 1) * 6 * 2 * t * 2 * (long)sizeof(T) <= 48 * 1024;
    return v == 1 ? (t > 1 ? t / 2 : 1) : (v == 2 && fits) ? 2 * t : t;
}
// rows are a power of two: they divide more mesh heights (the y-slab order of
// the x inverse needs that)
constexpr int floor_pow2(int n) { return n < 2 ? 1 : 2 * floor_pow2(n / 2); }
template <typename T>
constexpr int xfwd_rows(int LX, int v) {
    int r = floor_pow2((sizeof(T) == 4 ? 2048 : 1024) / (LX > 0 ? LX : 1));
    r = r < 1 ? 1 : (r > 16 ? 16 : r);
    // variant 2 doubles the rows while the tile stays within 48 KiB of LDS
    const bool fits = 2L * r * (LX + 1) * 2 * (long)sizeof(T) <= 48 * 1024;
    return v == 1 ? (r > 1 ? r / 2 : 1) : (v == 2 && fits) ? 2 * r : r;
}
template <typename T>
constexpr int xinv_rows(int LX, int v) {
    int r = floor_pow2((sizeof(T) == 4 ? 1024 : 512) / (LX > 0 ? LX : 1));
    r = r < 1 ? 1 : (r > 8 ? 8 : r);
    const bool fits = 2L * 3 * r * (LX + 1) * 2 * (long)sizeof(T) <= 48 * 1024;
    return v == 1 ? (r > 1 ? r / 2 : 1) : (v == 2 && fits) ? 2 * r : r;
}

// Eq. (4) terms: a loop over c.nf (kernel arguments, indexed in place), or
// with STATIC_NF unrolled to MAX_F with static indices (arguments held in
// registers); the same terms in the same order either way
template <typename T, bool STATIC_NF = false>
__device__ __forceinline__ T combo_at(const Combo<T>& c, long i) {
    T v = c.base[i];
    if constexpr (STATIC_NF) {
#pragma unroll
        for (int l = 0; l < MAX_F; ++l) {
            if (l >= c.nf) break;
            v += c.coef[l] * c.f[l][i];
        }
    } else {
        for (int l = 0; l < c.nf; ++l) v += c.coef[l] * c.f[l][i];
    }
    return v;
}

// ------------------------------------------------------------------------
// forward x pass: real rows of length nin (zero padded to 2 LX) -> LX+1 complex
// A real sequence of length P = 2 LX is packed as z[j] = x[2j] + i x[2j+1],
// transformed with a length-LX complex FFT and split with
//   X[k] = (Z[k] + Z*[LX-k])/2 - i e^{-2 pi i k/P} (Z[k] - Z*[LX-k])/2.
// LDS of one x forward tile
template <typename T, int LX, int ROWS>
struct XfwdShared {  // every array 16-byte aligned: 128-bit LDS accesses stay single instructions
    using F = RowFFT<T, LX, false, ROWS, NT>;
    alignas(16) cx<T> buf[F::LDS_ELEMS];
    alignas(16) cx<T> twl[LX];
    alignas(16) cx<T> twp[LX + 1];
};
template <typename T, int ROWS>
struct XfwdShared<T, 0, ROWS> {
    int unused;
};

// rows row0 .. row0 + ROWS - 1 (one workgroup)
template <typename T, typename S, int LX, int ROWS, bool HALF, bool STATIC_NF = false, bool BLK = false>
__device__ __forceinline__ void xfwd_tile(const Combo<T>& in, T* __restrict__ mk_out, int nin, long nrows,
                                          typename Spec<T, S>::elem* __restrict__ spec, int SX,
                                          const cx<T>* __restrict__ twL, const cx<T>* __restrict__ twP, T fscale,
                                          long row0, XfwdShared<T, LX, ROWS>& sh, long blk_stride = 0) {
    using C = cx<T>;
    if constexpr (LX == 0) {
        for (int r = threadIdx.x; r < ROWS; r += NT) {
            const long g = row0 + r;
            if (g < nrows) {
                const T v = combo_at<T, STATIC_NF>(in, g);
                if (mk_out) mk_out[g] = v;
                spec[g * SX] = Spec<T, S>::put(C{v * fscale, T(0)});
            }
        }
        return;
    } else {
        // HALF (nin <= LX, a mesh row): packed inputs z[i] = x[2i] + i x[2i+1]
        // with i >= LX/2 lie in the zero padding
        using F = RowFFT<T, LX, false, ROWS, NT, HALF, false>;
        C* buf = sh.buf;
        C* twl = sh.twl;
        C* twp = sh.twp;
        TwStage<T, LX, NT> tw1;
        TwStage<T, LX + 1, NT> tw2;
        tw1.fetch(twL);
        tw2.fetch(twP);
        // stage-0 inputs z[i] = x[2i] + i x[2i+1] of the stage combination,
        // straight from global memory: all loads of one operand are issued
        // before they are used.  Addresses are the tile's first real and a 32-bit
        // offset in bytes (ROWS nin <= 2^15).
        const int left = (int)(nrows - row0 < ROWS ? nrows - row0 : ROWS);  // rows of the tile
        const long tile0 = left > 0 ? row0 * nin : 0;
        auto put_tables = [&] {
            tw1.put(twl);
            tw2.put(twp);
        };
        // A wave without a butterfly (fewer than NT of them) goes to the barrier: half of
        // the waves of a 640-long tile of two rows formed addresses and loaded for
        // nothing (640x320x4 12.3 -> 11.8 us, 160x80x8 5.0 -> 4.3; with 256-long rows,
        // where every wave has one, 11.0 both).
        if (F::U0 > 1 || F::NU0 >= NT || (int)threadIdx.x < F::NU0) {
            C v[F::U0][F::R0];
            unsigned off[F::U0][F::R0];
            bool ok[F::U0][F::R0];
            bool two[F::U0][F::R0];
#pragma unroll
            for (int m = 0; m < F::U0; ++m) {
                const int u = threadIdx.x + m * NT;
#pragma unroll
                for (int q = 0; q < F::R0; ++q) {
                    int r, i;
                    F::first_input(u, q, r, i);
                    ok[m][q] = F::live0(u) && r < left && 2 * i < nin;
                    off[m][q] = ok[m][q] ? (__umul24((unsigned)r, (unsigned)nin) + 2 * i) * (unsigned)sizeof(T) : 0;
                    two[m][q] = 2 * i + 1 < nin;
                }
            }
            const bool pairs = (nin & 1) == 0;  // rows start 8/16-byte aligned: load both reals at once
            // every load is issued, from a clamped offset (element 0 for an empty
            // slot), so a wave keeps all of them in flight; a load under a branch
            // would be waited for at the branch's end.  Empty slots and the
            // missing odd element of a row are zeroed after the combination.
            auto load2 = [&](const T* __restrict__ p, int m, int q) -> C {
                const T* a = (const T*)((const char*)p + off[m][q]);
                C w;
                if (pairs) {
                    w = *(const C*)a;
                } else {
                    w.x = a[0];
                    w.y = a[two[m][q] ? 1 : 0];
                }
                return w;
            };
            constexpr int QN = HALF ? (F::R0 + 1) / 2 : F::R0;  // inputs q >= QN lie in the zero half
            const T* base = in.base + tile0;
#pragma unroll
            for (int m = 0; m < F::U0; ++m)
#pragma unroll
                for (int q = 0; q < F::R0; ++q) v[m][q] = q < QN ? load2(base, m, q) : C{T(0), T(0)};
            auto add_term = [&](int l) {
                C w[F::U0][F::R0];
                const T* f = in.f[l] + tile0;
#pragma unroll
                for (int m = 0; m < F::U0; ++m)
#pragma unroll
                    for (int q = 0; q < F::R0; ++q) w[m][q] = q < QN ? load2(f, m, q) : C{T(0), T(0)};
                const T cf = in.coef[l];
#pragma unroll
                for (int m = 0; m < F::U0; ++m)
#pragma unroll
                    for (int q = 0; q < F::R0; ++q) {
                        v[m][q].x += cf * w[m][q].x;
                        v[m][q].y += cf * w[m][q].y;
                    }
            };
            if constexpr (STATIC_NF) {
#pragma unroll
                for (int l = 0; l < MAX_F; ++l) {
                    if (l >= in.nf) break;
                    add_term(l);
                }
            } else {
                for (int l = 0; l < in.nf; ++l) add_term(l);
            }
#pragma unroll
            for (int m = 0; m < F::U0; ++m)
#pragma unroll
                for (int q = 0; q < QN; ++q) {
                    if (!ok[m][q]) v[m][q] = C{T(0), T(0)};
                    if (!two[m][q]) v[m][q].y = T(0);
                }
            if (mk_out) {
                T* mo = mk_out + tile0;
#pragma unroll
                for (int m = 0; m < F::U0; ++m)
#pragma unroll
                    for (int q = 0; q < QN; ++q)
                        if (ok[m][q]) {
                            T* a = (T*)((char*)mo + off[m][q]);
                            a[0] = v[m][q].x;
                            if (two[m][q]) a[1] = v[m][q].y;
                        }
            }
#pragma unroll
            for (int m = 0; m < F::U0; ++m)
#pragma unroll
                for (int q = 0; q < QN; ++q) {
                    v[m][q].x *= fscale;
                    v[m][q].y *= fscale;
                }
            put_tables();
            F::first_to_lds(v, buf);
        } else {
            put_tables();
        }
        __syncthreads();
        F::rest(buf, twl);
        // X[k] for k < LX; the lane of k = 0 also writes X[LX], which takes
        // the same z_0 (LX - k and k both wrap to 0)
        using E = typename Spec<T, S>::elem;
        E* tile = spec + row0 * (BLK ? SpecBlock<E>::KB : SX);
        for (int e = threadIdx.x; e < ROWS * LX; e += NT) {
            const int r = e / LX, k = e - r * LX;
            if (r >= left) continue;
            const C* rb = buf + r * F::RS;
            const C zk = rb[F::P(k)];
            const C zc = cconj(rb[F::P(k == 0 ? 0 : LX - k)]);
            const C ev{(zk.x + zc.x) * T(0.5), (zk.y + zc.y) * T(0.5)};
            const C od{(zk.y - zc.y) * T(0.5), (zc.x - zk.x) * T(0.5)};  // -i (zk - zc)/2
            const SpecRow<BLK, E> out{tile + __umul24((unsigned)r, (unsigned)(BLK ? SpecBlock<E>::KB : SX)), blk_stride};
            out[k] = Spec<T, S>::put(cadd(ev, cmul(od, twp[k])));
            if (k == 0) out[LX] = Spec<T, S>::put(cadd(ev, cmul(od, twp[LX])));
        }
    }
}

template <typename T, typename S, int LX, int ROWS, bool HALF, bool BLK>
__global__ __launch_bounds__(NT) void k_xfwd(Combo<T> in, T* __restrict__ mk_out, int nin, long nrows,
                                             typename Spec<T, S>::elem* __restrict__ spec, int SX, long blk_stride,
                                             const cx<T>* __restrict__ twL, const cx<T>* __restrict__ twP,
                                             T fscale) {
    __shared__ XfwdShared<T, LX, ROWS> sh;
    xfwd_tile<T, S, LX, ROWS, HALF, false, BLK>(in, mk_out, nin, nrows, spec, SX, twL, twP, fscale,
                                                (long)blockIdx.x * ROWS, sh, blk_stride);
}

// ------------------------------------------------------------------------
// inverse x pass: LX+1 complex -> real, keep x < nx; then per cell
//   Z[k] = (X[k] + X*[LX-k]) + i e^{+2 pi i k/P} (X[k] - X*[LX-k]),
//   z = IDFT_LX(Z), x[2j] = Re z[j], x[2j+1] = Im z[j].
// LDS of one x inverse tile
template <typename T, int LX, int ROWS>
struct XinvShared {
    static constexpr int LXE = LX > 0 ? LX : 2;
    static constexpr int RS = LX > 0 ? RowFFT<T, LXE, true, 3 * ROWS, NT>::RS : 1;
    alignas(16) cx<T> buf[3 * ROWS * RS];
    alignas(16) cx<T> twl[LXE];
};

// row block bx of gx (the row blocks of one sample) of sample b
template <typename T, typename S, int LX, int ROWS, int MODE, bool BLK = false>
__device__ __forceinline__ void xinv_tile(const typename Spec<T, S>::elem* __restrict__ spec, int SX,
                                          const T* __restrict__ M, const Phys<T>& ph, const XinvOut& out,
                                          const cx<T>* __restrict__ twL, const cx<T>* __restrict__ twP, T hscale,
                                          int bx, int gx, int b, XinvShared<T, LX, ROWS>& sh, long blk_stride = 0) {
    using C = cx<T>;
    constexpr int LXE = LX > 0 ? LX : 2;
    // only x < nx <= LX is kept: packed outputs z[j] with j < LX/2
    using F = RowFFT<T, LXE, true, 3 * ROWS, NT, false, true>;
    constexpr int RS = XinvShared<T, LX, ROWS>::RS;
    C* buf = sh.buf;
    C* twl = sh.twl;
    const long nrow = (long)ph.ny * ph.nz;
    const long N = nrow * ph.nx;
    // the exchange stencil of the fused H_eff reads neighbour rows: y-slab
    // block order (xcd_run, yslab) when the row blocks tile each plane
    long row0 = (long)bx * ROWS;
    const bool tiled = ph.ny % ROWS == 0;
    int plane = 0, y0 = 0;  // z and first y of the block's rows when tiled
    if (tiled) {
        int yg;
        yslab(xcd_run(bx, gx), ph.ny / ROWS, ph.nz, plane, yg);
        y0 = yg * ROWS;
        row0 = (long)plane * ph.ny + y0;
    }
    spec += (long)b * 3 * nrow * (BLK ? SpecBlock<typename Spec<T, S>::elem>::KB : SX);
    if (M) M += (long)b * 3 * N;
    const long vo = (long)b * 3 * N;
    if constexpr (LX == 0) {
        for (int lr = threadIdx.x; lr < 3 * ROWS; lr += NT) {
            const int r = lr / 3, c = lr - 3 * r;
            const long g = row0 + r;
            if (g < nrow) buf[lr * RS] = Spec<T, S>::get(spec[(c * nrow + g) * SX]);
        }
        __syncthreads();
    } else {
        TwStage<T, LX, NT> tw1;
        tw1.fetch(twL);
        // stage-0 inputs Z[k] = (X[k] + X*[LX-k]) + i e^{+2 pi i k/P} (X[k] - X*[LX-k])
        // of tile row lr = 3 r + c (component c of mesh row row0 + r), from
        // global memory
        C xa[F::U0][F::R0], xb[F::U0][F::R0], wk[F::U0][F::R0];
#pragma unroll
        for (int m = 0; m < F::U0; ++m) {
            const int u = threadIdx.x + m * NT;
#pragma unroll
            for (int q = 0; q < F::R0; ++q) {
                int lr, k;
                F::first_input(u, q, lr, k);
                const int r = lr / 3, c = lr - 3 * r;
                const long g = row0 + r;
                xa[m][q] = C{T(0), T(0)};
                xb[m][q] = C{T(0), T(0)};
                wk[m][q] = twP[k];
                if (F::live0(u) && g < nrow) {
                    // (c nrow + g) < 3 ny nz <= 3 * 2^19 and SX <= 1040: exact in 32 bits
                    using E = const typename Spec<T, S>::elem;
                    const SpecRow<BLK, E> row{spec + __umul24((unsigned)(c * (int)nrow + (int)g),
                                                              (unsigned)(BLK ? SpecBlock<E>::KB : SX)),
                                              blk_stride};
                    xa[m][q] = Spec<T, S>::get(row[k]);
                    xb[m][q] = Spec<T, S>::get(row[LX - k]);
                }
            }
        }
        C z[F::U0][F::R0];
#pragma unroll
        for (int m = 0; m < F::U0; ++m)
#pragma unroll
            for (int q = 0; q < F::R0; ++q) {
                const C xk = xa[m][q];
                const C xc = cconj(xb[m][q]);
                const C sm = cadd(xk, xc);
                const C wd = cmulc(csub(xk, xc), wk[m][q]);
                z[m][q] = C{sm.x - wd.y, sm.y + wd.x};
            }
        tw1.put(twl);
        F::first_to_lds(z, buf);
        __syncthreads();
        F::rest(buf, twl);
    }
    const int nx = ph.nx;
    const float rnx = 1.0f / (float)nx;
    for (int e = threadIdx.x; e < ROWS * nx; e += NT) {
        // e / nx through a float reciprocal: (e + 1/2) / nx lies at least
        // 1/(2 nx) >= 2^-12 from an integer, and the rounding error is below
        // 2^-22 (e < 2^15, nx <= 2^10)
        const int r = (int)(((float)e + 0.5f) * rnx), x = e - (int)__umul24((unsigned)r, (unsigned)nx);
        const long g = row0 + r;
        if (g >= nrow) continue;
        T hd[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const C v = buf[(3 * r + c) * RS + (LX > 0 ? F::P(x >> 1) : 0)];
            hd[c] = ((x & 1) ? v.y : v.x) * hscale;
        }
        const long cell = g * nx + x;
        if constexpr (MODE == XINV_DEMAG) {
            T* H = (T*)out.h + vo;
#pragma unroll
            for (int c = 0; c < 3; ++c) H[c * N + cell] = hd[c];
        } else {
            const int y = tiled ? y0 + r : (int)g % ph.ny, z = tiled ? plane : (int)g / ph.ny;
            T m[3], H[3];
            // Eq. (3) operands, loaded with the stencil (terms past nl read m0 and are
            // left out)
            T v[3], fl[3][3];
            if constexpr (MODE == XINV_UPDATE) {
#pragma unroll
                for (int c = 0; c < 3; ++c) v[c] = ((const T*)out.m0)[vo + c * N + cell];
#pragma unroll
                for (int l = 0; l < 3; ++l) {
                    const T* p = (const T*)(l < out.nl ? out.fl[l] : out.m0) + vo;
#pragma unroll
                    for (int c = 0; c < 3; ++c) fl[l][c] = p[c * N + cell];
                }
            }
            heff_at(PtrField<T>{M}, N, cell, x, y, z, b, ph, hd, m, H);
            if constexpr (MODE == XINV_HEFF) {
                T* Ho = (T*)out.h + vo;
#pragma unroll
                for (int c = 0; c < 3; ++c) Ho[c * N + cell] = H[c];
            } else if constexpr (MODE == XINV_UPDATE) {
                T F[3];
                llg_at(m, H, ph, F);
                T* Mn = (T*)out.mnew + vo;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
#pragma unroll
                    for (int l = 0; l < 3; ++l) {
                        const T s = v[c] + (T)out.cb[l] * fl[l][c];
                        v[c] = l < out.nl ? s : v[c];
                    }
                    Mn[c * N + cell] = v[c] + (T)out.cb[out.nl] * F[c];
                }
            } else {
                T F[3];
                llg_at(m, H, ph, F);
                T* Fo = (T*)out.f + vo;
#pragma unroll
                for (int c = 0; c < 3; ++c) Fo[c * N + cell] = F[c];
                if (out.mnext) {
                    T* Mn = (T*)out.mnext + vo;
                    const T cn = (T)out.cnext;
#pragma unroll
                    for (int c = 0; c < 3; ++c) Mn[c * N + cell] = m[c] + cn * F[c];
                }
                if (out.g) {
                    T* G = (T*)out.g + vo;
#pragma unroll
                    for (int c = 0; c < 3; ++c) G[c * N + cell] = hd[c] + ph.n00[c] * m[c];
                }
                if (out.h) {
                    T* Ho = (T*)out.h + vo;
#pragma unroll
                    for (int c = 0; c < 3; ++c) Ho[c * N + cell] = hd[c];
                }
            }
        }
    }
}

template <typename T, typename S, int LX, int ROWS, int MODE, bool BLK>
__global__ __launch_bounds__(NT) void k_xinv(const typename Spec<T, S>::elem* __restrict__ spec, int SX,
                                             long blk_stride, const T* __restrict__ M, Phys<T> ph, XinvOut out,
                                             const cx<T>* __restrict__ twL, const cx<T>* __restrict__ twP,
                                             T hscale) {
    __shared__ XinvShared<T, LX, ROWS> sh;
    xinv_tile<T, S, LX, ROWS, MODE, BLK>(spec, SX, M, ph, out, twL, twP, hscale, blockIdx.x, gridDim.x, blockIdx.y, sh,
                                         blk_stride);
}

// ------------------------------------------------------------------------
// strided column FFT: element (comp, outer, i, kx) at comp*cs + outer*os + i*is + kx
// HALF: the forward transform's input rows >= L/2 are zero (n_in <= L/2) or
// the inverse transform keeps only rows < L/2 (n_out <= L/2)
// LDS of one column-pass tile
template <typename T, typename S, int L, int TK>
struct ColShared {
    using F = ColFFT<T, S, L, false, TK, 1, col_threads(L, TK)>;
    alignas(16) cx<T> buf[F::NSTAGE > 1 ? F::LDS_ELEMS : 1];
    alignas(16) cx<T> twl[L];
};

// tile lin of ntx x nby x nbz tiles (kx tiles, outer index, component)
template <typename T, typename S, int L, bool INV, int TK, bool HALF>
__device__ __forceinline__ void colfft_tile(const typename Spec<T, S>::elem* __restrict__ src, long s_cs, long s_os,
                                            long s_is, int n_in, typename Spec<T, S>::elem* __restrict__ dst,
                                            long d_cs, long d_os, long d_is, int n_out, int Kx,
                                            const cx<T>* __restrict__ tw, T scale, int lin, int ntx, int nby, int nbz,
                                            ColShared<T, S, L, TK>& sh) {
    using C = cx<T>;
    constexpr int NTC = col_threads(L, TK);
    using F = ColFFT<T, S, L, INV, TK, 1, NTC, !INV && HALF, INV && HALF>;
    using E = typename Spec<T, S>::elem;
    // each XCD takes a contiguous run of tiles (xcd_run): when a tile row is
    // shorter than a 128-byte line, the neighbouring tiles that share its
    // lines are mostly fetched into the same L2
    const int pos = xcd_run(lin, ntx * nby * nbz);
    const int bx = pos % ntx, by = (pos / ntx) % nby, bz = pos / (ntx * nby);
    const int kx0 = bx * TK;
    const Base1<const E> sp{src + bz * s_cs + by * s_os + kx0};
    const Base1<E> dp{dst + bz * d_cs + by * d_os + kx0};
    typename F::Regs rg;
    if constexpr (F::NSTAGE == 1) {
        F::load_first(rg, sp, s_is, n_in, Kx - kx0, 1);
        F::single(rg, dp, d_is, n_out, Kx - kx0, 1, scale);
    } else {
        C* buf = sh.buf;
        C* twl = sh.twl;
        TwStage<T, L, NTC> tws;
        tws.fetch(tw);
        F::load_first(rg, sp, s_is, n_in, Kx - kx0, 1);
        tws.put(twl);
        F::first_to_lds(rg, buf);
        __syncthreads();
        F::middle(buf, twl);
        F::last_to_global(buf, twl, dp, d_is, n_out, Kx - kx0, 1, scale);
    }
}

template <typename T, typename S, int L, bool INV, int TK, bool HALF>
__global__ __launch_bounds__(col_threads(L, TK)) void k_colfft(const typename Spec<T, S>::elem* __restrict__ src, long s_cs,
                                               long s_os, long s_is, int n_in,
                                               typename Spec<T, S>::elem* __restrict__ dst, long d_cs, long d_os,
                                               long d_is, int n_out, int Kx, const cx<T>* __restrict__ tw,
                                               T scale) {
    __shared__ ColShared<T, S, L, TK> sh;
    colfft_tile<T, S, L, INV, TK, HALF>(src, s_cs, s_os, s_is, n_in, dst, d_cs, d_os, d_is, n_out, Kx, tw, scale,
                                        blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z), gridDim.x,
                                        gridDim.y, gridDim.z, sh);
}

// ------------------------------------------------------------------------
// z forward, k-space product H^ = K^ M^ (K^ = -N^/(Px Py Pz), real and
// symmetric, stored for |ky| <= Py/2, |kz| <= Pz/2; the components odd in y
// (xy, yz) change sign for ky > Py/2, those odd in z (xz, yz) for kz > Pz/2),
// z inverse.  In place on rows z < nz of the [3][nz][nyrows][SX] buffer.
// One workgroup takes the rows ky = q and ky = Py - q, which share the folded
// kernel, so every folded value is read from memory once.  Tile groups
// g = w * 3 + c: component c of row ky = (w ? Py - q : q).
//
template <typename E>
struct ZBases {
    E* row0;  // (ky = q, component 0, z = 0, kx0)
    E* row1;  // (ky = Py - q, ...)
    unsigned cs;  // component stride nz * nyrows * SX (< 2^31 for every supported mesh)
    __device__ __forceinline__ E* operator()(int g) const {
        // one multiply-add; a chain of selects compiles to branches
        const unsigned c = g >= 3 ? g - 3 : g;
        return (g >= 3 ? row1 : row0) + (unsigned long)c * cs;
    }
};

// H = K M of one (column, kz) with the values k of the folded kernel; yneg and
// zneg: rows ky > Py/2, kz > Pz/2, where the components odd along that axis
// change sign
template <typename T>
__device__ __forceinline__ void apply_kernel(const T (&k)[6], bool yneg, bool zneg, cx<T>& px, cx<T>& py, cx<T>& pz) {
    using C = cx<T>;
    const T nxx = k[0], nyy = k[1], nzz = k[2];
    const T nxy = yneg ? -k[3] : k[3], nxz = zneg ? -k[4] : k[4];
    const T yz = zneg ? -k[5] : k[5], nyz = yneg ? -yz : yz;
    const C mx = px, my = py, mz = pz;
    px = C{nxx * mx.x + nxy * my.x + nxz * mz.x, nxx * mx.y + nxy * my.y + nxz * mz.y};
    py = C{nxy * mx.x + nyy * my.x + nyz * mz.x, nxy * mx.y + nyy * my.y + nyz * mz.y};
    pz = C{nxz * mx.x + nyz * my.x + nzz * mz.x, nxz * mx.y + nyz * my.y + nzz * mz.y};
}

// FP32 z passes with a radix-8 stage take the product in registers between the
// last forward and the first inverse stage (zmul_tile); in FP64 the thread's
// values and kernel values fill 230 registers and the waves left hide less than
// the LDS passes cost (256x256x16 46 us against 41.8, 200x120x10 27.7 against 19.4).
// FP32, back to back, before and after: 256x256x16 24.8 -> 23.4 us, 128x128x32 19.9 ->
// 15.8, 200x200x6 15.4 -> 13.2, 128x64x128 (LZ 256) 54 -> 39, 60x60x200 (LZ 512) 92 ->
// 46 (the last two mostly by zmul_place), 512x512x64 546 -> 526 and BF16 560 -> 463.
// The pass moves its bytes (within 3 %) at 5.6 TB/s where spectrum B stays in the
// 256 MB cache in front of HBM and at 3.9 TB/s where it does not (512x512x64: 64-byte
// rows read and written in place); its vector ALUs are 60-75 % busy.
template <typename T>
constexpr bool zmul_in_regs(int LZ) { return sizeof(T) == 4 && LZ >= 16; }

// threads of a z tile: with the product in registers one thread per (ky, column,
// eight kz) in whole waves, else NT
template <typename T>
constexpr int zmul_threads(int LZ, int TK) {
    if (!zmul_in_regs<T>(LZ)) return NT;
    const int n = (LZ / 8) * 2 * TK;
    return n < 64 ? 64 : (n + 63) / 64 * 64;
}

// LDS of one z-pass tile
template <typename T, int LZ, int TK>
struct ZmulShared {
    static constexpr int L = LZ > 1 ? LZ : 2;
    alignas(16) cx<T> lb[LZ * 6 * TK];
    alignas(16) cx<T> twl[L];
};

// kx tile `tile`, folded row pair q, sample `sample`
//
// FP32, lengths of 16 and more: the last forward stage (radix 8, outputs kz = j + r
// LZ/8) and the first inverse stage (radix 8 with inputs j + r LZ/8, or radix R0
// with inputs j' + q LZ/R0, 8/R0 of its butterflies) take the same elements, so one
// thread does both and the product between them in registers, for the three
// components of one (ky, column, j).  The tile then crosses the LDS four times
// (eight with a third stage) instead of eight to twelve.  The thread's 8 x 6 kernel
// values are loaded with the tile, whole packs a lane.  The inverse starts with
// radix 8 where the spectra are stored in FP32; 16-bit spectra keep the order
// of the other passes (R0 first; col_radix), bit for bit that of the tile in LDS.
template <typename T, typename S, int LZ, int TK>
__device__ __forceinline__ void zmul_tile(typename Spec<T, S>::elem* __restrict__ buf, int SX, int Kx, int nz,
                                          int nyrows, int Py, const T* __restrict__ kfold,
                                          const cx<T>* __restrict__ tw, int tile, int q, int sample,
                                          ZmulShared<T, LZ, TK>& sh) {
    using C = cx<T>;
    using E = typename Spec<T, S>::elem;
    constexpr int L = LZ > 1 ? LZ : 2;  // LZ = 1 uses no transform
    constexpr int KZF = LZ / 2 + 1;
    constexpr int NTZ = zmul_threads<T>(LZ, TK), W = 6 * TK;
    // rows z >= nz of the forward input are the zero padding and only rows
    // z < nz of the inverse output are kept; nz <= Pz/2 always
    using Ff = ColFFT<T, S, L, false, TK, 6, NTZ, true, false>;
    using Fi = ColFFT<T, S, L, true, TK, 6, NTZ, false, true>;
    C* lb = sh.lb;
    C* twl = sh.twl;
    const int kx0 = tile * TK;
    const int ng = (2 * q == Py || q == 0) ? 3 : 6;  // 0 <= q <= Py/2
    const int ncol = Kx - kx0;
    const long cs = (long)nz * nyrows * SX, zs = (long)nyrows * SX;
    E* sb = buf + (long)sample * 3 * cs;
    const ZBases<E> bases{sb + (long)q * SX + kx0, sb + (long)(Py - q) * SX + kx0, (unsigned)cs};
    const T* __restrict__ krow = kfold + kernel_row(q, SX, KZF);  // uniform
    // A tile may reach past Kx: columns >= ncol read the kernel of column Kx - 1
    // instead, so every load stays in bounds and is issued unconditionally.
    // Those columns are never stored.
    auto kcol = [&](int col) { return kx0 + (col < ncol ? col : ncol - 1); };
    if constexpr (zmul_in_regs<T>(LZ)) {
        constexpr int L8 = LZ / 8, NU = L8 * 2 * TK;
        TwStage<T, LZ, NTZ> tws;
        tws.fetch(tw);
        typename Ff::Regs rg;
        Ff::load_first(rg, bases, zs, nz, ncol, ng);
        const bool live = NU % NTZ == 0 || (int)threadIdx.x < NU;
        const int e = live ? threadIdx.x : NU - 1;
        const int col = e % TK, w = (e / TK) & 1, j = e / (2 * TK);
        const int kc = kcol(col);
        T k[8][6];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int kz = j + r * L8;  // j < L8: above LZ/2 for r > 4, and for r = 4 unless j = 0
            kernel_load<T>(krow, kc, r < 4 || (r == 4 && j == 0) ? kz : LZ - kz, SX, k[r]);
        }
        tws.put(twl);
        Ff::first_to_lds(rg, lb);
        __syncthreads();
        Ff::middle(lb, twl);
        C v[3][8];
        C* p = lb + w * 3 * TK + col;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const C t = twl[r * j];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const C a = p[(j + r * L8) * W + c * TK];
                v[c][r] = r == 0 ? a : cmul(a, t);
            }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) dft8<false>(v[c]);
#pragma unroll
        for (int r = 0; r < 8; ++r)
            apply_kernel(k[r], w != 0, r > 4 || (r == 4 && j != 0), v[0][r], v[1][r], v[2][r]);
        constexpr int IR = std::is_same<T, S>::value ? 8 : Fi::R0, NB = 8 / IR;
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                C x[IR];
#pragma unroll
                for (int i = 0; i < IR; ++i) x[i] = v[c][b + i * NB];
                dft_r<IR, true>(x);
#pragma unroll
                for (int i = 0; i < IR; ++i) v[c][b + i * NB] = x[i];
            }
        __syncthreads();
        if (live) {
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int i = 0; i < IR; ++i) p[((j + b * L8) * IR + i) * W + c * TK] = v[c][b + i * NB];
        }
        __syncthreads();
        if constexpr (std::is_same<T, S>::value) {
            Fi::rest_to_global(lb, twl, bases, zs, nz, ncol, ng, T(1));
        } else {
            Fi::middle(lb, twl);
            Fi::last_to_global(lb, twl, bases, zs, nz, ncol, ng, T(1));
        }
    } else {
        // the transform in LDS in natural order, the kernel values of this
        // thread's product units (both ky rows of a column and kz) in registers
        using PU = typename Ff::PU;
        using RW = typename Ff::RW;
        constexpr int PN = Ff::PN;
        constexpr int NUP = LZ * TK, PER = (NUP + NTZ - 1) / NTZ;
        T k[PER][6];
        auto load_k = [&]() {
#pragma unroll
            for (int m = 0; m < PER; ++m) {
                const int e0 = threadIdx.x + m * NTZ, e = e0 < NUP ? e0 : NUP - 1;
                const int kz = e / TK;
                kernel_load<T>(krow, kcol(e % TK), 2 * kz <= LZ ? kz : LZ - kz, SX, k[m]);
            }
        };
        if constexpr (LZ == 1) {
            constexpr int NU = 6 * (TK / PN);
            load_k();
            for (int u = threadIdx.x; u < NU; u += NTZ) {
                const int p = u % (TK / PN), g = u / (TK / PN);
                if (g < ng && p * PN < ncol) {
                    PU v;
                    v.raw = *(const RW*)(bases(g) + p * PN);
#pragma unroll
                    for (int i = 0; i < PN; ++i) lb[g * TK + p * PN + i] = Spec<T, S>::get(v.e[i]);
                }
            }
        } else {
            TwStage<T, LZ, NTZ> tws;
            tws.fetch(tw);
            typename Ff::Regs rg;
            Ff::load_first(rg, bases, zs, nz, ncol, ng);
            load_k();
            tws.put(twl);
            Ff::first_to_lds(rg, lb);
            if constexpr (Ff::NSTAGE > 1) {
                __syncthreads();
                Ff::middle(lb, twl);
                Ff::last_in_lds(lb, twl);
            }
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < PER; ++m) {
            const int e = threadIdx.x + m * NTZ;
            if (NUP % NTZ == 0 || e < NUP) {
                const int kz = e / TK;
                const bool zneg = 2 * kz > LZ;
                C* p = lb + kz * W + e % TK;
                apply_kernel(k[m], false, zneg, p[0], p[TK], p[2 * TK]);
                if (ng == 6) apply_kernel(k[m], true, zneg, p[3 * TK], p[4 * TK], p[5 * TK]);
            }
        }
        __syncthreads();
        if constexpr (LZ > 1) Fi::first_in_lds(lb);
        if constexpr (Fi::NSTAGE > 1) {
            Fi::middle(lb, twl);
            Fi::last_to_global(lb, twl, bases, zs, nz, ncol, ng, T(1));
            return;
        }
        constexpr int NU = LZ * 6 * (TK / PN);
        for (int u = threadIdx.x; u < NU; u += NTZ) {
            const int p = u % (TK / PN), t = u / (TK / PN), g = t % 6, z = t / 6;
            if (g < ng && p * PN < ncol && z < nz) {
                PU v;
#pragma unroll
                for (int i = 0; i < PN; ++i) v.e[i] = Spec<T, S>::put(lb[z * W + g * TK + p * PN + i]);
                *(RW*)(bases(g) + z * zs + p * PN) = v.raw;
            }
        }
    }
}

// Tiles of one 128-byte line of a spectrum row (G of them when a tile row is
// shorter) are placed on one XCD, one dispatch round apart, so the line is
// fetched into one L2: position lin of ntile x nq (ntile a multiple of G, XCD
// lin % 8) -> tile and row pair.
template <typename E, int TK>
constexpr int zmul_group() { return TK * (int)sizeof(E) >= 128 ? 1 : 128 / (TK * (int)sizeof(E)); }
template <typename E, int TK>
__device__ __forceinline__ void zmul_place(int lin, int ntile, int nq, int& tile, int& q) {
    constexpr int G = zmul_group<E, TK>(), B = 8 * G;
    if (G > 1 && lin < ntile * nq / B * B) {
        const int r = lin % B;
        lin = lin - r + (r % 8) * G + r / 8;
    }
    q = lin / ntile;
    tile = lin - q * ntile;
}

template <typename T, typename S, int LZ, int TK>
__global__ __launch_bounds__(zmul_threads<T>(LZ, TK)) void k_zmul(typename Spec<T, S>::elem* __restrict__ buf, int SX, int Kx, int nz,
                                             int nyrows, int Py, const T* __restrict__ kfold,
                                             const cx<T>* __restrict__ tw) {
    __shared__ ZmulShared<T, LZ, TK> sh;
    int tile, q;
    zmul_place<typename Spec<T, S>::elem, TK>(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x, gridDim.y, tile, q);
    if (tile * TK >= Kx) return;
    zmul_tile<T, S, LZ, TK>(buf, SX, Kx, nz, nyrows, Py, kfold, tw, tile, q, blockIdx.z, sh);
}

}  // namespace llgx

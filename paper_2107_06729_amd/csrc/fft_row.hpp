// FFTs along contiguous rows held in LDS, for the x passes.
//
// NR rows of length L; element i of row r lives at buf[r * RS + P(i)].  Powers
// of two have P(i) = i + i / 16 (FP64: i / 8): the LDS serves 128 bytes a cycle,
// 16 complex values (8), so runs of consecutive elements, two thirds of the
// accesses, stay free of conflicts, and the stride-8 writes of the first stage
// spread over the banks.  (One padding element after every 8 FP32 values made
// every run take two rounds: 256x1000x4, 43 % of the LDS cycles of the fused
// pass.)  Other lengths are not padded (their R0 is a multiple of 3 or 5: at
// most a few lanes share a bank, in that stage alone, and the padded index of
// every element cost more: a third of the instructions of a 640-row tile were
// index arithmetic).  The stages address element x0 + r S of a unit as P(x0) +
// dP(r S), one index per unit: exact when S is a multiple of the padding step, or
// when S divides it and x0 mod S + r S crosses no step that r S does not.  The stage
// schedule is that of fft_lds.hpp (radix R0, then radix 8).
//
// Work unit of every stage: one butterfly j of one row, j fastest, so
// consecutive threads touch consecutive elements.  The first stage takes its
// inputs from the caller in registers (x[m][q] = element j + q L/R0 of the
// unit's row, unit u = threadIdx.x + m NT), so a caller can load them straight
// from global memory (coalesced along the row) and fuse any pre-processing.
// The last stage runs in place in LDS (each unit rewrites its own elements).
// HALF_IN: elements >= L/2 of every row are zero (a zero padded forward
// transform), so stage 0 drops them at compile time.  HALF_OUT: only
// elements < L/2 are read afterwards, so the last stage forms only the first
// half of its radix-8 outputs.
#pragma once
#include <hip/hip_runtime.h>

#include "fft_lds.hpp"

namespace llgx {

template <typename T, int L, bool INV, int NR, int NT, bool HALF_IN = false, bool HALF_OUT = false>
struct RowFFT {
    using C = cx<T>;
    static constexpr int R0 = first_radix(L);
    static constexpr int NSTAGE = fft_stages(L, R0);
    static constexpr bool PAD = (L & (L - 1)) == 0;
    static constexpr int PS = sizeof(T) == 4 ? 4 : 3;          // a padding element after 2^PS
    static constexpr int RS = L + (PAD ? L >> PS : 0) + 1;  // row stride (complex)
    static constexpr int LDS_ELEMS = NR * RS;
    static constexpr int NU0 = NR * (L / R0), U0 = (NU0 + NT - 1) / NT;
    static constexpr int NU8 = NR * (L / 8), U8 = (NU8 + NT - 1) / NT;
    static_assert(L >= 2, "length");

    static __device__ __forceinline__ int P(int i) { return PAD ? i + (i >> PS) : i; }
    // P(x0 + d) - P(x0) for the strides of the stages
    static constexpr int dP(int d) { return PAD ? d + (d >> PS) : d; }

    // unit u of a stage with L/R butterflies per row
    template <int R>
    static __device__ __forceinline__ void unit(int u, int& row, int& j) {
        row = u / (L / R);
        j = u - row * (L / R);
    }

    // element index of input q of stage-0 unit u (for the caller's loads)
    static __device__ __forceinline__ void first_input(int u, int q, int& row, int& i) {
        int j;
        unit<R0>(u, row, j);
        i = j + q * (L / R0);
    }

    static __device__ __forceinline__ bool live0(int u) { return NU0 % NT == 0 || u < NU0; }

    // stage 0 on the caller's values, outputs to rows j R0 + q
    static __device__ __forceinline__ void first_to_lds(C (&x)[U0][R0], C* buf) {
#pragma unroll
        for (int m = 0; m < U0; ++m) {
            const int u = threadIdx.x + m * NT;
            if (live0(u)) {
                int row, j;
                unit<R0>(u, row, j);
                if constexpr (HALF_IN) {
#pragma unroll
                    for (int q = (R0 + 1) / 2; q < R0; ++q) x[m][q] = C{T(0), T(0)};
                }
                dft_r<R0, INV>(x[m]);
                C* rb = buf + row * RS + P(j * R0);
#pragma unroll
                for (int q = 0; q < R0; ++q) rb[dP(q)] = x[m][q];
            }
        }
    }

    template <int NS>
    static __device__ __forceinline__ void mid_stage(C* buf, const C* __restrict__ tw) {
        C x[U8][8];
#pragma unroll
        for (int m = 0; m < U8; ++m) {
            const int u = threadIdx.x + m * NT;
            if (NU8 % NT == 0 || u < NU8) {
                int row, j;
                unit<8>(u, row, j);
                const int k = j % NS;
                const C* rb = buf + row * RS + P(j);
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const C a = rb[dP(r * (L / 8))];
                    const C w = tw[r * k * (L / (NS * 8))];
                    x[m][r] = r == 0 ? a : (INV ? cmulc(a, w) : cmul(a, w));
                }
                dft_r<8, INV>(x[m]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < U8; ++m) {
            const int u = threadIdx.x + m * NT;
            if (NU8 % NT == 0 || u < NU8) {
                int row, j;
                unit<8>(u, row, j);
                const int k = j % NS;
                C* rb = buf + row * RS + P((j / NS) * NS * 8 + k);
#pragma unroll
                for (int r = 0; r < 8; ++r) rb[dP(r * NS)] = x[m][r];
            }
        }
        __syncthreads();
    }

    template <int NS>
    static __device__ __forceinline__ void mid_from(C* buf, const C* __restrict__ tw) {
        if constexpr (NS * 8 < L) {
            mid_stage<NS>(buf, tw);
            mid_from<NS * 8>(buf, tw);
        }
    }

    // stages between the first and the last (a barrier before, one at the end)
    static __device__ __forceinline__ void middle(C* buf, const C* __restrict__ tw) {
        if constexpr (NSTAGE > 2) mid_from<R0>(buf, tw);
    }

    // stage 0 from LDS (data in natural order, a barrier before); ends with a barrier
    static __device__ __forceinline__ void first_in_lds(C* buf) {
        C x[U0][R0];
#pragma unroll
        for (int m = 0; m < U0; ++m) {
            const int u = threadIdx.x + m * NT;
            if (live0(u)) {
                int row, j;
                unit<R0>(u, row, j);
                const C* rb = buf + row * RS + P(j);
#pragma unroll
                for (int q = 0; q < R0; ++q) x[m][q] = rb[dP(q * (L / R0))];
            }
        }
        __syncthreads();
        first_to_lds(x, buf);
        __syncthreads();
    }

    // outputs x[8] of the last stage (elements j + r L/8) of one unit, rb at P(j)
    static __device__ __forceinline__ void last_regs(const C* rb, const C* __restrict__ tw, int j, C (&x)[8]) {
        constexpr int NS = L / 8;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const C a = rb[dP(r * NS)];
            const C w = tw[r * j];
            x[r] = r == 0 ? a : (INV ? cmulc(a, w) : cmul(a, w));
        }
        dft_r<8, INV>(x);
    }

    // last stage, each kept output handed to f(row, element, value); NSTAGE >= 2
    template <typename Fn>
    static __device__ __forceinline__ void last_each(const C* buf, const C* __restrict__ tw, const Fn& f) {
#pragma unroll
        for (int m = 0; m < U8; ++m) {
            const int u = threadIdx.x + m * NT;
            if (NU8 % NT == 0 || u < NU8) {
                int row, j;
                unit<8>(u, row, j);
                C x[8];
                last_regs(buf + row * RS + P(j), tw, j, x);
#pragma unroll
                for (int r = 0; r < (HALF_OUT ? 4 : 8); ++r) f(row, j + r * (L / 8), x[r]);
            }
        }
    }

    // every stage after the first; callers put a barrier after first_to_lds,
    // and this ends with one
    static __device__ __forceinline__ void rest(C* buf, const C* __restrict__ tw) {
        if constexpr (NSTAGE > 1) {
            middle(buf, tw);
#pragma unroll
            for (int m = 0; m < U8; ++m) {
                const int u = threadIdx.x + m * NT;
                if (NU8 % NT == 0 || u < NU8) {
                    int row, j;
                    unit<8>(u, row, j);
                    C* rb = buf + row * RS + P(j);
                    C x[8];
                    last_regs(rb, tw, j, x);
#pragma unroll
                    for (int r = 0; r < (HALF_OUT ? 4 : 8); ++r) rb[dP(r * (L / 8))] = x[r];
                }
            }
            __syncthreads();
        }
    }
};

}  // namespace llgx

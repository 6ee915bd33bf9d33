// Kernel declarations and launch helpers shared by the HIP sources.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

#include "fft_lds.hpp"

namespace llgx {

constexpr int MAX_F = 8;       // stage derivatives an Eq. (4) combination may read
constexpr int MAX_HIST = 6;    // Eq. (6) nodes: p + 1 with p <= 5
constexpr int MAX_LEN = 2048;  // largest padded FFT length per axis

// Stage input of Eq. (4): M_k = base + sum_l coef[l] * f[l] (coef = h b_kl).
template <typename T>
struct Combo {
    const T* base;
    const T* f[MAX_F];
    T coef[MAX_F];
    int nf;
};

// Eq. (6) at one sub-step: H_d = sum_i w[i] g[i] - N00 M_k.
template <typename T>
struct Extrap {
    const T* g[MAX_HIST];
    T w[MAX_HIST];
    int n;
};

// Eq. (6) for several sub-step times at once: out[j] = sum_i w[j][i] g[i].
template <typename T>
struct EPoly {
    const T* g[MAX_HIST];
    T w[MAX_F][MAX_HIST];
    T* out[MAX_F];
    int ng, nd;
};

// 2-D launch of the per-cell kernels (x along threads, mesh rows along blocks).
struct CellGrid {
    dim3 grid, block;
    long nblocks;
};
CellGrid cell_grid(int nx, int ny, int nz, int nb);

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own
// L2): block b runs on XCD b % 8.  Give each XCD one contiguous run of row
// groups, so the y and z neighbours a stencil reads were mostly fetched into
// the same L2 by the same XCD.
__device__ __forceinline__ int xcd_run(int b, int nblk) {
    const int q = nblk >> 3, r = nblk & 7, x = b & 7, i = b >> 3;
    return x * q + (x < r ? x : r) + i;
}

// Order of the row blocks of the stencil kernels: the run of positions that
// xcd_run gives one XCD is a range of y-groups over all planes (z and
// samples), not a range of planes, so the stencil's z neighbours come from
// the same XCD's L2 and only the rows at the two ends of a y range are
// fetched by two XCDs.  Maps position p to (plane, y-group) for gy y-groups
// per plane, y fastest within a range; a bijection on [0, gy * planes).
__device__ __forceinline__ void yslab(int p, int gy, int planes, int& plane, int& yg) {
    const int q = gy >> 3, r = gy & 7;  // ranges 0..r-1 hold q + 1 groups, the rest q
    const int big = planes * (q + 1);
    int c, o, g;
    if (p < r * big) {
        c = p / big;
        o = p - c * big;
        g = q + 1;
    } else {  // only reached when q > 0
        const int small = planes * q, pp = p - r * big;
        c = r + pp / small;
        o = pp - (c - r) * small;
        g = q;
    }
    plane = o / g;
    yg = c * q + (c < r ? c : r) + (o - plane * g);
}

// Eq. (3): M = M0 + sum_k cb[k] f[k] (cb = h c_k) and, when err is set, the
// per-cell estimate |sum_k ce[k] f[k]| (ce = h (c_k - c^_k)) over the union of
// the stage derivatives either sum uses.
template <typename T>
struct Final {
    const T* f[MAX_F];
    T cb[MAX_F];
    double ce[MAX_F];
    int n;
    int err;
};

// Material and field constants of the H_eff terms and the LLG right-hand side.
template <typename T>
struct Phys {
    T exx, exy, exz;   // 2A/(mu0 Ms^2) / d^2 per axis
    T ani;             // 2K/(mu0 Ms^2)
    T u[3];            // anisotropy axis
    T gp;              // gamma / (1 + alpha^2)
    T gpa;             // gamma alpha / ((1 + alpha^2) Ms)
    T n00[3];          // self term of Eq. (6)
    const T* hab;      // applied field of each sample [nb][3] (device)
    const int* empty;  // device flag: nonzero when some cell has M = 0 (no material), or nobody looked
    int nx, ny, nz;
    int nb;            // samples of this mesh processed by one launch
};

// Output selection of the inverse x pass.
enum XinvMode { XINV_DEMAG = 0, XINV_HEFF = 1, XINV_RHS = 2, XINV_UPDATE = 3 };

struct XinvOut {
    void* h;       // demag field (XINV_DEMAG) or H_eff (XINV_HEFF), may be null in XINV_RHS
    void* f;       // dM/dt (XINV_RHS)
    void* g;       // stored field G = H_d + N00 M of Eq. (6) (optional)
    void* mnext;   // XINV_RHS, optional: next stage input M + cnext F (Eq. 4, a stage
                   // row whose only entry is the stage just formed)
    double cnext;
    // XINV_UPDATE, the last stage of a step: Eq. (3), mnew = m0 + sum_l cb[l] fl[l]
    // + cb[nl] F (nl <= 3 earlier stages), instead of f; mnew may be m0
    const void* m0 = nullptr;
    const void* fl[3] = {nullptr, nullptr, nullptr};
    void* mnew = nullptr;
    double cb[4] = {0.0, 0.0, 0.0, 0.0};
    int nl = 0;
};

// Host-side launchers of the FFT passes (pass_x.hip, pass_col.hip, pass_z.hip)
// and of the tensor setup (newell.hip).  Lengths as listed in fft_lds.hpp.  Spectra
// are passed untyped (SpecPtr) and stored as S: the working precision T, or
// _Float16 / __bf16 pairs for T = float.  fscale, scale and hscale multiply
// the x-pass input, the y-pass output and the final field (all 1 for storage
// in the working precision); the folded k-space kernel carries its own scale.
using SpecPtr = void*;
template <typename T, typename S>
hipError_t launch_xfwd(hipStream_t s, int LX, const Combo<T>& in, T* mk_out, int nin, long nrows, SpecPtr spec,
                       int SX, long blk_stride, const cx<T>* twL, const cx<T>* twP, T fscale, int variant);
template <typename T, typename S>
hipError_t launch_xinv(hipStream_t s, int LX, int mode, SpecPtr spec, int SX, long blk_stride, const T* M,
                       const Phys<T>& ph,
                       const XinvOut& out, const cx<T>* twL, const cx<T>* twP, T hscale, int variant);
template <typename T, typename S>
hipError_t launch_colfft(hipStream_t s, int L, bool inv, SpecPtr src, long s_cs, long s_os, long s_is, int n_in,
                         SpecPtr dst, long d_cs, long d_os, long d_is, int n_out, int Kx, int nouter, int ncomp,
                         const cx<T>* tw, T scale, int variant);
template <typename T, typename S>
hipError_t launch_zmul(hipStream_t s, int LZ, SpecPtr buf, int SX, int Kx, int nz, int nyrows, int Py, int Pz,
                       const T* kfold, int Kyf, int Kzf, const cx<T>* tw, int nb, int variant);
// Fused y/z pass of thin meshes (pass_yzy.hip): spectrum A blocked by 32
// bytes of kx (SpecBlock), blk_stride elements apart (0 in the x passes above:
// plain rows of SX); kcol is the folded kernel as [kx][kz][component][KYS].
template <typename T, typename S>
hipError_t launch_yzy(hipStream_t s, int LY, SpecPtr spec, long blk_stride, int Kx, int ny, int nz, int nb,
                      const T* kcol, int KYS, const cx<T>* tw, T yscale, int variant);
// whether the fused pass takes a mesh of nz cells padded to LY along y (native:
// spectra stored in the working precision)
template <typename T>
bool yzy_ok(int LY, int nz, bool native);
// its variant on a new handle, for so many columns (all samples)
int yzy_default(int LY, int nz, long columns);
hipError_t launch_newell_octant(hipStream_t s, int nx, int ny, int nz, double dx, double dy, double dz,
                                double* octant);
hipError_t launch_scatter_tensor(hipStream_t s, const double* octant, int comp, int nx, int ny, int nz,
                                 int Px, int Py, int Pz, double* real);
template <typename T>
hipError_t launch_fold(hipStream_t s, const cx<double>* spec, int SX, int Kx, int Py, int Pz, int Kyf, int Kzf,
                       double scale, int comp, T* kfold, T* kcol, int KYS, double* imag_max_parts, int nparts);

// Folded k-space kernel layout: for each (ky, kz) the six components of SX
// columns in planes of 16-byte packs, FP32 [kx][xx yy zz xy] and [kx][xz yz] (8
// bytes), FP64 [kx][xx yy], [kx][zz xy], [kx][xz yz].  A lane per column reads
// whole packs and consecutive columns are contiguous; a tile of 16 FP32 (8
// FP64) columns reads whole 128-byte lines of every plane.
// kernel_index = kernel_row (start of the ky row, 64-bit) + kernel_off (within
// the row, < 6 Kzf SX, 32-bit).
__host__ __device__ __forceinline__ long kernel_row(int kyf, int SX, int Kzf) { return (long)kyf * SX * Kzf * 6; }
template <typename T>
__host__ __device__ __forceinline__ int kernel_off(int kx, int kzf, int comp, int SX) {
    const int row = kzf * SX * 6;
    if (sizeof(T) == 8) return row + (comp / 2) * SX * 2 + kx * 2 + comp % 2;
    return comp < 4 ? row + kx * 4 + comp : row + SX * 4 + kx * 2 + comp - 4;
}
template <typename T>
__host__ __device__ __forceinline__ long kernel_index(int kyf, int kx, int kzf, int comp, int SX, int Kzf) {
    return kernel_row(kyf, SX, Kzf) + kernel_off<T>(kx, kzf, comp, SX);
}
// the six components of one (ky, kz, column): off = kernel_off(kx, kzf, 0, SX)
template <typename T>
__device__ __forceinline__ void kernel_load(const T* __restrict__ row, int kx, int kzf, int SX, T (&k)[6]) {
    if constexpr (sizeof(T) == 4) {
        const float4 a = *(const float4*)(row + kernel_off<T>(kx, kzf, 0, SX));
        const float2 b = *(const float2*)(row + kernel_off<T>(kx, kzf, 4, SX));
        k[0] = a.x, k[1] = a.y, k[2] = a.z, k[3] = a.w, k[4] = b.x, k[5] = b.y;
    } else {
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const double2 a = *(const double2*)(row + kernel_off<T>(kx, kzf, 2 * p, SX));
            k[2 * p] = a.x, k[2 * p + 1] = a.y;
        }
    }
}

// Launch variants per FFT pass (bit-identical results, different tiles).
constexpr int NVAR_XFWD = 3, NVAR_COL = 3, NVAR_ZMUL = 3, NVAR_XINV = 3;

// Stage kernels (llg.hip).
template <typename T>
hipError_t launch_combine(hipStream_t s, long n, const Combo<T>& c, T* out);
// Optional second output of a sub-step kernel: the next stage input of Eq. (4),
// mnext = m0 + sum_l coef[l] f[l] + cnext F (nf terms of earlier stages, then the
// stage just formed), so no combination pass is needed for it.
template <typename T>
struct NextStage {
    const T* m0;
    T* mnext;
    T cnext;
    int nf;
    const T* f[MAX_F - 1];
    T coef[MAX_F - 1];
    // na > 0 (at most 2): in place of F the kernel writes Eq. (3) up to this
    // stage, m0 + sum_l ca[l] fa[l] + cown F
    int na;
    const T* fa[2];
    T ca[2], cown;
};

// Sub-step F at the stage input mk.base (mk.nf must be 0: a stage input with
// terms is formed once by launch_combine; forming M_k inside the 7-point
// stencil re-reads every term at the neighbours, which measured slower than
// one combine pass on gfx950 even for a single term).
template <typename T>
hipError_t launch_extrap_rhs(hipStream_t s, const Combo<T>& mk, const Extrap<T>& ex, const Phys<T>& ph, T* F,
                             const NextStage<T>& nx);
template <typename T>
hipError_t launch_epoly(hipStream_t s, long n, const EPoly<T>& ep);
// launch_extrap_rhs fused with launch_epoly: writes every ep.out[j] and
// takes this stage's field from E_jself (jself < 0: ex.g[0]); ep.ng <= 6,
// ep.nd <= 2 (else hipErrorInvalidValue)
template <typename T>
hipError_t launch_stage_ep(hipStream_t s, const Combo<T>& mk, const Extrap<T>& ex, const EPoly<T>& ep, int jself,
                           const Phys<T>& ph, T* F, const NextStage<T>& nx);
template <typename T>
hipError_t launch_stage_final(hipStream_t s, const Combo<T>& mk, const Extrap<T>& ex, const Phys<T>& ph, const T* M0,
                              const Final<T>& fs, double inv_ms, T* mnew, double* parts);
// Whether the sub-steps of a mesh form Eq. (6) themselves (ex.n stored fields)
// instead of reading fields that launch_epoly or launch_stage_ep formed
bool eq6_inside(long cells, size_t real_bytes);
// ABM2's sub-step at the predicted state mk (1 or 2 terms), formed inside
template <typename T>
hipError_t launch_predicted(hipStream_t s, const Combo<T>& mk, const Extrap<T>& ex, const Phys<T>& ph, T* F);
template <typename T>
hipError_t launch_final(hipStream_t s, long ncell, int nb, const T* base, const Final<T>& fs, double inv_ms, T* mnew,
                        double* parts, int nparts);
// nout partials of the maximum of nparts values (NaN propagates)
hipError_t launch_reduce_max(hipStream_t s, const double* parts, int nparts, double* out, int nout);
// per-block partials (nparts blocks) of max over cells |v| / Ms, for launch_reduce_max
template <typename T>
hipError_t launch_max_norm(hipStream_t s, long ncell, int nb, const T* v, double inv_ms, double* parts, int nparts);
// flag = 1 if any of the n cells ([nb][3][ncell] layout) has M = 0 (flag is
// not cleared here)
template <typename T>
hipError_t launch_detect_empty(hipStream_t s, long ncell, int nb, const T* M, int* flag);
template <typename T>
hipError_t launch_renorm(hipStream_t s, long ncell, int nb, T* M, double Ms);
// p[0..n) = v by a kernel (no hipMemsetAsync)
hipError_t launch_fill_int(hipStream_t s, int* p, int n, int v);
template <typename T>
hipError_t launch_mean(hipStream_t s, long ncell, const T* M, double* parts, int nparts);
hipError_t launch_reduce_sum3(hipStream_t s, const double* parts, int nparts, double* out);
template <typename T>
hipError_t launch_cast(hipStream_t s, long n, const double* src, T* dst);

}  // namespace llgx

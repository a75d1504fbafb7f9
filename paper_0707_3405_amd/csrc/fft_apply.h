// Plane-wave H.X apply, kinetic + local part (hot-path rows a2-a6).
//
// Sec. 2.2 (iii) and sec. 4.1: the local potential is applied by transforming
// each band to real space on the FFT grid (coefficients zero-padded outside
// the sphere), multiplying by V(r), and transforming back.  Here the 3-D
// transform is pruned to the sphere and split into three passes over a
// "stick" buffer S[band][z][stick] (a stick is one (n_x, n_y) column of the
// sphere):
//
//   pass 1 (k_zinv):  per (band, group of sticks): scatter the sphere
//                     coefficients of each stick into LDS, inverse z-FFT,
//                     write S (only sticks, not the full grid).
//   pass 2 (k_plane): per (band, z-plane): scatter the plane's sticks into the
//                     kept x-columns, inverse y-FFT on those columns, then on
//                     groups of rows inverse x-FFT (its first stage reading the
//                     kept columns directly), multiply by V(r)/N^3, forward
//                     x-FFT (keeping only the kept columns), forward y-FFT,
//                     gather the sticks back into S.
//   pass 3 (k_zfwd):  per (band, group of sticks): forward z-FFT, gather the
//                     sphere points, add the kinetic term 1/2|k+G|^2 X.
//
// Sign convention: grid <- G uses exp(+2 pi i n.j/N) with no scale, G <- grid
// uses exp(-2 pi i n.j/N) with 1/N^3 (folded into the stored potential).
#pragma once

#include <algorithm>
#include <type_traits>

#include "fft_core.h"
#include "pw_internal.h"

namespace pw {

// the k-point items of one launch, passed by value (blockIdx.z picks one)
template <class T>
struct ApplyItems {
    FftApplyItem<T> it[kMaxApplyBatch];
};

// FFT sizes, in two lists so that they compile side by side
#define PW_FFT_SIZES_SMALL(X) X(16) X(20) X(24) X(32) X(36) X(40) X(48) X(60) X(64)
#define PW_FFT_SIZES_LARGE(X) X(72) X(80) X(96) X(108) X(120) X(128)
#define PW_FFT_SIZES(X) PW_FFT_SIZES_SMALL(X) PW_FFT_SIZES_LARGE(X)

// the three passes for one FFT size (false: not a size of the list)
bool run_apply_small(const ApplyItems<double> &items, int nk, const double *v, int nb, hipStream_t st);
bool run_apply_small(const ApplyItems<float> &items, int nk, const float *v, int nb, hipStream_t st);
bool run_apply_large(const ApplyItems<double> &items, int nk, const double *v, int nb, hipStream_t st);
bool run_apply_large(const ApplyItems<float> &items, int nk, const float *v, int nb, hipStream_t st);

namespace {

using namespace fft;

constexpr int kThreads = 256;       // z passes
constexpr int kPlaneWaves = 12;     // most waves of a plane workgroup (three per SIMD: 168 VGPRs each)
constexpr size_t kLdsMax = 160 * 1024;

template <class T>
__device__ __forceinline__ void load_twiddles(cpx<T> *tw_s, const double *tw_g, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        tw_s[i] = cpx<T>{T(tw_g[2 * i]), T(tw_g[2 * i + 1])};
}

// ---- pass 1: inverse z-FFT per stick ---------------------------------------
template <class P, class T>
__global__ void __launch_bounds__(kThreads) k_zinv(const ApplyItems<T> items, int spb) {
    const FftApplyItem<T> &item = items.it[blockIdx.z];
    const SphereDev &sp = item.sp;
    const cpx<T> *__restrict__ X = item.X;
    const int64_t ldx = item.ldx;
    cpx<T> *__restrict__ S = item.S;
    constexpr int N = P::N, LD = N + 1;
    constexpr int R1 = P::R1, R2 = P::R2;
    extern __shared__ unsigned char smem_raw[];
    cpx<T> *tw = reinterpret_cast<cpx<T> *>(smem_raw);
    cpx<T> *buf = tw + N;

    const int band = blockIdx.y;
    const int s0 = blockIdx.x * spb;
    const int ns = min(spb, sp.nst - s0);
    if (ns <= 0) return;
    const cpx<T> *Xb = X + (int64_t)band * ldx;

    load_twiddles(tw, sp.twid, N);
    for (int i = threadIdx.x; i < ns * LD; i += blockDim.x) buf[i] = cpx<T>{T(0), T(0)};
    __syncthreads();
    const int g0 = sp.st_start[s0];
    const int g1 = sp.st_start[s0 + ns - 1] + sp.st_len[s0 + ns - 1];
    for (int g = g0 + threadIdx.x; g < g1; g += blockDim.x) {
        const int pos = sp.g_map[g];
        const int s = pos / N, z = pos - s * N;
        buf[(s - s0) * LD + z] = Xb[g];
    }
    __syncthreads();
    for (int it = threadIdx.x; it < ns * R2; it += blockDim.x) {
        const int seq = it % ns, n2 = it / ns;
        dit_a<P, +1>(buf + seq * LD, n2, tw);
    }
    __syncthreads();
    cpx<T> *Sb = S + (int64_t)band * N * sp.ldst + s0;
    for (int it = threadIdx.x; it < ns * R1; it += blockDim.x) {
        const int seq = it % ns, k1 = it / ns;
        cpx<T> out[R2];
        dit_b<P, +1>(buf + seq * LD, k1, out);
#pragma unroll
        for (int k2 = 0; k2 < R2; ++k2) Sb[(int64_t)(k1 + R1 * k2) * sp.ldst + seq] = out[k2];
    }
}

// ---- pass 2: per z-plane xy transforms with the potential in between -------
// XCD-aware mapping: consecutive hardware workgroup ids go round-robin over
// the 8 XCDs; each XCD is given a contiguous range of (plane, band) work so
// that all bands of one plane share that XCD's L2 copy of V(z, :, :).
__device__ __forceinline__ int xcd_logical(int lin, int total) {
    const int q = total / 8, r = total % 8;
    const int xcd = lin % 8, local = lin / 8;
    return xcd * q + min(xcd, r) + local;
}

// How a wave works on a plane of split P.  Rows go in groups of RG (the second
// stage then has RG * R1 <= 64 items, one per lane); the first stage's RG * R2
// items take IT passes of RPI rows, lane l holding item n2 = l % R2 of row
// l / R2 in every pass, so its twiddles and column offsets stay in registers.
template <class P>
struct PlaneWave {
    static constexpr int RG = 64 / P::R1 < P::N ? 64 / P::R1 : P::N;
    static constexpr int RPIMAX = 64 / P::R2 < RG ? 64 / P::R2 : RG;
    static constexpr int IT = (RG + RPIMAX - 1) / RPIMAX;
    static constexpr int RPI = (RG + IT - 1) / IT;
    static constexpr int NG = (P::N + RG - 1) / RG;
    // Row stride of the kept columns and of the exchange buffer, by the banks
    // (16-byte reads run 16 lanes at a time, writes 8; 8-byte ones 32 and 16).
    // Columns: 1 modulo the 256 bytes of all banks, so that the first stages'
    // items (n2 columns apart, rows R2 apart) meet consecutive slots; above
    // N = 96 LDS has no room for the padding.  Exchange: R2 modulo the banks, for
    // the same reason.  In FP64 a slot of the exchange holds one component (two
    // rounds), in FP32 a whole value: 8 bytes either way, the cheapest write.
    template <class T>
    static constexpr int ld() {
        constexpr int m = 128 / (int)sizeof(T);
        int l = P::N + 1;
        while (P::N <= 96 && l % m != 1) ++l;
        return l;
    }
    static constexpr int ldx() {
        constexpr int m = P::N <= 96 ? 32 : 16;
        int l = P::N;
        while (l % m != P::R2 % m) ++l;
        return l;
    }
    static constexpr size_t xbytes() { return (size_t)RPI * ldx() * 8; }   // per wave
};

// bytes of the kept columns, to a multiple of 16
template <class P, class T>
__host__ __device__ constexpr size_t plane_columns(int ncx) {
    return ((size_t)ncx * PlaneWave<P>::template ld<T>() * 2 * sizeof(T) + 15) & ~size_t(15);
}

// Orders one wave's LDS accesses: they complete in program order, so this only
// keeps the compiler from moving them.
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// R2 consecutive slots of the exchange buffer, in pairs where the offset allows
template <int R2>
__device__ __forceinline__ void xread(const double *x, double *v) {
    if constexpr (R2 % 2 == 0) {
        typedef double V2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int i = 0; i < R2; i += 2) {
            const V2 w = *reinterpret_cast<const V2 *>(x + i);
            v[i] = w[0];
            v[i + 1] = w[1];
        }
    } else {
#pragma unroll
        for (int i = 0; i < R2; ++i) v[i] = x[i];
    }
}
template <int R2>
__device__ __forceinline__ void xwrite(double *x, const double *v) {
    if constexpr (R2 % 2 == 0) {
        typedef double V2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int i = 0; i < R2; i += 2) *reinterpret_cast<V2 *>(x + i) = V2{v[i], v[i + 1]};
    } else {
#pragma unroll
        for (int i = 0; i < R2; ++i) x[i] = v[i];
    }
}
template <int R2>
__device__ __forceinline__ void xread(const cf *x, cf *v) {
    if constexpr (R2 % 2 == 0) {
        typedef float V4 __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int i = 0; i < R2; i += 2) {
            const V4 w = *reinterpret_cast<const V4 *>(x + i);
            v[i] = cf{w[0], w[1]};
            v[i + 1] = cf{w[2], w[3]};
        }
    } else {
#pragma unroll
        for (int i = 0; i < R2; ++i) v[i] = x[i];
    }
}
template <int R2>
__device__ __forceinline__ void xwrite(cf *x, const cf *v) {
    if constexpr (R2 % 2 == 0) {
        typedef float V4 __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int i = 0; i < R2; i += 2)
            *reinterpret_cast<V4 *>(x + i) = V4{v[i].x, v[i].y, v[i + 1].x, v[i + 1].y};
    } else {
#pragma unroll
        for (int i = 0; i < R2; ++i) x[i] = v[i];
    }
}
// what a slot of the exchange buffer holds
template <class T>
struct Slot;
template <>
struct Slot<double> {
    using type = double;
};
template <>
struct Slot<float> {
    using type = cf;
};

// One wave's state over the planes of its workgroup: lane mapping, twiddles and
// the offsets of its x columns.  HALF: R1 = 8 and every kept frequency of the
// sphere lies in [-N/4, N/4), so that of the R1 inputs n1 R2 + n2 of a first
// stage (and outputs of a last one) only n1 = 0, 1, 6, 7 can be non-zero.
template <class P, class T, bool HALF>
struct PlaneLane {
    using W = PlaneWave<P>;
    using X = typename Slot<T>::type;
    static constexpr int N = P::N, LD = W::template ld<T>(), LDX = W::ldx(), R1 = P::R1, R2 = P::R2;
    int lane, n2, rr;       // first stages: item n2, row (or column) rr of a pass
    int k1, r2;             // second stages: item k1, row r2 of the group
    bool act1, act2;
    cpx<T> tw[R1];          // exp(2 pi i n2 k1 / N)
    static constexpr bool kept(int n1) { return !HALF || n1 < R1 / 4 || n1 >= R1 - R1 / 4; }

    __device__ __forceinline__ void init(const double *twid) {
        lane = threadIdx.x & 63;
        n2 = lane % R2;
        rr = lane / R2;
        act1 = rr < W::RPI;
        k1 = lane % R1;
        r2 = lane / R1;
        act2 = r2 < W::RG;
#pragma unroll
        for (int k = 1; k < R1; ++k) {
            const int i = n2 * k;   // < N
            tw[k] = cpx<T>{T(twid[2 * i]), T(twid[2 * i + 1])};
        }
    }
    // first stage of an inverse transform on u (natural order in)
    __device__ __forceinline__ void first(cpx<T> *u) const {
        if constexpr (HALF) dft8_quarters_in<+1>(u);
        else Dft<R1, +1, T>::run(u);
#pragma unroll
        for (int k = 1; k < R1; ++k) u[k] = cmul(u[k], tw[k]);
    }
    // last stage of a forward transform on u (natural order out)
    __device__ __forceinline__ void last(cpx<T> *u) const {
#pragma unroll
        for (int k = 1; k < R1; ++k) u[k] = cmul(u[k], cpx<T>{tw[k].x, -tw[k].y});
        if constexpr (HALF) dft8_quarters_out<-1>(u);
        else Dft<R1, -1, T>::run(u);
    }
    // The sticks of columns [c0, c1) into A and inverse y-FFT of those columns,
    // in place (natural -> digit-reversed).
    __device__ __forceinline__ void columns_in(const SphereDev &sp, const cpx<T> *Sp, cpx<T> *A, int c0, int c1) const {
        if (c0 >= c1) return;
        const int s0 = sp.xc_start[c0], s1 = sp.xc_start[c1];
        // the first sticks are on their way while the columns are cleared
        const int sa = s0 + lane, sb = sa + 64;
        const int qa = min(sa, s1 - 1), qb = min(sb, s1 - 1);
        const T vax = Sp[qa].x, vay = Sp[qa].y, vbx = Sp[qb].x, vby = Sp[qb].y;
        const int pa = sp.st_xc[qa] * LD + sp.st_y[qa], pb = sp.st_xc[qb] * LD + sp.st_y[qb];
        for (int c = c0; c < c1; ++c)
            for (int y = lane; y < N; y += 64)
                if (!HALF || y < N / 4 || y >= N - N / 4) A[c * LD + y] = cpx<T>{T(0), T(0)};
        wave_order();
        if (sa < s1) A[pa] = cpx<T>{vax, vay};
        if (sb < s1) A[pb] = cpx<T>{vbx, vby};
        for (int s = s0 + 128 + lane; s < s1; s += 64) A[sp.st_xc[s] * LD + sp.st_y[s]] = Sp[s];
        wave_order();
        for (int c = c0 + rr; c < c1; c += 64 / R2) {
            if (rr >= 64 / R2) break;
            cpx<T> u[R1];
#pragma unroll
            for (int n1 = 0; n1 < R1; ++n1)
                if (kept(n1)) u[n1] = A[c * LD + n1 * R2 + n2];
            first(u);
#pragma unroll
            for (int k = 0; k < R1; ++k) A[c * LD + k * R2 + n2] = u[k];
        }
        wave_order();
        column_stage<+1>(A, c0, c1);
    }
    // The second stage of an inverse transform (or the first of a forward one)
    // of columns [c0, c1), in place.  Columns run fastest over the lanes, four
    // at a time or eight, so that the items, R2 apart, fall into different banks.
    template <int S>
    __device__ __forceinline__ void column_stage(cpx<T> *A, int c0, int c1) const {
        const int cp = (R1 <= 8 && c1 - c0 > 4) ? 8 : 4;
        const int j = lane & (cp - 1), k = cp == 8 ? lane >> 3 : lane >> 2;
        for (int c = c0 + j; c < c1; c += cp) {
            if (k >= R1) break;
            cpx<T> out[R2];
            cpx<T> *x = A + c * LD + k * R2;
#pragma unroll
            for (int i = 0; i < R2; ++i) out[i] = x[i];
            Dft<R2, S, T>::run(out);
#pragma unroll
            for (int i = 0; i < R2; ++i) x[i] = out[i];
        }
    }
    // Forward y-FFT of columns [c0, c1) (digit-reversed -> natural) and back to the sticks.
    __device__ __forceinline__ void columns_out(const SphereDev &sp, cpx<T> *Sp, cpx<T> *A, int c0, int c1) const {
        if (c0 >= c1) return;
        column_stage<-1>(A, c0, c1);
        wave_order();
        for (int c = c0 + rr; c < c1; c += 64 / R2) {
            if (rr >= 64 / R2) break;
            cpx<T> u[R1];
#pragma unroll
            for (int k = 0; k < R1; ++k) u[k] = A[c * LD + k * R2 + n2];
            last(u);
#pragma unroll
            for (int n1 = 0; n1 < R1; ++n1)
                if (kept(n1)) A[c * LD + n1 * R2 + n2] = u[n1];
        }
        wave_order();
        for (int s = sp.xc_start[c0] + lane; s < sp.xc_start[c1]; s += 64) Sp[s] = A[sp.st_xc[s] * LD + sp.st_y[s]];
    }
    // offset in A of x column n1 R2 + n2, or -1 where it is not kept
    __device__ __forceinline__ void x_columns(const SphereDev &sp, int (&off)[R1]) const {
        const int xmin_g = ((sp.xmin % N) + N) % N;
#pragma unroll
        for (int n1 = 0; n1 < R1; ++n1) {
            int xc = n1 * R2 + n2 - xmin_g;
            xc += (xc < 0) ? N : 0;
            off[n1] = (kept(n1) && xc < sp.ncx) ? xc * LD : -1;
        }
    }
    // Inverse x-FFT of the rows of group g, their inputs read straight from the
    // kept columns: leaves the R2 values of item k1 of row RG g + r2 in out (lanes
    // with act2).  The values change lanes through the wave's own buffer xb, RPI
    // rows at a time.
    __device__ __forceinline__ void rows_in(const cpx<T> *A, const int (&off)[R1], X *xb, int g, cpx<T> *out) const {
        X va[R2], vb[R2];
        X *xw = xb + rr * LDX + n2;
#pragma unroll
        for (int i = 0; i < W::IT; ++i) {
            const int r = i * W::RPI + rr;
            const int y = g * W::RG + r;
            const int ypos = digit_rev<P>(y);
            cpx<T> u[R1];
            const bool on = act1 && r < W::RG && y < N;
            if (on) {
#pragma unroll
                for (int n1 = 0; n1 < R1; ++n1)
                    if (kept(n1)) u[n1] = off[n1] >= 0 ? A[off[n1] + ypos] : cpx<T>{T(0), T(0)};
                first(u);
            }
            const bool mine = act2 && r2 / W::RPI == i;
            const X *xr = xb + (r2 - i * W::RPI) * LDX + k1 * R2;
            wave_order();
            if (on) {
#pragma unroll
                for (int k = 0; k < R1; ++k) {
                    if constexpr (sizeof(T) == 8) xw[k * R2] = u[k].x;
                    else xw[k * R2] = u[k];
                }
            }
            wave_order();
            if (mine) xread<R2>(xr, va);
            if constexpr (sizeof(T) == 8) {
                wave_order();
                if (on) {
#pragma unroll
                    for (int k = 0; k < R1; ++k) xw[k * R2] = u[k].y;
                }
                wave_order();
                if (mine) xread<R2>(xr, vb);
            }
        }
#pragma unroll
        for (int k = 0; k < R2; ++k) {
            if constexpr (sizeof(T) == 8) out[k] = cpx<T>{va[k], vb[k]};
            else out[k] = va[k];
        }
        Dft<R2, +1, T>::run(out);
    }
    // the adjoint of rows_in: forward x-FFT from out back into the kept columns
    __device__ __forceinline__ void rows_out(cpx<T> *A, const int (&off)[R1], X *xb, int g, cpx<T> *out) const {
        Dft<R2, -1, T>::run(out);
        X va[R2], vb[R2];
#pragma unroll
        for (int k = 0; k < R2; ++k) {
            if constexpr (sizeof(T) == 8) {
                va[k] = out[k].x;
                vb[k] = out[k].y;
            } else {
                va[k] = out[k];
            }
        }
        const X *xr = xb + rr * LDX + n2;
#pragma unroll
        for (int i = 0; i < W::IT; ++i) {
            const int r = i * W::RPI + rr;
            const int y = g * W::RG + r;
            const int ypos = digit_rev<P>(y);
            const bool on = act1 && r < W::RG && y < N;
            const bool mine = act2 && r2 / W::RPI == i;
            X *xw = xb + (r2 - i * W::RPI) * LDX + k1 * R2;
            cpx<T> u[R1];
            wave_order();
            if (mine) xwrite<R2>(xw, va);
            wave_order();
            if (on) {
#pragma unroll
                for (int k = 0; k < R1; ++k) {
                    if constexpr (sizeof(T) == 8) u[k].x = xr[k * R2];
                    else u[k] = xr[k * R2];
                }
            }
            if constexpr (sizeof(T) == 8) {
                wave_order();
                if (mine) xwrite<R2>(xw, vb);
                wave_order();
                if (on) {
#pragma unroll
                    for (int k = 0; k < R1; ++k) u[k].y = xr[k * R2];
                }
            }
            if (on) {
                last(u);
#pragma unroll
                for (int n1 = 0; n1 < R1; ++n1)
                    if (kept(n1) && off[n1] >= 0) A[off[n1] + ypos] = u[n1];
            }
        }
    }
};

// A wave owns whole columns for the y transforms and whole rows for the x
// transforms, and passes values between its lanes through LDS of its own, so a
// plane takes two workgroup barriers (columns to rows and back) and the waves
// drift apart: one wave's LDS accesses run under another's arithmetic.  Per plane
// at N = 96 ~13.6k VALU wave instructions and about as many LDS cycles, mostly
// writes (8 bytes a lane at best 85 B per cycle; reads run at 256).  Against the
// form with a barrier after each of ~14 stages, 64 bands: N = 96 413 -> 307 us
// FP64, 198 -> 176 FP32; N = 72, 92 bands, 290 -> 172 FP64.
// The bound of 12 waves holds every instance to 168 VGPRs, those launched with four
// waves too: in FP64 the default splits spill 28 of them (100 bytes of scratch a
// lane) at N = 120, 22 at 128, 8 at 108 and, unpruned, 13 at 96; the density's
// register form 9 at 96, 35 at 120 and 53 at 128.
template <class P, class T, bool HALF>
__global__ void __launch_bounds__(64 * kPlaneWaves) k_plane(const ApplyItems<T> items, const T *__restrict__ vperm,
                                                            int nb) {
    const FftApplyItem<T> &item = items.it[blockIdx.z];
    const SphereDev &sp = item.sp;
    cpx<T> *__restrict__ S = item.S;
    using W = PlaneWave<P>;
    constexpr int N = P::N, LD = W::template ld<T>(), R2 = P::R2;
    extern __shared__ unsigned char smem_raw[];
    cpx<T> *A = reinterpret_cast<cpx<T> *>(smem_raw);   // [ncx][LD], y along the row

    const int total = N * nb;
    const int lid = xcd_logical(blockIdx.x, total);
    const int z = lid / nb, band = lid % nb;
    const int ncx = sp.ncx, nw = blockDim.x >> 6, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto *xb = reinterpret_cast<typename Slot<T>::type *>(smem_raw + plane_columns<P, T>(ncx)) + wave * (W::RPI * W::ldx());
    cpx<T> *Sp = S + ((int64_t)band * N + z) * sp.ldst;
    const T *Vz = vperm + (int64_t)z * N * N;

    PlaneLane<P, T, HALF> L;
    L.init(sp.twid);
    const int cg = (ncx + nw - 1) / nw;
    const int c0 = min(ncx, wave * cg), c1 = min(ncx, c0 + cg);
    L.columns_in(sp, Sp, A, c0, c1);
    int off[P::R1];
    L.x_columns(sp, off);
    __syncthreads();
    for (int g = wave; g < W::NG; g += nw) {
        // V of this lane's item: on its way during the inverse transform
        const int y = min(g * W::RG + L.r2, N - 1);
        T v[R2];
#pragma unroll
        for (int k = 0; k < R2; ++k) v[k] = Vz[y * N + L.k1 * R2 + k];
        cpx<T> out[R2];
        L.rows_in(A, off, xb, g, out);
#pragma unroll
        for (int k = 0; k < R2; ++k) out[k] = cscale(out[k], v[k]);
        L.rows_out(A, off, xb, g, out);
    }
    __syncthreads();
    L.columns_out(sp, Sp, A, c0, c1);
}

// ---- pass 3: forward z-FFT per stick, gather, kinetic -----------------------
template <class P, class T>
__global__ void __launch_bounds__(kThreads) k_zfwd(const ApplyItems<T> items, int spb) {
    const FftApplyItem<T> &item = items.it[blockIdx.z];
    const SphereDev &sp = item.sp;
    const cpx<T> *__restrict__ S = item.S;
    const cpx<T> *__restrict__ X = item.X;
    const int64_t ldx = item.ldx;
    cpx<T> *__restrict__ Y = item.Y;
    const int64_t ldy = item.ldy;
    constexpr int N = P::N, LD = N + 1;
    constexpr int R1 = P::R1, R2 = P::R2;
    extern __shared__ unsigned char smem_raw[];
    cpx<T> *tw = reinterpret_cast<cpx<T> *>(smem_raw);
    cpx<T> *buf = tw + N;

    const int band = blockIdx.y;
    const int s0 = blockIdx.x * spb;
    const int ns = min(spb, sp.nst - s0);
    if (ns <= 0) return;
    load_twiddles(tw, sp.twid, N);
    const cpx<T> *Sb = S + (int64_t)band * N * sp.ldst + s0;
    for (int i = threadIdx.x; i < ns * N; i += blockDim.x) {
        const int z = i / ns, seq = i - z * ns;
        buf[seq * LD + digit_rev<P>(z)] = Sb[(int64_t)z * sp.ldst + seq];
    }
    __syncthreads();
    for (int it = threadIdx.x; it < ns * R1; it += blockDim.x) {
        const int seq = it % ns, k1 = it / ns;
        dif_b<P, -1>(buf + seq * LD, k1);
    }
    __syncthreads();
    for (int it = threadIdx.x; it < ns * R2; it += blockDim.x) {
        const int seq = it % ns, n2 = it / ns;
        cpx<T> out[R1];
        dif_a<P, -1>(buf + seq * LD, n2, tw, out);
#pragma unroll
        for (int n1 = 0; n1 < R1; ++n1) buf[seq * LD + n1 * R2 + n2] = out[n1];
    }
    __syncthreads();
    const int g0 = sp.st_start[s0];
    const int g1 = sp.st_start[s0 + ns - 1] + sp.st_len[s0 + ns - 1];
    const cpx<T> *Xb = X + (int64_t)band * ldx;
    cpx<T> *Yb = Y + (int64_t)band * ldy;
    for (int g = g0 + threadIdx.x; g < g1; g += blockDim.x) {
        const int pos = sp.g_map[g];
        const int s = pos / N, zz = pos - s * N;
        const cpx<T> v = buf[(s - s0) * LD + zz];
        const cpx<T> x = Xb[g];
        const T t = T(sp.kin[g]);
        Yb[g] = cpx<T>{v.x + t * x.x, v.y + t * x.y};
    }
}

// ---- dispatch ---------------------------------------------------------------
constexpr int kSticksPerBlock = 16;   // default sticks per workgroup of the z passes

// Waves of a plane workgroup.  Four, one per SIMD, where LDS (kept columns and
// an exchange buffer per wave) holds enough such workgroups, two in FP64, in FP32
// four (three above N = 96): workgroups out of step with each other fill the LDS
// phases of one with the arithmetic of another, which waves behind one barrier do
// not (N = 96, FP64, 64 bands: 2 x 4 waves 333 us, 1 x 12 379; N = 72: 3 x 4 140,
// 1 x 9 218; counts that are no multiple of 4 load the SIMDs unevenly).  FP32
// where they don't fit: eight or six waves, two workgroups (64 bands, 2 x 8 and
// otherwise: N = 72, 45 columns 148 and, 3 x 4, 159 us; 63 columns 220 and, 1 x 12,
// 272; N = 96, 61 columns 287 and 377; 2 x 6: N = 108, 53 columns 405 and 447).
// With one workgroup up to 12 waves (N = 120, FP32: 2 x 4 458, 1 x 12 402), but
// for R2 = 16, whose items collide in the banks whatever the waves (N = 128, FP32:
// 533 and 558).  few: no more planes than compute units, so nothing else runs beside
// a workgroup, and up to 12 waves shorten it (one band, 12 / 4 waves: N = 72 FP64
// 23.2 / 27.0 us, N = 80 26.4 / 30.6, N = 96 FP32 23.5 / 30.0).
// most > 0: a cap from the tuning, below these.  0 if even one wave does not fit.
template <class P, class T>
int plane_waves(int ncx, int most, bool few) {
    using W = PlaneWave<P>;
    constexpr bool F32 = sizeof(T) == 4 && P::R2 != 16;
    auto lds = [&](int nw) { return plane_columns<P, T>(ncx) + nw * W::xbytes(); };
    int nw = kPlaneWaves;
    if (!few) {
        if (lds(4) * (!F32 ? 2 : P::N <= 96 ? 4 : 3) <= kLdsMax) nw = 4;
        else if (F32 && lds(6) * 2 <= kLdsMax) nw = lds(8) * 2 <= kLdsMax ? 8 : 6;
    }
    nw = std::min(nw, W::NG);
    while (nw > 0 && lds(nw) > kLdsMax) --nw;
    return most > 0 ? std::min(nw, most) : nw;
}

template <class P, class T>
void run_apply_split(const ApplyItems<T> &items, int nk, const T *vperm, int nb, hipStream_t st) {
    constexpr int N = P::N;
    using W = PlaneWave<P>;
    const Tuning &tune = thread_tuning();
    const int spb = tune.fft_spb > 0 ? tune.fft_spb : kSticksPerBlock;
    const size_t e = sizeof(cpx<T>);
    const size_t sm13 = (size_t)N * e + (size_t)spb * (N + 1) * e;
    int nst_max = 0;
    for (int k = 0; k < nk; ++k) nst_max = std::max(nst_max, items.it[k].sp.nst);
    dim3 g13((nst_max + spb - 1) / spb, nb, nk);
    // rows in flight asked for by the tuning: a cap on the waves
    const int most = tune.fft_rb > 0 ? std::max(1, std::min(kPlaneWaves, tune.fft_rb / W::RG)) : 0;
    // The plane pass of the items with spheres inside the middle half (h) or not: a
    // launch for each kind that there is.  The pruned form and the full one round
    // differently, so an item's form may not depend on the others of its batch.
    auto plane = [&](auto h, bool launch) {
        constexpr bool H = decltype(h)::value;
        int n = 0, ncx_max = 0, of[kMaxApplyBatch];
        for (int k = 0; k < nk; ++k)
            if (H == (P::R1 == 8 && items.it[k].sp.quarter)) {
                of[n++] = k;
                ncx_max = std::max(ncx_max, items.it[k].sp.ncx);
            }
        if (!n) return;
        const int nw = plane_waves<P, T>(ncx_max, most, (int64_t)N * nb * n <= device_cu_count());
        PW_REQUIRE(nw >= 1, PW_ERR_ARG, "FFT plane does not fit in LDS");
        const size_t sm2 = plane_columns<P, T>(ncx_max) + nw * W::xbytes();
        if (!launch) return ensure_smem_limit((const void *)k_plane<P, T, H>, sm2);
        auto go = [&](const ApplyItems<T> &kind) {
            hipLaunchKernelGGL((k_plane<P, T, H>), dim3(N * nb, 1, n), dim3(64 * nw), sm2, st, kind, vperm, nb);
        };
        if (n == nk) return go(items);
        ApplyItems<T> kind;
        for (int k = 0; k < n; ++k) kind.it[k] = items.it[of[k]];
        go(kind);
    };
    auto planes = [&](bool launch) {
        if constexpr (P::R1 == 8) plane(std::true_type{}, launch);
        plane(std::false_type{}, launch);
    };
    planes(false);   // refuse before anything is launched
    ensure_smem_limit((const void *)k_zinv<P, T>, sm13);
    ensure_smem_limit((const void *)k_zfwd<P, T>, sm13);
    hipLaunchKernelGGL((k_zinv<P, T>), g13, dim3(kThreads), sm13, st, items, spb);
    planes(true);
    hipLaunchKernelGGL((k_zfwd<P, T>), g13, dim3(kThreads), sm13, st, items, spb);
    PW_HIP(hipGetLastError());
}

// host-side compile-time loop over the candidate second factors 2..16
template <int B, int E, class F>
void host_for(F &&f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        host_for<B + 1, E>(static_cast<F &&>(f));
    }
}

// the split a context's tuning selects for length N (0: the default)
int effective_r2(int n, int r2) { return r2 > 0 ? r2 : choose_r2(n); }

template <int N, class T>
void run_apply(const ApplyItems<T> &items, int nk, const T *vperm, int nb, hipStream_t st) {
    const int r2 = effective_r2(N, thread_tuning().fft_r2);
    bool done = false;
    host_for<2, 17>([&](auto R) {
        constexpr int r = R;
        if constexpr (split_ok(N, r)) {
            if (!done && r == r2) {
                run_apply_split<Split<N, r>, T>(items, nk, vperm, nb, st);
                done = true;
            }
        }
    });
    PW_REQUIRE(done, PW_ERR_ARG, "radix split not available for this FFT length");
}

}  // namespace
}  // namespace pw

// FFT side of the runtime: potential layout, density, sizes and the launchers of
// the H.X passes (fft_apply.h; compiled per precision and list of sizes in
// fft_f64_*.hip and fft_f32_*.hip).
#include "fft_apply.h"

namespace pw {
namespace {

// ---- density: per z-plane inverse xy transforms, occ |psi|^2 accumulated -----
// part[group][z][y][x position] = sum of occ[b] |psi_b(x, y, z)|^2 over the bands
// of the group (psi without the 1/sqrt(Omega) factor; band b of the launch is in
// group (first + b) % groups and has occupation occ[b * ostride]), added to what
// `part` holds.  One workgroup owns one plane of one group and adds its bands in
// order, so no two threads write one element and the sum is deterministic.  REG: a wave per row group, its sums in registers over the
// bands; else any count of waves, the sums in memory.  256 bands at N = 96: 4652
// us in one group with the bands in series and a barrier per stage, 790 us so;
// 842 with four waves and the sums in L2 (three groups of sums per wave spill).
template <class P, class T, bool HALF, bool REG>
__global__ void __launch_bounds__(64 * kPlaneWaves)
    k_plane_rho(const ApplyItems<T> items, int nb, const double *__restrict__ occ, int ostride, double *__restrict__ part,
                int groups, int first) {
    const SphereDev &sp = items.it[0].sp;
    const cpx<T> *__restrict__ S = items.it[0].S;
    using W = PlaneWave<P>;
    constexpr int N = P::N, R2 = P::R2;
    extern __shared__ unsigned char smem_raw[];
    cpx<T> *A = reinterpret_cast<cpx<T> *>(smem_raw);
    const int z = blockIdx.x, ncx = sp.ncx, nw = blockDim.x >> 6, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto *xb = reinterpret_cast<typename Slot<T>::type *>(smem_raw + plane_columns<P, T>(ncx)) + wave * (W::RPI * W::ldx());
    double *rz = part + ((int64_t)((first + blockIdx.y) % groups) * N + z) * N * N;
    PlaneLane<P, T, HALF> L;
    L.init(sp.twid);
    const int cg = (ncx + nw - 1) / nw;
    const int c0 = min(ncx, wave * cg), c1 = min(ncx, c0 + cg);
    int off[P::R1];
    L.x_columns(sp, off);
    auto row = [&](int g) { return g * W::RG + L.r2; };
    double acc[R2];
    if constexpr (REG) {
#pragma unroll
        for (int k = 0; k < R2; ++k) acc[k] = (L.act2 && row(wave) < N) ? rz[row(wave) * N + L.k1 * R2 + k] : 0.0;
    }
    for (int band = blockIdx.y; band < nb; band += groups) {
        const double f = occ[(int64_t)band * ostride];
        L.columns_in(sp, S + ((int64_t)band * N + z) * sp.ldst, A, c0, c1);
        __syncthreads();
        for (int g = wave; g < W::NG; g += nw) {
            cpx<T> out[R2];
            L.rows_in(A, off, xb, g, out);
            double *rho = rz + row(g) * N + L.k1 * R2;
            const bool ok = L.act2 && row(g) < N;
#pragma unroll
            for (int k = 0; k < R2; ++k) {
                const double a = (double)out[k].x, b = (double)out[k].y;
                if constexpr (REG) acc[k] += f * (a * a + b * b);
                else if (ok) rho[k] += f * (a * a + b * b);
            }
        }
        __syncthreads();
    }
    if constexpr (REG) {
        if (L.act2 && row(wave) < N) {
#pragma unroll
            for (int k = 0; k < R2; ++k) rz[row(wave) * N + L.k1 * R2 + k] = acc[k];
        }
    }
}

// rho[x][y][z] = scale * sum of the groups' part[group][z][y][position of x], on top
// of what rho holds if `add`
template <class P>
__global__ void k_rho_permute(const double *__restrict__ part, int groups, double scale, double *__restrict__ rho,
                              bool add) {
    constexpr int N = P::N;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)N * N * N) return;
    const int z = (int)(i % N), y = (int)((i / N) % N), x = (int)(i / ((int64_t)N * N));
    double s = add ? rho[i] : 0.0;
    for (int g = 0; g < groups; ++g) s += part[(((int64_t)g * N + z) * N + y) * N + digit_rev<P>(x)];
    rho[i] = s * scale;
}

// ---- potential layout: vperm[z][y][p] = scale * V[x(p)][y][z] ---------------
// p is the digit-reversed x position produced by the inverse x-FFT of pass 2
// (it depends on the radix split P), so the multiply in pass 2 reads V
// contiguously.
template <class P>
__global__ void k_permute_v(const double *__restrict__ v, double scale, double *__restrict__ out,
                            int *bad) {
    constexpr int N = P::N;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)N * N * N) return;
    const int p = (int)(i % N), y = (int)((i / N) % N), z = (int)(i / ((int64_t)N * N));
    const int x = freq_at<P>(p);
    const double val = v[((int64_t)x * N + y) * N + z];
    if (!isfinite(val)) atomicOr(bad, 1);
    out[i] = val * scale;
}

// the same potential moved from the layout of split PF to that of split PT
template <class PF, class PT>
__global__ void k_repermute_v(const double *__restrict__ in, double *__restrict__ out) {
    constexpr int N = PT::N;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)N * N * N) return;
    const int p = (int)(i % N);
    const int64_t row = i - p;
    out[i] = in[row + digit_rev<PF>(freq_at<PT>(p))];
}


}  // namespace

bool fft_size_supported(int n) {
#define PW_CASE(NN) if (n == NN) return true;
    PW_FFT_SIZES(PW_CASE)
#undef PW_CASE
    return false;
}

std::vector<int> fft_supported_sizes() {
    std::vector<int> v;
#define PW_CASE(NN) v.push_back(NN);
    PW_FFT_SIZES(PW_CASE)
#undef PW_CASE
    return v;
}

template <int N>
void permute_for(int r2, const double *v, double scale, double *v_zyx, int *bad, hipStream_t st) {
    const int64_t tot = (int64_t)N * N * N;
    const dim3 grid((unsigned)((tot + 255) / 256));
    bool done = false;
    host_for<2, 17>([&](auto R) {
        constexpr int r = R;
        if constexpr (split_ok(N, r)) {
            if (!done && r == r2) {
                hipLaunchKernelGGL((k_permute_v<Split<N, r>>), grid, dim3(256), 0, st, v, scale, v_zyx, bad);
                done = true;
            }
        }
    });
    PW_REQUIRE(done, PW_ERR_ARG, "radix split not available for this FFT length");
}

template <int N>
void repermute_for(int r2_from, int r2_to, const double *in, double *out, hipStream_t st) {
    const int64_t tot = (int64_t)N * N * N;
    const dim3 grid((unsigned)((tot + 255) / 256));
    bool done = false;
    host_for<2, 17>([&](auto RF) {
        constexpr int rf = RF;
        if constexpr (split_ok(N, rf)) {
            host_for<2, 17>([&](auto RT) {
                constexpr int rt = RT;
                if constexpr (split_ok(N, rt)) {
                    if (!done && rf == r2_from && rt == r2_to) {
                        hipLaunchKernelGGL((k_repermute_v<Split<N, rf>, Split<N, rt>>), grid, dim3(256), 0, st,
                                           in, out);
                        done = true;
                    }
                }
            });
        }
    });
    PW_REQUIRE(done, PW_ERR_ARG, "radix split not available for this FFT length");
}

void launch_permute_potential(const double *v, int n, double scale, double *v_zyx, int *bad, int r2,
                              hipStream_t st) {
    switch (n) {
#define PW_CASE(NN)                                                              \
    case NN:                                                                     \
        permute_for<NN>(effective_r2(NN, r2), v, scale, v_zyx, bad, st);        \
        break;
        PW_FFT_SIZES(PW_CASE)
#undef PW_CASE
        default:
            throw Error{PW_ERR_ARG, "unsupported FFT size"};
    }
    PW_HIP(hipGetLastError());
}

void launch_repermute_potential(const double *in, int n, int r2_from, int r2_to, double *out,
                                hipStream_t st) {
    switch (n) {
#define PW_CASE(NN)                                                                                 \
    case NN:                                                                                        \
        repermute_for<NN>(effective_r2(NN, r2_from), effective_r2(NN, r2_to), in, out, st);         \
        break;
        PW_FFT_SIZES(PW_CASE)
#undef PW_CASE
        default:
            throw Error{PW_ERR_ARG, "unsupported FFT size"};
    }
    PW_HIP(hipGetLastError());
}

std::vector<int> fft_radix_splits(int n) {
    std::vector<int> v;
    for (int r = 2; r <= 16; ++r)
        if (split_ok(n, r)) v.push_back(r);
    return v;
}

int fft_default_r2(int n) { return choose_r2(n); }

// waves of the density's plane workgroups: one per row group where that fits
template <int N>
struct DensityShape {
    using P = Split<N>;
    using W = PlaneWave<P>;
    static size_t lds(int ncx, int nw) { return plane_columns<P, double>(ncx) + nw * W::xbytes(); }
    static bool reg(int ncx) { return W::NG <= kPlaneWaves && lds(ncx, W::NG) <= kLdsMax; }
    static int waves(int ncx) { return reg(ncx) ? W::NG : plane_waves<P, double>(ncx, 0, false); }
};

template <int N>
void run_density(const SphereDev &sp, const cd *X, int64_t ldx, int nb, const double *occ, int ostride, double *part,
                 int groups, int first, cd *S, hipStream_t st) {
    using P = Split<N>;
    using D = DensityShape<N>;
    const int spb = kSticksPerBlock;
    const size_t e = sizeof(cd);
    const size_t sm1 = (size_t)N * e + (size_t)spb * (N + 1) * e;
    const int nw = D::waves(sp.ncx);
    PW_REQUIRE(nw >= 1, PW_ERR_ARG, "FFT plane does not fit in LDS");
    const size_t sm2 = D::lds(sp.ncx, nw);
    ensure_smem_limit((const void *)k_zinv<P, double>, sm1);
    ApplyItems<double> items{};
    items.it[0] = FftApplyItem<double>{sp, X, ldx, nullptr, 0, S};
    hipLaunchKernelGGL((k_zinv<P, double>), dim3((sp.nst + spb - 1) / spb, nb), dim3(kThreads), sm1, st, items, spb);
    auto rho = [&](auto h, auto r) {
        constexpr bool H = decltype(h)::value, R = decltype(r)::value;
        ensure_smem_limit((const void *)k_plane_rho<P, double, H, R>, sm2);
        hipLaunchKernelGGL((k_plane_rho<P, double, H, R>), dim3(N, std::min(groups, nb)), dim3(64 * nw), sm2, st, items,
                           nb, occ, ostride, part, groups, first);
    };
    auto by_sum = [&](auto h) {
        if (D::reg(sp.ncx)) rho(h, std::true_type{});
        else rho(h, std::false_type{});
    };
    if constexpr (P::R1 == 8) {
        if (sp.quarter) by_sum(std::true_type{});
        else by_sum(std::false_type{});
    } else {
        by_sum(std::false_type{});
    }
    PW_HIP(hipGetLastError());
}

int density_resident(const SphereDev &sp) {
    switch (sp.n) {
#define PW_CASE(NN)                                                                               \
    case NN: {                                                                                    \
        const int nw = DensityShape<NN>::waves(sp.ncx);                                           \
        return nw ? std::min<int>((int)(kLdsMax / DensityShape<NN>::lds(sp.ncx, nw)), 12 / nw) : 1; \
    }
        PW_FFT_SIZES(PW_CASE)
#undef PW_CASE
        default:
            return 1;
    }
}

void launch_density_accumulate(const SphereDev &sp, const cd *X, int64_t ldx, int nb, const double *occ, int ostride,
                               double *part, int groups, int first, cd *S, hipStream_t st) {
    if (nb <= 0) return;
    switch (sp.n) {
#define PW_CASE(NN)                                                         \
    case NN:                                                                        \
        run_density<NN>(sp, X, ldx, nb, occ, ostride, part, groups, first, S, st);  \
        return;
        PW_FFT_SIZES(PW_CASE)
#undef PW_CASE
        default:
            throw Error{PW_ERR_ARG, "unsupported FFT size"};
    }
}

void launch_density_finish(const double *part, int n, int groups, double scale, double *rho, bool add, hipStream_t st) {
    const int64_t tot = (int64_t)n * n * n;
    const dim3 grid((unsigned)((tot + 255) / 256));
    switch (n) {
#define PW_CASE(NN)                                                                                         \
    case NN:                                                                                                    \
        hipLaunchKernelGGL((k_rho_permute<Split<NN>>), grid, dim3(256), 0, st, part, groups, scale, rho, add);  \
        break;
        PW_FFT_SIZES(PW_CASE)
#undef PW_CASE
        default:
            throw Error{PW_ERR_ARG, "unsupported FFT size"};
    }
    PW_HIP(hipGetLastError());
}

template <class T>
void fft_apply_impl(const ApplyItems<T> &items, int nk, const T *v_zyx, int nb, hipStream_t st) {
    if (nb <= 0 || nk <= 0) return;
    if (!run_apply_small(items, nk, v_zyx, nb, st) && !run_apply_large(items, nk, v_zyx, nb, st))
        throw Error{PW_ERR_ARG, "unsupported FFT size"};
}

template <class T>
void fft_apply_batch(const FftApplyItem<T> *items, int nk, const T *v_zyx, int nb, hipStream_t st) {
    PW_REQUIRE(nk >= 1 && nk <= kMaxApplyBatch, PW_ERR_ARG, "k-points per batched apply must be in [1, 16]");
    ApplyItems<T> all{};
    for (int k = 0; k < nk; ++k) {
        PW_REQUIRE(items[k].sp.n == items[0].sp.n, PW_ERR_ARG, "batched apply needs one FFT grid");
        all.it[k] = items[k];
    }
    fft_apply_impl(all, nk, v_zyx, nb, st);
}

void launch_fft_apply(const SphereDev &sp, const double *v_zyx, const cd *X, int64_t ldx, cd *Y,
                      int64_t ldy, int nb, cd *S, hipStream_t st) {
    const FftApplyItem<double> it{sp, X, ldx, Y, ldy, S};
    fft_apply_batch(&it, 1, v_zyx, nb, st);
}
void launch_fft_apply(const SphereDev &sp, const float *v_zyx, const cf *X, int64_t ldx, cf *Y,
                      int64_t ldy, int nb, cf *S, hipStream_t st) {
    const FftApplyItem<float> it{sp, X, ldx, Y, ldy, S};
    fft_apply_batch(&it, 1, v_zyx, nb, st);
}
void launch_fft_apply_batch(const FftApplyItem<double> *items, int nk, const double *v_zyx, int nb,
                            hipStream_t st) {
    fft_apply_batch(items, nk, v_zyx, nb, st);
}
void launch_fft_apply_batch(const FftApplyItem<float> *items, int nk, const float *v_zyx, int nb,
                            hipStream_t st) {
    fft_apply_batch(items, nk, v_zyx, nb, st);
}

}  // namespace pw

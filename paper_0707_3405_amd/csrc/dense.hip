// Small dense FP64 steps of the iteration.
//
//  * k_chol_inv (one workgroup): Cholesky factor of a Gram matrix G = R^H R and
//    R^-1, used to orthonormalise a block (W <- W R^-1; BLOPEX-style LOBPCG, sec. 3.2).
//  * launch_heev_f64: lowest k eigenpairs of a Hermitian matrix -- the Rayleigh-Ritz
//    eigenproblem of the LOBPCG iteration (sec. 3.2, Algorithm 1; size 3m) and of the final
//    Rayleigh-Ritz over all bands (sec. 3.2, sec. 4.2).  Householder
//    reduction to real tridiagonal form (many workgroups down to 96 rows, then
//    one), bisection with Sturm counts (a workgroup per eigenvalue), inverse
//    iteration (a wave per eigenvalue), re-orthogonalisation (CholQR or Gram-Schmidt
//    twice), back-transform (a wave per vector).
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <type_traits>

#include "pw_internal.h"

namespace pw {
namespace {

__device__ __forceinline__ cd cconj(cd a) { return {a.x, -a.y}; }
__device__ __forceinline__ cd cmulz(cd a, cd b) { return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__device__ __forceinline__ cf cconj(cf a) { return {a.x, -a.y}; }
__device__ __forceinline__ cf cmulz(cf a, cf b) { return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }

// 1 / d to within an ulp without the division sequence: the hardware
// reciprocal refined by two Newton steps (d finite and normal).  Measured on
// gfx950 over 4M samples: v_rcp_f64 alone is off by up to 4.6e-8 relative,
// one step leaves up to 14 ulp, two steps at most 1 ulp.
__device__ __forceinline__ double rcp_nr(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = fma(r, fma(-d, r, 1.0), r);
    r = fma(r, fma(-d, r, 1.0), r);
    return r;
}

// d^-1/2: the hardware value refined by two Newton steps (d positive and normal)
__device__ __forceinline__ double rsqrt_nr(double d) {
    double r = __builtin_amdgcn_rsq(d);
    r = fma(0.5 * r, fma(-d * r, r, 1.0), r);
    r = fma(0.5 * r, fma(-d * r, r, 1.0), r);
    return r;
}

// FP32: the hardware reciprocal (within 1 ulp) and square root
__device__ __forceinline__ float rcp_nr(float d) { return __builtin_amdgcn_rcpf(d); }
__device__ __forceinline__ double sqrt_r(double x) { return sqrt(x); }
__device__ __forceinline__ float sqrt_r(float x) { return __builtin_sqrtf(x); }

// value of v in lane `lane` (uniform), as a wave-uniform value
__device__ __forceinline__ double lane_read(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}
__device__ __forceinline__ float lane_read(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

template <int CTRL>
__device__ __forceinline__ double dpp_mov(double x) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x) {   // one 32-bit move
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}
// sum over the 16 lanes of a DPP row; every lane of the row gets the same value
template <class R>
__device__ __forceinline__ R row16_sum(R x) {
    x += dpp_mov<0xB1>(x);    // quad_perm [1,0,3,2]
    x += dpp_mov<0x4E>(x);    // quad_perm [2,3,0,1]
    x += dpp_mov<0x141>(x);   // row_half_mirror
    x += dpp_mov<0x140>(x);   // row_mirror
    return x;
}
template <class R>
__device__ __forceinline__ R quad_sum(R x) {
    x += dpp_mov<0xB1>(x);
    x += dpp_mov<0x4E>(x);
    return x;
}
// lanes whose DPP row is disabled by ROW_MASK read 0
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_rows(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, ROW_MASK, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, ROW_MASK, 0xF, false);
    return __hiloint2double(hi, lo);
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_rows(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROW_MASK, 0xF, false));
}
// Wave sum returned as a wave-uniform value, without LDS: the row sums, then
// row_bcast:15 adds row 0 into row 1 and row 2 into row 3, row_bcast:31 adds
// rows 0 + 1 into rows 2 and 3, and lane 63 holds the total (same order of
// additions in every wave).
template <class R>
__device__ __forceinline__ R wave_total(R x) {
    x = row16_sum(x);
    x += dpp_rows<0x142, 0xA>(x);   // row_bcast:15
    x += dpp_rows<0x143, 0xC>(x);   // row_bcast:31
    return lane_read(x, 63);
}

// sum over the lanes with the same lane % TR (TR = 4, 8, 16, 32); every lane gets it
template <int TR>
__device__ __forceinline__ double stride_sum(double x) {
    if constexpr (TR <= 4) x += dpp_mov<0x124>(x);   // row_ror:4
    if constexpr (TR <= 8) x += dpp_mov<0x128>(x);   // row_ror:8
    auto swap_sum = [&](auto swap) {
        const auto lo = swap((unsigned)__double2loint(x)), hi = swap((unsigned)__double2hiint(x));
        x = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
    };
    if constexpr (TR <= 16) swap_sum([](unsigned v) { return __builtin_amdgcn_permlane16_swap(v, v, false, false); });
    swap_sum([](unsigned v) { return __builtin_amdgcn_permlane32_swap(v, v, false, false); });
    return x;
}

// Block-wide sum of one double per thread: wave shuffles, then the wave
// partials added in wave order by every thread (deterministic, 2 barriers).
__device__ double block_sum(double v, double *red) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    if (lane == 0) red[wave] = v;
    __syncthreads();
    double s = 0.0;
    for (int q = 0; q < nw; ++q) s += red[q];
    __syncthreads();
    return s;
}

template <int B, int E, class F>
__device__ __forceinline__ void unroll_for(F &&f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        unroll_for<B + 1, E>(static_cast<F &&>(f));
    }
}

// ---- Cholesky + inverse of the factor (n <= 64) --------------------------------
// Gaussian elimination without pivoting on the augmented matrix [G | I]: the
// row operations that reduce G (Hermitian positive definite, G = L D L^H) to
// the upper triangle D L^H turn I into L^-1; scaling row j of both by d_j^-1/2
// gives [R | R^-H] with G = R^H R.  Rows and columns >= n are padded with the
// identity.
// Bound by the chain of n pivots (reciprocal, multiplier, next pivot: about
// 250 cycles each), so 16 pivots at a time are eliminated inside a wave, without
// a barrier.  A panel is 16 rows of the augmented matrix, 16 + 64 columns: the
// diagonal block and, for each of the four column blocks i, the block of G
// right of it (i > k), of the inverse left of it (i < k), or the identity
// (i = k).  Waves 0 and 1 each hold the diagonal block, one column per lane in
// lanes 0-15, and half of the 64 others in lanes 16-47; the pivot row's entries
// in lanes j and a > j are the pivot and the multipliers, read as scalars.
// The blocks of the later panels stay in the matrix cores' accumulators: wave
// 2 + i holds column block i of panels 1-3, which receive
// M(c, i) -= R(k, c)^H M(k, i) after panel k; the four blocks of the next panel do so
// ahead of it, one on each SIMD, the others beside it.
// Measured at n = 16 / 64: 6.6 / 23.8 us (12.7 / 47.7 us with a pair of pivots per
// barrier on a 32 x 32 grid of threads).  About 470 cycles per pivot, of them
// 250 the chain; 6 waves, so that the panel's registers don't spill (14 waves
// with one block each: 33 us).
constexpr int kCholMax = 64;
constexpr int kCholP = 16;   // rows of a panel
constexpr int kCholWaves = 6;

int chol_panels(int n) { return (n + kCholP - 1) / kCholP; }
// row block, then the staged G, later reused for the other two row blocks
size_t chol_lds(int n) {
    const size_t N = kCholP * (size_t)chol_panels(n), block = kCholP * kCholMax;
    return (block + std::max(N * (N + 1), N > kCholP ? 2 * block : 0)) * 16;
}

__global__ void __launch_bounds__(64 * kCholWaves) k_chol_inv(const cd *__restrict__ G, int64_t ldg, int n,
                                                      cd *__restrict__ Rinv, int64_t ldr, int *status) {
    extern __shared__ double chol_smem[];
    typedef double v4 __attribute__((ext_vector_type(4)));
    constexpr int P = kCholP, W = kCholMax;
    const int np = (n + P - 1) / P, N = P * np, LS = N + 1;
    cd *const out0 = reinterpret_cast<cd *>(chol_smem);   // panels 0, 2: [16][64]
    cd *const sg = out0 + P * W;                          // G as stored, [column][LS]
    cd *const in = sg, *const out1 = sg + P * W;          // next panel; panel 1
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    if (lane < N) {
        constexpr int Q = (W + kCholWaves - 1) / kCholWaves;
        cd x[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int b = wave + kCholWaves * q;
            x[q] = lane < n && b < n ? G[(int64_t)b * ldg + lane] : cd{lane == b ? 1.0 : 0.0, 0.0};
        }
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (wave + kCholWaves * q < N) sg[(wave + kCholWaves * q) * LS + lane] = x[q];
    }
    __syncthreads();
    double dmax = lane < n ? fmax(sg[lane * LS + lane].x, 0.0) : 0.0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) dmax = fmax(dmax, __shfl_xor(dmax, o));
    // a tiny diagonal shift keeps a numerically semi-definite Gram factorable
    const double shift = 1e-15 * dmax * n;
    auto herm = [&](int a, int b) {   // Hermitian part of the stored Gram, shifted
        const cd x = sg[b * LS + a], y = sg[a * LS + b];
        return cd{0.5 * (x.x + y.x) + (a == b ? shift : 0.0), 0.5 * (x.y - y.y)};
    };
    if (wave < 2) {
        const bool diag = lane < P, other = !diag && lane < 3 * P;
        const int o = 2 * P * wave + (lane - P) % (2 * P), slot = o / P;   // column of [inverse | G]
        cd g[P];
        {
            const int col = diag ? lane : min(o, N - 1);
#pragma unroll
            for (int r = 0; r < P; ++r) g[r] = herm(r, col);
        }
        bool fail = false;
        for (int k = 0;; ++k) {
            int ln = lane;
            asm volatile("" : "+v"(ln));   // keeps the masks of the lanes out of registers across panels
            const int unit = !diag && slot == k ? ln % P : -1;   // this lane's row of the identity
#pragma unroll
            for (int r = 0; r < P; ++r) {
                g[r].x = unit < 0 ? g[r].x : unit == r ? 1.0 : 0.0;
                g[r].y = unit < 0 ? g[r].y : 0.0;
            }
            double dp = 1.0;   // lane r: pivot of row r
            auto pivot = [&](int j) {   // 1 / d_j
                const double d = lane_read(g[j].x, j);
                const bool bad = !(d > 1e-300) | !(d <= DBL_MAX);
                fail |= bad;
                dp = ln == j ? (bad ? 1.0 : d) : dp;
                return bad ? 1.0 : rcp_nr(d);
            };
            double inv = pivot(0);
            unroll_for<0, P>([&](auto j_) {
                constexpr int j = j_;
                if (P * k + j >= n) return;   // only padding left
                const cd tj = {g[j].x * inv, g[j].y * inv};
                // row a -= conj(g_ja) / d_j row j; the next pivot as soon as its row is there.
                // Four rows at a time, or the multipliers of all rows spill
                unroll_for<j + 1, P>([&](auto a_) {
                    constexpr int a = a_;
                    const double mr = lane_read(g[j].x, a), mi = lane_read(g[j].y, a);
                    g[a].x = fma(-mi, tj.y, fma(-mr, tj.x, g[a].x));
                    g[a].y = fma(mi, tj.x, fma(-mr, tj.y, g[a].y));
                    if constexpr (a == j + 1) inv = pivot(a);
                    if constexpr ((a - j) % 4 == 0) __builtin_amdgcn_sched_barrier(0);
                });
                __builtin_amdgcn_sched_barrier(0);
            });
            const double isd = rsqrt_nr(dp);
            cd *const out = k & 1 ? out1 : out0;
#pragma unroll
            for (int r = 0; r < P; ++r) {
                const double sc = lane_read(isd, r);
                g[r].x *= sc;
                g[r].y *= sc;
                if (other && k + 1 < np) out[r * W + o] = g[r];
            }
            if (k + 1 < np) __syncthreads();
            // R^-1 (upper) = (R^-H)^H with R^-H = D^-1/2 L^-1
            cd *dst = Rinv + (int64_t)P * k * ldr + o;
#pragma unroll
            for (int r = 0; r < P; ++r) {
                if (other && P * k + r < n && o < n) *dst = slot <= k ? cd{g[r].x, -g[r].y} : cd{0.0, 0.0};
                dst += ldr;
            }
            if (k + 1 == np) break;
            __syncthreads();
            const int src = diag ? P * (k + 1) + ln : o;
#pragma unroll
            for (int r = 0; r < P; ++r) g[r] = in[r * W + src];
        }
        if (fail && t == 0) atomicOr(status, 1);
        return;
    }
    // blocks (c, i) of the later panels; i < c: of the inverse (zero so far), else of G
    const int i = wave - 2, li = lane & 15, gr = lane >> 4;
    v4 re[3], im[3];
    auto init = [&](auto c_) {
        constexpr int c = c_;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const cd v = i >= c && i < np ? herm(P * c + gr + 4 * r, P * i + li) : cd{0.0, 0.0};
            re[c - 1][r] = v.x;
            im[c - 1][r] = v.y;
        }
    };
    // M(c, i) -= R(k, c)^H M(k, i); the inverse's blocks i > k are still zero
    auto update = [&](auto c_, auto k_) {
        constexpr int c = c_, k = k_;
        if (c >= np || i >= np || (i > k && i < c)) return;
        const cd *const m = k & 1 ? out1 : out0;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int row = (4 * s + gr) * W;
            const cd a = m[row + P * c + li], b = m[row + P * i + li];
            re[c - 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.x, b.x, re[c - 1], 0, 0, 0);
            im[c - 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.x, b.y, im[c - 1], 0, 0, 0);
            re[c - 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, re[c - 1], 0, 0, 0);
            im[c - 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, im[c - 1], 0, 0, 0);
        }
    };
    unroll_for<1, 4>(init);
    if (np > 1) __syncthreads();   // panel 0 done
    unroll_for<1, 4>([&](auto k_) {
        constexpr int k = k_;
        if (k >= np) return;
        std::integral_constant<int, k - 1> last;
        update(k_, last);
#pragma unroll
        for (int r = 0; r < 4; ++r) in[(gr + 4 * r) * W + P * i + li] = cd{re[k - 1][r], im[k - 1][r]};
        __syncthreads();
        unroll_for<k + 1, 4>([&](auto c_) { update(c_, last); });
        if (k + 1 < np) __syncthreads();
    });
}

// ---- Hermitian eigensolver ---------------------------------------------------
// Five stages on the stream:
//   reduction  A = Q T Q^H, T real tridiagonal (lower Householder):
//              k_trd_col (a launch per column) down to 96 rows, k_hetrd_la (1 workgroup)
//   k_stebz    (k groups)      lowest k eigenvalues of T by 256-point multisection
//   k_stein_w  (k waves)       eigenvectors of T by inverse iteration, in registers
//   k_orth_chol2 / k_orth_chol / k_orth (1 workgroup), k_orth_clusters  re-orthogonalisation
//   k_unmtr_w  (k waves)       back-transform V = Q Z
//
// ---- multi-workgroup reduction for n > 96 --------------------------------------
// H_j = I - tau_j v_j v_j^H, A <- H_j^H A H_j, w = tau y - (|tau|^2 / 2)
// Re(v^H y) v, A -= w v^H + v w^H, both triangles of the trailing square kept.
// One launch per column (k_trd_col): a column is a serial chain of two
// reductions over the chip, bound by launch and memory latency, not by the
// bytes (a 512^2 matrix is 4 MB).  Launch j
//   - every workgroup by itself: y_{j-1} = sum of the chunk partials (fixed
//     order, so all workgroups get the same bits), w_{j-1}, the pivot column j
//     with the update of step j - 1 on the fly, d_j and the reflector v_j; one
//     thread per row (n <= 1024);
//   - then on its tile of TR rows x 128 columns of the trailing square
//     [j + 1, n)^2, loaded at the start behind the vectors: the update of step
//     j - 1 and the partial of A v_j over the tile's columns.
// Repeating the vector work in every workgroup (its loads: 64 KB at n = 512)
// costs less than the launch and the round trip through memory that a kernel
// of its own takes: 13.0 us per column with the vector work in a kernel of one
// workgroup, 4.4 us so (mean over n = 512; 7.4 -> 3.0 ms for the whole
// eigensolve without its vectors).  Of these about 1 us each are the launch and
// the loads; the rest is the serial chain of the two sums.
// Threads: one per row left (256, 512 or 1024), since waves without rows only
// delay the others' scalar work.  Tile rows: the fewest for which the repeated
// vector loads don't show.  Measured on 193 / 256 / 512 / 1024 columns, whole
// eigensolve with few vectors: 1.06 / 1.40 / 2.96 / 8.3 ms with 4, 8 and 32 rows
// at 256, 512 and 1024 threads; 16 rows at 512 threads 3.1 ms, 32 rows 3.2 ms;
// 16 rows at 1024 threads 9.2 ms, 8 rows 11.2 ms.
// The last kTrRest columns are left to k_hetrd_la, whose columns get cheaper with
// the rows left: 4.0 us at 96 against 4.1 here, 1.4 at 32 (whole eigensolve with 64
// vectors at n = 192: 1185 us with k_hetrd_la alone, 953 with the last 128
// columns, 884 with 96; n = 129: 723, 598, 570).  The launch before them (`last`)
// only applies the update of its predecessor.  96 launches where there was one
// are no loss for single solves or four at a time (eight at a time: +2 %).
// Tiles lie on a fixed grid and are numbered in shells of 128 x 128 blocks from
// the bottom right corner, so that the live ones are a prefix and a tile keeps
// its workgroup number, hence its XCD and L2, for the whole reduction.
// v and the partials alternate between two buffers (a launch reads the last
// one's and writes its own); v is zero outside the reflector's rows.  Column
// j - 1 of A receives its reflector in launch j: in launch j - 1 every
// workgroup still reads that column.
constexpr int kTrCols = 128;
constexpr int kTrRest = 96;   // the last columns are left to k_hetrd_la
constexpr int kTrR256 = 4, kTrR512 = 8, kTrR1024 = 32;

struct TrdState {
    cd *v[2];      // [n] reflectors of even / odd steps
    cd *yp[2];     // [nblocks][n] partials of A v over 128 columns
};

__global__ void k_herm_sym(cd *__restrict__ A, int64_t lda, int n) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)n * n) return;
    const int r = (int)(idx % n), c = (int)(idx / n);
    if (r > c) {
        const cd a = A[(int64_t)c * lda + r], b = A[(int64_t)r * lda + c];
        const cd m = {0.5 * (a.x + b.x), 0.5 * (a.y - b.y)};
        A[(int64_t)c * lda + r] = m;
        A[(int64_t)r * lda + c] = cconj(m);
    } else if (r == c) {
        A[(int64_t)c * lda + r].y = 0.0;
    }
}

template <int NT, int TR>
__global__ void __launch_bounds__(NT)
    k_trd_col(cd *__restrict__ A, int64_t lda, int n, int j, TrdState S, double *__restrict__ dd,
              double *__restrict__ ee, cd *__restrict__ tau_out, bool last) {
    // a wave's load covers TR rows x CS columns, a wave of the tile CS NQ columns
    constexpr int NW = NT / 64, CS = 64 / TR, NQ = kTrCols / (CS * NW), NB = NT / kTrCols;
    __shared__ cd svp[NT], sw[NT], sv[NT];   // v_{j-1}, w_{j-1}, v_j (from row r0)
    __shared__ cd yw[NW][64];
    __shared__ double red[2][NW];
    __shared__ cd s_y, s_v, s_alpha;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const bool first = blockIdx.x == 0;
    // this workgroup's tile
    const int nb = (n + kTrCols - 1) / kTrCols;
    const int q = blockIdx.x / (kTrCols / TR), sub = blockIdx.x % (kTrCols / TR);
    int s = 0;
    while ((s + 1) * (s + 1) <= q) ++s;
    const int rs = q - s * s;
    const int br = nb - 1 - (rs <= s ? s : rs - s - 1), bc = nb - 1 - (rs <= s ? rs : s);
    const int i0 = kTrCols * br + TR * sub, c0 = kTrCols * bc;
    const int lo = last ? j - 1 : j;   // the tiles cover rows and columns > lo
    if (!first && (i0 >= n || i0 + TR - 1 <= lo)) return;   // no live row
    const int kb = j / kTrCols, r0 = kTrCols * kb, row = r0 + t;   // this thread's row
    // loads: the vectors first, the tile behind them
    const bool in = row >= j && row < n;
    cd yq[NB], vi = {0.0, 0.0}, c = {0.0, 0.0}, tau1 = {0.0, 0.0};
#pragma unroll
    for (int k = 0; k < NB; ++k) yq[k] = cd{0.0, 0.0};
    double beta1 = 0.0;
    if (j > 0) {
        tau1 = tau_out[j - 1];
        beta1 = ee[j - 1];
        const cd *yp = S.yp[(j - 1) & 1];
        if (in) vi = S.v[(j - 1) & 1][row];
#pragma unroll
        for (int k = 0; k < NB; ++k)
            if (in && kb + k < nb) yq[k] = yp[(int64_t)(kb + k) * n + row];
    }
    if (in && !last) c = A[(int64_t)j * lda + row];
    const int i = i0 + lane % TR, cw = c0 + CS * NQ * wave + lane / TR;
    const bool rok = i > lo && i < n;
    cd a[NQ];
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
        const int col = cw + CS * k;
        a[k] = rok && col > lo && col < n ? A[(int64_t)col * lda + i] : cd{0.0, 0.0};
    }
    // w_{j-1} and column j
#pragma unroll
    for (int h = 1; h < NB; h *= 2)   // pairwise: fixed order, short chain
#pragma unroll
        for (int k = 0; k + h < NB; k += 2 * h) {
            yq[k].x += yq[k + h].x;
            yq[k].y += yq[k + h].y;
        }
    const cd y = yq[0];
    const double vy = wave_total(vi.x * y.x + vi.y * y.y);
    if (lane == 0) red[0][wave] = vy;
    if (row == j) {
        s_y = y;
        s_v = vi;
    }
    __syncthreads();
    auto total = [&](const double *r) {   // pairwise over the waves
        double x = r[lane % NW];
        x += dpp_mov<0xB1>(x);
        x += dpp_mov<0x4E>(x);
        if (NW > 4) x += dpp_mov<0x141>(x);
        if (NW > 8) x += dpp_mov<0x140>(x);
        return x;
    };
    const double nu = 0.5 * (tau1.x * tau1.x + tau1.y * tau1.y) * total(red[0]);
    const cd ty = cmulz(tau1, y), typ = cmulz(tau1, s_y), vj = s_v;
    const cd w = {ty.x - nu * vi.x, ty.y - nu * vi.y};
    const cd wj = {typ.x - nu * vj.x, typ.y - nu * vj.y};
    if (j > 0) {
        const cd u1 = cmulz(vi, cconj(wj)), u2 = cmulz(w, cconj(vj));
        c.x -= u1.x + u2.x;
        c.y -= u1.y + u2.y;
    }
    if (first) {
        if (row == j && !last) dd[j] = c.x;
        if (j > 0) {
            if (row > j && in) A[(int64_t)(j - 1) * lda + row] = vi;   // kept for the back-transform
            if (row == j) A[(int64_t)(j - 1) * lda + j] = cd{beta1, 0.0};
        }
    }
    svp[t] = vi;
    sw[t] = w;
    // reflector j
    if (!last) {
        const double cc = wave_total(row > j + 1 ? c.x * c.x + c.y * c.y : 0.0);
        if (lane == 0) red[1][wave] = cc;
        if (row == j + 1) s_alpha = c;
        __syncthreads();
        const double sigma = total(red[1]);
        const cd alpha = s_alpha;
        cd tau = {0.0, 0.0}, scale = {0.0, 0.0};
        double beta = alpha.x;
        const bool reflect = !(sigma == 0.0 && alpha.y == 0.0);
        if (reflect) {
            const double nrm = sqrt(alpha.x * alpha.x + alpha.y * alpha.y + sigma);
            beta = alpha.x >= 0.0 ? -nrm : nrm;
            const double dr = alpha.x - beta, di = alpha.y;
            const double ib = rcp_nr(beta), iden = rcp_nr(dr * dr + di * di);
            tau = cd{-dr * ib, -di * ib};
            scale = cd{dr * iden, -di * iden};
        }
        cd v = {0.0, 0.0};
        if (reflect && row == j + 1) v = cd{1.0, 0.0};
        else if (reflect && row > j + 1 && row < n) v = cmulz(c, scale);
        sv[t] = v;
        if (first) {
            if (in) S.v[j & 1][row] = v;
            if (t == 0) {
                tau_out[j] = tau;
                ee[j] = beta;
            }
        }
    }
    __syncthreads();
    // the tile: update of step j - 1, partial of A v_j
    const cd vpi = svp[i - r0], wpi = sw[i - r0];
    cd acc = {0.0, 0.0};
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
        const int col = cw + CS * k;
        const cd u1 = cmulz(wpi, cconj(svp[col - r0])), u2 = cmulz(vpi, cconj(sw[col - r0]));
        a[k].x -= u1.x + u2.x;
        a[k].y -= u1.y + u2.y;
        if (rok && col > lo && col < n) A[(int64_t)col * lda + i] = a[k];
        if (!last) {
            const cd vc = sv[col - r0];
            acc.x += a[k].x * vc.x - a[k].y * vc.y;
            acc.y += a[k].x * vc.y + a[k].y * vc.x;
        }
    }
    if (last) return;
    yw[wave][lane] = acc;
    __syncthreads();
    if (wave == 0) {   // the waves' partials in pairs, then the CS lanes of a row
        cd x[NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) x[k] = yw[k][lane];
#pragma unroll
        for (int h = 1; h < NW; h *= 2)
#pragma unroll
            for (int k = 0; k + h < NW; k += 2 * h) {
                x[k].x += x[k + h].x;
                x[k].y += x[k + h].y;
            }
        const cd sum = {stride_sum<TR>(x[0].x), stride_sum<TR>(x[0].y)};
        if (lane < TR && rok) S.yp[j & 1][(int64_t)bc * n + i] = sum;
    }
}

// ---- register-resident reduction for n <= 32 T (T <= 3; FP32: T <= 6) --------
// The same Householder sequence as k_trd_col, but the whole
// matrix stays in registers: 1024 threads on a 32 x 32 grid, each holding one
// element of every tile b <= a (off-diagonal tiles are stored once and used
// for both triangles of y = A v; diagonal tiles are stored in full).  Tiles
// whose rows or columns are all finished are skipped.  All sums run in a fixed
// order (deterministic).  The kernel is k_hetrd_la below.
constexpr int kRfMaxT = 6;
constexpr int kRfMaxN = 32 * kRfMaxT;

// Look-ahead form of the register-resident reduction (same Householder
// sequence and storage of the reflectors): thread (ti, tj) = (t % 32, t / 32)
// holds A(ti + 32a, tj + 32b) for tiles b <= a, so column c of the matrix is
// held by the 32 lanes of one half-wave.  Step j: every wave applies the rank-2
// update of step j - 1 to its live tiles; the wave holding column j does so
// with raised priority, then forms reflector j from its own registers (norm by
// DPP over the half-wave) and writes it to LDS while the other waves are still
// updating.  Then the partials of y = A v (row partials one per half-wave,
// column partials summed over lane quads by DPP, both in LDS) and w = tau y -
// nu v by four threads per row: three barriers per column instead of four.
// R is the arithmetic type: double, or float for the Rayleigh-Ritz problems of
// the complex64 stage of the mixed iteration (the input is rounded to float,
// the outputs are stored as double).
template <int T, class R>
__global__ void __launch_bounds__(1024)
    k_hetrd_la(cd *__restrict__ A, int64_t lda, int n, double *__restrict__ dd,
               double *__restrict__ ee, cd *__restrict__ tau_out) {
    using C = cpx<R>;
    constexpr int NR = 32 * T;
    constexpr int NE = T * (T + 1) / 2;
    __shared__ C vs[2][NR];          // reflectors of steps of both parities
    __shared__ C ws[NR];             // w of the last step, zero outside its live rows
    __shared__ C pr[32][NR + 1];     // row sums of y, one per half-wave (padded)
    __shared__ C pc[8][NR + 1];      // column sums of y, one per lane quad (padded)
    __shared__ R sv[16];             // per-wave partials of Re(v^H A v)
    __shared__ C s_tau[2];
    const int t = threadIdx.x, ti = t & 31, tj = t >> 5, wave = t >> 6, lane = t & 63;

    C E[NE];
    unroll_for<0, T>([&](auto a_) {
        constexpr int a = a_;
        unroll_for<0, a + 1>([&](auto b_) {
            constexpr int b = b_;
            const int i = ti + 32 * a, c = tj + 32 * b;
            C m = {R(0), R(0)};
            if (i < n && c < n) {   // exact Hermitian part (A + A^H) / 2
                const cd x = A[(int64_t)c * lda + i], y = A[(int64_t)i * lda + c];
                m = C{R(0.5 * (x.x + y.x)), R(0.5 * (x.y - y.y))};
                if (i == c) m.y = R(0);
            }
            E[a * (a + 1) / 2 + b] = m;
        });
    });
    for (int i = t; i < NR; i += 1024) vs[0][i] = vs[1][i] = ws[i] = C{R(0), R(0)};
    __syncthreads();
    // A -= w v^H + v w^H on the live tiles of step jm (v = vs[par], w = ws)
    auto update = [&](int jm, int par) {
        unroll_for<0, T>([&](auto a_) {
            constexpr int a = a_;
            if (32 * a + 31 <= jm) return;
            const C vi = vs[par][ti + 32 * a], wi = ws[ti + 32 * a];
            unroll_for<0, a + 1>([&](auto b_) {
                constexpr int b = b_;
                if (32 * b + 31 <= jm) return;
                const C vj = cconj(vs[par][tj + 32 * b]), wj = cconj(ws[tj + 32 * b]);
                const C u1 = cmulz(wi, vj), u2 = cmulz(vi, wj);
                // whole-element update (member-wise updates kept FP32 elements in scratch)
                const C e = E[a * (a + 1) / 2 + b];
                E[a * (a + 1) / 2 + b] = C{e.x - (u1.x + u2.x), e.y - (u1.y + u2.y)};
            });
        });
    };
    // entry (ti + 32 a, col) of this lane for the column tile jb (zero above it)
    auto col_entry = [&](auto a_, int jb) -> C {
        constexpr int a = decltype(a_)::value;
        // selects by component (an element-wise pick became a dynamically indexed
        // stack array in FP32)
        R xr = R(0), xi = R(0);
        unroll_for<0, a + 1>([&](auto b_) {
            constexpr int b = b_;
            const bool hit = b == jb;
            xr = hit ? E[a * (a + 1) / 2 + b].x : xr;
            xi = hit ? E[a * (a + 1) / 2 + b].y : xi;
        });
        return C{xr, xi};
    };
    for (int j = 0; j + 1 < n; ++j) {
        const int par = j & 1, own = j & 31, jb = j >> 5;
        const bool owner = wave == (own >> 1);   // uniform per wave
        if (owner) __builtin_amdgcn_s_setprio(2);
        if (j > 0) update(j - 1, par ^ 1);
        if (owner) {
            // ---- reflector j from column j, held by half-wave `own` ----
            const int base = (own & 1) * 32;
            R sg = R(0);
            unroll_for<0, T>([&](auto a_) {
                constexpr int a = a_;
                const int r = ti + 32 * a;
                if (r >= j + 2 && r < n) {
                    const C x = col_entry(a_, jb);
                    sg += x.x * x.x + x.y * x.y;
                }
            });
            sg = row16_sum(sg);
            sg += dpp_rows<0x142, 0xA>(sg);   // lanes 31 and 63: the two half-wave totals
            const R sigma = lane_read(sg, base + 31);
            const int a1 = (j + 1) >> 5;
            C xa = {R(0), R(0)}, xd = {R(0), R(0)};
            unroll_for<0, T>([&](auto a_) {
                constexpr int a = a_;
                if (a == a1) xa = col_entry(a_, jb);
                if (a == jb) xd = col_entry(a_, jb);
            });
            const C alpha = {lane_read(xa.x, base + ((j + 1) & 31)), lane_read(xa.y, base + ((j + 1) & 31))};
            const R djj = lane_read(xd.x, base + own);
            C tau, scale;
            R beta;
            if (sigma == R(0) && alpha.y == R(0)) {
                tau = C{R(0), R(0)};
                beta = alpha.x;
                scale = C{R(0), R(0)};
            } else {
                const R nrm = sqrt_r(alpha.x * alpha.x + alpha.y * alpha.y + sigma);
                beta = alpha.x >= R(0) ? -nrm : nrm;
                const R dr = alpha.x - beta, di = alpha.y;
                const R ib = rcp_nr(beta), iden = rcp_nr(dr * dr + di * di);
                tau = C{-dr * ib, -alpha.y * ib};
                scale = C{dr * iden, -di * iden};
            }
            const bool reflect = !(tau.x == R(0) && tau.y == R(0));
            if (tj == own) {   // the owning half-wave writes the whole reflector
                unroll_for<0, T>([&](auto a_) {
                    constexpr int a = a_;
                    const int r = ti + 32 * a;
                    C vv = {R(0), R(0)};
                    if (reflect && r > j && r < n) vv = r == j + 1 ? C{R(1), R(0)} : cmulz(col_entry(a_, jb), scale);
                    vs[par][r] = vv;
                    if (r > j + 1 && r < n) A[(int64_t)j * lda + r] = cd{vv.x, vv.y};   // kept for the back-transform
                });
                if (ti == own) {
                    dd[j] = djj;
                    ee[j] = beta;
                    tau_out[j] = cd{tau.x, tau.y};
                    A[(int64_t)j * lda + j + 1] = cd{beta, 0.0};
                    s_tau[par] = tau;
                }
            }
            __builtin_amdgcn_s_setprio(0);
        }
        __syncthreads();
        // ---- partials of y = A v ----
        {
            R vpart = R(0);
            unroll_for<0, T>([&](auto a_) {   // row sums over this lane's tiles of row ti + 32a
                constexpr int a = a_;
                if (32 * a + 31 <= j) return;
                R rr = R(0), ri = R(0);
                unroll_for<0, a + 1>([&](auto b_) {
                    constexpr int b = b_;
                    if (32 * b + 31 <= j) return;
                    const C e = E[a * (a + 1) / 2 + b];
                    const C vj = vs[par][tj + 32 * b];
                    rr += e.x * vj.x - e.y * vj.y;
                    ri += e.x * vj.y + e.y * vj.x;
                });
                const C vi = vs[par][ti + 32 * a];
                vpart += vi.x * rr + vi.y * ri;
                pr[tj][ti + 32 * a] = C{rr, ri};
            });
            unroll_for<0, T - 1>([&](auto b_) {   // conj(e) v_i into y_j, off-diagonal tiles
                constexpr int b = b_;
                if (32 * b + 31 <= j) return;
                R cr = R(0), ci = R(0);
                unroll_for<b + 1, T>([&](auto a_) {
                    constexpr int a = a_;
                    const C e = E[a * (a + 1) / 2 + b];
                    const C vi = vs[par][ti + 32 * a];
                    cr += e.x * vi.x + e.y * vi.y;
                    ci += e.x * vi.y - e.y * vi.x;
                });
                const C vj = vs[par][tj + 32 * b];
                vpart += vj.x * cr + vj.y * ci;
                cr = quad_sum(cr);   // the eight quad sums of a column are added in the w step
                ci = quad_sum(ci);
                if ((ti & 3) == 0) pc[ti >> 2][tj + 32 * b] = C{cr, ci};
            });
            vpart = wave_total(vpart);
            if (lane == 0) sv[wave] = vpart;
        }
        __syncthreads();
        // ---- w = tau y - nu v, four threads per row ----
        if (t < 4 * NR) {
            const int r = t >> 2, q = t & 3;
            const bool live = r > j && r < n;
            R sr = R(0), si = R(0);
            if (live) {
                R er = R(0), ei = R(0);
#pragma unroll
                for (int h = 0; h < 8; h += 2) {
                    sr += pr[8 * q + h][r].x;
                    si += pr[8 * q + h][r].y;
                    er += pr[8 * q + h + 1][r].x;
                    ei += pr[8 * q + h + 1][r].y;
                }
                if (r < 32 * (T - 1)) {   // the last column tile has no tile below the diagonal
                    sr += pc[2 * q][r].x;
                    si += pc[2 * q][r].y;
                    er += pc[2 * q + 1][r].x;
                    ei += pc[2 * q + 1][r].y;
                }
                sr += er;
                si += ei;
            }
            sr = quad_sum(sr);
            si = quad_sum(si);
            R vhy = (sv[4 * q] + sv[4 * q + 1]) + (sv[4 * q + 2] + sv[4 * q + 3]);
            vhy = quad_sum(vhy);
            const C tau = s_tau[par];
            const R nu = R(0.5) * (tau.x * tau.x + tau.y * tau.y) * vhy;
            if (q == 0) {
                C wr = {R(0), R(0)};
                if (live) {
                    const C ty = cmulz(tau, C{sr, si});
                    const C vr = vs[par][r];
                    wr = C{ty.x - nu * vr.x, ty.y - nu * vr.y};
                }
                ws[r] = wr;
            }
        }
        __syncthreads();
    }
    if (n >= 2) update(n - 2, (n - 2) & 1);
    {   // d_{n-1}: element (n-1, n-1) after the last update
        const int m = n - 1, mb = m >> 5;
        if (ti == (m & 31) && tj == (m & 31)) {
            unroll_for<0, T>([&](auto a_) {
                constexpr int a = a_;
                if (a == mb) dd[m] = E[a * (a + 1) / 2 + a].x;
            });
        }
    }
}

struct TriBounds {
    double gl, gu, pivmin, tnorm;
};

// Gershgorin interval, pivot floor and norm of the tridiagonal matrix, by the
// whole workgroup (min and max: exact in any order).  red: 3 doubles per wave.
// fmin and fmax drop a NaN, so an entry that is not finite makes the norm
// infinite (the interval is meaningless then).
__device__ TriBounds tri_bounds(const double *__restrict__ dd, const double *__restrict__ ee, int n, double *red) {
    double gl = DBL_MAX, gu = -DBL_MAX, tnorm = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const double r = (i > 0 ? fabs(ee[i - 1]) : 0.0) + (i + 1 < n ? fabs(ee[i]) : 0.0);
        gl = fmin(gl, dd[i] - r);
        gu = fmax(gu, dd[i] + r);
        const double a = fabs(dd[i]) + r;
        tnorm = fmax(tnorm, a <= DBL_MAX ? a : HUGE_VAL);
    }
    for (int off = 32; off > 0; off >>= 1) {
        gl = fmin(gl, __shfl_xor(gl, off));
        gu = fmax(gu, __shfl_xor(gu, off));
        tnorm = fmax(tnorm, __shfl_xor(tnorm, off));
    }
    const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[3 * wave] = gl;
        red[3 * wave + 1] = gu;
        red[3 * wave + 2] = tnorm;
    }
    __syncthreads();
    for (int q = 0; q < nw; ++q) {
        gl = fmin(gl, red[3 * q]);
        gu = fmax(gu, red[3 * q + 1]);
        tnorm = fmax(tnorm, red[3 * q + 2]);
    }
    const double pivmin = DBL_MIN * fmax(1.0, tnorm * tnorm);
    const double span = fmax(gu - gl, DBL_EPSILON * fmax(1.0, tnorm));
    return {gl - 2.0 * DBL_EPSILON * span - 1e-300, gu + 2.0 * DBL_EPSILON * span + 1e-300, pivmin, tnorm};
}

// Number of eigenvalues below x from the ratios q_i = d_i - x - e_{i-1}^2 /
// q_{i-1}: needs no scaling, but every step waits on a refined reciprocal.
// de[i] = (d_i, e_{i-1}^2).
__device__ int sturm_ratio(const double2 *de, int n, double x, double pivmin) {
    double q = de[0].x - x;
    if (fabs(q) < pivmin) q = -pivmin;
    int c = q < 0;
    for (int i = 1; i < n; ++i) {
        // the hardware reciprocal refined to an ulp, as the count's
        // backward-error argument needs; |q| >= pivmin keeps it finite
        q = de[i].x - x - de[i].y * rcp_nr(q);
        if (fabs(q) < pivmin) q = -pivmin;
        c += q < 0;
    }
    return c;
}

// The same count as the sign changes of the leading principal minors
//   p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2},
// one dependent FMA per step instead of a reciprocal chain.  A computed p_i is
// the exact one for d_i - x and e_{i-1}^2 changed by a few ulps, as in the
// ratio form.  The entries are scaled by a power of two to norm <= 1, so |p|
// grows at most 3x per step; every 16 steps the pair (p_i, p_{i-1}) is scaled
// back to about 1.  A zero p_i needs no care (the next minor is then
// -e^2 p_{i-1} and the pair counts one change in either sign of zero), but a
// pair that has all but vanished (a split matrix with an eigenvalue at x) sets
// `lost`, and the caller counts by ratios.
__device__ int sturm_minors(const double2 *de, int n, double x, bool &lost) {
    double p0 = 1.0, p1 = de[0].x - x;
    int c = (unsigned)__double2hiint(p1) >> 31;
    auto step = [&](int i) {
        const double2 v = de[i];
        const double p = fma(v.x - x, p1, -(v.y * p0));
        c += (unsigned)(__double2hiint(p) ^ __double2hiint(p1)) >> 31;
        p0 = p1;
        p1 = p;
    };
    lost = false;
    int i = 1;
    for (; i + 16 <= n; i += 16) {
#pragma unroll
        for (int u = 0; u < 16; ++u) step(i + u);
        const double m = fmax(fabs(p0), fabs(p1));
        lost |= !(m > 0x1p-900);
        const int ex = -__builtin_amdgcn_frexp_exp(m);
        p0 = __builtin_amdgcn_ldexp(p0, ex);
        p1 = __builtin_amdgcn_ldexp(p1, ex);
    }
    for (; i < n; ++i) step(i);
    lost |= !(fmax(fabs(p0), fabs(p1)) > 0x1p-900);
    return c;
}

// Lowest k eigenvalues, one workgroup of 256 threads per eigenvalue: each
// round counts at 256 interior points of the bracket (one per thread) and keeps
// the sub-interval where the count crosses the index: 8 bits a round, 7
// rounds from the Gershgorin interval to double precision.  The first point
// with count > idx is found by per-wave ballots and a minimum over the waves.
// Bound by the chain of n dependent steps per round; the minors take one FMA
// there, so one point per thread and one wave per SIMD (more points per round
// save fewer rounds than their issue slots cost).  Lowest 64 of n = 192:
// 133 us with the ratio form at 512 points, 36 us with the minors; all of
// n = 512: 532 -> 117 us.
// rel_tol: relative width at which a bracket stops (DBL_EPSILON; FLT_EPSILON
// for a tridiagonal matrix from the FP32 reduction, whose eigenvalues carry
// FP32 rounding anyway).
constexpr int kStebzThreads = 256;
__global__ void __launch_bounds__(kStebzThreads) k_stebz(const double *__restrict__ dd,
                                                          const double *__restrict__ ee, int n,
                                                          double *__restrict__ w, double rel_tol,
                                                          int *__restrict__ status) {
    extern __shared__ double2 de[];   // [n] (d_i, e_{i-1}^2), scaled
    __shared__ double red[3 * kStebzThreads / 64];
    __shared__ int wfirst[2][kStebzThreads / 64];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    constexpr int NP = kStebzThreads;   // interior points per round
    const TriBounds tb = tri_bounds(dd, ee, n, red);
    const int idx = blockIdx.x;
    if (!(tb.tnorm <= DBL_MAX)) {   // NaN or infinity in the matrix, or norms past the range
        if (t == 0) {
            w[idx] = NAN;
            atomicOr(status, 4);
        }
        return;
    }
    // exact scaling to norm <= 1 (none for a zero norm)
    const int ex = tb.tnorm > 0.0 ? __builtin_amdgcn_frexp_exp(tb.tnorm) : 0;
    for (int i = t; i < n; i += kStebzThreads) {
        const double e = i > 0 ? __builtin_amdgcn_ldexp(ee[i - 1], -ex) : 0.0;
        de[i] = double2{__builtin_amdgcn_ldexp(dd[i], -ex), e * e};
    }
    __syncthreads();
    double lo = tb.gl, hi = tb.gu;
    for (int round = 0; round < 18; ++round) {
        const double width = hi - lo;
        if (width <= 2.0 * rel_tol * fmax(fabs(lo), fabs(hi)) + tb.pivmin) break;
        // thread t counts at point t + 1 (point p at lo + width p / (NP + 1))
        const double x = __builtin_amdgcn_ldexp(lo + width * (double)(t + 1) / (double)(NP + 1), -ex);
        bool lost;
        int c = sturm_minors(de, n, x, lost);
        if (__any(lost)) c = sturm_ratio(de, n, x, DBL_MIN);   // uniform per wave
        const uint64_t b = __ballot(c > idx);
        const int buf = round & 1;
        if (lane == 0) wfirst[buf][wave] = b ? 64 * wave + __ffsll((unsigned long long)b) - 1 : NP;
        __syncthreads();
        int first = NP;   // the first point (0-based) whose count exceeds idx; NP if none
#pragma unroll
        for (int q = 0; q < kStebzThreads / 64; ++q) first = min(first, wfirst[buf][q]);
        const double nlo = first == 0 ? lo : lo + width * (double)first / (double)(NP + 1);
        const double nhi = first == NP ? hi : lo + width * (double)(first + 1) / (double)(NP + 1);
        lo = nlo;
        hi = nhi;
    }
    if (t == 0) {
        const double v = 0.5 * (lo + hi);
        w[idx] = v;
        if (!isfinite(v)) atomicOr(status, 4);
    }
}

// Inverse iteration, one eigenvalue per wave, with no memory access inside the
// recurrences: every lane runs the same (wave-uniform) LU factorisation and
// solves, entry i of each per-step array (the LU factors, the iterate, d and e)
// is kept by lane i % 64 in register slot i / 64, written with a lane select and
// read back with readlane.  LU with partial pivoting of T - lambda I (dlagtf
// order, the pivot choice taken by selects), two solves from a hashed start
// vector, unit 2-norm.  n <= 64 RPL; all of n = 512: 237 us (385 us with the
// factors in LDS and up to four eigenvalues in a workgroup).
template <int RPL>
__global__ void __launch_bounds__(64) k_stein_w(const double *__restrict__ dd,
                                                const double *__restrict__ ee, int n, int k,
                                                const double *__restrict__ w, double *__restrict__ Z) {
    const int L = threadIdx.x;
    const int idx = blockIdx.x;
    double dv[RPL], ev[RPL];   // d_i and e_i (e_{n-1} = 0) of entry i = L + 64 q
    double tn = 0.0;           // max_i |d_i| + |e_{i-1}| + |e_i|, as in tri_bounds
#pragma unroll
    for (int q = 0; q < RPL; ++q) {
        const int i = L + 64 * q;
        dv[q] = i < n ? dd[i] : 0.0;
        ev[q] = i + 1 < n ? ee[i] : 0.0;
        if (i < n) {
            const double r = (i > 0 ? fabs(ee[i - 1]) : 0.0) + (i + 1 < n ? fabs(ee[i]) : 0.0);
            tn = fmax(tn, fabs(dd[i]) + r);
        }
    }
    for (int off = 32; off > 0; off >>= 1) tn = fmax(tn, __shfl_xor(tn, off));
    const double lam = w[idx];
    const double eps_t = DBL_EPSILON * fmax(tn, 1e-300);
    double fdd[RPL], fdl[RPL], fdu[RPL], fdu2[RPL], zz[RPL];
    int fpiv[RPL];
#pragma unroll
    for (int q = 0; q < RPL; ++q) {
        fdd[q] = fdl[q] = fdu[q] = fdu2[q] = 0.0;
        fpiv[q] = 0;
        const int i = L + 64 * q;
        uint64_t h = (uint64_t)(i + 1) * 0x9E3779B97F4A7C15ull ^ (uint64_t)(idx + 7) * 0xD1B54A32D192ED03ull;
        h ^= h >> 31;
        h *= 0xBF58476D1CE4E5B9ull;
        h ^= h >> 29;
        zz[q] = (double)(h >> 11) * (2.0 / 9007199254740992.0) - 1.0;
    }
    // ---- LU of T - lambda I: step i eliminates row i + 1 ----
    double d_cur = lane_read(dv[0], 0) - lam, u_cur = lane_read(ev[0], 0), sub = u_cur;
    // step i (slot Q, lane l) with the entries i + 1 read from slot QN, lane ln
    auto lu_step = [&](auto Q_, auto QN_, int l, int ln) {
        constexpr int Q = decltype(Q_)::value, QN = decltype(QN_)::value;
        double d_nx = 0.0, u_nx = 0.0;
        if constexpr (QN < RPL) {
            d_nx = lane_read(dv[QN], ln) - lam;
            u_nx = lane_read(ev[QN], ln);
        }
        const bool piv = fabs(d_cur) < fabs(sub);
        const double dp = fabs(d_cur) < eps_t ? (d_cur < 0 ? -eps_t : eps_t) : d_cur;
        const double r = rcp_nr(piv ? sub : dp);
        const double m = (piv ? d_cur : sub) * r;
        const double du = piv ? d_nx : u_cur;
        const bool me = L == l;
        fdd[Q] = me ? r : fdd[Q];
        fdl[Q] = me ? m : fdl[Q];
        fdu[Q] = me ? du : fdu[Q];
        fdu2[Q] = me ? (piv ? u_nx : 0.0) : fdu2[Q];
        fpiv[Q] = me ? (int)piv : fpiv[Q];
        d_cur = fma(-m, du, piv ? u_cur : d_nx);
        u_cur = piv ? -m * u_nx : u_nx;
        sub = u_nx;
    };
    unroll_for<0, RPL>([&](auto q_) {
        constexpr int q = q_;
        const int lim = min(63, n - 1 - 64 * q);   // steps i = 64 q + l <= n - 2 with i + 1 in slot q
        for (int l = 0; l < lim; ++l) lu_step(std::integral_constant<int, q>{}, std::integral_constant<int, q>{}, l, l + 1);
        if (64 * q + 63 < n - 1)
            lu_step(std::integral_constant<int, q>{}, std::integral_constant<int, q + 1>{}, 63, 0);
    });
    {   // row n - 1
        const int qn = (n - 1) >> 6, ln = (n - 1) & 63;
        const double r = 1.0 / (fabs(d_cur) < eps_t ? eps_t : d_cur);
        const bool me = L == ln;
#pragma unroll
        for (int q = 0; q < RPL; ++q) {
            if (q != qn) continue;
            fdd[q] = me ? r : fdd[q];
            fdu[q] = me ? 0.0 : fdu[q];
            fdu2[q] = me ? 0.0 : fdu2[q];
            fpiv[q] = me ? 0 : fpiv[q];
        }
    }
    // ---- two solves; the first one's 1 / max-norm is applied as the second reads it ----
    double scale = 1.0, n2 = 0.0;
    for (int iter = 0; iter < 2; ++iter) {
        // L solve with the row interchanges: z is the running entry of row i
        double z = lane_read(zz[0], 0) * scale;
        auto l_step = [&](auto Q_, auto QN_, int l, int ln) {
            constexpr int Q = decltype(Q_)::value, QN = decltype(QN_)::value;
            double znx = 0.0;
            if constexpr (QN < RPL) znx = lane_read(zz[QN], ln) * scale;
            const double lm = lane_read(fdl[Q], l);
            const bool piv = __builtin_amdgcn_readlane(fpiv[Q], l) != 0;
            const double out = piv ? znx : z;
            zz[Q] = L == l ? out : zz[Q];
            z = fma(-lm, out, piv ? z : znx);
        };
        unroll_for<0, RPL>([&](auto q_) {
            constexpr int q = q_;
            const int lim = min(63, n - 1 - 64 * q);
            for (int l = 0; l < lim; ++l) l_step(std::integral_constant<int, q>{}, std::integral_constant<int, q>{}, l, l + 1);
            if (64 * q + 63 < n - 1)
                l_step(std::integral_constant<int, q>{}, std::integral_constant<int, q + 1>{}, 63, 0);
        });
        {
            const int qn = (n - 1) >> 6, ln = (n - 1) & 63;
#pragma unroll
            for (int q = 0; q < RPL; ++q)
                if (q == qn) zz[q] = L == ln ? z : zz[q];
        }
        // U solve from the bottom; z1, z2 are the two entries below
        double nrm = 0.0, z1 = 0.0, z2 = 0.0;
        n2 = 0.0;
        unroll_for<0, RPL>([&](auto qr_) {
            constexpr int q = RPL - 1 - decltype(qr_)::value;
            const int top = min(63, n - 1 - 64 * q);
            for (int l = top; l >= 0; --l) {
                const double zi = lane_read(zz[q], l), du = lane_read(fdu[q], l), du2 = lane_read(fdu2[q], l),
                             rd = lane_read(fdd[q], l);
                const double sv = (zi - du * z1 - du2 * z2) * rd;
                zz[q] = L == l ? sv : zz[q];
                nrm = fmax(nrm, fabs(sv));
                n2 += sv * sv;
                z2 = z1;
                z1 = sv;
            }
        });
        scale = nrm > 0 ? 1.0 / nrm : 1.0;
    }
    const double inv = n2 > 0 ? 1.0 / sqrt(n2) : 1.0;
#pragma unroll
    for (int q = 0; q < RPL; ++q) {
        const int i = L + 64 * q;
        if (i < n) Z[(int64_t)i * k + idx] = zz[q] * inv;
    }
}

// Gram-Schmidt (twice) of column j of Z [rows r, leading dimension ldz] against
// columns [i0, j), with normalisation after each pass, by the whole workgroup.
// coef: [j - i0] doubles, red: one double per wave.
__device__ void gs_column(double *Z, int64_t ldz, int n, int i0, int j, double *coef, double *red) {
    const int t = threadIdx.x, nt = blockDim.x, lane = t & 63, wave = t >> 6, nw = nt >> 6;
    for (int pass = 0; pass < 2; ++pass) {
        if (j > i0) {
            // coef[i - i0] = z_i . z_j, one wave per i, lanes over rows
            for (int i = i0 + wave; i < j; i += nw) {
                double sacc = 0.0;
                for (int r = lane; r < n; r += 64) sacc += Z[r * ldz + i] * Z[r * ldz + j];
                for (int off = 32; off > 0; off >>= 1) sacc += __shfl_xor(sacc, off);
                if (lane == 0) coef[i - i0] = sacc;
            }
            __syncthreads();
            for (int r = t; r < n; r += nt) {
                double sv = Z[r * ldz + j];
                for (int i = i0; i < j; ++i) sv -= coef[i - i0] * Z[r * ldz + i];
                Z[r * ldz + j] = sv;
            }
            __syncthreads();
        }
        double pn = 0.0;
        for (int r = t; r < n; r += nt) {
            const double vv = Z[r * ldz + j];
            pn += vv * vv;
        }
        const double nn = block_sum(pn, red);
        const double inv = nn > 0 ? 1.0 / sqrt(nn) : 0.0;
        for (int r = t; r < n; r += nt) Z[r * ldz + j] *= inv;
        __syncthreads();
    }
}

// Every column against all earlier ones, Z in LDS (k > 64 with n k small).
__global__ void __launch_bounds__(1024) k_orth(double *__restrict__ Zg, int n, int k) {
    extern __shared__ unsigned char smem_raw[];
    double *coef = reinterpret_cast<double *>(smem_raw);   // [k]
    double *red = coef + k;                                 // [16]
    double *Z = red + 16;                                   // [n][k + 1] (padded rows: no bank conflicts)
    for (int i = threadIdx.x; i < n * k; i += blockDim.x) Z[(i / k) * (k + 1) + i % k] = Zg[i];
    __syncthreads();
    for (int j = 0; j < k; ++j) gs_column(Z, k + 1, n, 0, j, coef, red);
    for (int i = threadIdx.x; i < n * k; i += blockDim.x) Zg[i] = Z[(i / k) * (k + 1) + i % k];
}

// Larger Z: only within clusters of eigenvalues closer than ctol (vectors of
// separated eigenvalues are already orthogonal to ~ n eps ||T|| / gap, the
// backward error of the inverse-iteration solves over the gap, and unit).  One
// workgroup per column, the one of a cluster's first column takes the whole
// cluster and the others leave, so clusters run side by side and a column
// on its own costs nothing and is left as the inverse iteration made it, a unit
// vector (all of n = 512, no clusters: 2066 us as one workgroup over every column,
// 6.2 us so).
__global__ void __launch_bounds__(1024) k_orth_clusters(double *__restrict__ Z, int n, int k,
                                                        const double *__restrict__ w, double ctol_rel,
                                                        const double *__restrict__ dd,
                                                        const double *__restrict__ ee) {
    extern __shared__ double coef[];   // [k]
    __shared__ double red[48];
    const int j0 = blockIdx.x;
    const double ctol = ctol_rel * fmax(tri_bounds(dd, ee, n, red).tnorm, 1e-300);
    __syncthreads();   // red is used again
    if (j0 > 0 && w[j0] - w[j0 - 1] <= ctol) return;
    int j1 = j0 + 1;
    while (j1 < k && w[j1] - w[j1 - 1] <= ctol) ++j1;
    if (j1 == j0 + 1) return;
    for (int j = j0; j < j1; ++j) gs_column(Z, k, n, j0, j, coef, red);
}

// CholQR, twice, of the columns of Z [n][k] (k <= 64, n <= 256, all in LDS):
// G = Z^T Z, G = R^T R, Z <- Z R^-1.  Equivalent to Gram-Schmidt in column
// (eigenvalue) order; one thread per row for the triangular multiply.
constexpr int kOrthMaxK = 64;
__global__ void __launch_bounds__(256) k_orth_chol(double *__restrict__ Zg, int n, int k,
                                                   int *__restrict__ status) {
    extern __shared__ unsigned char smem_raw[];
    const int ldz = k + 1, ldg = k + 1;
    double *Z = reinterpret_cast<double *>(smem_raw);   // [n][k+1]
    double *G = Z + (size_t)n * ldz;                     // [k][k+1]: G, then R, then R^-1
    double *rowt = G + (size_t)k * ldg;                  // [k]
    const int t = threadIdx.x, nt = blockDim.x;
    for (int i = t; i < n * k; i += nt) Z[(i / k) * ldz + i % k] = Zg[i];
    __syncthreads();
    bool fail = false;
    for (int pass = 0; pass < 2; ++pass) {
        // G = Z^T Z (upper triangle), four independent partial sums per dot
        const int npair = k * (k + 1) / 2;
        for (int pidx = t; pidx < npair; pidx += nt) {
            int a = 0, rem = pidx;
            while (rem >= k - a) {
                rem -= k - a;
                ++a;
            }
            const int b = a + rem;
            double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
            int r = 0;
            for (; r + 3 < n; r += 4) {
                s0 += Z[r * ldz + a] * Z[r * ldz + b];
                s1 += Z[(r + 1) * ldz + a] * Z[(r + 1) * ldz + b];
                s2 += Z[(r + 2) * ldz + a] * Z[(r + 2) * ldz + b];
                s3 += Z[(r + 3) * ldz + a] * Z[(r + 3) * ldz + b];
            }
            for (; r < n; ++r) s0 += Z[r * ldz + a] * Z[r * ldz + b];
            G[a * ldg + b] = (s0 + s1) + (s2 + s3);
        }
        __syncthreads();
        // Cholesky G = R^T R (upper); the trailing update uses the unscaled pivot row
        for (int j = 0; j < k; ++j) {
            double d = G[j * ldg + j];
            if (!(d > 1e-300)) {
                fail = true;
                d = 1.0;
            }
            const double inv_d = 1.0 / d;
            const int m = k - j - 1;
            for (int i = t; i < m * m; i += nt) {
                const int a = j + 1 + i % m, b = j + 1 + i / m;
                if (b >= a) G[a * ldg + b] -= G[j * ldg + a] * G[j * ldg + b] * inv_d;
            }
            __syncthreads();
            const double isd = 1.0 / sqrt(d);
            for (int c = j + 1 + t; c < k; c += nt) G[j * ldg + c] *= isd;
            if (t == 0) G[j * ldg + j] = d * isd;
        }
        __syncthreads();
        // R^-1 in place, rows from the bottom: X_ic = (delta_ic - sum_{q=i+1..c} R_iq X_qc) / R_ii
        for (int i = k - 1; i >= 0; --i) {
            for (int c = i + t; c < k; c += nt) rowt[c] = G[i * ldg + c];
            __syncthreads();
            for (int c = i + t; c < k; c += nt) {
                double sacc = (c == i) ? 1.0 : 0.0;
                for (int q = i + 1; q <= c; ++q) sacc -= rowt[q] * G[q * ldg + c];
                G[i * ldg + c] = sacc / rowt[i];
            }
            __syncthreads();
        }
        // Z <- Z R^-1, one thread per row (row in registers)
        for (int r = t; r < n; r += nt) {
            double z[kOrthMaxK];
#pragma unroll
            for (int i = 0; i < kOrthMaxK; ++i) z[i] = i < k ? Z[r * ldz + i] : 0.0;
            for (int j = 0; j < k; ++j) {
                double s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int i = 0; i < kOrthMaxK; i += 2) {
                    if (i <= j) s0 += z[i] * G[i * ldg + j];
                    if (i + 1 <= j) s1 += z[i + 1] * G[(i + 1) * ldg + j];
                }
                Z[r * ldz + j] = s0 + s1;
            }
        }
        __syncthreads();
    }
    for (int i = t; i < n * k; i += nt) Zg[i] = Z[(i / k) * ldz + i % k];
    if (t == 0 && fail) atomicOr(status, 2);
}

// CholQR applied twice to the real eigenvector block Z [n x k] (k <= 64,
// n <= 208), in LDS, 1024 threads.  G = Z^T Z and Z R^-1 run on the FP64
// matrix cores (16 x 16 output tiles, one to three per wave).  The factor
// comes from elimination on [G | I] as in k_chol_inv (pivot row broadcast
// through LDS, one barrier per step, rows kept unscaled until the end: the
// augmented half becomes L^-1 and R^-T = D^-1/2 L^-1), with 2 x 2 tiles per
// thread on a 32 x 32 grid.  Columns >= k carry an identity block of G, whose
// pivots change nothing: the elimination ends at k.
// The elimination, k/2 barrier steps of latency, was most of the time, and it
// is left out where G is within kOc2Near of the identity: there R^-1 = I - F
// with F the strict upper part of G - I plus half its diagonal, off by F^2,
// below (64 kOc2Near)^2 = 4e-17, and one pass is enough.  Inverse
// iteration gives that for eigenvalues with relative gaps above ~1e-6, that is
// nearly every Rayleigh-Ritz problem; a cluster takes the elimination, and its
// second pass is near the identity again.  n = 192, k = 64: 92 -> 20 us;
// n = 48, k = 16: 67 -> 6.3 us.
constexpr double kOc2Near = 1e-10;
// upper 16 x 16 tiles of G, then the lower ones (left zero)
__constant__ const unsigned char kOc2Tile[16] = {0x00, 0x01, 0x02, 0x03, 0x11, 0x12, 0x13, 0x22,
                                                 0x23, 0x33, 0x10, 0x20, 0x30, 0x21, 0x31, 0x32};
constexpr int kOc2Ld = 68;   // LDS row stride of Z (doubles)
constexpr int kOc2Lr = 65;   // LDS row stride of G and of R^-1
__host__ __device__ constexpr size_t orth_chol2_lds(int n) {
    return ((size_t)((n + 15) / 16 * 16) * kOc2Ld + 64 * kOc2Lr + 8 * 64) * sizeof(double);
}
__global__ void __launch_bounds__(1024) k_orth_chol2(double *__restrict__ Zg, int n, int k,
                                                     int *__restrict__ status) {
    typedef double v4d __attribute__((ext_vector_type(4)));
    extern __shared__ double smd[];
    const int n16 = (n + 15) / 16 * 16;     // rows padded with zeros to whole tiles
    double *Z = smd;                        // [n16][kOc2Ld], columns >= k zero
    double *Gs = Z + (size_t)n16 * kOc2Ld;  // [64][kOc2Lr]: G, then R^-1
    double *pg = Gs + 64 * kOc2Lr;          // [2][2][64] pivot row pairs of G
    double *pu = pg + 4 * 64;               // [2][2][64] pivot row pairs of the augmented half
    const int t = threadIdx.x, nt = blockDim.x;
    const int ti = t >> 5, tj = t & 31, a0 = 2 * ti, b0 = 2 * tj;
    const int wave = t >> 6, lane = t & 63, li = lane & 15, lg = lane >> 4;
    const int wrow_last = 4 * wave + 3;
    for (int i = t; i < n16 * kOc2Ld; i += nt) {
        const int r = i / kOc2Ld, c = i % kOc2Ld;
        Z[i] = (r < n && c < k) ? Zg[(size_t)r * k + c] : 0.0;
    }
    __syncthreads();
    bool fail = false;
    for (int pass = 0; pass < 2; ++pass) {
        const int tile = kOc2Tile[wave], ra = 16 * (tile >> 4), cg = 16 * (tile & 15);
        v4d gacc = {0.0, 0.0, 0.0, 0.0};
        if (ra <= cg && cg < k) {   // G = Z^T Z, upper tiles, one per wave
            v4d odd = {0.0, 0.0, 0.0, 0.0};
            for (int k0 = 0; k0 < n16; k0 += 8) {
                const double *z0 = Z + (size_t)(k0 + lg) * kOc2Ld;
                gacc = __builtin_amdgcn_mfma_f64_16x16x4f64(z0[ra + li], z0[cg + li], gacc, 0, 0, 0);
                const double *z1 = z0 + 4 * kOc2Ld;
                odd = __builtin_amdgcn_mfma_f64_16x16x4f64(z1[ra + li], z1[cg + li], odd, 0, 0, 0);
            }
            gacc += odd;
        }
        bool away = false;   // some element of G not within kOc2Near of the identity (or not finite)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int a = ra + lg + 4 * r, b = cg + li;
            away |= a <= b && b < k && !(fabs(gacc[r] - (a == b ? 1.0 : 0.0)) <= kOc2Near);
        }
        const bool near = !__syncthreads_or(away);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int a = ra + lg + 4 * r, b = cg + li;
            double v = gacc[r];
            if (near) v = a < b ? -v : a == b ? 1.5 - 0.5 * v : 0.0;   // I - F
            Gs[a * kOc2Lr + b] = v;
        }
        __syncthreads();
        if (!near) {
        double g[2][2], u[2][2], dpiv[2] = {1.0, 1.0};
#pragma unroll
        for (int ia = 0; ia < 2; ++ia)
#pragma unroll
            for (int ib = 0; ib < 2; ++ib) {
                const int a = a0 + ia, b = b0 + ib;
                g[ia][ib] = (a == b && a >= k) ? 1.0 : Gs[a * kOc2Lr + b];
                u[ia][ib] = a == b ? 1.0 : 0.0;
                if (ti == 0) {   // rows 0 and 1: the first pivot pair
                    pg[64 * ia + b] = g[ia][ib];
                    pu[64 * ia + b] = u[ia][ib];
                }
            }
        __syncthreads();
        // two pivots per barrier (as in k_chol_inv): rows j, j + 1 arrive with
        // the pivots < j applied; row j + 1 after pivot j is formed locally
        for (int j = 0; j < k; j += 2) {
            const int bsel = (j >> 1) & 1;
            const double *r0g = pg + 128 * bsel, *r1g = r0g + 64, *r0u = pu + 128 * bsel, *r1u = r0u + 64;
            double d0 = r0g[j];
            if (!(d0 > 1e-300) || !isfinite(d0)) {
                fail = true;
                d0 = 1.0;
            }
            const double inv0 = rcp_nr(d0);
            const double l = r0g[j + 1] * inv0;
            double d1 = r1g[j + 1] - l * r0g[j + 1];
            if (!(d1 > 1e-300) || !isfinite(d1)) {
                fail = true;
                d1 = 1.0;
            }
#pragma unroll
            for (int ia = 0; ia < 2; ++ia) {
                if (a0 + ia == j) dpiv[ia] = d0;
                if (a0 + ia == j + 1) dpiv[ia] = d1;
            }
            if (wrow_last > j) {   // rows below pivot j in this wave (uniform per wave)
                const double inv1 = rcp_nr(d1);
                double m0[2], m1[2];
#pragma unroll
                for (int ia = 0; ia < 2; ++ia) {
                    const int a = a0 + ia;
                    m0[ia] = a > j ? r0g[a] * inv0 : 0.0;
                    m1[ia] = a > j + 1 ? (r1g[a] - l * r0g[a]) * inv1 : 0.0;
                }
                double g0[2], g1[2], u0[2], u1[2];
#pragma unroll
                for (int ib = 0; ib < 2; ++ib) {
                    const int b = b0 + ib;
                    g0[ib] = r0g[b];
                    g1[ib] = r1g[b] - l * g0[ib];
                    u0[ib] = r0u[b];
                    u1[ib] = r1u[b] - l * u0[ib];
                }
#pragma unroll
                for (int ia = 0; ia < 2; ++ia) {
                    const int a = a0 + ia;
#pragma unroll
                    for (int ib = 0; ib < 2; ++ib) {
                        if (b0 + ib >= a) g[ia][ib] -= m0[ia] * g0[ib] + m1[ia] * g1[ib];
                        u[ia][ib] -= m0[ia] * u0[ib] + m1[ia] * u1[ib];
                    }
                }
                if (j + 2 < k && a0 == j + 2) {
                    double *ng = pg + 128 * (bsel ^ 1), *nu = pu + 128 * (bsel ^ 1);
#pragma unroll
                    for (int ia = 0; ia < 2; ++ia) {
                        ng[64 * ia + b0] = g[ia][0];
                        ng[64 * ia + b0 + 1] = g[ia][1];
                        nu[64 * ia + b0] = u[ia][0];
                        nu[64 * ia + b0 + 1] = u[ia][1];
                    }
                }
            }
            __syncthreads();
        }
        // R^-1 (c, a) = (D^-1/2 L^-1)(a, c)
#pragma unroll
        for (int ia = 0; ia < 2; ++ia) {
            const double isd = 1.0 / sqrt(dpiv[ia]);
#pragma unroll
            for (int ib = 0; ib < 2; ++ib) Gs[(b0 + ib) * kOc2Lr + a0 + ia] = u[ia][ib] * isd;
        }
        __syncthreads();
        }
        {   // Z <- Z R^-1: wave w computes one column tile of row tiles w / 4 + 4 i
            // (rows of R^-1 down to the tile's last column; the column tiles are
            // dealt so that every SIMD gets each of them once)
            const int cb = 16 * ((wave + (wave >> 2)) & 3);
            v4d acc[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = v4d{0.0, 0.0, 0.0, 0.0};
            for (int k0 = 0; k0 < cb + 16; k0 += 4) {
                const double b = Gs[(k0 + lg) * kOc2Lr + cb + li];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int rt = 16 * ((wave >> 2) + 4 * i);
                    if (rt < n16)
                        acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(Z[(size_t)(rt + li) * kOc2Ld + k0 + lg], b,
                                                                      acc[i], 0, 0, 0);
                }
            }
            __syncthreads();   // every read of Z done before it is overwritten
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int rt = 16 * ((wave >> 2) + 4 * i);
                if (rt < n16)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int row = rt + lg + 4 * r, col = cb + li;
                        Z[(size_t)row * kOc2Ld + col] = (row < n && col < k) ? acc[i][r] : 0.0;
                    }
            }
        }
        __syncthreads();
        if (near) break;
    }
    for (int i = t; i < n * k; i += nt) Zg[i] = Z[(i / k) * kOc2Ld + i % k];
    if (t == 0 && fail) atomicOr(status, 2);
}

// V[:, c] = H_0 ... H_{n-2} Z[:, c] for n <= 64 RPL: one wave per kUwCols
// columns, RPL rows per lane, column sums by DPP alone (wave_total), no barriers.
// Reflectors are applied in groups of kUwRing with a ring of kUwRing
// reflectors loaded ahead, so the loads of one group overlap the work of the
// previous one.
// The ring is 8 deep up to n = 256 and shorter above, by registers.  One
// reflector is a chain of ~1000 cycles up to n = 512, so a wave of its own per
// column beats workgroups with 32 columns in LDS and four barriers a reflector
// (n = k = 512: 1884 -> 481 us).
constexpr int kUwCols = 1;
template <int RPL>
__global__ void __launch_bounds__(64) k_unmtr_w(const cd *__restrict__ A, int64_t lda, int n, int k,
                                                const cd *__restrict__ tau,
                                                const double *__restrict__ Z, cd *__restrict__ V,
                                                int64_t ldv) {
    constexpr int kUwRing = RPL <= 4 ? 8 : RPL <= 8 ? 4 : 2;
    const int l = threadIdx.x;
    const int c0 = blockIdx.x * kUwCols;
    cd x[RPL][kUwCols];
#pragma unroll
    for (int q = 0; q < RPL; ++q)
#pragma unroll
        for (int c = 0; c < kUwCols; ++c) {
            const int r = l + 64 * q;
            x[q][c] = cd{(r < n && c0 + c < k) ? Z[(int64_t)r * k + c0 + c] : 0.0, 0.0};
        }
    cd ring[kUwRing][RPL];
    cd rtau[kUwRing];
    // reflector j (0 <= j <= n-2): rows j+1..n-1, v_{j+1} = 1; j < 0 is a no-op
    auto load = [&](int slot_j, cd (&v)[RPL], cd &tj) {
        const int j = slot_j;
#pragma unroll
        for (int q = 0; q < RPL; ++q) {
            const int r = l + 64 * q;
            v[q] = (j >= 0 && r == j + 1) ? cd{1.0, 0.0}
                                          : ((j >= 0 && r > j + 1 && r < n) ? A[(int64_t)j * lda + r]
                                                                            : cd{0.0, 0.0});
        }
        tj = j >= 0 ? tau[j] : cd{0.0, 0.0};
    };
    const int jtop = n - 2;
#pragma unroll
    for (int s = 0; s < kUwRing; ++s) load(jtop - s, ring[s], rtau[s]);
    for (int jg = jtop; jg >= 0; jg -= kUwRing) {
#pragma unroll
        for (int s = 0; s < kUwRing; ++s) {
            const cd tj = rtau[s];
            cd v[RPL];
#pragma unroll
            for (int q = 0; q < RPL; ++q) v[q] = ring[s][q];
            load(jg - s - kUwRing, ring[s], rtau[s]);   // refill the slot for the next group
            if (tj.x == 0.0 && tj.y == 0.0) continue;
#pragma unroll
            for (int c = 0; c < kUwCols; ++c) {
                double dr = 0.0, di = 0.0;   // v^H x_c
#pragma unroll
                for (int q = 0; q < RPL; ++q) {
                    dr += v[q].x * x[q][c].x + v[q].y * x[q][c].y;
                    di += v[q].x * x[q][c].y - v[q].y * x[q][c].x;
                }
                dr = wave_total(dr);
                di = wave_total(di);
                const cd sc = cmulz(tj, cd{dr, di});
#pragma unroll
                for (int q = 0; q < RPL; ++q) {
                    const cd u = cmulz(v[q], sc);
                    x[q][c].x -= u.x;
                    x[q][c].y -= u.y;
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < kUwCols; ++c) {
        if (c0 + c >= k) break;
#pragma unroll
        for (int q = 0; q < RPL; ++q) {
            const int r = l + 64 * q;
            if (r < n) V[(int64_t)(c0 + c) * ldv + r] = x[q][c];
        }
    }
}

}  // namespace

void launch_chol_inv_f64(const cd *G, int64_t ldg, int n, cd *Rinv, int64_t ldr, int *status,
                         hipStream_t st) {
    PW_REQUIRE(n >= 1 && n <= kCholMax, PW_ERR_ARG, "block size must be in [1, 64]");
    const size_t sm = chol_lds(n);
    ensure_smem_limit((const void *)k_chol_inv, sm);
    hipLaunchKernelGGL(k_chol_inv, dim3(1), dim3(64 * kCholWaves), sm, st, G, ldg, n, Rinv, ldr, status);
    PW_HIP(hipGetLastError());
}

size_t heev_scratch_bytes(int n, int k) {
    const size_t nch = (size_t)(n + 63) / 64;
    return 8 * 256 + (size_t)n * 16 + 2 * (size_t)n * 8 + (size_t)n * k * 8 +
           (3 + nch) * (size_t)n * 16;   // n > 96: reflector pair and two sets of ceil(n / 128) partials
}

void launch_heev_f64(cd *A, int64_t lda, int n, int k, double *w, cd *V, int64_t ldv, void *scratch,
                     int *status, hipStream_t st, bool fp32_reduction) {
    PW_REQUIRE(n >= 1 && n <= 1024 && k >= 1 && k <= n, PW_ERR_ARG, "heev: need 1 <= k <= n <= 1024");
    auto align = [](size_t x) { return (x + 255) & ~size_t(255); };
    char *p = static_cast<char *>(scratch);
    cd *tau = reinterpret_cast<cd *>(p);
    p += align((size_t)n * 16);
    double *d = reinterpret_cast<double *>(p);
    p += align((size_t)n * 8);
    double *e = reinterpret_cast<double *>(p);
    p += align((size_t)n * 8);
    double *Z = reinterpret_cast<double *>(p);
    p += align((size_t)n * k * 8);
    // 1. tridiagonalisation (the trailing block of A is overwritten in both triangles)
    int j0 = 0;   // columns done before the single-workgroup form takes the rest
    if (n > (fp32_reduction ? kRfMaxN : kTrRest)) {
        TrdState S;
        S.v[0] = reinterpret_cast<cd *>(p);
        p += align((size_t)n * 16);
        S.v[1] = reinterpret_cast<cd *>(p);
        p += align((size_t)n * 16);
        const int nb = (n + kTrCols - 1) / kTrCols;
        S.yp[0] = reinterpret_cast<cd *>(p);
        S.yp[1] = S.yp[0] + (size_t)nb * n;
        hipLaunchKernelGGL(k_herm_sym, dim3((unsigned)(((int64_t)n * n + 255) / 256)), dim3(256), 0, st, A, lda,
                           n);
        j0 = n - kTrRest;
        for (int j = 0; j <= j0; ++j) {
            const bool last = j == j0;   // only the update of the column before
            const int live = nb - (last ? j : j + 1) / kTrCols;   // blocks of 128 rows or columns
            auto col = [&](auto nt, auto tr) {
                constexpr int NT = decltype(nt)::value, TR = decltype(tr)::value;
                hipLaunchKernelGGL((k_trd_col<NT, TR>), dim3(live * live * (kTrCols / TR)), dim3(NT), 0, st, A, lda,
                                   n, j, S, d, e, tau, last);
            };
            const int rows = kTrCols * (nb - j / kTrCols);   // rows of the kernel, one per thread
            if (rows <= 256)
                col(std::integral_constant<int, 256>{}, std::integral_constant<int, kTrR256>{});
            else if (rows <= 512)
                col(std::integral_constant<int, 512>{}, std::integral_constant<int, kTrR512>{});
            else
                col(std::integral_constant<int, 1024>{}, std::integral_constant<int, kTrR1024>{});
        }
    }
    {
        cd *const Ar = A + (int64_t)j0 * (lda + 1);
        const int nr = n - j0;
        auto go = [&](auto t_, auto r_) {
            constexpr int T = decltype(t_)::value;
            hipLaunchKernelGGL((k_hetrd_la<T, decltype(r_)>), dim3(1), dim3(1024), 0, st, Ar, lda, nr, d + j0, e + j0,
                               tau + j0);
        };
        const int T = (nr + 31) / 32;
        if (fp32_reduction && n <= kRfMaxN) {
            switch (T) {
                case 1: go(std::integral_constant<int, 1>{}, 0.0f); break;
                case 2: go(std::integral_constant<int, 2>{}, 0.0f); break;
                case 3: go(std::integral_constant<int, 3>{}, 0.0f); break;
                case 4: go(std::integral_constant<int, 4>{}, 0.0f); break;
                case 5: go(std::integral_constant<int, 5>{}, 0.0f); break;
                default: go(std::integral_constant<int, 6>{}, 0.0f); break;
            }
        } else {
            static_assert(kTrRest == 96, "cases below");
            switch (T) {
                case 1: go(std::integral_constant<int, 1>{}, 0.0); break;
                case 2: go(std::integral_constant<int, 2>{}, 0.0); break;
                default: go(std::integral_constant<int, 3>{}, 0.0); break;
            }
        }
    }
    // 2. eigenvalues, one workgroup each, spread over k CUs
    const bool lowp = fp32_reduction && n <= kRfMaxN;
    hipLaunchKernelGGL(k_stebz, dim3(k), dim3(kStebzThreads), (size_t)n * 16, st, d, e, n, w,
                       lowp ? (double)FLT_EPSILON : DBL_EPSILON, status);
    // 3. inverse iteration, one wave per eigenvalue
    const int rpl = (n + 63) / 64;
    auto by_rpl = [&](auto &&f) {
        switch (rpl) {
            case 1: f(std::integral_constant<int, 1>{}); break;
            case 2: f(std::integral_constant<int, 2>{}); break;
            case 3: f(std::integral_constant<int, 3>{}); break;
            case 4: f(std::integral_constant<int, 4>{}); break;
            case 5: case 6: f(std::integral_constant<int, 6>{}); break;
            case 7: case 8: f(std::integral_constant<int, 8>{}); break;
            case 9: case 10: case 11: case 12: f(std::integral_constant<int, 12>{}); break;
            default: f(std::integral_constant<int, 16>{}); break;
        }
    };
    by_rpl([&](auto q) { hipLaunchKernelGGL(k_stein_w<decltype(q)::value>, dim3(k), dim3(64), 0, st, d, e, n, k, w, Z); });
    // 4. orthogonalisation
    const size_t smc = ((size_t)n * (k + 1) + (size_t)k * (k + 1) + k) * 8;
    const size_t sml = ((size_t)n * (k + 1) + k + 16) * 8;
    if (k <= 64 && orth_chol2_lds(n) <= 150 * 1024) {
        const size_t sm = orth_chol2_lds(n);
        ensure_smem_limit((const void *)k_orth_chol2, sm);
        hipLaunchKernelGGL(k_orth_chol2, dim3(1), dim3(1024), sm, st, Z, n, k, status);
    } else if (k <= kOrthMaxK && n <= 256 && smc <= 150 * 1024) {
        ensure_smem_limit((const void *)k_orth_chol, smc);
        hipLaunchKernelGGL(k_orth_chol, dim3(1), dim3(256), smc, st, Z, n, k, status);
    } else if (sml <= 132 * 1024) {
        ensure_smem_limit((const void *)k_orth, sml);
        hipLaunchKernelGGL(k_orth, dim3(1), dim3(1024), sml, st, Z, n, k);
    } else {
        hipLaunchKernelGGL(k_orth_clusters, dim3(k), dim3(1024), (size_t)k * 8, st, Z, n, k, w, 2e-5, d, e);
    }
    // 5. back-transform
    by_rpl([&](auto q) {
        hipLaunchKernelGGL(k_unmtr_w<decltype(q)::value>, dim3((k + kUwCols - 1) / kUwCols), dim3(64), 0, st, A, lda, n,
                           k, tau, Z, V, ldv);
    });
    PW_HIP(hipGetLastError());
}

}  // namespace pw

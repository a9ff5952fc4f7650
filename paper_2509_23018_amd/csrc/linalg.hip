// Dense complex FP64 linear algebra on gfx950 (linalg.hpp): a GEMM on the
// FP64 matrix cores, an elementwise axpby and a Hermitian Jacobi eigensolver.
#include <algorithm>
#include <cmath>
#include <vector>

#include "common.hpp"
#include "linalg.hpp"
#include "prof.hpp"

namespace gw {
namespace {

// ---------------------------------------------------------------- GEMM
//
// One workgroup of 4 waves (2 x 2) per 32 BX x 32 tile of C; each wave owns BX
// blocks of the 16x16x4 FP64 MFMA.  The k dimension is staged through LDS 16
// at a time, in two buffers: stage t + 2 is loaded into registers while stage
// t is multiplied, and written to LDS a stage before its use, one barrier per
// stage.  Rows and columns past the edge of C are clamped: they feed only
// entries that are not stored.  Only the last, partial stage masks its k.
// Each complex multiply-add takes three real products (p1 = ar br, p2 = ai bi,
// p3 = (ar + ai)(br + bi); Re = p1 - p2, Im = p3 - p1 - p2).  Every entry of C
// is summed in the same order whatever the tile, so the tile does not change a
// bit of the result.
//
// Bound by the FP64 matrix pipe where the grid fills the chip, by the chain of
// stages where it does not.  Measured against 64 x 64 tiles of one LDS buffer,
// loads one stage ahead and clamps and masks in every stage (TFLOP/s count the
// six flops executed per complex multiply-add):
//   2048 x 2048 x 2048        960 ->  800 us (53.7 -> 64.4 TFLOP/s), BX = 2
//   4 of 2007 x 2007 x 512    914 ->  815 us (54.2 -> 60.7)
//   3840 x 603 x 6031        2630 -> 1424 us (31.9 -> 58.9)
//   3840 x 400 x 2007         445 ->  352 us (41.6 -> 52.5), BX = 1
//   1189 x 135 x 1189         154 ->   38 us,                BX = 1
//   135 x 135 x 1189          158 ->   37 us,                BX = 1
// Writing stage t + 1 to LDS before the MFMAs of stage t (915 us for the
// first) and 32-deep stages (47 us for the fifth) were slower.

template <int OPA, int OPB, int BX>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void zgemm_kernel(
    ZGemm g) {
    constexpr int TM = 32 * BX, TN = 32, KT = 16, PD = 2;
    constexpr int NA = TM * KT / 256, NB = TN * KT / 256;
    __shared__ double2 s_a[2][TM][KT + 1];  // [m][k]
    __shared__ double2 s_b[2][KT][TN + 1];  // [k][n]
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, row = lane & 15, kq = lane >> 4;
    const int wi = wave >> 1, wj = wave & 1;
    const int64_t bz = blockIdx.z;
    const int i0 = blockIdx.y * TM, j0 = blockIdx.x * TN;

    dbl4 p1[BX], p2[BX], p3[BX];
#pragma unroll
    for (int x = 0; x < BX; ++x) p1[x] = p2[x] = p3[x] = zero4();

    // staged element e = tid + 256 u: (m, k) of the A side, (k, n) of the B side
    auto a_mk = [&](int u, int& mm, int& kk) {
        const int e = tid + 256 * u;
        mm = OPA == kOpN ? e / KT : e % TM;
        kk = OPA == kOpN ? e % KT : e / TM;
    };
    auto b_kn = [&](int u, int& kk, int& nn) {
        const int e = tid + 256 * u;
        nn = OPB == kOpN ? e % TN : e / KT;
        kk = OPB == kOpN ? e / TN : e % KT;
    };
    const double2 *pa[NA], *pb[NB];  // element u of the next stage to load
#pragma unroll
    for (int u = 0; u < NA; ++u) {
        int mm, kk;
        a_mk(u, mm, kk);
        const int64_t im = min(i0 + mm, g.m - 1);
        pa[u] = g.a + bz * g.stride_a + (OPA == kOpN ? im * g.lda + kk : kk * g.lda + im);
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        int kk, nn;
        b_kn(u, kk, nn);
        const int64_t in = min(j0 + nn, g.n - 1);
        pb[u] = g.b + bz / g.b_repeat * g.stride_b + (OPB == kOpN ? kk * g.ldb + in : in * g.ldb + kk);
    }
    const int64_t da = OPA == kOpN ? KT : KT * g.lda, db = OPB == kOpN ? KT * g.ldb : KT;
    double2 ra[PD][NA], rb[PD][NB];
    // component loads: a whole-struct copy would be fused with the LDS write
    // into one copy behind the MFMAs
    auto load = [&](int slot, int e) {  // element e of NA + NB
        if (e < NA) {
            ra[slot][e].x = pa[e]->x;
            ra[slot][e].y = pa[e]->y;
            pa[e] += da;
        } else {
            rb[slot][e - NA].x = pb[e - NA]->x;
            rb[slot][e - NA].y = pb[e - NA]->y;
            pb[e - NA] += db;
        }
    };
    auto fetch = [&](int slot) {
#pragma unroll
        for (int e = 0; e < NA + NB; ++e) load(slot, e);
    };
    const int nfull = g.k / KT, rem = g.k % KT;
    auto fetch_rem = [&](int slot) {  // the last, partial stage: k past the end is zero
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            int mm, kk;
            a_mk(u, mm, kk);
            ra[slot][u] = kk < rem ? *pa[u] : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            int kk, nn;
            b_kn(u, kk, nn);
            rb[slot][u] = kk < rem ? *pb[u] : make_double2(0.0, 0.0);
        }
    };
    auto store1 = [&](int slot, int buf, int e) {
        if (e < NA) {
            int mm, kk;
            a_mk(e, mm, kk);
            const double2 v = ra[slot][e];
            s_a[buf][mm][kk] = make_double2(v.x, OPA == kOpC ? -v.y : v.y);
        } else {
            int kk, nn;
            b_kn(e - NA, kk, nn);
            const double2 v = rb[slot][e - NA];
            s_b[buf][kk][nn] = make_double2(v.x, OPB == kOpC ? -v.y : v.y);
        }
    };
    auto store = [&](int slot, int buf) {
#pragma unroll
        for (int e = 0; e < NA + NB; ++e) store1(slot, buf, e);
    };
    // fragments of k-step q, and the sums of the third product
    auto read = [&](int buf, int q, double2 (&a)[BX], double2& b) {
#pragma unroll
        for (int x = 0; x < BX; ++x) a[x] = s_a[buf][wi * (16 * BX) + x * 16 + row][q * 4 + kq];
        b = s_b[buf][q * 4 + kq][wj * 16 + row];
    };
    auto sums = [&](const double2 (&a)[BX], double2 b, double (&as)[BX], double& bs) {
#pragma unroll
        for (int x = 0; x < BX; ++x) as[x] = a[x].x + a[x].y;
        bs = b.x + b.y;
    };
    auto mfma1 = [&](int i, const double2 (&a)[BX], double2 b, const double (&as)[BX], double bs) {
        const int x = i / 3;
        if (i % 3 == 0) p1[x] = mfma_f64(a[x].x, b.x, p1[x]);
        if (i % 3 == 1) p2[x] = mfma_f64(a[x].y, b.y, p2[x]);
        if (i % 3 == 2) p3[x] = mfma_f64(as[x], bs, p3[x]);
    };
    auto multiply = [&](int buf) {
#pragma unroll
        for (int q = 0; q < KT / 4; ++q) {
            double2 a[BX], b;
            double as[BX], bs;
            read(buf, q, a, b);
            sums(a, b, as, bs);
#pragma unroll
            for (int i = 0; i < 3 * BX; ++i) mfma1(i, a, b, as, bs);
        }
    };
    const int nst = nfull + (rem > 0);
    auto fetch_any = [&](int st, int slot) {
        if (st < nfull) fetch(slot);
        else if (st < nst) fetch_rem(slot);
    };
    if (nst > 0) {
        fetch_any(0, 0);
        store(0, 0);
        __syncthreads();
#pragma unroll
        for (int d = 1; d < PD; ++d) fetch_any(d, d % PD);
        // Stage st is multiplied from buffer st & 1, stage st + PD loaded
        // (always a whole one here) and stage st + 1 written to LDS.  Every
        // instruction between the MFMAs is placed: one load per two MFMAs from
        // the start of the stage, one LDS write per MFMA at its end, the next
        // k-step's fragments and sums before the current one ends.  In runs
        // before and after the MFMAs the same instructions made the fifth
        // product above take 44 us where it now takes 38, the first 842 and
        // 800 us on one box.
        int st = 0;
        for (; st + PD + PD - 1 < nfull; st += PD) {
#pragma unroll
            for (int d = 0; d < PD; ++d) {
                const int buf = d & 1;
                constexpr int NM = 3 * BX, NQ = KT / 4, NE = NA + NB;
                double2 a[2][BX], b[2];
                double as[2][BX], bs[2];
                read(buf, 0, a[0], b[0]);
                sums(a[0], b[0], as[0], bs[0]);
                __builtin_amdgcn_s_setprio(2);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const int f = q & 1;
#pragma unroll
                    for (int i = 0; i < NM; ++i) {
                        mfma1(i, a[f], b[f], as[f], bs[f]);
                        __builtin_amdgcn_sched_barrier(0);
                        const int t = q * NM + i;
                        const int w = t - (NQ * NM - NE - 1);
                        if (t % 2 == 1 && t / 2 < NE) load(d, t / 2);
                        if (w >= 0 && w < NE) store1((d + 1) % PD, buf ^ 1, w);
                        if (i == (NM - 2) / 2 && q + 1 < NQ) read(buf, q + 1, a[f ^ 1], b[f ^ 1]);
                        if (i == NM - 2 && q + 1 < NQ) sums(a[f ^ 1], b[f ^ 1], as[f ^ 1], bs[f ^ 1]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                __builtin_amdgcn_s_setprio(0);
                __syncthreads();
            }
        }
        for (; st < nst; st += PD) {
#pragma unroll
            for (int d = 0; d < PD; ++d) {
                if (st + d >= nst) break;
                const int buf = d & 1;
                fetch_any(st + d + PD, d);
                multiply(buf);
                if (st + d + 1 < nst) store((d + 1) % PD, buf ^ 1);
                __syncthreads();
            }
        }
    }
    double2* C = g.c + bz * g.stride_c;
    const bool use_beta = g.beta.x != 0.0 || g.beta.y != 0.0;
#pragma unroll
    for (int x = 0; x < BX; ++x)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int r = i0 + wi * (16 * BX) + x * 16 + 4 * t + kq;
            const int c = j0 + wj * 16 + row;
            if (r >= g.m || c >= g.n) continue;
            const double2 acc =
                make_double2(p1[x][t] - p2[x][t], p3[x][t] - p1[x][t] - p2[x][t]);
            double2 v = cmul(g.alpha, acc);
            double2* dst = C + static_cast<int64_t>(r) * g.ldc + c;
            if (use_beta) {
                const double2 o = cmul(g.beta, *dst);
                v.x += o.x;
                v.y += o.y;
            }
            *dst = v;
        }
}

template <int OPA, int OPB, int BX>
void zgemm_tile_launch(const ZGemm& g, hipStream_t s) {
    const dim3 grid(static_cast<unsigned>(ceil_div(g.n, 32)),
                    static_cast<unsigned>(ceil_div(g.m, 32 * BX)), static_cast<unsigned>(g.batch));
    ProfScope ps("zgemm", s);
    hipLaunchKernelGGL((zgemm_kernel<OPA, OPB, BX>), grid, dim3(256), 0, s, g);
    GW_HIP_TRY(hipGetLastError());
}

// 64 x 32 tiles read fewer bytes per flop; 32 x 32 tiles make twice the
// workgroups.  Below four 64 x 32 tiles per CU the second counts for more: 780
// tiles (3840 x 400 x 2007) take 394 us wide and 359 us narrow, 1140
// (3840 x 603 x 6031) 1516 and 1631 us.
template <int OPA, int OPB>
void zgemm_launch(const ZGemm& g, hipStream_t s) {
    const int64_t wide = static_cast<int64_t>(ceil_div(g.n, 32)) * ceil_div(g.m, 64) * g.batch;
    if (wide >= 1024)
        zgemm_tile_launch<OPA, OPB, 2>(g, s);
    else
        zgemm_tile_launch<OPA, OPB, 1>(g, s);
}

// z may alias x or y (elementwise), so the pointers are not restrict
__global__ __launch_bounds__(256) void zaxpby_kernel(int64_t n, double2 a, const double2* x,
                                                     double2 b, const double2* y, double2* z) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const double2 u = cmul(a, x[i]);
        const double2 v = cmul(b, y[i]);
        z[i] = make_double2(u.x + v.x, u.y + v.y);
    }
}

__global__ __launch_bounds__(256) void scale_rows_kernel(const double2* in, double2* out,
                                                         const double* __restrict__ w,
                                                         int64_t n, int64_t cols) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const double f = w[i / cols];
        const double2 x = in[i];
        out[i] = make_double2(f * x.x, f * x.y);
    }
}

__global__ __launch_bounds__(256) void diag_re_kernel(const double2* __restrict__ a, int n,
                                                      double* __restrict__ out) {
    const int64_t b = blockIdx.y;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < n) out[b * n + j] = a[b * n * n + static_cast<int64_t>(j) * n + j].x;
}

// ---------------------------------------------------------------- Cholesky

constexpr int kCB = 64;  // Cholesky block

// out[0] = the largest real diagonal entry of g (one workgroup)
__global__ __launch_bounds__(256) void diag_max_kernel(const double2* __restrict__ g, int n,
                                                       double* __restrict__ out) {
    __shared__ double s[256];
    double m = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) m = fmax(m, g[static_cast<int64_t>(i) * n + i].x);
    s[threadIdx.x] = m;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) s[threadIdx.x] = fmax(s[threadIdx.x], s[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = s[0];
}

// Diagonal block K = [k0, k0 + kb) of g: the upper Cholesky factor R_KK of
// g[K][K] (g[K][K] = R_KK^H R_KK) written back over it (lower part zero), and
// X = R_KK^-1 into x ([kCB][kCB], upper; rows and columns of lost directions
// zero).  A pivot at or below 1e-26 * gmax[0] is a lost direction.
//
// One workgroup, so the latency of its dependent steps is the whole cost.  The
// block lives in registers (thread (ti, tj) holds rows ti + 16 r and columns
// tj + 16 c; blocks below the diagonal are not touched) and a step passes only
// the pivot row through LDS: its owners write it as it stands, and behind the
// step's one barrier each wave scales it for itself, an element per lane.  X is
// solved by two waves, half a column entry per lane, so that every lane reads the
// same entries of R; the order of each sum is that of plain back substitution.
// With the block in LDS, three barriers per step and each column's rows read at
// a pace of its own a 64 x 64 block took 107 us; with X by one wave, a column per
// lane, and a choice between an LDS place and a zero's place (flat loads) 75 us
// against 66 us.
__global__ __launch_bounds__(256) void chol_block_kernel(double2* __restrict__ g, int n, int k0,
                                                         int kb, const double* __restrict__ gmax,
                                                         double2* __restrict__ x) {
    constexpr int R = kCB / 16;
    __shared__ double2 s_r[kCB][kCB + 1];
    __shared__ double s_x[2][kCB][64];
    __shared__ double s_diag[kCB];
    __shared__ double2 s_piv[2][kCB];
    __shared__ double2 s_row[4][kCB];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int ti = threadIdx.x >> 4, tj = threadIdx.x & 15;
    const double thr = 1e-26 * gmax[0];
    const double2 zero = make_double2(0.0, 0.0);
    for (int e = threadIdx.x; e < 2 * kCB * 64; e += 256) (&s_x[0][0][0])[e] = 0.0;
    for (int e = threadIdx.x; e < kCB * (kCB + 1); e += 256) (&s_r[0][0])[e] = zero;
    double2 a[R][R];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < R; ++c) {
            const int i = ti + 16 * r, j = tj + 16 * c;
            const bool in = i < kb && j < kb;
            const double2 v = g[in ? static_cast<int64_t>(k0 + i) * n + k0 + j
                                   : static_cast<int64_t>(k0) * n + k0];
            a[r][c] = make_double2(in ? v.x : 0.0, in ? v.y : 0.0);
        }
#pragma unroll
    for (int pr = 0; pr < R; ++pr) {
#pragma unroll 1
        for (int pt = 0; pt < 16; ++pt) {
            const int k = 16 * pr + pt, buf = k & 1;
            if (k >= kb) break;
            if (ti == pt)
#pragma unroll
                for (int c = 0; c < R; ++c) s_piv[buf][tj + 16 * c] = a[pr][c];
            __syncthreads();
            const double piv = s_piv[buf][k].x;
            const bool lost = !(piv > thr);
            const double rk = lost ? 1.0 : sqrt(piv);
            const double2 u = s_piv[buf][lane];
            const double2 sc = lost || lane < k ? zero
                               : lane == k      ? make_double2(rk, 0.0)
                                                : make_double2(u.x / rk, u.y / rk);
            s_row[wave][lane] = sc;
            if (wave == 0) s_r[k][lane] = make_double2(lane == k ? 0.0 : sc.x, sc.y);
            if (wave == 0 && lane == k) s_diag[k] = sc.x;
            __builtin_amdgcn_wave_barrier();
            // trailing rows: a[i][j] -= conj(r[k][i]) r[k][j], i > k, the upper
            // 16 x 16 blocks
            double2 rj[R];
#pragma unroll
            for (int c = pr; c < R; ++c) rj[c] = s_row[wave][tj + 16 * c];
#pragma unroll
            for (int r = pr; r < R; ++r) {
                double2 p = s_row[wave][ti + 16 * r];  // a choice of values, not of places
                const bool below = ti + 16 * r > k;
                p.x = below ? p.x : 0.0;
                p.y = below ? p.y : 0.0;
#pragma unroll
                for (int c = r; c < R; ++c) {
                    a[r][c].x -= p.x * rj[c].x + p.y * rj[c].y;  // conj(p) r
                    a[r][c].y -= p.x * rj[c].y - p.y * rj[c].x;
                }
            }
        }
    }
    __syncthreads();
    // X = R^-1 by back substitution upwards: column j = 32 wave + lane/2, its real
    // part in the even lane and its imaginary part in the odd one: Re p x =
    // fma(p.x, x.x, p.y (-x.y)), Im p x = fma(p.y, x.x, p.x x.y).  The sum of row i
    // runs upwards from k = i + 1, by whole groups of 8: the k before it meet
    // zeros of R (s_r has no diagonal), those past kb zeros of X.
    if (wave < 2) {
        const int j = 32 * wave + (lane >> 1);
        const bool im = lane & 1;
        double* xl = &s_x[wave][0][lane];
        const double2* xj = reinterpret_cast<const double2*>(&s_x[wave][0][lane & ~1]);
        const double* pr = reinterpret_cast<const double*>(&s_r[0][0]) + im;
        const double* pi = reinterpret_cast<const double*>(&s_r[0][0]) + !im;
        const long long sign = im ? 0 : 1ll << 63;
#pragma unroll
        for (int ib = kCB / 8 - 1; ib >= 0; --ib) {
#pragma unroll 1
            for (int ii = 7; ii >= 0; --ii) {
                const int i = 8 * ib + ii;
                if (i >= kb || i >= 32 * (wave + 1)) continue;  // uniform; X[i][j] = 0
                double sum = 0.0;
#pragma unroll
                for (int k = 8 * ib; k < kCB; ++k) {
                    const int e = 2 * (i * (kCB + 1) + k);
                    const double2 q = xj[32 * k];
                    const double qi = __longlong_as_double(__double_as_longlong(q.y) ^ sign);
                    sum += fma(pr[e], q.x, pi[e] * qi);
                }
                const double rii = s_diag[i];
                double v = 0.0;
                if (rii > 0.0 && i <= j && j < kb)
                    v = i == j ? (im ? 0.0 : 1.0 / rii) : -sum / rii;
                xl[64 * i] = v;
            }
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kb * kb; e += 256) {
        const int i = e / kb, j = e % kb;
        g[static_cast<int64_t>(k0 + i) * n + k0 + j] =
            i == j ? make_double2(s_diag[i], 0.0) : s_r[i][j];
        x[i * kCB + j] = *reinterpret_cast<const double2*>(&s_x[j >> 5][i][2 * (j & 31)]);
    }
}

// dst[i][j] = src[i][j] for an [rows][cols] block (leading dimensions lds, ldd)
__global__ __launch_bounds__(256) void copy_block_kernel(const double2* __restrict__ src,
                                                         int64_t lds, double2* __restrict__ dst,
                                                         int64_t ldd, int rows, int cols) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= static_cast<int64_t>(rows) * cols) return;
    const int64_t i = t / cols, j = t % cols;
    dst[i * ldd + j] = src[i * lds + j];
}

__global__ __launch_bounds__(256) void zero_fill_kernel(double2* __restrict__ p, int64_t n) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        p[i] = make_double2(0.0, 0.0);
}

// ---------------------------------------------------------------- Jacobi
//
// Round-robin order on n' = n rounded up to even: in step r (r < n' - 1) the
// n'/2 pairs are (L[k], L[n'-1-k]) with L[0] = 0 and
// L[j] = 1 + (j - 1 + r) mod (n' - 1); every pair meets once per sweep.  An
// index n (odd n) is a phantom: its pair does not rotate.
//
// Rotation of pair (p, q) (p < q), from h_pp, h_qq and b = h_pq = |b| e^{i phi}:
// tau = (h_qq - h_pp) / (2 |b|), t = sign(tau) / (|tau| + sqrt(1 + tau^2)),
// c = 1 / sqrt(1 + t^2), S = t c e^{i phi}; J = [[c, S], [-conj(S), c]] on
// (p, q) makes (J^H H J)_pq = 0.  One step applies the n'/2 disjoint
// rotations at once: A <- J^H A J and V <- V J.

// From n = kBJMin on by blocks of kBJ indices, below that by elements.
constexpr int kBJ = 16, kBP = 2 * kBJ, kBJMin = 64;

__device__ __forceinline__ int rr_index(int j, int r, int np) {  // j < np, r < np - 1
    const int x = j - 1 + r;
    return j == 0 ? 0 : 1 + (x >= np - 1 ? x - (np - 1) : x);
}

__device__ __forceinline__ void rr_pair(int k, int r, int np, int& p, int& q) {
    const int a = rr_index(k, r, np), b = rr_index(np - 1 - k, r, np);
    p = min(a, b);
    q = max(a, b);
}

struct Rot {
    double c;
    double2 s;  // S
};

__device__ __forceinline__ Rot rotation_of(double hpp, double hqq, double2 b) {
    Rot r{1.0, make_double2(0.0, 0.0)};
    const double ab = hypot(b.x, b.y);
    if (ab == 0.0) return r;
    const double tau = (hqq - hpp) / (2.0 * ab);
    const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
    // c = 1 / sqrt(1 + t^2), then one Newton step on c^2 (1 + t^2) = 1 with the
    // products kept exact by fma: for small t the rounded c alone leaves
    // c^2 + |S|^2 - 1 at about +eps/2 on average, a bias that thousands of
    // rotations per entry turn into a (1 + O(1e-13)) scaling of the spectrum
    const double c0 = 1.0 / sqrt(1.0 + t * t);
    const double pp = c0 * c0, pe = fma(c0, c0, -pp);
    const double qq = t * t, qe = fma(t, t, -qq);
    const double res = (pp - 1.0) + pe + fma(pp, qq, pp * qe + pe * qq);
    const double c = c0 - 0.5 * c0 * res;
    const double sc = t * c / ab;  // S = t c b / |b|
    r.c = c;
    r.s = make_double2(sc * b.x, sc * b.y);
    return r;
}

// The same rotation with one square root, one division and one reciprocal
// square root in the chain: with d = h_qq - h_pp, u = t / |b| =
// 2 sign(d) / (|d| + sqrt(d^2 + 4 |b|^2)), so that t^2 = u^2 |b|^2 and
// S = c u b need no |b|.  1 + t^2 lies in [1, 2]: c from the hardware's
// reciprocal square root and two Newton steps, then the exact one above.
__device__ __forceinline__ Rot rotation_short(double hpp, double hqq, double2 b) {
    Rot r{1.0, make_double2(0.0, 0.0)};
    const double b2 = b.x * b.x + b.y * b.y;
    if (b2 == 0.0) return r;
    const double d = hqq - hpp;
    const double u = (d >= 0.0 ? 2.0 : -2.0) / (fabs(d) + sqrt(fma(d, d, 4.0 * b2)));
    const double ub = u * b2, qq = u * ub, x = 1.0 + qq;  // qq = t^2
    double c0 = __builtin_amdgcn_rsq(x);
    c0 = fma(c0, 0.5 * fma(-x * c0, c0, 1.0), c0);
    c0 = fma(c0, 0.5 * fma(-x * c0, c0, 1.0), c0);
    const double qe = fma(u, ub, -qq);
    const double pp = c0 * c0, pe = fma(c0, c0, -pp);
    const double res = (pp - 1.0) + pe + fma(pp, qq, pp * qe + pe * qq);
    const double c = c0 - 0.5 * c0 * res;
    const double sc = u * c;
    r.c = c;
    r.s = make_double2(sc * b.x, sc * b.y);
    return r;
}

// Whole eigen-decomposition of one n x n matrix (n < kBJMin) by one workgroup,
// A and V in LDS: element sweeps in round-robin order until the off-diagonal
// norm is below tol of the norm or has stopped falling at roundoff (the
// criterion of jacobi_eigh), at most max_sweeps.  SHORT picks the rotation; NT
// threads are at least one per 2 x 2 block of A.
//
// A chain of n - 1 dependent steps per sweep, each the latency of a rotation
// (one wave) and of the update of A (every wave); V is updated with the
// previous step's rotations beside the next ones.  As a launch per step, with
// A and V in global memory and a host wait per sweep, a step took 5.4 us (24
// matrices of n = 48: 2,340 us) against 1.35 us here (670 us).  Updating only
// the upper blocks of A and writing their mirror images took as long.
template <bool SHORT, int NT>
__global__ __launch_bounds__(NT) void jacobi_lds_kernel(double2* __restrict__ a_io,
                                                         double2* __restrict__ v_io, int n,
                                                         double tol, int max_sweeps,
                                                         double* __restrict__ sweeps_out) {
    extern __shared__ double2 jl[];
    constexpr int NW = NT / 64;
    __shared__ double s_red[2 * NW];
    __shared__ double rc[2][kBJMin / 2];
    __shared__ double2 rs[2][kBJMin / 2];
    const int ld = n | 1;  // odd row length: columns fall on different banks
    double2* a = jl;
    double2* v = jl + n * ld;
    const int np = n + (n & 1), half = np / 2;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    a_io += static_cast<int64_t>(blockIdx.x) * n * n;
    v_io += static_cast<int64_t>(blockIdx.x) * n * n;
    for (int e = tid; e < n * n; e += NT) {
        const int i = e / n, j = e % n;
        a[i * ld + j] = a_io[e];
        v[i * ld + j] = make_double2(i == j ? 1.0 : 0.0, 0.0);
    }
    __syncthreads();
    auto rotations = [&](int r, int buf) {  // one wave
        if (lane >= half) return;
        int p, q;
        rr_pair(lane, r, np, p, q);
        Rot ro{1.0, make_double2(0.0, 0.0)};
        if (q < n) {
            const double hpp = a[p * ld + p].x, hqq = a[q * ld + q].x;
            ro = SHORT ? rotation_short(hpp, hqq, a[p * ld + q])
                       : rotation_of(hpp, hqq, a[p * ld + q]);
        }
        rc[buf][lane] = ro.c;
        rs[buf][lane] = ro.s;
    };
    // right: [x_p, x_q] <- [c x_p - conj(S) x_q, S x_p + c x_q]
    auto right = [](double c, double2 sx, double2 xp, double2 xq, double2& op, double2& oq) {
        const double2 u = cmul(make_double2(sx.x, -sx.y), xq), w = cmul(sx, xp);
        op = make_double2(c * xp.x - u.x, c * xp.y - u.y);
        oq = make_double2(w.x + c * xq.x, w.y + c * xq.y);
    };
    // left: rows p' = c row_p - S row_q, q' = conj(S) row_p + c row_q
    auto left = [](double c, double2 sx, double2 xp, double2 xq, double2& op, double2& oq) {
        const double2 u = cmul(sx, xq), w = cmul(make_double2(sx.x, -sx.y), xp);
        op = make_double2(c * xp.x - u.x, c * xp.y - u.y);
        oq = make_double2(w.x + c * xq.x, w.y + c * xq.y);
    };
    const double2 zero = make_double2(0.0, 0.0);
    auto update_block = [&](int k1, int k2, int r, int buf) {  // 2 x 2 block of A, in place
        int p1, q1, p2, q2;
        rr_pair(k1, r, np, p1, q1);
        rr_pair(k2, r, np, p2, q2);
        const bool q1ok = q1 < n, q2ok = q2 < n;
        const double2 app = a[p1 * ld + p2], apq = q2ok ? a[p1 * ld + q2] : zero;
        const double2 aqp = q1ok ? a[q1 * ld + p2] : zero;
        const double2 aqq = q1ok && q2ok ? a[q1 * ld + q2] : zero;
        double2 bpp, bpq, bqp, bqq, cpp, cqp, cpq, cqq;
        right(rc[buf][k2], rs[buf][k2], app, apq, bpp, bpq);
        right(rc[buf][k2], rs[buf][k2], aqp, aqq, bqp, bqq);
        left(rc[buf][k1], rs[buf][k1], bpp, bqp, cpp, cqp);
        left(rc[buf][k1], rs[buf][k1], bpq, bqq, cpq, cqq);
        if (k1 == k2) {  // the rotated pair: exact zeros off the diagonal, real diagonal
            cpq = cqp = zero;
            cpp.y = 0.0;
            cqq.y = 0.0;
        }
        a[p1 * ld + p2] = cpp;
        if (q2ok) a[p1 * ld + q2] = cpq;
        if (q1ok) a[q1 * ld + p2] = cqp;
        if (q1ok && q2ok) a[q1 * ld + q2] = cqq;
    };
    // one of the half^2 <= NT blocks of A; column pair kv and every iv-th row of
    // V for the threads of waves 1 and up
    const int ta = tid / half, tb = tid % half;
    auto update_a = [&](int r, int buf) {
        if (ta < half) update_block(ta, tb, r, buf);
    };
    const int tv = (tid + NT - 64) % NT;
    const int kv = tv % half, i0v = tv / half, iv = (NT - 64) / half;
    auto update_v = [&](int r, int buf) {
        int p, q;
        rr_pair(kv, r, np, p, q);
        if (q >= n || i0v >= iv) return;
        const double c = rc[buf][kv];
        const double2 sx = rs[buf][kv];
        for (int i = i0v; i < n; i += iv) {
            double2 op, oq;
            right(c, sx, v[i * ld + p], v[i * ld + q], op, oq);
            v[i * ld + p] = op;
            v[i * ld + q] = oq;
        }
    };
    double prev = -1.0;
    int sweeps = 0;
    for (; sweeps < max_sweeps && n > 1; ++sweeps) {
        double off = 0.0, all = 0.0;
        for (int e = tid; e < n * n; e += NT) {
            const int i = e / n, j = e % n;
            const double2 x = a[i * ld + j];
            const double m2 = x.x * x.x + x.y * x.y;
            all += m2;
            if (i != j) off += m2;
        }
        for (int w = 32; w > 0; w >>= 1) {
            off += __shfl_xor(off, w);
            all += __shfl_xor(all, w);
        }
        if (lane == 0) {
            s_red[wave] = off;
            s_red[NW + wave] = all;
        }
        __syncthreads();
        off = all = 0.0;
        for (int w = 0; w < NW; ++w) {
            off += s_red[w];
            all += s_red[NW + w];
        }
        off = sqrt(off);
        all = sqrt(all);
        const bool stalled = sweeps >= 3 && prev >= 0.0 && off >= 0.25 * prev && off <= 1e-12 * all;
        prev = off;
        if (off <= tol * all || stalled) break;  // the same in every thread
        if (wave == 0) rotations(0, 0);
        for (int r = 0; r < np - 1; ++r) {
            __syncthreads();  // the rotations of step r are there
            update_a(r, r & 1);
            __syncthreads();
            if (wave > 0)
                update_v(r, r & 1);
            else if (r + 1 < np - 1)
                rotations(r + 1, (r + 1) & 1);
        }
        __syncthreads();
    }
    for (int e = tid; e < n * n; e += NT) {
        const int i = e / n, j = e % n;
        a_io[e] = a[i * ld + j];
        v_io[e] = v[i * ld + j];
    }
    if (tid == 0) sweeps_out[blockIdx.x] = sweeps;
}

// ---------------------------------------------------------------- block Jacobi
//
// For n >= kBJMin the same rotations are grouped by blocks of kBJ = 16
// indices.  The blocks (n rounded up to whole blocks, then to an even count;
// a block past n is a phantom) meet in the round-robin order above, and in
// one block step each pair of blocks (I, J) owns the 32 x 32 Hermitian
// sub-matrix S = A[I u J, I u J]:
//   1. one workgroup per pair runs one cyclic sweep of the element rotations
//      on S in LDS (31 steps of 16 disjoint rotations) and accumulates them
//      into the unitary Q = J_1 J_2 ... J_31;
//   2. one launch applies every pair's Q at once: the tile of A on rows
//      I_k u J_k and columns I_l u J_l becomes Q_k^H A[., .] Q_l, and the
//      columns I_l u J_l of V become V[:, .] Q_l.
// A tile depends only on its own entries and two Q's, so step 2 is in place;
// the tiles with k <= l are computed and the others written as their
// conjugate transposes, which keeps A exactly Hermitian.  A block sweep
// (blocks - 1 steps) meets every pair of indices at least once, as an element
// sweep does, but reads and writes A and V once per block step instead of
// once per element step.  Entries past n are zero in S, so their rotations
// are the identity and never couple them with the others; they are neither
// read nor written.

struct Quad {  // a 2 x 2 block of complex entries
    double2 a00, a01, a10, a11;
};

__device__ __forceinline__ double2 cfma(double2 a, double2 b, double2 c) {  // c + a b
    return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
__device__ __forceinline__ double2 cfma_conj_a(double2 a, double2 b, double2 c) {  // c + conj(a) b
    return make_double2(fma(a.x, b.x, fma(a.y, b.y, c.x)), fma(a.x, b.y, fma(-a.y, b.x, c.y)));
}

__device__ __forceinline__ int bj_row(int t, int bp, int bq) {  // local index -> global index
    return t < kBJ ? bp * kBJ + t : bq * kBJ + (t - kBJ);
}

// one pair's sweep; q_out[pair] = Q (32 x 32, row-major)
//
// A chain of 31 dependent steps: the rotations (16 lanes of one wave), then the
// update of S (waves 0 to 3, a 2 x 2 block per thread); waves 4 to 7 apply each
// step's rotations to Q beside the next step's, off the chain.  41 us per
// launch with one set of waves for all of it, 32 us so (n = 135).  The long form
// of the rotation for every caller: rotation_short's other roundings add up over
// the sweeps in the phases of the eigenvectors (1e-12 apart at n = 90, 1e-7 at
// 300, both equally good eigenvectors).
__global__ __launch_bounds__(512) void bj_inner_kernel(const double2* __restrict__ a, int n,
                                                       int nbp, int r,
                                                       double2* __restrict__ q_out,
                                                       int64_t a_stride, int64_t q_stride) {
    const int64_t bz = blockIdx.z;
    a += bz * a_stride;
    q_out += bz * q_stride + static_cast<int64_t>(blockIdx.x) * kBP * kBP;
    const int bp = rr_index(blockIdx.x, r, nbp), bq = rr_index(nbp - 1 - blockIdx.x, r, nbp);
    __shared__ double2 sm[kBP][kBP + 1];
    __shared__ double2 qm[kBP][kBP + 1];
    __shared__ double rc[2][kBP / 2];
    __shared__ double2 rs[2][kBP / 2];
    for (int e = threadIdx.x; e < kBP * kBP; e += 512) {
        const int i = e / kBP, j = e % kBP;
        const int gi = bj_row(i, bp, bq), gj = bj_row(j, bp, bq);
        sm[i][j] = gi < n && gj < n ? a[static_cast<int64_t>(gi) * n + gj] : make_double2(0.0, 0.0);
        qm[i][j] = make_double2(i == j ? 1.0 : 0.0, 0.0);
    }
    __syncthreads();
    const int t = threadIdx.x & 255, k1 = t / (kBP / 2), k2 = t % (kBP / 2);
    const bool on_s = threadIdx.x < 256;
    auto rotations = [&](int r2) {  // lanes 0 to 15 of wave 0
        if (threadIdx.x >= kBP / 2) return;
        int p, q;
        rr_pair(t, r2, kBP, p, q);
        const Rot ro = rotation_of(sm[p][p].x, sm[q][q].x, sm[p][q]);
        rc[r2 & 1][t] = ro.c;
        rs[r2 & 1][t] = ro.s;
    };
    rotations(0);
    __syncthreads();
    for (int r2 = 0; r2 < kBP - 1; ++r2) {
        int p2, q2;
        rr_pair(k2, r2, kBP, p2, q2);
        const double c2 = rc[r2 & 1][k2];
        const double2 s2 = rs[r2 & 1][k2], s2c = make_double2(s2.x, -s2.y);
        // right: [x_p, x_q] <- [c x_p - conj(S) x_q, S x_p + c x_q]
        auto right = [&](double2 xp, double2 xq, double2& op, double2& oq) {
            const double2 u = cmul(s2c, xq), w = cmul(s2, xp);
            op = make_double2(c2 * xp.x - u.x, c2 * xp.y - u.y);
            oq = make_double2(w.x + c2 * xq.x, w.y + c2 * xq.y);
        };
        if (on_s) {
            int p1, q1;
            rr_pair(k1, r2, kBP, p1, q1);
            const double c1 = rc[r2 & 1][k1];
            const double2 s1 = rs[r2 & 1][k1], s1c = make_double2(s1.x, -s1.y);
            // left: rows p' = c row_p - S row_q, q' = conj(S) row_p + c row_q
            auto left = [&](double2 xp, double2 xq, double2& op, double2& oq) {
                const double2 u = cmul(s1, xq), w = cmul(s1c, xp);
                op = make_double2(c1 * xp.x - u.x, c1 * xp.y - u.y);
                oq = make_double2(w.x + c1 * xq.x, w.y + c1 * xq.y);
            };
            double2 bpp, bpq, bqp, bqq, cpp, cpq, cqp, cqq;
            right(sm[p1][p2], sm[p1][q2], bpp, bpq);
            right(sm[q1][p2], sm[q1][q2], bqp, bqq);
            left(bpp, bqp, cpp, cqp);
            left(bpq, bqq, cpq, cqq);
            if (k1 == k2) {  // the rotated pair: exact zeros off the diagonal, real diagonal
                cpq = cqp = make_double2(0.0, 0.0);
                cpp.y = 0.0;
                cqq.y = 0.0;
            }
            sm[p1][p2] = cpp;
            sm[p1][q2] = cpq;
            sm[q1][p2] = cqp;
            sm[q1][q2] = cqq;
        }
        __syncthreads();
        if (on_s) {
            if (r2 + 1 < kBP - 1) rotations(r2 + 1);
        } else {
            // Q <- Q J on rows k1 and k1 + 16, columns (p2, q2)
            for (int h = 0; h < 2; ++h) {
                const int i = k1 + h * (kBP / 2);
                double2 op, oq;
                right(qm[i][p2], qm[i][q2], op, oq);
                qm[i][p2] = op;
                qm[i][q2] = oq;
            }
        }
        __syncthreads();
    }
    for (int e = threadIdx.x; e < kBP * kBP; e += 512) q_out[e] = qm[e / kBP][e % kBP];
}

// Workgroups [0, na): tiles (k, l), k <= l, of A, numbered row by row of the
// upper triangle of pairs; [na, na + ceil(n / 32) * npair): tiles (row chunk,
// pair l) of V.  Each thread owns a 2 x 2 block of the 32 x 32 tile.
__global__ __launch_bounds__(256) void bj_update_kernel(double2* __restrict__ a,
                                                        double2* __restrict__ v, int n, int nbp,
                                                        int r, const double2* __restrict__ qs,
                                                        int64_t a_stride, int64_t q_stride,
                                                        int na) {
    const int64_t bz = blockIdx.z;
    a += bz * a_stride;
    v += bz * a_stride;
    qs += bz * q_stride;
    const int npair = nbp / 2;
    __shared__ double2 xm[kBP][kBP + 1];
    __shared__ double2 ym[kBP][kBP + 1];
    __shared__ double2 qk[kBP][kBP + 1];
    __shared__ double2 ql[kBP][kBP + 1];
    const int t = threadIdx.x;
    const int i0 = 2 * (t / (kBP / 2)), j0 = 2 * (t % (kBP / 2));
    const double2 zero = make_double2(0.0, 0.0);
    // (x q_l)[i0.., j0..]
    auto mul_right = [&]() {
        const double2 z = make_double2(0.0, 0.0);
        Quad acc{z, z, z, z};
#pragma unroll 4
        for (int c = 0; c < kBP; ++c) {
            const double2 x0 = xm[i0][c], x1 = xm[i0 + 1][c];
            const double2 b0 = ql[c][j0], b1 = ql[c][j0 + 1];
            acc.a00 = cfma(x0, b0, acc.a00);
            acc.a01 = cfma(x0, b1, acc.a01);
            acc.a10 = cfma(x1, b0, acc.a10);
            acc.a11 = cfma(x1, b1, acc.a11);
        }
        return acc;
    };
    int blk = blockIdx.x;
    if (blk < na) {
        int k = 0;
        while (blk >= npair - k) {
            blk -= npair - k;
            ++k;
        }
        const int l = k + blk;
        const int bpk = rr_index(k, r, nbp), bqk = rr_index(nbp - 1 - k, r, nbp);
        const int bpl = rr_index(l, r, nbp), bql = rr_index(nbp - 1 - l, r, nbp);
        for (int e = t; e < kBP * kBP; e += 256) {
            const int i = e / kBP, j = e % kBP;
            const int gi = bj_row(i, bpk, bqk), gj = bj_row(j, bpl, bql);
            xm[i][j] = gi < n && gj < n ? a[static_cast<int64_t>(gi) * n + gj] : make_double2(0.0, 0.0);
            qk[i][j] = qs[static_cast<int64_t>(k) * kBP * kBP + e];
            ql[i][j] = qs[static_cast<int64_t>(l) * kBP * kBP + e];
        }
        __syncthreads();
        const Quad y = mul_right();
        ym[i0][j0] = y.a00;
        ym[i0][j0 + 1] = y.a01;
        ym[i0 + 1][j0] = y.a10;
        ym[i0 + 1][j0 + 1] = y.a11;
        __syncthreads();
        // T = q_k^H y
        Quad tt{zero, zero, zero, zero};
#pragma unroll 4
        for (int c = 0; c < kBP; ++c) {
            const double2 h0 = qk[c][i0], h1 = qk[c][i0 + 1];
            const double2 y0 = ym[c][j0], y1 = ym[c][j0 + 1];
            tt.a00 = cfma_conj_a(h0, y0, tt.a00);
            tt.a01 = cfma_conj_a(h0, y1, tt.a01);
            tt.a10 = cfma_conj_a(h1, y0, tt.a10);
            tt.a11 = cfma_conj_a(h1, y1, tt.a11);
        }
        // xm is free (every thread has read it in mul_right before the barrier)
        xm[i0][j0] = tt.a00;
        xm[i0][j0 + 1] = tt.a01;
        xm[i0 + 1][j0] = tt.a10;
        xm[i0 + 1][j0 + 1] = tt.a11;
        __syncthreads();
        for (int e = t; e < kBP * kBP; e += 256) {
            const int i = e / kBP, j = e % kBP;
            if (k == l) {  // Hermitian part of the diagonal tile
                const int gi = bj_row(i, bpk, bqk), gj = bj_row(j, bpk, bqk);
                if (gi < n && gj < n) {
                    const double2 x = xm[i][j], y = xm[j][i];
                    a[static_cast<int64_t>(gi) * n + gj] =
                        make_double2(0.5 * (x.x + y.x), i == j ? 0.0 : 0.5 * (x.y - y.y));
                }
            } else {
                const int gi = bj_row(i, bpk, bqk), gj = bj_row(j, bpl, bql);
                if (gi < n && gj < n) a[static_cast<int64_t>(gi) * n + gj] = xm[i][j];
                // row i of the mirrored tile: rows I_l u J_l, columns I_k u J_k
                const int hi = bj_row(i, bpl, bql), hj = bj_row(j, bpk, bqk);
                if (hi < n && hj < n) {
                    const double2 x = xm[j][i];
                    a[static_cast<int64_t>(hi) * n + hj] = make_double2(x.x, -x.y);
                }
            }
        }
        return;
    }
    blk -= na;
    const int chunk = blk / npair, l = blk % npair;
    const int bpl = rr_index(l, r, nbp), bql = rr_index(nbp - 1 - l, r, nbp);
    const int row0 = chunk * kBP;
    for (int e = t; e < kBP * kBP; e += 256) {
        const int i = e / kBP, j = e % kBP;
        const int gj = bj_row(j, bpl, bql);
        xm[i][j] = row0 + i < n && gj < n ? v[static_cast<int64_t>(row0 + i) * n + gj] : make_double2(0.0, 0.0);
        ql[i][j] = qs[static_cast<int64_t>(l) * kBP * kBP + e];
    }
    __syncthreads();
    const Quad y = mul_right();
    const double2 out[4] = {y.a00, y.a01, y.a10, y.a11};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int gi = row0 + i0 + e / 2, gj = bj_row(j0 + e % 2, bpl, bql);
        if (gi < n && gj < n) v[static_cast<int64_t>(gi) * n + gj] = out[e];
    }
}

__global__ __launch_bounds__(256) void eye_kernel(double2* __restrict__ v, int n, int64_t stride) {
    const int64_t bz = blockIdx.z;
    const int64_t nn = static_cast<int64_t>(n) * n;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < nn;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        v[bz * stride + i] = make_double2(i / n == i % n ? 1.0 : 0.0, 0.0);
}

// Partial sums of (off-diagonal |a|^2, all |a|^2) per workgroup, then one
// workgroup adds the partials: out[2*b], out[2*b + 1] per batch entry b.
constexpr int kRedBlocks = 256;

__global__ __launch_bounds__(256) void offnorm_partial_kernel(const double2* __restrict__ a,
                                                              int n, int64_t stride,
                                                              double* __restrict__ part) {
    const int64_t bz = blockIdx.z;
    const int64_t nn = static_cast<int64_t>(n) * n;
    double off = 0.0, all = 0.0;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < nn;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const double2 x = a[bz * stride + i];
        const double m2 = x.x * x.x + x.y * x.y;
        all += m2;
        if (i / n != i % n) off += m2;
    }
    __shared__ double s_off[256], s_all[256];
    s_off[threadIdx.x] = off;
    s_all[threadIdx.x] = all;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            s_off[threadIdx.x] += s_off[threadIdx.x + w];
            s_all[threadIdx.x] += s_all[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[(bz * kRedBlocks + blockIdx.x) * 2] = s_off[0];
        part[(bz * kRedBlocks + blockIdx.x) * 2 + 1] = s_all[0];
    }
}

__global__ __launch_bounds__(256) void offnorm_final_kernel(const double* __restrict__ part,
                                                            double* __restrict__ out) {
    const int64_t bz = blockIdx.x;
    __shared__ double s_off[256], s_all[256];
    s_off[threadIdx.x] = part[(bz * kRedBlocks + threadIdx.x) * 2];
    s_all[threadIdx.x] = part[(bz * kRedBlocks + threadIdx.x) * 2 + 1];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            s_off[threadIdx.x] += s_off[threadIdx.x + w];
            s_all[threadIdx.x] += s_all[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[2 * bz] = s_off[0];
        out[2 * bz + 1] = s_all[0];
    }
}

__global__ __launch_bounds__(256) void gather_cols_batched_kernel(
    const double2* __restrict__ in, double2* __restrict__ out, int rows, int n_in, int n_out,
    const int* __restrict__ perm) {
    const int64_t bz = blockIdx.z;
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= static_cast<int64_t>(rows) * n_out) return;
    const int64_t i = t / n_out;
    const int j = static_cast<int>(t % n_out);
    out[bz * rows * n_out + t] = in[bz * rows * n_in + i * n_in + perm[bz * n_out + j]];
}

}  // namespace

void launch_gather_cols(const double2* in, double2* out, int rows, int n_in, int n_out,
                        const int* perm, int batch, hipStream_t s) {
    const int64_t n = static_cast<int64_t>(rows) * n_out;
    if (n <= 0 || batch <= 0) return;
    hipLaunchKernelGGL(gather_cols_batched_kernel,
                       dim3(static_cast<unsigned>(ceil_div64(n, 256)), 1, batch), dim3(256), 0, s,
                       in, out, rows, n_in, n_out, perm);
    GW_HIP_TRY(hipGetLastError());
}

void launch_zgemm(ZOp opa, ZOp opb, const ZGemm& g, hipStream_t s) {
    if (g.m <= 0 || g.n <= 0 || g.batch <= 0) return;
    switch (opa * 3 + opb) {
        case 0: zgemm_launch<kOpN, kOpN>(g, s); break;
        case 1: zgemm_launch<kOpN, kOpT>(g, s); break;
        case 2: zgemm_launch<kOpN, kOpC>(g, s); break;
        case 3: zgemm_launch<kOpT, kOpN>(g, s); break;
        case 4: zgemm_launch<kOpT, kOpT>(g, s); break;
        case 5: zgemm_launch<kOpT, kOpC>(g, s); break;
        case 6: zgemm_launch<kOpC, kOpN>(g, s); break;
        case 7: zgemm_launch<kOpC, kOpT>(g, s); break;
        default: zgemm_launch<kOpC, kOpC>(g, s); break;
    }
}

void launch_zaxpby(int64_t n, double2 a, const double2* x, double2 b, const double2* y,
                   double2* z, hipStream_t s) {
    if (n <= 0) return;
    const int64_t blocks = std::min<int64_t>(ceil_div64(n, 256), 8192);
    hipLaunchKernelGGL(zaxpby_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, n, a,
                       x, b, y, z);
    GW_HIP_TRY(hipGetLastError());
}

void launch_diag_re(const double2* a, int n, int batch, double* out, hipStream_t s) {
    if (n <= 0 || batch <= 0) return;
    hipLaunchKernelGGL(diag_re_kernel, dim3(ceil_div(n, 256), batch), dim3(256), 0, s, a, n, out);
    GW_HIP_TRY(hipGetLastError());
}

void launch_scale_rows(const double2* in, double2* out, const double* w, int64_t rows,
                       int64_t cols, hipStream_t s) {
    const int64_t n = rows * cols;
    if (n <= 0) return;
    const int64_t blocks = std::min<int64_t>(ceil_div64(n, 256), 8192);
    hipLaunchKernelGGL(scale_rows_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s,
                       in, out, w, n, cols);
    GW_HIP_TRY(hipGetLastError());
}

size_t chol_work_bytes(int n) {
    auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
    // x (kCB x kCB), panel t (kCB x n), column block u (n x kCB), gmax
    return al(sizeof(double2) * kCB * kCB) + 2 * al(sizeof(double2) * kCB * static_cast<size_t>(n)) + 256;
}

void chol_inverse(double2* g, double2* rinv, int n, void* work, hipStream_t s) {
    if (n <= 0) return;
    auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
    char* w = static_cast<char*>(work);
    double2* x = reinterpret_cast<double2*>(w);
    double2* t = reinterpret_cast<double2*>(w + al(sizeof(double2) * kCB * kCB));
    double2* u = reinterpret_cast<double2*>(w + al(sizeof(double2) * kCB * kCB) +
                                            al(sizeof(double2) * kCB * static_cast<size_t>(n)));
    double* gmax = reinterpret_cast<double*>(w + al(sizeof(double2) * kCB * kCB) +
                                             2 * al(sizeof(double2) * kCB * static_cast<size_t>(n)));
    const int64_t nn = static_cast<int64_t>(n) * n;
    hipLaunchKernelGGL(zero_fill_kernel, dim3(static_cast<unsigned>(std::min<int64_t>(ceil_div64(nn, 256), 4096))),
                       dim3(256), 0, s, rinv, nn);
    hipLaunchKernelGGL(diag_max_kernel, dim3(1), dim3(256), 0, s, g, n, gmax);
    GW_HIP_TRY(hipGetLastError());
    const double2 one = make_double2(1.0, 0.0), mone = make_double2(-1.0, 0.0);
    for (int k0 = 0; k0 < n; k0 += kCB) {
        const int kb = std::min(kCB, n - k0), rest = n - k0 - kb;
        hipLaunchKernelGGL(chol_block_kernel, dim3(1), dim3(256), 0, s, g, n, k0, kb, gmax, x);
        GW_HIP_TRY(hipGetLastError());
        if (rest > 0) {
            // panel of R: T = X^H g[K][K+], then g[K][K+] = T
            ZGemm p;
            p.m = kb;
            p.n = rest;
            p.k = kb;
            p.a = x;
            p.lda = kCB;
            p.b = g + static_cast<int64_t>(k0) * n + k0 + kb;
            p.ldb = n;
            p.c = t;
            p.ldc = n;
            launch_zgemm(kOpC, kOpN, p, s);
            hipLaunchKernelGGL(copy_block_kernel, dim3(static_cast<unsigned>(ceil_div64(static_cast<int64_t>(kb) * rest, 256))),
                               dim3(256), 0, s, t, static_cast<int64_t>(n),
                               g + static_cast<int64_t>(k0) * n + k0 + kb, static_cast<int64_t>(n), kb, rest);
            GW_HIP_TRY(hipGetLastError());
            // trailing update g[K+][K+] -= T^H T
            ZGemm q;
            q.m = rest;
            q.n = rest;
            q.k = kb;
            q.a = t;
            q.lda = n;
            q.b = t;
            q.ldb = n;
            q.c = g + static_cast<int64_t>(k0 + kb) * n + k0 + kb;
            q.ldc = n;
            q.alpha = mone;
            q.beta = one;
            launch_zgemm(kOpC, kOpN, q, s);
        }
        // R^-1 column block K: diagonal block X, above it -R^-1[<K][<K] R[<K][K] X
        hipLaunchKernelGGL(copy_block_kernel, dim3(static_cast<unsigned>(ceil_div64(static_cast<int64_t>(kb) * kb, 256))),
                           dim3(256), 0, s, x, static_cast<int64_t>(kCB),
                           rinv + static_cast<int64_t>(k0) * n + k0, static_cast<int64_t>(n), kb, kb);
        GW_HIP_TRY(hipGetLastError());
        if (k0 > 0) {
            ZGemm a;  // U = R^-1[<K][<K] R[<K][K]
            a.m = k0;
            a.n = kb;
            a.k = k0;
            a.a = rinv;
            a.lda = n;
            a.b = g + k0;
            a.ldb = n;
            a.c = u;
            a.ldc = kCB;
            launch_zgemm(kOpN, kOpN, a, s);
            ZGemm b;  // R^-1[<K][K] = -U X
            b.m = k0;
            b.n = kb;
            b.k = kb;
            b.a = u;
            b.lda = kCB;
            b.b = x;
            b.ldb = kCB;
            b.c = rinv + k0;
            b.ldc = n;
            b.alpha = mone;
            launch_zgemm(kOpN, kOpN, b, s);
        }
    }
}

size_t jacobi_work_bytes(int n, int batch) {
    // reduction partials and the two results per entry
    const size_t red = static_cast<size_t>(batch) * kRedBlocks * 2 * 8 +
                       static_cast<size_t>(batch) * 2 * 8 + 512;
    if (n >= kBJMin) {  // one Q per pair of blocks
        const int nblk = ceil_div(n, kBJ), nbp = nblk + (nblk & 1);
        const size_t qb = static_cast<size_t>(nbp / 2) * kBP * kBP * sizeof(double2) * batch;
        return ((qb + 255) & ~size_t(255)) + red;
    }
    return (static_cast<size_t>(batch) * sizeof(double) + 255) & ~size_t(255);  // sweep counts
}

int jacobi_eigh(double2* a, double2* v, int n, int batch, double tol, int max_sweeps, void* work,
                hipStream_t s, bool same_bits) {
    if (n <= 0 || batch <= 0) return 0;
    if (n < kBJMin) {
        double* count = static_cast<double*>(work);
        const size_t lds = 2 * static_cast<size_t>(n) * (n | 1) * sizeof(double2);
        // one thread per 2 x 2 block of A: 512 up to n = 44, 1,024 above
        const int half = (n + 1) / 2, nt = half * half <= 512 ? 512 : 1024;
        const auto kernel = nt == 512 ? (same_bits ? jacobi_lds_kernel<false, 512> : jacobi_lds_kernel<true, 512>)
                                      : (same_bits ? jacobi_lds_kernel<false, 1024> : jacobi_lds_kernel<true, 1024>);
        GW_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       static_cast<int>(lds)));
        {
            ProfScope ps("jacobi_sweep", s);
            hipLaunchKernelGGL(kernel, dim3(batch), dim3(nt), lds, s, a, v, n, tol, max_sweeps, count);
            GW_HIP_TRY(hipGetLastError());
        }
        std::vector<double> h(batch);
        GW_HIP_TRY(hipMemcpyAsync(h.data(), count, h.size() * sizeof(double), hipMemcpyDeviceToHost, s));
        GW_HIP_TRY(hipStreamSynchronize(s));
        return static_cast<int>(*std::max_element(h.begin(), h.end()));
    }
    const int64_t nn = static_cast<int64_t>(n) * n;
    const int nblk = ceil_div(n, kBJ), nbp = nblk + (nblk & 1), npair = nbp / 2;
    const int64_t q_stride = static_cast<int64_t>(npair) * kBP * kBP;
    const size_t first = (static_cast<size_t>(q_stride) * batch * sizeof(double2) + 255) & ~size_t(255);
    char* w = static_cast<char*>(work);
    double* part = reinterpret_cast<double*>(w + first);
    double* res = part + static_cast<size_t>(batch) * kRedBlocks * 2;
    const unsigned eb = static_cast<unsigned>(std::min<int64_t>(ceil_div64(nn, 256), 4096));
    hipLaunchKernelGGL(eye_kernel, dim3(eb, 1, batch), dim3(256), 0, s, v, n, nn);
    GW_HIP_TRY(hipGetLastError());
    // block sweeps: in place, Q's in the work area
    double2* qs = reinterpret_cast<double2*>(w);
    const int na_bl = npair * (npair + 1) / 2;
    const int nv_bl = ceil_div(n, kBP) * npair;
    std::vector<double> h(2 * static_cast<size_t>(batch));
    std::vector<double> prev(batch, -1.0);
    int sweeps = 0;
    for (; sweeps < max_sweeps; ++sweeps) {
        hipLaunchKernelGGL(offnorm_partial_kernel, dim3(kRedBlocks, 1, batch), dim3(256), 0, s, a,
                           n, nn, part);
        hipLaunchKernelGGL(offnorm_final_kernel, dim3(batch), dim3(256), 0, s, part, res);
        GW_HIP_TRY(hipGetLastError());
        GW_HIP_TRY(hipMemcpyAsync(h.data(), res, h.size() * sizeof(double), hipMemcpyDeviceToHost, s));
        GW_HIP_TRY(hipStreamSynchronize(s));
        // done when the off-diagonal norm is below tol of the norm, or when it
        // has stopped falling (the convergence is quadratic until rounding
        // re-creates off-diagonal entries at the level of the unit roundoff)
        bool done = true;
        for (int b = 0; b < batch; ++b) {
            const double off = std::sqrt(h[2 * b]), all = std::sqrt(h[2 * b + 1]);
            const bool small = off <= tol * all;
            const bool stalled = sweeps >= 3 && prev[b] >= 0.0 && off >= 0.25 * prev[b] &&
                                 off <= 1e-12 * all;
            if (!small && !stalled) done = false;
            prev[b] = off;
        }
        if (done) break;
        ProfScope ps("jacobi_sweep", s);
        for (int r = 0; r < nbp - 1; ++r) {
            hipLaunchKernelGGL(bj_inner_kernel, dim3(npair, 1, batch), dim3(512), 0, s, a, n, nbp, r,
                               qs, nn, q_stride);
            hipLaunchKernelGGL(bj_update_kernel, dim3(na_bl + nv_bl, 1, batch), dim3(256), 0, s, a,
                               v, n, nbp, r, qs, nn, q_stride, na_bl);
        }
        GW_HIP_TRY(hipGetLastError());
    }
    return sweeps;
}

}  // namespace gw

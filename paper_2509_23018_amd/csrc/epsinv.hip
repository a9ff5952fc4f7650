// Inverse dielectric matrix of Eq. (3): eps^-1(z) = [I - v chi(z)]^-1, v the
// diagonal Coulomb matrix, for every frequency, on the device.
//
// eps = I - v chi is built in the output buffer and inverted there by block
// Gauss-Jordan elimination without pivoting, 512 columns at a time (at most
// N_G rounded up to 64).  For the block K of columns/rows:
//   D^-1   the inverse of the diagonal block A[K,K]: a copy of the block
//          inverted by the same elimination 64 columns at a time, whose
//          64 x 64 pivot blocks are inverted by one workgroup in registers
//          (scalar Gauss-Jordan);
//   L      = A[:, K] with its K rows zeroed (saved), then A[not K, K] = 0;
//   R      = D^-1 A[K, :], with R[:, K] = D^-1, written back as A[K, :];
//   A     -= L R  (one GEMM of N_G x 512 x N_G on FP64 MFMA: 64 flops per
//          byte of A read and written, against 16 at 64 columns).
// After the last block A holds eps^-1.  Without pivoting the elimination
// needs nonsingular leading blocks: eps = v^1/2 eps~ v^-1/2 with
// eps~ = I - v^1/2 chi v^1/2 Hermitian positive definite (eigenvalues >= 1)
// whenever chi is Hermitian negative semidefinite (zero and imaginary
// frequencies), so there every pivot block is well conditioned; on the real
// axis eps is not guaranteed to be.
#include <algorithm>

#include "common.hpp"
#include "epsinv.hpp"
#include "linalg.hpp"
#include "prof.hpp"

namespace gw {
namespace {

constexpr int kB = 64;   // width of the pivot blocks inverted by one workgroup
constexpr int kW = 512;  // width of the elimination's blocks

// out[w] = I - diag(v) chi[w]
__global__ __launch_bounds__(256) void build_eps_kernel(const double2* __restrict__ chi,
                                                        const double* __restrict__ v, int ng,
                                                        double2* __restrict__ out) {
    const int64_t w = blockIdx.z;
    const int64_t nn = static_cast<int64_t>(ng) * ng;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; t < nn;
         t += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int i = static_cast<int>(t / ng), j = static_cast<int>(t % ng);
        const double2 c = chi[w * nn + t];
        out[w * nn + t] = make_double2((i == j ? 1.0 : 0.0) - v[i] * c.x, -v[i] * c.y);
    }
}

// Matrices below are row-major n x n with leading dimension n, matrix w of the
// batch at a + w * sa.

__device__ __forceinline__ double2 crecip(double2 a) {  // 1 / a
    const double den = a.x * a.x + a.y * a.y;
    return make_double2(a.x / den, -a.y / den);
}
// a - b c, a rounded once (as a chain of FMAs onto a it would be twice)
__device__ __forceinline__ double2 csub_mul(double2 a, double2 b, double2 c) {
    const double2 v = cmul(b, c);
    return make_double2(a.x - v.x, a.y - v.y);
}

// Workgroup 0 of matrix w: d[w] = A[w][K,K]^-1 for the bk x bk block at
// (k0, k0) (bk <= 64), scalar Gauss-Jordan without pivoting; d[w] at d +
// w * kB * kB, leading dimension kB.  The others: L[w] = A[w][:, K] (rows in K
// zero), then A[w][i, K] = 0 for the rows i not in K, which workgroup 0 does
// not read; L[w] at l + w * n * kB, leading dimension kB.
//
// The inverse is a chain of bk dependent steps on one workgroup, so the latency
// of a step is the whole cost.  The block lives in registers (thread (ti, tj)
// holds rows ti + 16 r and columns tj + 16 c).  Two steps go together: the two
// pivot rows and columns pass through LDS as they stand, in two buffers, and
// every thread takes its own part of the second row and column through the first
// step itself, so that two steps cost one barrier and one round of LDS reads.
// A launch with a 64 x 64 block: 182 us with the block in LDS (four barriers and
// three passes over it per step), 44 us by single steps, 39 us by two.  35 us
// with FMAs straight onto the entry, which rounds it twice per step: the
// inverse's error grows by 10 to 70 %, not kept.  Two or four threads per 2 x 4
// or 2 x 2 entries, and forming only the next pivot's row and column before the
// barrier, did not help.
__global__ __launch_bounds__(256) void pivot_kernel(double2* __restrict__ a, int n, int64_t sa,
                                                    int k0, int bk, double2* __restrict__ d,
                                                    double2* __restrict__ l) {
    constexpr int R = kB / 16;
    __shared__ double2 s_row[2][2][kB], s_col[2][2][kB];  // [buffer][step]
    const int64_t w = blockIdx.y;
    double2* aw = a + w * sa;
    if (blockIdx.x > 0) {
        const int64_t t = static_cast<int64_t>(blockIdx.x - 1) * 256 + threadIdx.x;
        if (t >= static_cast<int64_t>(n) * bk) return;
        const int i = static_cast<int>(t / bk), j = static_cast<int>(t % bk);
        const bool in_k = i >= k0 && i < k0 + bk;
        double2* src = aw + static_cast<int64_t>(i) * n + k0 + j;
        l[w * static_cast<int64_t>(n) * kB + static_cast<int64_t>(i) * kB + j] =
            in_k ? make_double2(0.0, 0.0) : *src;
        if (!in_k) *src = make_double2(0.0, 0.0);
        return;
    }
    const int ti = threadIdx.x >> 4, tj = threadIdx.x & 15;
    double2 x[R][R];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < R; ++c) {
            const int i = ti + 16 * r, j = tj + 16 * c;
            const bool in = i < bk && j < bk;
            const double2 v = aw[in ? static_cast<int64_t>(k0 + i) * n + k0 + j
                                    : static_cast<int64_t>(k0) * n + k0];
            // past the block the identity: the second step of an odd bk
            x[r][c] = make_double2(in ? v.x : i == j ? 1.0 : 0.0, in ? v.y : 0.0);
        }
#pragma unroll
    for (int pr = 0; pr < R; ++pr) {
#pragma unroll 1
        for (int pt = 0; pt < 16; pt += 2) {
            const int p = 16 * pr + pt, buf = (pt >> 1) & 1;
            if (p >= bk) break;
            if ((tj & ~1) == pt)
#pragma unroll
                for (int r = 0; r < R; ++r) s_col[buf][tj & 1][ti + 16 * r] = x[r][pr];
            if ((ti & ~1) == pt)
#pragma unroll
                for (int c = 0; c < R; ++c) s_row[buf][ti & 1][tj + 16 * c] = x[pr][c];
            __syncthreads();
            // a step: row p scaled, its pivot 1 / pivot; a_ij -= a_ip a_pj for the
            // other rows (column p: 0 - a_ip / pivot).  r1, r2: the scaled rows.
            const double2 inv1 = crecip(s_row[buf][0][p]);
            const double2 f = s_row[buf][1][p];  // a_{p+1,p}
            const double2 h = cmul(inv1, s_row[buf][0][p + 1]);  // r1 in column p + 1
            const double2 inv2 = crecip(csub_mul(s_row[buf][1][p + 1], f, h));
            double2 r1[R], r2[R];
#pragma unroll
            for (int c = 0; c < R; ++c) {
                const int j = tj + 16 * c;
                r1[c] = cmul(inv1, s_row[buf][0][j]);
                r2[c] = s_row[buf][1][j];
            }
            if (tj == pt) {
                r1[pr] = inv1;
                r2[pr] = make_double2(0.0, 0.0);
            }
#pragma unroll
            for (int c = 0; c < R; ++c) r2[c] = cmul(inv2, csub_mul(r2[c], f, r1[c]));
            if (tj == pt + 1) {
                r1[pr] = make_double2(0.0, 0.0);
                r2[pr] = inv2;
            }
            if ((tj & ~1) == pt)  // columns p and p + 1 start from zero
#pragma unroll
                for (int r = 0; r < R; ++r) x[r][pr] = make_double2(0.0, 0.0);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const double2 c1 = s_col[buf][0][ti + 16 * r];
                const double2 c2 = csub_mul(s_col[buf][1][ti + 16 * r], c1, h);
#pragma unroll
                for (int c = 0; c < R; ++c)
                    x[r][c] = csub_mul(csub_mul(x[r][c], c1, r1[c]), c2, r2[c]);
            }
            if ((ti & ~1) == pt)
#pragma unroll
                for (int c = 0; c < R; ++c)
                    x[pr][c] = ti == pt ? csub_mul(r1[c], h, r2[c]) : r2[c];
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < R; ++c) {
            const int i = ti + 16 * r, j = tj + 16 * c;
            if (i < bk && j < bk) d[w * kB * kB + i * kB + j] = x[r][c];
        }
}

// R[w] = D^-1 A[w][K, :] with R[w][:, K] = D^-1, to r + w * kB * n (leading
// dimension n) and back into A[w][K, :], for blocks of at most 64 rows: one
// workgroup per 16 columns, 4 waves of 16 x 16, three real MFMA products per
// complex one.  Both operands fit LDS whole, so it is one load, one barrier
// and 16 k-steps; the columns are read before they are overwritten.  On the
// chain of an inverse, where each launch costs its latency (64 of these for
// 2,007 G): 9 us at n = 512 against 5 + 5 us as a GEMM and a copy; 7 us with
// the choices past the edges made between values (no flat loads).
__global__ __launch_bounds__(256) void pivot_rows_kernel(double2* __restrict__ a, int n, int64_t sa,
                                                         int k0, int bk,
                                                         const double2* __restrict__ d,
                                                         double2* __restrict__ r) {
    __shared__ double2 s_d[kB][kB + 1];  // [m][k]
    __shared__ double2 s_a[kB][17];      // [k][n]
    const int64_t w = blockIdx.y;
    const int j0 = blockIdx.x * 16;
    double2* aw = a + w * sa + static_cast<int64_t>(k0) * n;
    double2 vd[16], va[4];  // every load in flight before the first is used
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = threadIdx.x + 256 * u, k = e / 16, j = j0 + e % 16;
        const bool in = k < bk && j < n;
        const double2 v = aw[in ? static_cast<int64_t>(k) * n + j : 0];
        va[u] = make_double2(in ? v.x : 0.0, in ? v.y : 0.0);
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int e = threadIdx.x + 256 * u, i = e / kB, k = e % kB;
        const bool in = i < bk && k < bk;
        const double2 v = d[w * kB * kB + (in ? e : 0)];
        vd[u] = make_double2(in ? v.x : 0.0, in ? v.y : 0.0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = threadIdx.x + 256 * u;
        s_a[e / 16][e % 16] = va[u];
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int e = threadIdx.x + 256 * u;
        s_d[e / kB][e % kB] = vd[u];
    }
    __syncthreads();
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, row = lane & 15, kq = lane >> 4;
    dbl4 p1 = zero4(), p2 = zero4(), p3 = zero4();
#pragma unroll
    for (int k = 0; k < kB; k += 4) {
        const double2 b = s_a[k + kq][row], v = s_d[wave * 16 + row][k + kq];
        p1 = mfma_f64(v.x, b.x, p1);
        p2 = mfma_f64(v.y, b.y, p2);
        p3 = mfma_f64(v.x + v.y, b.x + b.y, p3);
    }
    const int j = j0 + row;
    const bool in_k = j >= k0 && j < k0 + bk;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int i = wave * 16 + 4 * t + kq;
        if (i >= bk || j >= n) continue;
        const double2 v = in_k ? s_d[i][j - k0]
                               : make_double2(p1[t] - p2[t], p3[t] - p1[t] - p2[t]);
        r[w * static_cast<int64_t>(kB) * n + static_cast<int64_t>(i) * n + j] = v;
        aw[static_cast<int64_t>(i) * n + j] = v;
    }
}

// L[w] = A[w][:, K] (rows in K zeroed), then A[w][i, K] = 0 for rows i not in
// K; L[w] at l + w * n * kb, leading dimension kb
__global__ __launch_bounds__(256) void take_panel_kernel(double2* __restrict__ a, int n,
                                                         int64_t sa, int k0, int bk, int kb,
                                                         double2* __restrict__ l) {
    const int64_t w = blockIdx.z;
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= static_cast<int64_t>(n) * bk) return;
    const int i = static_cast<int>(t / bk), j = static_cast<int>(t % bk);
    double2* src = a + w * sa + static_cast<int64_t>(i) * n + k0 + j;
    const bool in_k = i >= k0 && i < k0 + bk;
    l[w * static_cast<int64_t>(n) * kb + static_cast<int64_t>(i) * kb + j] =
        in_k ? make_double2(0.0, 0.0) : *src;
    if (!in_k) *src = make_double2(0.0, 0.0);
}

// R[w][:, K] = D^-1, then A[w][K, :] = R[w]; R[w] at r + w * kb * n (leading
// dimension n), D^-1 of w at d + w * sd (leading dimension ldd)
__global__ __launch_bounds__(256) void put_rows_kernel(double2* __restrict__ a, int n, int64_t sa,
                                                       int k0, int bk, int kb,
                                                       double2* __restrict__ r,
                                                       const double2* __restrict__ d, int64_t sd,
                                                       int ldd) {
    const int64_t w = blockIdx.z;
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= static_cast<int64_t>(bk) * n) return;
    const int i = static_cast<int>(t / n), j = static_cast<int>(t % n);
    double2* rr = r + w * static_cast<int64_t>(kb) * n + static_cast<int64_t>(i) * n + j;
    double2 x = *rr;
    if (j >= k0 && j < k0 + bk) {
        x = d[w * sd + static_cast<int64_t>(i) * ldd + (j - k0)];
        *rr = x;
    }
    a[w * sa + static_cast<int64_t>(k0 + i) * n + j] = x;
}

// D[w] = A[w][K, K] (bk x bk, leading dimension bk, at d + w * sd)
__global__ __launch_bounds__(256) void copy_pivot_kernel(const double2* __restrict__ a, int n,
                                                         int64_t sa, int k0, int bk,
                                                         double2* __restrict__ d, int64_t sd) {
    const int64_t w = blockIdx.z;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= bk * bk) return;
    const int i = t / bk, j = t % bk;
    d[w * sd + t] = a[w * sa + static_cast<int64_t>(k0 + i) * n + k0 + j];
}

size_t al256(size_t b) { return (b + 255) & ~size_t(255); }

// scratch of one gj_invert level with blocks of width kb on n x n matrices
size_t level_bytes(int n, int nz, int kb) {
    const size_t p = static_cast<size_t>(nz) * n * kb * sizeof(double2);
    const size_t d = static_cast<size_t>(nz) * kb * kb * sizeof(double2);
    return al256(d) + 2 * al256(p);
}

// In-place Gauss-Jordan inversion of nz matrices (n x n, batch stride sa),
// blocks of width kb: 64 (pivot blocks inverted by one workgroup) or more
// (pivot blocks copied and inverted by this routine at width 64).
void gj_invert(double2* a, int n, int64_t sa, int nz, int kb, char* ws, hipStream_t s) {
    double2* d = reinterpret_cast<double2*>(ws);
    double2* l = reinterpret_cast<double2*>(ws + al256(static_cast<size_t>(nz) * kb * kb * 16));
    double2* r = reinterpret_cast<double2*>(ws + al256(static_cast<size_t>(nz) * kb * kb * 16) +
                                            al256(static_cast<size_t>(nz) * n * kb * 16));
    char* inner = ws + level_bytes(n, nz, kb);
    for (int k0 = 0; k0 < n; k0 += kb) {
        const int bk = std::min(kb, n - k0);
        if (kb == kB) {
            hipLaunchKernelGGL(pivot_kernel,
                               dim3(static_cast<unsigned>(1 + ceil_div64(static_cast<int64_t>(n) * bk, 256)), nz),
                               dim3(256), 0, s, a, n, sa, k0, bk, d, l);
            GW_HIP_TRY(hipGetLastError());
            hipLaunchKernelGGL(pivot_rows_kernel, dim3(static_cast<unsigned>(ceil_div(n, 16)), nz),
                               dim3(256), 0, s, a, n, sa, k0, bk, d, r);
            GW_HIP_TRY(hipGetLastError());
        } else {
            const int64_t sd = static_cast<int64_t>(kb) * kb;
            hipLaunchKernelGGL(copy_pivot_kernel, dim3(ceil_div(bk * bk, 256), 1, nz), dim3(256), 0,
                               s, a, n, sa, k0, bk, d, sd);
            GW_HIP_TRY(hipGetLastError());
            gj_invert(d, bk, sd, nz, kB, inner, s);
            hipLaunchKernelGGL(take_panel_kernel,
                               dim3(static_cast<unsigned>(ceil_div64(static_cast<int64_t>(n) * bk, 256)), 1, nz),
                               dim3(256), 0, s, a, n, sa, k0, bk, kb, l);
            GW_HIP_TRY(hipGetLastError());
            ZGemm g1;  // R = D^-1 A[K, :]
            g1.m = bk;
            g1.n = n;
            g1.k = bk;
            g1.a = d;
            g1.lda = bk;
            g1.stride_a = sd;
            g1.b = a + static_cast<int64_t>(k0) * n;
            g1.ldb = n;
            g1.stride_b = sa;
            g1.c = r;
            g1.ldc = n;
            g1.stride_c = static_cast<int64_t>(kb) * n;
            g1.batch = nz;
            launch_zgemm(kOpN, kOpN, g1, s);
            hipLaunchKernelGGL(put_rows_kernel,
                               dim3(static_cast<unsigned>(ceil_div64(static_cast<int64_t>(bk) * n, 256)), 1, nz),
                               dim3(256), 0, s, a, n, sa, k0, bk, kb, r, d, sd, bk);
            GW_HIP_TRY(hipGetLastError());
        }
        ZGemm g2;  // A -= L R
        g2.m = n;
        g2.n = n;
        g2.k = bk;
        g2.a = l;
        g2.lda = kb;
        g2.stride_a = static_cast<int64_t>(n) * kb;
        g2.b = r;
        g2.ldb = n;
        g2.stride_b = static_cast<int64_t>(kb) * n;
        g2.c = a;
        g2.ldc = n;
        g2.stride_c = sa;
        g2.alpha = make_double2(-1.0, 0.0);
        g2.beta = make_double2(1.0, 0.0);
        g2.batch = nz;
        launch_zgemm(kOpN, kOpN, g2, s);
    }
}

// the elimination's block width for N_G: kW, or N_G rounded up to kB if less
int block_width(int ng) { return std::min(kW, ceil_div(ng, kB) * kB); }

}  // namespace

size_t epsinv_bytes(int ng, int nz) {
    const int kb = block_width(ng);
    return level_bytes(ng, nz, kb) + (kb > kB ? level_bytes(kb, nz, kB) : 0);
}

void run_epsinv(const double2* chi, int ng, int nz, const double* v, double2* out, char* base,
                hipStream_t s) {
    if (ng <= 0 || nz <= 0) return;
    const int64_t nn = static_cast<int64_t>(ng) * ng;
    {
        ProfScope ps("eps_build", s);
        hipLaunchKernelGGL(build_eps_kernel,
                           dim3(static_cast<unsigned>(std::min<int64_t>(ceil_div64(nn, 256), 4096)), 1, nz),
                           dim3(256), 0, s, chi, v, ng, out);
        GW_HIP_TRY(hipGetLastError());
    }
    ProfScope ps("eps_invert", s);
    gj_invert(out, ng, nn, nz, block_width(ng), base, s);
}

}  // namespace gw

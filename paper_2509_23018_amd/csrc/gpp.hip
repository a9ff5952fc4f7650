// The GPP off-diagonal self-energy kernel (Optimized GPP Kernel for
// Off-Diagonal Self-Energy Matrix Elements section of the paper): the full
// matrix Sigma_lm(E) on a grid of energies,
//     Sigma_lm(E) = sum_n sum_GG' conj(M_ln(G)) P^{nE}_GG' M_mn(G'),
// as the paper casts it, two complex GEMMs per (band n, energy E):
//   T = conj(M_n) P^{nE}        (N_Sigma x N_G x N_G)
//   Sigma(E) += T M_n^T         (N_Sigma x N_G x N_Sigma).
// The plasmon-pole inner matrix is
//     P_GG' = Omega2_GG' v_G' / (2 wt_GG' (E - E_n - s_n wt_GG')),
// s_n = -1 (occupied) or +1 (empty).  Here it is never stored: the first
// GEMM forms each 16 x 64 stage of P from Omega2, wt and v as it writes the
// stage to LDS (a division per element), so P costs no HBM traffic.  Both
// GEMMs run over the pairs of many bands and all energies of a batch in one
// launch each.
#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "gpp.hpp"
#include "linalg.hpp"
#include "prof.hpp"

namespace gw {
namespace {

constexpr int kMaxBands = 64;  // bands of one launch

// The bands of one launch.
struct GppBands {
    double en[kMaxBands];
    uint64_t occupied;  // bit per band
};

// T[q][l][G'] = sum_G conj(M_n[l][G]) P_ne[G][G'] for the pairs q = (band n,
// energy e), e fastest: 16 BX (l) x 64 (G') tiles, 4 waves of 16 BX x 16 on the
// 16x16x4 FP64 MFMA, three real products per complex multiply-add.  G is
// staged 16 at a time through LDS, in two buffers, with the loads two stages
// ahead; the stage's P is formed as it is written to LDS, a stage before its
// use, between the MFMAs of the stage before.
//
// Bound by the FP64 pipes: the MFMAs, and about 19 FP64 instructions per
// element of P, which keep the matrix pipe from issuing and are paid once per
// row tile.  So a tile holds all rows of N_Sigma where it can (BX up to 4),
// and no more rows than are there.  One launch holds the pairs of many bands:
// with one band and 16 energies it had 192 workgroups (739 G), fewer than the
// chip has CUs.  48 x 739, 64 bands x 16 energies: 64 launches of 115 us on
// 64 x 64 tiles against 3.2 ms in all.  The pairs are the fastest grid index,
// so that the workgroups that run together share 64 columns of Omega2 and wt
// in every L2.
template <int BX>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void gpp_t_kernel(
    const double2* __restrict__ m, int ns, int ng, const double2* __restrict__ omega2,
    const double* __restrict__ wt, const double* __restrict__ v,
    const double2* __restrict__ energies, int ne, GppBands bands, double2* __restrict__ t) {
    constexpr int TM = 16 * BX, KT = 16, NP = KT / 4;
    constexpr int PD = BX <= 2 ? 2 : 1;  // stages between a load and its use, as registers allow
    __shared__ double2 s_a[2][TM][KT + 1];  // [l][G]
    __shared__ double2 s_b[2][KT][65];      // [G][G']
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, row = lane & 15, kq = lane >> 4;
    const int64_t q = blockIdx.x;
    const int n = static_cast<int>(q / ne);
    const double2 ee = energies[q % ne];
    const double sn = (bands.occupied >> n) & 1 ? -1.0 : 1.0;
    const double x0 = ee.x - bands.en[n];
    const int i0 = blockIdx.y * TM, j0 = blockIdx.z * 64;
    m += static_cast<int64_t>(n) * ns * ng;

    dbl4 p1[BX], p2[BX], p3[BX];
#pragma unroll
    for (int x = 0; x < BX; ++x) p1[x] = p2[x] = p3[x] = zero4();

    // staged: rows l = i0 + (tid + 256 u) / 16 of M, G = k0 + tid % 16; rows
    // G = k0 + wave + 4 u of Omega2 and wt, column j0 + lane.  Rows and columns
    // past the edge are clamped: they feed only entries that are not stored.
    const int kk = tid % KT;
    const double2* pa[BX];
#pragma unroll
    for (int u = 0; u < BX; ++u)
        pa[u] = m + static_cast<int64_t>(min(i0 + tid / KT + 16 * u, ns - 1)) * ng + kk;
    const int64_t jc = min(j0 + lane, ng - 1);
    const double vj = 0.5 * v[jc], y2 = ee.y * ee.y;
    double2 ra[PD][BX], ro[PD][NP];
    double rw[PD][NP];
    auto load = [&](int st, int slot, int e) {  // element e of BX + 2 NP of a whole stage
        if (e < BX) {
            ra[slot][e].x = pa[e][st * KT].x;
            ra[slot][e].y = pa[e][st * KT].y;
            return;
        }
        const int u = (e - BX) / 2;
        const int64_t g0 = static_cast<int64_t>(st * KT + wave + 4 * u) * ng;
        if ((e - BX) % 2 == 0) {
            ro[slot][u].x = (omega2 + g0)[jc].x;
            ro[slot][u].y = (omega2 + g0)[jc].y;
        } else {
            rw[slot][u] = (wt + g0)[jc];
        }
    };
    const int nfull = ng / KT, nst = (ng + KT - 1) / KT;
    auto fetch = [&](int st, int slot) {
        if (st < nfull) {
#pragma unroll
            for (int e = 0; e < BX + 2 * NP; ++e) load(st, slot, e);
        } else if (st < nst) {  // the last, partial stage
#pragma unroll
            for (int u = 0; u < BX; ++u)
                ra[slot][u] = st * KT + kk < ng ? pa[u][st * KT] : make_double2(0.0, 0.0);
#pragma unroll
            for (int u = 0; u < NP; ++u) {
                const int64_t g0 = static_cast<int64_t>(min(st * KT + wave + 4 * u, ng - 1)) * ng;
                ro[slot][u] = (omega2 + g0)[jc];
                rw[slot][u] = (wt + g0)[jc];
            }
        }
    };
    // P = Omega2 v / (2 wt (x + i y)), x + i y = E - E_n - s wt; zero past the last G
    auto store_p = [&](int slot, int buf, int u, bool there) {
        const double2 o = ro[slot][u];
        const double w = rw[slot][u];
        const double x = x0 - sn * w;
        const double inv = vj / (w * (x * x + y2));
        const double2 p = make_double2((o.x * x + o.y * ee.y) * inv, (o.y * x - o.x * ee.y) * inv);
        s_b[buf][wave + 4 * u][lane] = there ? p : make_double2(0.0, 0.0);
    };
    auto store_a = [&](int slot, int buf, int u) {
        s_a[buf][tid / KT + 16 * u][kk] = make_double2(ra[slot][u].x, -ra[slot][u].y);
    };
    auto store = [&](int st, int slot, int buf) {
#pragma unroll
        for (int u = 0; u < BX; ++u) store_a(slot, buf, u);
#pragma unroll
        for (int u = 0; u < NP; ++u) store_p(slot, buf, u, st * KT + wave + 4 * u < ng);
    };
    auto read = [&](int buf, int k, double2 (&a)[BX], double2& b) {
#pragma unroll
        for (int x = 0; x < BX; ++x) a[x] = s_a[buf][x * 16 + row][k * 4 + kq];
        b = s_b[buf][k * 4 + kq][wave * 16 + row];
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
    fetch(0, 0);
    store(0, 0, 0);
    __syncthreads();
    if (PD == 2) fetch(1, 1);
    // Stage st is multiplied, st + PD loaded, and st + 1 formed and written to
    // LDS: spread over the stage where its operands came a stage ago (PD = 2),
    // else over the second half, behind the loads.
    int st = 0;
    for (; st + 2 * PD - 1 < nfull; st += PD) {
#pragma unroll
        for (int d = 0; d < PD; ++d) {
            constexpr int NM = 3 * BX, NQ = KT / 4, NT = NM * NQ, NE = BX + 2 * NP;
            constexpr int EV = PD == 1 || NT >= 2 * NE ? 2 : 1;  // MFMAs per load
            static_assert(NT >= EV * NE, "no room for a stage's loads");
            const int buf = PD == 2 ? d : st & 1;
            constexpr int P0 = PD == 2 ? 0 : NT / 2, PS = (NT - P0) / NP;
            double2 a[2][BX], b[2];
            double as[2][BX], bs[2];
            read(buf, 0, a[0], b[0]);
            sums(a[0], b[0], as[0], bs[0]);
            __builtin_amdgcn_s_setprio(2);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < NQ; ++k) {
                const int f = k & 1;
#pragma unroll
                for (int i = 0; i < NM; ++i) {
                    mfma1(i, a[f], b[f], as[f], bs[f]);
                    __builtin_amdgcn_sched_barrier(0);
                    const int x = k * NM + i;
                    if (x % EV == EV - 1 && x / EV < NE) load(st + d + PD, d, x / EV);
                    if (i == (NM - 2) / 2 && k + 1 < NQ) read(buf, k + 1, a[f ^ 1], b[f ^ 1]);
                    if (i == NM - 2 && k + 1 < NQ) sums(a[f ^ 1], b[f ^ 1], as[f ^ 1], bs[f ^ 1]);
                    if (x >= P0 && (x - P0) % PS == PS / 2 && (x - P0) / PS < NP)
                        store_p((d + 1) % PD, buf ^ 1, (x - P0) / PS, true);
                    if (x >= NT - 1 - BX && x < NT - 1) store_a((d + 1) % PD, buf ^ 1, x - (NT - 1 - BX));
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
            const int buf = PD == 2 ? d : st & 1;
            fetch(st + d + PD, d);
#pragma unroll
            for (int k = 0; k < KT / 4; ++k) {
                double2 a[BX], b;
                double as[BX], bs;
                read(buf, k, a, b);
                sums(a, b, as, bs);
#pragma unroll
                for (int i = 0; i < 3 * BX; ++i) mfma1(i, a, b, as, bs);
            }
            if (st + d + 1 < nst) store(st + d + 1, (d + 1) % PD, buf ^ 1);
            __syncthreads();
        }
    }
    double2* tq = t + q * static_cast<int64_t>(ns) * ng;
#pragma unroll
    for (int x = 0; x < BX; ++x)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int l = i0 + x * 16 + 4 * r + kq, c = j0 + wave * 16 + row;
            if (l < ns && c < ng)
                tq[static_cast<int64_t>(l) * ng + c] =
                    make_double2(p1[x][r] - p2[x][r], p3[x][r] - p1[x][r] - p2[x][r]);
        }
}

// sigma[i] += the sum over bands of part[band][i], in band order
__global__ __launch_bounds__(256) void sum_bands_kernel(const double2* __restrict__ part, int nband,
                                                        int64_t n, double2* __restrict__ sigma) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double2 acc = sigma[i];
    for (int b = 0; b < nband; ++b) {
        const double2 p = part[b * n + i];
        acc.x += p.x;
        acc.y += p.y;
    }
    sigma[i] = acc;
}

__global__ __launch_bounds__(256) void zero_kernel(double2* __restrict__ p, int64_t n) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        p[i] = make_double2(0.0, 0.0);
}

size_t al256(size_t b) { return (b + 255) & ~size_t(255); }

}  // namespace

GppLayout gpp_layout(int ns, int ng, int nb, int ne, size_t bytes) {
    GppLayout L;
    // T of one band within 1 GiB, at least one energy
    const size_t t1 = static_cast<size_t>(ns) * ng * sizeof(double2);
    const size_t s1 = static_cast<size_t>(ns) * ns * sizeof(double2);
    L.ec = std::max(1, std::min<int>(ne, static_cast<int>((size_t(1) << 30) / std::max<size_t>(t1, 1))));
    const size_t fixed = al256(static_cast<size_t>(ne) * sizeof(double2)) + 512;
    // As many bands as fit with a Sigma of their own per pair.  In the
    // library's scratch (bytes = 0): 256 MiB, the size of the last-level cache
    // that T is read back from.
    const size_t room = bytes ? bytes : (size_t(256) << 20) + fixed;
    const size_t pair = static_cast<size_t>(L.ec) * (t1 + s1);
    size_t bc = room > fixed ? (room - fixed) / std::max<size_t>(pair, 1) : 0;
    bc = std::min<size_t>(bc, std::min(nb, kMaxBands));
    bc = std::min<size_t>(bc, 65535 / L.ec);
    L.bc = std::max(1, static_cast<int>(bc));
    const size_t t = al256(static_cast<size_t>(L.bc) * L.ec * t1);
    L.off_part = t;
    L.off_e = t + (L.bc > 1 ? al256(static_cast<size_t>(L.bc) * L.ec * s1) : 0);
    L.total = L.off_e + al256(static_cast<size_t>(ne) * sizeof(double2));
    return L;
}

namespace {

template <int BX>
void launch_gpp_t(const double2* m, int ns, int ng, const double2* omega2, const double* wt,
                  const double* v, const double2* energies, int ec, int bc, const GppBands& bands,
                  double2* t, hipStream_t s) {
    ProfScope ps("gpp_t", s);
    hipLaunchKernelGGL((gpp_t_kernel<BX>),
                       dim3(static_cast<unsigned>(bc * ec), static_cast<unsigned>(ceil_div(ns, 16 * BX)),
                            static_cast<unsigned>(ceil_div(ng, 64))),
                       dim3(256), 0, s, m, ns, ng, omega2, wt, v, energies, ec, bands, t);
    GW_HIP_TRY(hipGetLastError());
}

}  // namespace

void run_gpp_sigma(const double2* m, int nb, int ns, int ng, const double* e_n,
                   const int32_t* occupied, int ne, const double2* omega2, const double* wt,
                   const double* v, double2* sigma, char* base, const GppLayout& L, hipStream_t s) {
    double2* t = reinterpret_cast<double2*>(base);
    double2* part = reinterpret_cast<double2*>(base + L.off_part);
    const double2* energies = reinterpret_cast<const double2*>(base + L.off_e);
    const int64_t sig = static_cast<int64_t>(ns) * ns;
    {
        const int64_t n = sig * ne;
        hipLaunchKernelGGL(zero_kernel, dim3(static_cast<unsigned>(std::min<int64_t>(ceil_div64(n, 256), 4096))),
                           dim3(256), 0, s, sigma, n);
        GW_HIP_TRY(hipGetLastError());
    }
    if (nb == 0 || ns == 0 || ng == 0) return;
    // row tiles of equal height, at most 64 rows each
    const int blocks = ceil_div(ns, 16), bx = ceil_div(blocks, ceil_div(blocks, 4));
    for (int e0 = 0; e0 < ne; e0 += L.ec) {
        const int ec = std::min(L.ec, ne - e0);
        for (int n0 = 0; n0 < nb; n0 += L.bc) {
            const int bc = std::min(L.bc, nb - n0);
            const double2* mn = m + static_cast<int64_t>(n0) * ns * ng;
            GppBands bands{};
            for (int n = 0; n < bc; ++n) {
                bands.en[n] = e_n[n0 + n];
                if (occupied[n0 + n]) bands.occupied |= uint64_t(1) << n;
            }
            const auto launch = bx == 1   ? launch_gpp_t<1>
                                : bx == 2 ? launch_gpp_t<2>
                                : bx == 3 ? launch_gpp_t<3>
                                          : launch_gpp_t<4>;
            launch(mn, ns, ng, omega2, wt, v, energies + e0, ec, bc, bands, t, s);
            // T M_n^T of every pair: added to Sigma(E) where the launch holds
            // one band, else summed over the bands by the kernel after it
            ZGemm g;
            g.m = ns;
            g.n = ns;
            g.k = ng;
            g.a = t;
            g.lda = ng;
            g.stride_a = static_cast<int64_t>(ns) * ng;
            g.b = mn;
            g.ldb = ng;
            g.stride_b = static_cast<int64_t>(ns) * ng;
            g.b_repeat = ec;
            g.c = bc > 1 ? part : sigma + e0 * sig;
            g.ldc = ns;
            g.stride_c = sig;
            g.beta = make_double2(bc > 1 ? 0.0 : 1.0, 0.0);
            g.batch = bc * ec;
            launch_zgemm(kOpN, kOpT, g, s);
            if (bc > 1) {
                const int64_t n = sig * ec;
                hipLaunchKernelGGL(sum_bands_kernel, dim3(static_cast<unsigned>(ceil_div64(n, 256))),
                                   dim3(256), 0, s, part, bc, n, sigma + e0 * sig);
                GW_HIP_TRY(hipGetLastError());
            }
        }
    }
}

}  // namespace gw

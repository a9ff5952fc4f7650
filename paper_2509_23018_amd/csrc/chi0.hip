// CHI0 on gfx950: chi_w += M^H diag(s*Delta_w) M over one streamed chunk of
// pairs (Eq. (4) of the paper), FP64 MFMA 16x16x4 tiles, plus the energy
// factor, the Hermitian mirror and the zero fill.
#include <algorithm>
#include <cstdlib>
#include <map>
#include <tuple>
#include <mutex>
#include <vector>

#include "chi0.hpp"
#include "items.hpp"
#include "lifetime.hpp"
#include "common.hpp"
#include "prof.hpp"

namespace gw {

namespace {

// ---------------------------------------------------------------- energy factor

__global__ __launch_bounds__(256) void delta_kernel(const double* __restrict__ e_v,
                                                    const double* __restrict__ e_c, PairMap pm,
                                                    int64_t npairs, ZArgs za, int w0,
                                                    double2* __restrict__ delta) {
    const int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= npairs) return;
    const int64_t lin = pm.k_off + k;
    const double de = e_v[pm.v0 + lin / pm.cw] - e_c[pm.c0 + lin % pm.cw];
    for (int w = 0; w < za.nz; ++w) {
        const double zr = za.re[w], zi = za.im[w];
        // 1/(de + z) + 1/(de - z), each as conj(d)/|d|^2
        const double ar = de + zr, br = de - zr;
        const double n1 = ar * ar + zi * zi, n2 = br * br + zi * zi;
        double re = ar / n1 + br / n2;
        double im = -zi / n1 + zi / n2;
        if (zr == 0.0) im = 0.0;  // imaginary axis / static: Delta is real
        delta[static_cast<int64_t>(w0 + w) * npairs + k] = make_double2(za.spin * re, za.spin * im);
    }
}

// ---------------------------------------------------------------- FP64 contraction

constexpr int kKt = 16;     // pairs per LDS stage

// One workgroup = one T x T tile of chi_w, WI x WJ waves, each a
// (T/WI) x (T/WJ) sub-tile of 16x16 MFMA blocks.  Per stage of kKt pairs the
// rows of M for the tile's G and G' are staged in LDS (double-buffered; rows
// padded by PAD elements), the G' side already multiplied by s*Delta_w(k);
// the MFMAs accumulate conj(M_i) (Delta M_j), with three real products per
// complex one on the 64x64 tile.  Pair rows past the chunk end (in the last
// stage) are clamped and carry Delta = 0, columns past N_G are clamped and only
// feed outputs that are not stored.
// mode: bit 0 accumulate, bit 1 (T = 64) also write the conjugate transpose to
// the mirrored tile.  PART: store the whole T x T tile instead, unmasked,
// row-major at cw (a partial sum over a range of pairs).
template <int T, int WI, int WJ, int PAD, bool PART = false>
__device__ __forceinline__ void f64_tile(double2* lds, const double2* __restrict__ m, int64_t kc,
                                         int ng, const double2* __restrict__ dw,
                                         double2* __restrict__ cw, int mode, int bi, int bj) {
    constexpr int NT = WI * WJ * 64;
    constexpr int BX = T / WI / 16, BY = T / WJ / 16;
    constexpr int LDR = T + PAD;                 // LDS row length (double2)
    constexpr int NLOAD = kKt * T / NT;          // staged elements per thread per side
    static_assert(NLOAD * NT == kKt * T && NT % T == 0, "tile / thread mismatch");
    double2* s_a = lds;                  // [2][kKt][LDR]
    double2* s_b = lds + 2 * kKt * LDR;  // [2][kKt][LDR]
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, row = lane & 15, kq = lane >> 4;
    const int wi = wave / WJ, wj = wave % WJ;
    const int i0 = bi * T, j0 = bj * T;

    // staging slots: element e = tid + NT*u -> row kk = e / T, column cc = e % T;
    // NT is a multiple of T, so cc is the same for every u and kk steps by NT/T
    constexpr int KSTEP = NT / T;
    const int cc = tid % T, kk0 = tid / T;
    const int ci = min(i0 + cc, ng - 1), cj = min(j0 + cc, ng - 1);

    // conj(a) b with three real products where the registers allow
    // (Karatsuba, K3): p1 = ar br, p2 = ai bi, p3 = (ar - ai)(br + bi);
    // Re = p1 + p2, Im = p3 - p1 + p2.  Otherwise four: p1 = Re, p2 = Im
    // (p3 unused).
    constexpr bool K3 = BX * BY <= 4;
    dbl4 p1[BX][BY], p2[BX][BY], p3[BX][BY];
#pragma unroll
    for (int a = 0; a < BX; ++a)
#pragma unroll
        for (int b = 0; b < BY; ++b) p1[a][b] = p2[a][b] = p3[a][b] = zero4();

    // Loads of a whole stage go through addresses that are uniform but for a
    // 32-bit offset per lane, fixed for the tile.
    const uint32_t voi = static_cast<uint32_t>((kk0 * ng + ci) * sizeof(double2));
    const uint32_t voj = static_cast<uint32_t>((kk0 * ng + cj) * sizeof(double2));
    const uint32_t vod = static_cast<uint32_t>(kk0 * sizeof(double2));
    const int64_t row_bytes = static_cast<int64_t>(ng) * sizeof(double2);
    double2 ra[NLOAD], rb[NLOAD], rd[NLOAD];
    // load l (of 3 NLOAD) of whole stage st: Delta, the G' and the G side of
    // staged row l / 3
    auto load = [&](int st, int l) {
        const int u = l / 3;
        const int64_t k = static_cast<int64_t>(st) * kKt + KSTEP * u;
        const char* pm = reinterpret_cast<const char*>(m) + k * row_bytes;
        if (l % 3 == 0) {
            rd[u] = *reinterpret_cast<const double2*>(reinterpret_cast<const char*>(dw + k) + vod);
        } else if (l % 3 == 1) {
            rb[u] = *reinterpret_cast<const double2*>(pm + voj);
        } else {
            // component loads: a whole-struct copy into LDS would be fused
            // into one global-to-LDS copy placed after the MFMAs, exposing
            // the load latency at every stage
            const double2* pa = reinterpret_cast<const double2*>(pm + voi);
            ra[u].x = pa->x;
            ra[u].y = pa->y;
        }
    };
    const int nfull = static_cast<int>(kc / kKt);
    const int nst = static_cast<int>((kc + kKt - 1) / kKt);
    auto fetch = [&](int st) {
        if (st < nfull) {
#pragma unroll
            for (int l = 0; l < 3 * NLOAD; ++l) load(st, l);
        } else if (st < nst) {  // the last, partial stage: rows past the end are clamped
#pragma unroll
            for (int u = 0; u < NLOAD; ++u) {
                const int64_t k = static_cast<int64_t>(st) * kKt + kk0 + KSTEP * u;
                const int64_t kr = k < kc ? k : kc - 1;
                rd[u] = k < kc ? dw[kr] : make_double2(0.0, 0.0);
                rb[u] = k < kc ? m[kr * ng + cj] : make_double2(0.0, 0.0);
                ra[u] = m[kr * ng + ci];
            }
        }
    };
    auto store = [&](int u, int buf) {
        s_a[(buf * kKt + kk0 + KSTEP * u) * LDR + cc] = make_double2(ra[u].x, ra[u].y);
        s_b[(buf * kKt + kk0 + KSTEP * u) * LDR + cc] = cmul(rd[u], rb[u]);
    };
    auto store_all = [&](int buf) {
#pragma unroll
        for (int u = 0; u < NLOAD; ++u) store(u, buf);
    };
    // fragments of k-step q, and the sums of the third product
    auto read = [&](int buf, int q, double2 (&a)[BX], double2 (&b)[BY]) {
        const double2* la = s_a + (buf * kKt + q * 4 + kq) * LDR + wi * (T / WI) + row;
        const double2* lb = s_b + (buf * kKt + q * 4 + kq) * LDR + wj * (T / WJ) + row;
#pragma unroll
        for (int x = 0; x < BX; ++x) a[x] = la[x * 16];
#pragma unroll
        for (int y = 0; y < BY; ++y) b[y] = lb[y * 16];
    };
    auto sums = [&](const double2 (&a)[BX], const double2 (&b)[BY], double (&as)[BX],
                    double (&bs)[BY]) {
#pragma unroll
        for (int x = 0; x < BX; ++x) as[x] = a[x].x - a[x].y;
#pragma unroll
        for (int y = 0; y < BY; ++y) bs[y] = b[y].x + b[y].y;
    };
    // MFMA i of the 3 BX BY of a k-step (K3)
    auto mfma_k3 = [&](int i, const double2 (&a)[BX], const double2 (&b)[BY],
                       const double (&as)[BX], const double (&bs)[BY]) {
        const int x = i / 3 / BY, y = i / 3 % BY;
        if (i % 3 == 0) p1[x][y] = mfma_f64(a[x].x, b[y].x, p1[x][y]);
        if (i % 3 == 1) p2[x][y] = mfma_f64(a[x].y, b[y].y, p2[x][y]);
        if (i % 3 == 2) p3[x][y] = mfma_f64(as[x], bs[y], p3[x][y]);
    };
    auto multiply = [&](int buf) {
#pragma unroll
        for (int q = 0; q < kKt / 4; ++q) {
            double2 a[BX], b[BY];
            read(buf, q, a, b);
            if constexpr (K3) {
                double as[BX], bs[BY];
                sums(a, b, as, bs);
#pragma unroll
                for (int i = 0; i < 3 * BX * BY; ++i) mfma_k3(i, a, b, as, bs);
            } else {
#pragma unroll
                for (int x = 0; x < BX; ++x)
#pragma unroll
                    for (int y = 0; y < BY; ++y)
                        cmfma_conj_a(p1[x][y], p2[x][y], a[x].x, a[x].y, b[y].x, b[y].y);
            }
        }
    };

    // Stage st + 1 is loaded while stage st is multiplied and written to the
    // other LDS buffer behind the loads.  The wave issues in order and shares
    // its SIMD with one other, so what stands between two MFMAs decides how
    // long the matrix pipe waits.
    fetch(0);
    store_all(0);
    __syncthreads();
    int st = 0;
    if constexpr (K3) {
        // Every instruction between the MFMAs of a whole stage is placed: six
        // loads in each of the first k-steps, one per two MFMAs; the next
        // k-step's fragments read after the ninth MFMA and their sums formed
        // before the last; in the last k-step one staged row written to LDS
        // per two MFMAs.  The same work with the loads and the LDS writes each
        // in one run before and after the MFMAs takes 64.0 ms where this takes
        // 58.7 (3,840 pairs of the 72^3 grid, 6,031 G, 8 frequencies, MTXEL
        // among them; 60.2 with the address arithmetic between the loads).
        constexpr int NM = 3 * BX * BY, NQ = kKt / 4, LD = NM / 2;
        static_assert(NQ * LD >= 3 * NLOAD && NM / 2 > NLOAD, "no room for a stage's loads");
        double2 a[2][BX], b[2][BY];
        double as[2][BX], bs[2][BY];
        for (; st + 1 < nfull; ++st) {
            const int buf = st & 1;
            read(buf, 0, a[0], b[0]);
            sums(a[0], b[0], as[0], bs[0]);
            __builtin_amdgcn_s_setprio(2);  // over the other workgroup's barrier and first reads
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int f = q & 1;
#pragma unroll
                for (int i = 0; i < NM; ++i) {
                    mfma_k3(i, a[f], b[f], as[f], bs[f]);
                    __builtin_amdgcn_sched_barrier(0);
                    const int l = q * LD + i / 2;
                    if (i % 2 == 1 && l < 3 * NLOAD) load(st + 1, l);
                    if (i == NM - 4 && q + 1 < NQ) read(buf, q + 1, a[f ^ 1], b[f ^ 1]);
                    if (i == NM - 2 && q + 1 < NQ) sums(a[f ^ 1], b[f ^ 1], as[f ^ 1], bs[f ^ 1]);
                    if (q + 1 == NQ && i % 2 == 0 && i >= 2 && i / 2 <= NLOAD)
                        store(i / 2 - 1, buf ^ 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_s_setprio(0);
            __syncthreads();
        }
    } else {
        for (; st + 1 < nfull; ++st) {
            __builtin_amdgcn_s_setprio(1);
            fetch(st + 1);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(2);
            multiply(st & 1);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(0);
            store_all((st & 1) ^ 1);
            __syncthreads();
        }
    }
    for (; st < nst; ++st) {  // the last whole stage and the partial one
        fetch(st + 1);
        multiply(st & 1);
        if (st + 1 < nst) store_all((st & 1) ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int x = 0; x < BX; ++x)
#pragma unroll
        for (int y = 0; y < BY; ++y)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int li = wi * (T / WI) + x * 16 + 4 * t + kq;
                const int lj = wj * (T / WJ) + y * 16 + row;
                const double re = K3 ? p1[x][y][t] + p2[x][y][t] : p1[x][y][t];
                const double im = K3 ? p3[x][y][t] - p1[x][y][t] + p2[x][y][t] : p2[x][y][t];
                if constexpr (PART) {
                    cw[li * T + lj] = make_double2(re, im);
                    continue;
                }
                const int gi = i0 + li, gj = j0 + lj;
                if (gi < ng && gj < ng) {
                    double2* p = cw + static_cast<int64_t>(gi) * ng + gj;
                    double2 v = make_double2(re, im);
                    if (mode & 1) {
                        const double2 o = *p;
                        v.x += o.x;
                        v.y += o.y;
                    }
                    *p = v;
                    // position li of row lj, permuted so that neither side of
                    // the transposition meets its own banks
                    if (T == 64 && (mode & 2)) lds[lj * T + (li ^ (lj & 7))] = v;
                }
            }
    if constexpr (T == 64 && !PART) {
        if (mode & 2) {  // the mirrored tile, a row per wave at a time
            __syncthreads();
            for (int lj = wave; lj < T; lj += NT / 64) {
                const int gj = j0 + lj, gi = i0 + lane;
                if (gj >= ng || gi >= ng) continue;
                const double2 v = lds[lj * T + (lane ^ (lj & 7))];
                cw[static_cast<int64_t>(gj) * ng + gi] = make_double2(v.x, -v.y);
            }
        }
    }
}

// Mode of a tile: the mirrored tile is written for Hermitian items off the
// diagonal (a tile on it holds both halves).
__device__ __forceinline__ int tile_mode(int mode, bool herm, int bi, int bj) {
    return herm && bi != bj ? mode : mode & 1;
}


// The first n_main items, one per workgroup, over all pairs of the chunk.
// Each of the remaining items (the last, partial round of workgroups) is cut
// into `parts` ranges of whole stages; workgroup n_main + j*parts + p writes
// item n_main + j's partial sum over range p to ws[j*parts + p] (T x T), and
// tail_reduce_kernel adds the parts into chi.
template <int T, int WI, int WJ, int PAD>
__global__ __launch_bounds__(WI * WJ * 64) void chi0_f64_kernel(
    const double2* __restrict__ m, int64_t kc, int ng, const double2* __restrict__ delta,
    WList wl, double2* __restrict__ chi, int mode, int nb, const int* __restrict__ order,
    int n_main, int parts, double2* __restrict__ ws) {
    extern __shared__ double2 lds[];
    const int b = blockIdx.x;
    int w, bi, bj;
    if (b < n_main) {
        const int t = xcd_item(b, n_main);
        item_tile(t, wl, nb, order, w, bi, bj);
        f64_tile<T, WI, WJ, PAD>(lds, m, kc, ng, delta + static_cast<int64_t>(w) * kc,
                                 chi + static_cast<int64_t>(w) * ng * ng,
                                 tile_mode(mode, hermitian_item(t, wl, nb), bi, bj), bi, bj);
        return;
    }
    const int u = b - n_main, j = u / parts, p = u % parts;
    item_tile(n_main + j, wl, nb, order, w, bi, bj);
    const int64_t nst = (kc + kKt - 1) / kKt;
    const int64_t k0 = p * nst / parts * kKt;
    const int64_t k1 = std::min<int64_t>(kc, (p + 1) * nst / parts * kKt);
    f64_tile<T, WI, WJ, PAD, true>(lds, m + k0 * ng, k1 - k0, ng,
                                   delta + static_cast<int64_t>(w) * kc + k0,
                                   ws + static_cast<int64_t>(u) * T * T, 0, bi, bj);
}

// chi_w[tile] (=|+=) the sum of the parts of tail item n_main + blockIdx.y,
// added in part order.
template <int T>
__global__ __launch_bounds__(256) void tail_reduce_kernel(const double2* __restrict__ ws,
                                                          int parts, int n_main, WList wl, int nb,
                                                          const int* __restrict__ order,
                                                          double2* __restrict__ chi, int ng,
                                                          int mode) {
    const int j = blockIdx.y, e = blockIdx.x * 256 + threadIdx.x;
    int w, bi, bj;
    item_tile(n_main + j, wl, nb, order, w, bi, bj);
    mode = tile_mode(mode, hermitian_item(n_main + j, wl, nb), bi, bj);
    const int gi = bi * T + e / T, gj = bj * T + e % T;
    if (gi >= ng || gj >= ng) return;
    const double2* src = ws + static_cast<int64_t>(j) * parts * T * T + e;
    double2 acc = src[0];
    for (int p = 1; p < parts; ++p) {
        const double2 v = src[static_cast<int64_t>(p) * T * T];
        acc.x += v.x;
        acc.y += v.y;
    }
    double2* cw = chi + static_cast<int64_t>(w) * ng * ng;
    double2* dst = cw + static_cast<int64_t>(gi) * ng + gj;
    if (mode & 1) {
        const double2 o = *dst;
        acc.x += o.x;
        acc.y += o.y;
    }
    *dst = acc;
    if (mode & 2) cw[static_cast<int64_t>(gj) * ng + gi] = make_double2(acc.x, -acc.y);
}

// Persistent form for batches of problems: every workgroup takes items
// (problem, frequency, tile) from an atomic counter until the list is
// exhausted, so problems of very different N_G share one launch without a
// tail per problem.  Items are sorted by decreasing cost on the host.
template <int T, int WI, int WJ, int PAD>
__global__ __launch_bounds__(WI * WJ * 64) void chi0_f64_batched_kernel(
    const QDesc* __restrict__ qd, const int4* __restrict__ items, int nitems,
    int* __restrict__ counter) {
    extern __shared__ double2 lds[];
    __shared__ int s_item;
    for (;;) {
        if (threadIdx.x == 0) s_item = atomicAdd(counter, 1);
        __syncthreads();
        const int it = __builtin_amdgcn_readfirstlane(s_item);
        __syncthreads();
        if (it >= nitems) break;
        const int4 itm = items[it];
        const QDesc d = qd[itm.x];
        f64_tile<T, WI, WJ, PAD>(lds, d.m, d.kc, d.ng, d.delta + static_cast<int64_t>(itm.y) * d.kc,
                                 d.chi + static_cast<int64_t>(itm.y) * d.ng * d.ng,
                                 tile_mode(d.mode, (itm.z & kItemHermitian) != 0,
                                           itm.z & ~kItemHermitian, itm.w),
                                 itm.z & ~kItemHermitian, itm.w);
    }
}

struct Chi0Variant {
    const void* fn;       // per-launch kernel
    const void* fn_batch; // persistent batched kernel
    const void* fn_tail;  // tail_reduce_kernel<T>
    int tile, threads;
    size_t lds;
};

template <int T, int WI, int WJ, int PAD>
Chi0Variant chi0_variant() {
    return {reinterpret_cast<const void*>(&chi0_f64_kernel<T, WI, WJ, PAD>),
            reinterpret_cast<const void*>(&chi0_f64_batched_kernel<T, WI, WJ, PAD>),
            reinterpret_cast<const void*>(&tail_reduce_kernel<T>), T, WI * WJ * 64,
            2 * 2 * kKt * (T + PAD) * sizeof(double2)};
}

// Tile shapes of the FP64 contraction, indexed by variant id (the autotuner
// chooses among them; GW_CHI0_VARIANT forces one).
const Chi0Variant& chi0_variant_by_id(int id) {
    static const Chi0Variant v[2] = {chi0_variant<64, 2, 2, 0>(), chi0_variant<128, 2, 4, 0>()};
    return v[id == 1 ? 1 : 0];
}

// chi[i][j] = conj(chi[j][i]) for every (i, j) in a tile strictly below the
// diagonal of tile x tile blocks (those the Hermitian contraction skipped),
// for every Hermitian frequency of wl.
__global__ __launch_bounds__(256) void mirror_kernel(double2* __restrict__ chi, int ng, int tile,
                                                     WList wl) {
    chi += static_cast<int64_t>(wl.w[blockIdx.z]) * ng * ng;
    const int j = blockIdx.x * 16 + (threadIdx.x & 15);
    const int i = blockIdx.y * 16 + (threadIdx.x >> 4);
    if (i >= ng || j >= ng) return;
    if (i / tile <= j / tile) return;
    const double2 u = chi[static_cast<int64_t>(j) * ng + i];
    chi[static_cast<int64_t>(i) * ng + j] = make_double2(u.x, -u.y);
}

__global__ __launch_bounds__(256) void fill_zero_kernel(double2* __restrict__ p, int64_t n) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        p[i] = make_double2(0.0, 0.0);
}

}  // namespace

void launch_delta(const double* e_v, const double* e_c, PairMap pm, int64_t npairs,
                  const double2* z, int nz, double spin, double2* delta, hipStream_t s) {
    if (npairs <= 0) return;
    for (int w0 = 0; w0 < nz; w0 += kMaxZ) {
        ZArgs za{};
        za.nz = std::min(kMaxZ, nz - w0);
        za.spin = spin;
        for (int w = 0; w < za.nz; ++w) {
            za.re[w] = z[w0 + w].x;
            za.im[w] = z[w0 + w].y;
        }
        ProfScope ps("delta", s);
        hipLaunchKernelGGL(delta_kernel, dim3(static_cast<unsigned>(ceil_div64(npairs, 256))),
                           dim3(256), 0, s, e_v, e_c, pm, npairs, za, w0, delta);
        GW_HIP_TRY(hipGetLastError());
    }
}

namespace {
// Workgroups of variant v resident on the current device at once.
int f64_slots(int variant) {
    static std::mutex mu;
    static std::map<std::pair<int, int>, int> cache;  // (device, variant) -> slots
    int dev = 0;
    GW_HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(mu);
    int& n = cache[{dev, variant}];
    if (n > 0) return n;
    const Chi0Variant& v = chi0_variant_by_id(variant);
    GW_HIP_TRY(hipFuncSetAttribute(v.fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   static_cast<int>(v.lds)));
    int per_cu = 0, cus = 0;
    GW_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, v.fn, v.threads, v.lds));
    GW_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    n = std::max(1, per_cu) * std::max(1, cus);
    return n;
}
}  // namespace

size_t chi0_f64_tail_bytes() {
    size_t b = 0;
    for (int v = 0; v < kNumChi0Variants; ++v) {
        const size_t t = static_cast<size_t>(chi0_variant_by_id(v).tile);
        b = std::max(b, static_cast<size_t>(f64_slots(v)) * t * t * sizeof(double2));
    }
    return b;
}

void launch_chi0_f64(const double2* m, int64_t kc, int ng, const double2* delta,
                     const WList& wl, double2* chi, bool accumulate, hipStream_t s, int variant,
                     double2* tail_ws, bool mirror) {
    if (kc <= 0 || wl.nh + wl.nf == 0) return;
    if (mirror && !chi0_variant_mirrors(variant)) throw Error{-5, "this tile does not mirror"};
    const Chi0Variant& v = chi0_variant_by_id(variant);
    const int nb = ceil_div(ng, v.tile);
    const int64_t nitems = static_cast<int64_t>(wl.nh) * (nb * (nb + 1) / 2) +
                           static_cast<int64_t>(wl.nf) * nb * nb;
    if (nitems >= (int64_t(1) << 30)) throw Error{-4, "too many chi tiles for one launch"};
    GW_HIP_TRY(hipFuncSetAttribute(v.fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   static_cast<int>(v.lds)));
    // A last round of workgroups that fills at most half the chip is cut
    // along the pairs: each of its items becomes `parts` workgroups over
    // ranges of stages, which together fill the round.
    int n_main = static_cast<int>(nitems), parts = 1, n_tail = 0;
    if (tail_ws) {
        const int slots = f64_slots(variant);
        const int rem = static_cast<int>(nitems % slots);
        const int64_t nst = (kc + kKt - 1) / kKt;
        const int pc = static_cast<int>(std::min<int64_t>(rem > 0 ? slots / rem : 0, nst));
        if (rem > 0 && 2 * rem <= slots && pc >= 2) {
            n_tail = rem;
            parts = pc;
            n_main = static_cast<int>(nitems) - rem;
        }
    }
    int mode = (accumulate ? 1 : 0) | (mirror ? 2 : 0);
    const int* order = tile_order(nb);
    {
        ProfScope ps("chi0_f64", s);
        void* args[] = {const_cast<double2**>(&m), &kc, &ng, const_cast<double2**>(&delta),
                        const_cast<WList*>(&wl), &chi, &mode, const_cast<int*>(&nb),
                        const_cast<int**>(&order), &n_main, &parts, &tail_ws};
        const unsigned grid = static_cast<unsigned>(n_main + n_tail * parts);
        GW_HIP_TRY(hipLaunchKernel(v.fn, dim3(grid), dim3(v.threads), args, v.lds, s));
    }
    if (n_tail > 0) {
        ProfScope ps("chi0_tail", s);
        void* args[] = {&tail_ws, &parts, &n_main, const_cast<WList*>(&wl),
                        const_cast<int*>(&nb), const_cast<int**>(&order), &chi, &ng, &mode};
        const unsigned gx = static_cast<unsigned>(v.tile * v.tile / 256);
        GW_HIP_TRY(hipLaunchKernel(v.fn_tail, dim3(gx, static_cast<unsigned>(n_tail)), dim3(256),
                                   args, 0, s));
    }
}

void launch_chi0_f64_batched(const QDesc* qd, const int4* items, int nitems, int* counter,
                             hipStream_t s, int variant, int grid) {
    if (nitems <= 0) return;
    const Chi0Variant& v = chi0_variant_by_id(variant);
    GW_HIP_TRY(hipFuncSetAttribute(v.fn_batch, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   static_cast<int>(v.lds)));
    ProfScope ps("chi0_f64_batched", s);
    void* args[] = {const_cast<QDesc**>(&qd), const_cast<int4**>(&items), &nitems, &counter};
    GW_HIP_TRY(hipLaunchKernel(v.fn_batch, dim3(static_cast<unsigned>(std::min(grid, nitems))),
                               dim3(v.threads), args, v.lds, s));
}

int chi0_variant_tile(int variant) { return chi0_variant_by_id(variant).tile; }
bool chi0_variant_mirrors(int variant) { return chi0_variant_tile(variant) == 64; }

int chi0_f64_batched_blocks_per_cu(int variant) {
    const Chi0Variant& v = chi0_variant_by_id(variant);
    GW_HIP_TRY(hipFuncSetAttribute(v.fn_batch, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   static_cast<int>(v.lds)));
    int n = 0;
    GW_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, v.fn_batch, v.threads, v.lds));
    return std::max(1, n);
}

int chi0_forced_variant() {
    static const int id = [] {
        const char* e = std::getenv("GW_CHI0_VARIANT");
        return e ? std::atoi(e) : -1;
    }();
    return id;
}

void launch_mirror(double2* chi, int ng, int tile, const WList& wl, hipStream_t s) {
    if (wl.nh == 0 || ng <= tile) return;  // one tile holds both halves
    ProfScope ps("mirror", s);
    hipLaunchKernelGGL(mirror_kernel, dim3(ceil_div(ng, 16), ceil_div(ng, 16), wl.nh), dim3(256), 0,
                       s, chi, ng, tile, wl);
    GW_HIP_TRY(hipGetLastError());
}

void launch_fill_zero(double2* p, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    const int64_t blocks = std::min<int64_t>(ceil_div64(n, 256), 65536);
    hipLaunchKernelGGL(fill_zero_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, p, n);
    GW_HIP_TRY(hipGetLastError());
}



namespace {
struct OrderCache {
    std::mutex mu;
    std::map<std::tuple<int, int, int>, int*> tables;  // (device, nb, super) -> device table
};
OrderCache& order_cache() {
    static OrderCache* c = new OrderCache();
    return *c;
}
}  // namespace

const int* tile_order(int nb, int kSuper) {
    int dev = 0;
    GW_HIP_TRY(hipGetDevice(&dev));
    OrderCache& oc = order_cache();
    std::lock_guard<std::mutex> lk(oc.mu);
    int*& t = oc.tables[{dev, nb, kSuper}];
    if (t) return t;
    std::vector<int> h, f;
    for (int si = 0; si < nb; si += kSuper)
        for (int sj = 0; sj < nb; sj += kSuper)
            for (int i = si; i < std::min(nb, si + kSuper); ++i)
                for (int j = sj; j < std::min(nb, sj + kSuper); ++j) {
                    f.push_back((i << 16) | j);
                    if (j >= i) h.push_back((i << 16) | j);
                }
    h.insert(h.end(), f.begin(), f.end());
    require_alloc("tile-order table for this G-list size");
    GW_HIP_TRY(hipMalloc(&t, h.size() * sizeof(int)));
    GW_HIP_TRY(hipMemcpy(t, h.data(), h.size() * sizeof(int), hipMemcpyHostToDevice));
    return t;
}

void release_tile_orders() {
    OrderCache& oc = order_cache();
    std::lock_guard<std::mutex> lk(oc.mu);
    for (auto& kv : oc.tables) {
        (void)hipSetDevice(std::get<0>(kv.first));
        (void)hipDeviceSynchronize();
        (void)hipFree(kv.second);
    }
    oc.tables.clear();
}



}  // namespace gw

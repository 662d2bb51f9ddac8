// Layout kernels: canonical complex128 host layouts <-> internal storage.
//
// Gauge packing folds the staggered phases into the links (Sec.2: the phase
// eta_mu(x) is multiplied into U_mu in advance), builds the eight hop links
// of every output site (sixteen for the improved operator; backward links
// daggered and negated, so the Dirac operator of Eq.5 becomes a plain sum),
// splits by parity and writes the word-major layout of common.h, rounding
// to the storage precision.
#include "kern.h"
#include "launch.h"

namespace stag {

__device__ __forceinline__ double eta_of(int mu, int x, int y, int z) {
    // eta_mu(x) = (-1)^(x_0 + ... + x_{mu-1})
    int s = 0;
    if (mu > 0) s += x;
    if (mu > 1) s += y;
    if (mu > 2) s += z;
    return (s & 1) ? -1.0 : 1.0;
}

// Hop pair pr of site s in the tiled link storage (common.h).
template <int P>
__device__ __forceinline__ char* pair_at(void* G, uint32_t s, int pr, int npairs, bool r12) {
    const uint32_t pb = link_pair_bytes(P, r12);
    return (char*)G + (size_t)(s / kLinkTile) * (kLinkTile * npairs * pb) + (size_t)pr * (kLinkTile * pb);
}

// A stored link has no NaN but the canonical one, of either sign: the resident
// kernel marks empty words with another, which links in memory filled with ones
// would pass on.
__device__ __forceinline__ double plain_nan(double v) { return v == v ? v : __longlong_as_double(0x7ff8ll << 48); }

// ------------------------------------------------------------------ fp64 and fp32 copies in one pass

// Where one field of links goes: U (or the fat links) to pairs 0..3 over one
// hop, the long links to pairs 4..7 over three.
struct ScatterArgs {
    const d2v* W;        // canonical links
    char* G64[2];        // copies by output parity, null: not stored
    char* G32[2];
    Geom g;
    int three;           // three-hop links
    int npairs;
    int* bad;            // r12: set when a link is not SU(3) within tol (null: no check)
    double tol;
};

// max |U U^+ - 1| and |det U - 1| of a 3x3 matrix.
__device__ __forceinline__ double su3_error(const double (&ur)[9], const double (&ui)[9]) {
    double err = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            // (U U^+)_ik = sum_j U_ij conj(U_kj)
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                re += ur[3 * i + j] * ur[3 * k + j] + ui[3 * i + j] * ui[3 * k + j];
                im += ui[3 * i + j] * ur[3 * k + j] - ur[3 * i + j] * ui[3 * k + j];
            }
            if (i == k) re -= 1.0;
            err = fmax(err, fmax(fabs(re), fabs(im)));
        }
    // det U = row0 . (row1 x row2)
    auto cm = [](double ar, double ai, double br, double bi, double& cr, double& ci) {
        cr = ar * br - ai * bi;
        ci = ar * bi + ai * br;
    };
    double dr = 0.0, di = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int k1 = (k + 1) % 3, k2 = (k + 2) % 3;
        double pr, pi, qr, qi;
        cm(ur[3 + k1], ui[3 + k1], ur[6 + k2], ui[6 + k2], pr, pi);
        cm(ur[3 + k2], ui[3 + k2], ur[6 + k1], ui[6 + k1], qr, qi);
        double tr, ti;
        cm(ur[k], ui[k], pr - qr, pi - qi, tr, ti);
        dr += tr;
        di += ti;
    }
    return fmax(err, fmax(fabs(dr - 1.0), fabs(di)));
}

// Entries HALF (0: forward, 1: backward half) of a hop pair at site s: NC / 2 of
// the pair's NC complex entries.
template <int NC>
__device__ __forceinline__ void store_half(char* G64, char* G32, uint32_t s, int pr, int npairs, int half,
                                           const double (&lr)[NC / 2], const double (&li)[NC / 2]) {
    constexpr int H = NC / 2;
    constexpr bool r12 = NC == 12;
    const uint32_t i = s % kLinkTile;
    if (G64) {
        d2v* o = (d2v*)pair_at<P64>(G64, s, pr, npairs, r12) + i + (uint32_t)half * (H * kLinkTile);
#pragma unroll
        for (int e = 0; e < H; ++e) {
            d2v v;
            v.x = lr[e];
            v.y = li[e];
            o[e * kLinkTile] = v;
        }
    }
    if (G32) {
        f4v* o = (f4v*)pair_at<P32>(G32, s, pr, npairs, r12);
        // words of two entries; with nine entries a half the middle word is shared
        auto two = [&](int w, int e) {
            f4v v;
            v.x = (float)lr[e];
            v.y = (float)li[e];
            v.z = (float)lr[e + 1];
            v.w = (float)li[e + 1];
            o[w * kLinkTile + i] = v;
        };
        if constexpr (r12) {
#pragma unroll
            for (int w = 0; w < 3; ++w) two(3 * half + w, 2 * w);
        } else {
            f2v v;
            v.x = (float)(half ? lr[0] : lr[8]);
            v.y = (float)(half ? li[0] : li[8]);
            ((f2v*)(o + 4 * kLinkTile + i))[half] = v;
            if (half) {
#pragma unroll
                for (int w = 0; w < 4; ++w) two(5 + w, 2 * w + 1);
            } else {
#pragma unroll
                for (int w = 0; w < 4; ++w) two(w, 2 * w);
            }
        }
    }
}

// Every canonical link read once and written to both of its places, in both
// precisions: the forward half of its own site's pair and the backward half
// (daggered, negated) of its forward neighbour's. A block takes 64 consecutive
// sites, whose links are one run of 36 KiB, through LDS (a site's 576 bytes
// are four links for four threads); a thread's stores then lie beside those of
// the other sites of its parity. Bound by the stores' traffic. Before it each
// copy and parity was packed by a kernel of its own that read the links twice,
// straight from each site's thread, and the SU(3) check read them once more:
// 24^3 x 48, fp64 and fp32 12-parameter copies, 4 x 152 + 96 us; this kernel 232 us
// (1.15 GB, 4.9 TB/s).
constexpr int kScatterSites = 64;
constexpr int kSitePitch = 37;  // 36 entries of a site and one of padding (LDS banks)
template <bool R12>
__global__ __launch_bounds__(kBlock) void k_gauge_scatter(ScatterArgs a) {
    __shared__ d2v run[kScatterSites * kSitePitch];
    const uint64_t V = 2ull * a.g.Vh;
    const uint64_t base = (uint64_t)blockIdx.x * kScatterSites;
    const uint32_t sites = (uint32_t)(V - base < (uint64_t)kScatterSites ? V - base : (uint64_t)kScatterSites);
    const d2v* W = a.W + base * 36;
#pragma unroll
    for (int k = 0; k < kScatterSites * 36 / kBlock; ++k) {
        const uint32_t i = k * kBlock + threadIdx.x;
        const uint32_t site = i / 36;
        if (site < sites) run[site * kSitePitch + (i - site * 36)] = __builtin_nontemporal_load(W + i);
    }
    __syncthreads();
    // thread: direction, parity, and which of the run's 32 sites of that parity
    const int mu = threadIdx.x >> 6, p = (threadIdx.x >> 5) & 1;
    const uint32_t s = (uint32_t)(base >> 1) + (threadIdx.x & 31);
    if (s >= a.g.Vh) return;
    int x, y, z, t;
    site_coords(a.g, s, p, x, y, z, t);
    uint32_t nf, nb;
    if (a.three) {
        neighbours3(a.g, s, x, y, z, t, mu, nf, nb);
    } else {
        neighbours(a.g, s, x, y, z, t, mu, nf, nb);
    }
    const uint32_t lex = 2 * s + ((y + z + t + p) & 1);
    const d2v* u = run + (lex - (uint32_t)base) * kSitePitch + mu * 9;
    double ur[9], ui[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        const d2v v = u[e];
        ur[e] = plain_nan(v.x);
        ui[e] = plain_nan(v.y);
    }
    if constexpr (R12) {
        if (a.bad && !(su3_error(ur, ui) <= a.tol)) *a.bad = 1;
    }
    const int pr = mu + (a.three ? 4 : 0);
    constexpr int NC = R12 ? 12 : 18, H = NC / 2;
    double fr[H], fi[H], br[H], bi[H];
    // 12-parameter links without phases; full ones with eta folded in
    const double eta = R12 ? 1.0 : eta_of(mu, x, y, z);
#pragma unroll
    for (int i = 0; i < H / 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            fr[3 * i + k] = eta * ur[3 * i + k];
            fi[3 * i + k] = eta * ui[3 * i + k];
            // U^dagger (12 parameters) or -(eta U)^dagger: entry (i, k) from U[k][i]
            br[3 * i + k] = R12 ? ur[3 * k + i] : -eta * ur[3 * k + i];
            bi[3 * i + k] = R12 ? -ui[3 * k + i] : eta * ui[3 * k + i];
        }
    store_half<NC>(a.G64[p], a.G32[p], s, pr, a.npairs, 0, fr, fi);
    store_half<NC>(a.G64[1 - p], a.G32[1 - p], nf, pr, a.npairs, 1, br, bi);
}

hipError_t launch_gauge_scatter(const void* W_dev, bool three, int npairs, void* const G64[2],
                                void* const G32[2], const Geom& g, bool r12, double tol, int* bad_dev,
                                hipStream_t st) {
    if (r12 && (three || npairs != 4)) return hipErrorInvalidValue;
    ScatterArgs a{};
    a.W = (const d2v*)W_dev;
    for (int q = 0; q < 2; ++q) {
        a.G64[q] = (char*)G64[q];
        a.G32[q] = (char*)G32[q];
    }
    a.g = g;
    a.three = three ? 1 : 0;
    a.npairs = npairs;
    a.bad = bad_dev;
    a.tol = tol;
    const dim3 grid((uint32_t)((2ull * g.Vh + kScatterSites - 1) / kScatterSites)), block(kBlock);
    if (r12) {
        hipLaunchKernelGGL((k_gauge_scatter<true>), grid, block, 0, st, a);
    } else {
        hipLaunchKernelGGL((k_gauge_scatter<false>), grid, block, 0, st, a);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ fp16 copies, check

// Hop pair pr of output site c (pairs 0..3: one-hop over U, pairs 4..7 of
// the improved operator: three-hop over Ulong): 18 complex in fp64, the
// forward link eta W(x) then -(eta W(x - h))^dagger.
__device__ __forceinline__ void hop_pair(const d2v* __restrict__ U, const d2v* __restrict__ Ulong,
                                         const Geom& g, const int (&c)[4], int pr, double (&lr)[18],
                                         double (&li)[18]) {
    const int mu = pr & 3;
    const int dist = pr < 4 ? 1 : 3;
    const d2v* W = pr < 4 ? U : Ulong;
    const int Lx = g.L[0], Ly = g.L[1], Lz = g.L[2];
    auto lex_of = [&](const int* q) -> size_t {
        return (size_t)q[0] + (size_t)Lx * ((size_t)q[1] + (size_t)Ly * ((size_t)q[2] + (size_t)Lz * q[3]));
    };
    int b[4] = {c[0], c[1], c[2], c[3]};
    b[mu] -= dist;
    while (b[mu] < 0) b[mu] += g.L[mu];
    const double ef = eta_of(mu, c[0], c[1], c[2]);
    const double eb = eta_of(mu, b[0], b[1], b[2]);
    const d2v* uf = W + (lex_of(c) * 4 + mu) * 9;
    const d2v* ub = W + (lex_of(b) * 4 + mu) * 9;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const d2v f = uf[i * 3 + k];
            lr[3 * i + k] = ef * plain_nan(f.x);
            li[3 * i + k] = ef * plain_nan(f.y);
            // -(eb W)^dagger: entry (i, k) = -eb conj(W[k][i])
            const d2v v = ub[k * 3 + i];
            lr[9 + 3 * i + k] = -eb * plain_nan(v.x);
            li[9 + 3 * i + k] = eb * plain_nan(v.y);
        }
}

// Divide the NC (12 or 18) complex entries of a hop pair by the site scale sc,
// round them to fp16 and write their words for site i of the tile.
template <int NC>
__device__ __forceinline__ void store_pair16(char* tile, uint32_t i, const double (&lr)[NC],
                                             const double (&li)[NC], float sc) {
    unsigned q[NC];
#pragma unroll
    for (int e = 0; e < NC; ++e)
        q[e] = sc == 0.f ? 0u : f2h_pair(__fdiv_rn((float)lr[e], sc), __fdiv_rn((float)li[e], sc));
    u4v* o = (u4v*)tile;
#pragma unroll
    for (int w = 0; w < NC / 4; ++w) {
        u4v v;
        v.x = q[4 * w];
        v.y = q[4 * w + 1];
        v.z = q[4 * w + 2];
        v.w = q[4 * w + 3];
        o[w * kLinkTile + i] = v;
    }
    if constexpr (NC % 4 != 0) {
        u2v v;
        v.x = q[NC - 2];
        v.y = q[NC - 1];
        ((u2v*)(o + (NC / 4) * kLinkTile))[i] = v;
    }
}

// Full (18-parameter) packing of every hop pair to fp16, whose scale needs all
// the links that an output site reads; Ulong null: Eq.5's four pairs, else the
// improved operator's eight.
__global__ __launch_bounds__(kBlock) void k_gauge_pack16(const d2v* __restrict__ U,
                                                         const d2v* __restrict__ Ulong, void* G,
                                                         float* gscale, Geom g, int p_out) {
    const uint32_t s = blockIdx.x * kBlock + threadIdx.x;
    if (s >= g.Vh) return;
    int c[4];
    site_coords(g, s, p_out, c[0], c[1], c[2], c[3]);
    const int np = Ulong ? 8 : 4;
    double lr[18], li[18];
    // one fp32 scale per output site over all the reals it reads
    float sc = 0.f;
#pragma unroll 1
    for (int pr = 0; pr < np; ++pr) {
        hop_pair(U, Ulong, g, c, pr, lr, li);
#pragma unroll
        for (int e = 0; e < 18; ++e) sc = fmaxf(sc, fmaxf(fabsf((float)lr[e]), fabsf((float)li[e])));
    }
    gscale[s] = sc;
#pragma unroll 1
    for (int pr = 0; pr < np; ++pr) {
        hop_pair(U, Ulong, g, c, pr, lr, li);
        store_pair16<18>(pair_at<P16S>(G, s, pr, np, false), s % kLinkTile, lr, li, sc);
    }
}

// 12-parameter packing to fp16: the first two rows of U_mu(x) and of
// U_mu(x - mu)^dagger per hop pair, without phases (layout in common.h),
// divided by the site scale of the full packing (the largest |Re| or
// |Im| over all 144 reals of the site's eight links, third rows included).
__global__ __launch_bounds__(kBlock) void k_gauge_pack12_16(const d2v* __restrict__ U, void* G,
                                                            float* gscale, Geom g, int p_out) {
    const uint32_t s = blockIdx.x * kBlock + threadIdx.x;
    if (s >= g.Vh) return;
    int c[4];
    site_coords(g, s, p_out, c[0], c[1], c[2], c[3]);
    const int Lx = g.L[0], Ly = g.L[1], Lz = g.L[2];
    auto lex_of = [&](const int* q) -> size_t {
        return (size_t)q[0] + (size_t)Lx * ((size_t)q[1] + (size_t)Ly * ((size_t)q[2] + (size_t)Lz * q[3]));
    };
    double lr[48], li[48];
    float sc = 0.f;
    const size_t lex = lex_of(c);
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        int b[4] = {c[0], c[1], c[2], c[3]};
        b[mu] = (b[mu] == 0) ? g.L[mu] - 1 : b[mu] - 1;
        const d2v* uf = U + (lex * 4 + mu) * 9;
        const d2v* ub = U + (lex_of(b) * 4 + mu) * 9;
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            const d2v f = uf[e], v = ub[e];
            sc = fmaxf(sc, fmaxf(fabsf((float)f.x), fabsf((float)f.y)));
            sc = fmaxf(sc, fmaxf(fabsf((float)v.x), fabsf((float)v.y)));
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const d2v f = uf[i * 3 + k];
                lr[12 * mu + 3 * i + k] = f.x;
                li[12 * mu + 3 * i + k] = f.y;
                // U^dagger: entry (i, k) = conj(U[k][i])
                const d2v v = ub[k * 3 + i];
                lr[12 * mu + 6 + 3 * i + k] = v.x;
                li[12 * mu + 6 + 3 * i + k] = -v.y;
            }
    }
    gscale[s] = sc;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        double pr[12], pi[12];
#pragma unroll
        for (int e = 0; e < 12; ++e) {
            pr[e] = lr[12 * mu + e];
            pi[e] = li[12 * mu + e];
        }
        store_pair16<12>(pair_at<P16S>(G, s, mu, 4, true), s % kLinkTile, pr, pi, sc);
    }
}

// Flag (bad = 1) every link with max |U U^+ - 1| or |det U - 1| above tol.
// All writers store the same value, so the race is benign.
__global__ __launch_bounds__(kBlock) void k_su3_check(const d2v* __restrict__ U, uint64_t nlinks,
                                                      double tol, int* bad) {
    const uint64_t l = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (l >= nlinks) return;
    double ur[9], ui[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        const d2v v = U[l * 9 + e];
        ur[e] = v.x;
        ui[e] = v.y;
    }
    const double err = su3_error(ur, ui);
    if (!(err <= tol)) *bad = 1;
}

hipError_t launch_su3_check(const void* U_dev, uint64_t nlinks, double tol, int* bad_dev,
                            hipStream_t st) {
    const uint64_t nb = (nlinks + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_su3_check, dim3((uint32_t)nb), dim3(kBlock), 0, st, (const d2v*)U_dev, nlinks,
                       tol, bad_dev);
    return hipGetLastError();
}

hipError_t launch_gauge_pack16(const void* U_dev, const void* Ulong_dev, void* G, float* gscale,
                               const Geom& g, int p_out, bool r12, hipStream_t st) {
    if (r12 && Ulong_dev) return hipErrorInvalidValue;
    const dim3 grid((g.Vh + kBlock - 1) / kBlock), block(kBlock);
    const d2v* U = (const d2v*)U_dev;
    if (r12) {
        hipLaunchKernelGGL(k_gauge_pack12_16, grid, block, 0, st, U, G, gscale, g, p_out);
    } else {
        hipLaunchKernelGGL(k_gauge_pack16, grid, block, 0, st, U, (const d2v*)Ulong_dev, G, gscale, g, p_out);
    }
    return hipGetLastError();
}

// Canonical spinors: complex128 [nrhs][Vh][3].
template <int P>
__global__ __launch_bounds__(kBlock) void k_import(const d2v* __restrict__ src, void* dst,
                                                   size_t dst_rs, uint32_t Vh) {
    using T = typename Real<P>::T;
    const uint32_t s = blockIdx.x * kBlock + threadIdx.x;
    const int r = blockIdx.y;
    if (s >= Vh) return;
    const d2v* p = src + ((size_t)r * Vh + s) * 3;
    T re[3], im[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const d2v v = p[c];
        re[c] = (T)v.x;
        im[c] = (T)v.y;
    }
    store_site<P>((char*)dst + (size_t)r * dst_rs, Vh, s, re, im);
}

// A block's 256 sites are one run of 12 KiB in the canonical layout, written
// in order from LDS: storing the three colours of a site from its own thread
// writes every 128-byte line of the run in three parts (32^3 x 64 fp32: 17.5 us;
// through LDS 12.7, 5.9 TB/s). Reading that way costs nothing extra (the
// import: 14 us either way).
template <int P>
__global__ __launch_bounds__(kBlock) void k_export(const void* src, size_t src_rs, d2v* dst,
                                                   uint32_t Vh) {
    using T = typename Real<P>::T;
    __shared__ d2v run[3 * kBlock];
    const uint32_t s = blockIdx.x * kBlock + threadIdx.x;
    const int r = blockIdx.y;
    if (s < Vh) {
        T re[3], im[3];
        load_site<P>((const char*)src + (size_t)r * src_rs, Vh, s, re, im);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            d2v v;
            v.x = (double)re[c];
            v.y = (double)im[c];
            run[3 * threadIdx.x + c] = v;
        }
    }
    __syncthreads();
    const uint32_t s0 = blockIdx.x * kBlock;
    const uint32_t n = 3 * (Vh - s0 < (uint32_t)kBlock ? Vh - s0 : (uint32_t)kBlock);
    d2v* p = dst + ((size_t)r * Vh + s0) * 3;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const uint32_t i = k * kBlock + threadIdx.x;
        if (i < n) p[i] = run[i];
    }
}

hipError_t launch_import(int prec, const void* src_dev, void* dst, size_t dst_rs, uint32_t Vh,
                         int nrhs, hipStream_t st) {
    const dim3 grid((Vh + kBlock - 1) / kBlock, nrhs), block(kBlock);
    const d2v* src = (const d2v*)src_dev;
    switch (prec) {
        case P64: hipLaunchKernelGGL((k_import<P64>), grid, block, 0, st, src, dst, dst_rs, Vh); break;
        case P32: hipLaunchKernelGGL((k_import<P32>), grid, block, 0, st, src, dst, dst_rs, Vh); break;
        case P16S: hipLaunchKernelGGL((k_import<P16S>), grid, block, 0, st, src, dst, dst_rs, Vh); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_export(int prec, const void* src, size_t src_rs, void* dst_dev, uint32_t Vh,
                         int nrhs, hipStream_t st) {
    const dim3 grid((Vh + kBlock - 1) / kBlock, nrhs), block(kBlock);
    d2v* dst = (d2v*)dst_dev;
    switch (prec) {
        case P64: hipLaunchKernelGGL((k_export<P64>), grid, block, 0, st, src, src_rs, dst, Vh); break;
        case P32: hipLaunchKernelGGL((k_export<P32>), grid, block, 0, st, src, src_rs, dst, Vh); break;
        case P16S: hipLaunchKernelGGL((k_export<P16S>), grid, block, 0, st, src, src_rs, dst, Vh); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace stag

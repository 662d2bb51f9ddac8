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
            lr[3 * i + k] = ef * f.x;
            li[3 * i + k] = ef * f.y;
            // -(eb W)^dagger: entry (i, k) = -eb conj(W[k][i])
            const d2v v = ub[k * 3 + i];
            lr[9 + 3 * i + k] = -eb * v.x;
            li[9 + 3 * i + k] = eb * v.y;
        }
}

// Hop pair pr of site s in the tiled link storage (common.h).
template <int P>
__device__ __forceinline__ char* pair_at(void* G, uint32_t s, int pr, int npairs, bool r12) {
    const uint32_t pb = link_pair_bytes(P, r12);
    return (char*)G + (size_t)(s / kLinkTile) * (kLinkTile * npairs * pb) + (size_t)pr * (kLinkTile * pb);
}

// Round the NC (12 or 18) complex entries of a hop pair to the storage
// precision and write their words for site i of the tile (P16S: divided by
// the site scale sc).
template <int P, int NC>
__device__ __forceinline__ void store_pair(char* tile, uint32_t i, const double (&lr)[NC],
                                           const double (&li)[NC], float sc) {
    if constexpr (P == P64) {
        d2v* o = (d2v*)tile + i;
#pragma unroll
        for (int e = 0; e < NC; ++e) {
            d2v v;
            v.x = lr[e];
            v.y = li[e];
            o[e * kLinkTile] = v;
        }
    } else if constexpr (P == P32) {
        f4v* o = (f4v*)tile + i;
#pragma unroll
        for (int w = 0; w < NC / 2; ++w) {
            f4v v;
            v.x = (float)lr[2 * w];
            v.y = (float)li[2 * w];
            v.z = (float)lr[2 * w + 1];
            v.w = (float)li[2 * w + 1];
            o[w * kLinkTile] = v;
        }
    } else {
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
}

// Full (18-parameter) packing of every hop pair; Ulong null: Eq.5's four
// pairs, else the improved operator's eight.
template <int P>
__global__ __launch_bounds__(kBlock) void k_gauge_pack(const d2v* __restrict__ U,
                                                       const d2v* __restrict__ Ulong, void* G,
                                                       float* gscale, Geom g, int p_out) {
    const uint32_t s = blockIdx.x * kBlock + threadIdx.x;
    if (s >= g.Vh) return;
    int c[4];
    site_coords(g, s, p_out, c[0], c[1], c[2], c[3]);
    const int np = Ulong ? 8 : 4;
    double lr[18], li[18];
    float sc = 0.f;
    if constexpr (P == P16S) {
        // one fp32 scale per output site over all the reals it reads
#pragma unroll 1
        for (int pr = 0; pr < np; ++pr) {
            hop_pair(U, Ulong, g, c, pr, lr, li);
#pragma unroll
            for (int e = 0; e < 18; ++e)
                sc = fmaxf(sc, fmaxf(fabsf((float)lr[e]), fabsf((float)li[e])));
        }
        gscale[s] = sc;
    }
#pragma unroll 1
    for (int pr = 0; pr < np; ++pr) {
        hop_pair(U, Ulong, g, c, pr, lr, li);
        store_pair<P, 18>(pair_at<P>(G, s, pr, np, false), s % kLinkTile, lr, li, sc);
    }
}

// 12-parameter packing: the first two rows of U_mu(x) and of
// U_mu(x - mu)^dagger per hop pair, without phases (layout in common.h).
// P16S divides by the site scale of the full packing (the largest |Re| or
// |Im| over all 144 reals of the site's eight links, third rows included).
template <int P>
__global__ __launch_bounds__(kBlock) void k_gauge_pack12(const d2v* __restrict__ U, void* G,
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
        if constexpr (P == P16S) {
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                const d2v f = uf[e], v = ub[e];
                sc = fmaxf(sc, fmaxf(fabsf((float)f.x), fabsf((float)f.y)));
                sc = fmaxf(sc, fmaxf(fabsf((float)v.x), fabsf((float)v.y)));
            }
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
    if constexpr (P == P16S) gscale[s] = sc;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        double pr[12], pi[12];
#pragma unroll
        for (int e = 0; e < 12; ++e) {
            pr[e] = lr[12 * mu + e];
            pi[e] = li[12 * mu + e];
        }
        store_pair<P, 12>(pair_at<P>(G, s, mu, 4, true), s % kLinkTile, pr, pi, sc);
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
    err = fmax(err, fmax(fabs(dr - 1.0), fabs(di)));
    if (!(err <= tol)) *bad = 1;
}

hipError_t launch_su3_check(const void* U_dev, uint64_t nlinks, double tol, int* bad_dev,
                            hipStream_t st) {
    const uint64_t nb = (nlinks + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_su3_check, dim3((uint32_t)nb), dim3(kBlock), 0, st, (const d2v*)U_dev, nlinks,
                       tol, bad_dev);
    return hipGetLastError();
}

hipError_t launch_gauge_pack(int prec, const void* U_dev, const void* Ulong_dev, void* G,
                             float* gscale, const Geom& g, int p_out, bool r12, hipStream_t st) {
    if (r12 && Ulong_dev) return hipErrorInvalidValue;
    if (r12) {
        const dim3 grid((g.Vh + kBlock - 1) / kBlock), block(kBlock);
        const d2v* U = (const d2v*)U_dev;
        switch (prec) {
            case P64: hipLaunchKernelGGL((k_gauge_pack12<P64>), grid, block, 0, st, U, G, gscale, g, p_out); break;
            case P32: hipLaunchKernelGGL((k_gauge_pack12<P32>), grid, block, 0, st, U, G, gscale, g, p_out); break;
            case P16S: hipLaunchKernelGGL((k_gauge_pack12<P16S>), grid, block, 0, st, U, G, gscale, g, p_out); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    const dim3 grid((g.Vh + kBlock - 1) / kBlock), block(kBlock);
    const d2v* U = (const d2v*)U_dev;
    const d2v* N = (const d2v*)Ulong_dev;
    switch (prec) {
        case P64: hipLaunchKernelGGL((k_gauge_pack<P64>), grid, block, 0, st, U, N, G, gscale, g, p_out); break;
        case P32: hipLaunchKernelGGL((k_gauge_pack<P32>), grid, block, 0, st, U, N, G, gscale, g, p_out); break;
        case P16S: hipLaunchKernelGGL((k_gauge_pack<P16S>), grid, block, 0, st, U, N, G, gscale, g, p_out); break;
        default: return hipErrorInvalidValue;
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

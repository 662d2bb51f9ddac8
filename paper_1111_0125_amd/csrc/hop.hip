// Hop kernel: the staggered Dirac operator of Eq.5 applied from one parity
// to the other, with optional second-stage epilogues that complete
// A = m^2 - D_eo D_oe (Eq.3). The phases of Sec.2 are folded into stored full
// links; with 12-parameter links they multiply each hop pair's outputs (as
// does the fp16 site scale: PairScale).
//
// The operator is a sum over NP hop pairs, each a forward and a backward hop
// whose two 3x3 links are stored contiguously per site: NP = 4 for Eq.5
// (pair mu: x +- mu), NP = 8 for the improved operator (pairs 4 + mu add the
// three-hops x +- 3mu over the long links). One output site is handled by S
// lanes of a wavefront (S = 1, 2 or 4); lane j of a site takes the pairs
// [j*NP/S, (j+1)*NP/S), and the S partial colour vectors are summed with
// cross-lane adds. With N > 1 right-hand sides every link is loaded once and
// applied to all of them (the block operator sharing gauge loads).
//
// This file is compiled once per storage precision (HOP_PREC) and pair
// count (HOP_NP).
#include <type_traits>

#include "kern.h"
#include "launch.h"

#ifndef HOP_PREC
#error "HOP_PREC must be defined"
#endif
#ifndef HOP_NP
#define HOP_NP 4
#endif
namespace stag {

// What an operand is made of at one site: the stored input and, for a
// deferred direction update, the stored residual.
template <int P>
struct Raw {
    typename Real<P>::T vr[3], vi[3], rr[3], ri[3];
};

// Load the raw operand of RHS r at site n (the residual only when `lazy`).
template <int P>
__device__ __forceinline__ void load_raw(const HopArgs& a, const char* in_r, int r, uint32_t n,
                                         bool lazy, Raw<P>& w) {
    load_site<P>(in_r, a.g.Vh, n, w.vr, w.vi);
    if (lazy) load_site<P>((const char*)a.lazy_r + (size_t)r * a.lazy_r_rs, a.g.Vh, n, w.rr, w.ri);
}

// The operand from its raw parts: the stored input, or d_new = q(r + beta d)
// for a deferred direction update; with `add_y` in the fp64 stages of a
// reliable update (x gathered by stage 1, x at stage 2's own site), x + y.
template <int P>
__device__ __forceinline__ void combine(const HopArgs& a, const Raw<P>& w, int r, uint32_t n,
                                        bool lazy, double beta, bool add_y,
                                        typename Real<P>::T (&vr)[3],
                                        typename Real<P>::T (&vi)[3]) {
    using T = typename Real<P>::T;
    if (lazy) {
        const T be = (T)beta;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            vr[c] = fma(be, w.vr[c], w.rr[c]);
            vi[c] = fma(be, w.vi[c], w.ri[c]);
        }
        round_site<P>(vr, vi);
    } else {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            vr[c] = w.vr[c];
            vi[c] = w.vi[c];
        }
    }
    if constexpr (P == P64) {
        if (add_y && a.lazy_y) {
            float yr[3], yi[3];
            load_site<P32>((const char*)a.lazy_y + (size_t)r * a.lazy_y_rs, a.g.Vh, n, yr, yi);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                vr[c] = vr[c] + (T)yr[c];
                vi[c] = vi[c] + (T)yi[c];
            }
        }
    }
}

// The own-site operand of stage 2 (x, formed like a stage-1 operand).
template <int P>
__device__ __forceinline__ void load_operand(const HopArgs& a, const char* in_r, int r, uint32_t n,
                                             bool lazy, double beta, typename Real<P>::T (&vr)[3],
                                             typename Real<P>::T (&vi)[3]) {
    Raw<P> w;
    load_raw<P>(a, in_r, r, n, lazy, w);
    combine<P>(a, w, r, n, lazy, beta, true, vr, vi);
}

// Neighbours of hop pair pr (pairs 4..7 are the three-hops of the improved operator).
template <int NP>
__device__ __forceinline__ void pair_neighbours(const Geom& g, uint32_t s, int x, int y, int z,
                                                int t, int pr, uint32_t& nf, uint32_t& nb) {
    if (NP == 4 || pr < 4) {
        neighbours(g, s, x, y, z, t, pr & 3, nf, nb);
    } else {
        neighbours3(g, s, x, y, z, t, pr & 3, nf, nb);
    }
}

// Load a colour vector from field f (a kernel argument, so uniform): the
// plane's address stays in scalar registers and the site is a 32-bit offset
// to it (sites per parity below kHop32MaxSites).
template <int P>
__device__ __forceinline__ void load_site32(const void* f, uint32_t Vh, uint32_t s,
                                            typename Real<P>::T (&re)[3],
                                            typename Real<P>::T (&im)[3]) {
    if constexpr (P == P16S) {
        f16s_decode(*(const u4v*)((const char*)f + s * 16u), re, im);
    } else {
        using V = std::conditional_t<P == P64, d2v, f2v>;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const V v = *(const V*)((const char*)f + (size_t)c * Vh * sizeof(V) + s * (uint32_t)sizeof(V));
            re[c] = v.x;
            im[c] = v.y;
        }
    }
}

// Planes of at most 4 GiB (16 bytes a site), for the 32-bit offsets above.
constexpr uint32_t kHop32MaxSites = 1u << 27;

// Where hop_all serves: the default launch shape (four pairs per lane) and
// blocks of up to 8; the improved operator's fp64 and fp32 blocks of 2 to 4 stay with
// the branching loop (16^3 x 32 fp64 with 4 RHS: 50.9 / 41.8 us there, 53.1 / 46.6
// here).
template <int P, int S, int N, int NP>
constexpr bool kUseHopAll = N > 1 && N <= 8 && S == NP / 4 && (NP == 4 || N == 8 || P == P16S);

// The pair sums of several right-hand sides, all of them active, at output
// site sl (every lane of the wavefront has one): the operands of right-hand
// side and pair i + AHEAD are requested before the products of i, with no
// branch per right-hand side in between, and the next pair's links before
// this pair's products (8 RHS: three ahead and the links with them, which
// leaves the registers). Stage 1 / stage 2 at 24^3 x 48 with 12-parameter links,
// us, against the branching loop of k_hop below: fp32 with 4 RHS 42.2 / 46.6
// (45.4 / 55.4), 8 RHS 65.1 / 79.3 (79.0 / 90.5); fp64 8 RHS 122.7 / 164.4 (177.1 /
// 211.4), 2 and 4 the same; fp16 2 RHS 20.2 / 23.5 (25.8 / 28.1), 8 RHS 56.0 / 69.3
// (76.7 / 75.6). fp32 with one request ahead: 4 RHS 43.5 / 49.2, 8 RHS 74.0 / 89.3.
template <int P, int S, int N, int EPI, bool NT, int NP, bool R12, bool LAZY>
__device__ __forceinline__ void hop_all(const HopArgs& a, uint32_t sl, int x, int y, int z, int t, int j,
                                        const RhsState* ls, typename Real<P>::T (&ar)[N][3],
                                        typename Real<P>::T (&ai)[N][3]) {
    using T = typename Real<P>::T;
    constexpr int B = NP / S;
    constexpr int AHEAD = N >= 8 ? 3 : 2;
    constexpr bool LINKS_AHEAD = N < 8;
    const uint32_t Vh = a.g.Vh;
    uint32_t nf[B], nb[B];
    static_for<0, B>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        pair_neighbours<NP>(a.g, sl, x, y, z, t, j * B + k, nf[k], nb[k]);
    });
    struct Op {
        T fr[3], fi[3], br[3], bi[3];
        T gr[LAZY ? 3 : 1], gi[LAZY ? 3 : 1], hr[LAZY ? 3 : 1], hi[LAZY ? 3 : 1];
    };
    Op q[AHEAD];
    auto request = [&](int i, Op& w) {
        const int k = i / N, r = i % N;
        const char* in_r = (const char*)a.in + (size_t)r * a.in_rs;
        load_site32<P>(in_r, Vh, nf[k], w.fr, w.fi);
        load_site32<P>(in_r, Vh, nb[k], w.br, w.bi);
        if constexpr (LAZY) {
            const char* z_r = (const char*)a.lazy_r + (size_t)r * a.lazy_r_rs;
            load_site32<P>(z_r, Vh, nf[k], w.gr, w.gi);
            load_site32<P>(z_r, Vh, nb[k], w.hr, w.hi);
        }
    };
    PairRaw<P> lw;
    load_pair_raw<P, NT, NP>(a.gauge, a.gscale, sl, j * B, R12, lw);
    static_for<0, AHEAD>([&](auto ic) { request(decltype(ic)::value, q[decltype(ic)::value]); });
    T pdr[3][N][3], pdi[3][N][3];
    T lr[18], li[18];
    PairScale<T> ps;
    static_for<0, B * N>([&](auto ic) {
        constexpr int i = decltype(ic)::value, k = i / N, r = i % N;
        if constexpr (r == 0) {
            finish_pair<P>(R12, eta_sign((j * B + k) & 3, x, y, z), lw, lr, li, ps);
            if constexpr (LINKS_AHEAD && k + 1 < B) {
#pragma unroll
                for (int e = 0; e < 18; ++e) asm volatile("" : "+v"(lr[e]), "+v"(li[e])::"memory");
                load_pair_raw<P, NT, NP>(a.gauge, a.gscale, sl, j * B + k + 1, R12, lw);
            }
        }
        Op& w = q[i % AHEAD];
        T pr[3], pi[3];
        if constexpr (LAZY) {
            const T be = (T)ls[r].beta;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                w.fr[c] = fma(be, w.fr[c], w.gr[c]);
                w.fi[c] = fma(be, w.fi[c], w.gi[c]);
                w.br[c] = fma(be, w.br[c], w.hr[c]);
                w.bi[c] = fma(be, w.bi[c], w.hi[c]);
            }
            round_site<P>(w.fr, w.fi);
            round_site<P>(w.br, w.bi);
        }
        pair_start(lr, li, w.fr, w.fi, pr, pi);
        pair_finish(lr, li, ps, w.br, w.bi, pr, pi);
        // requests stay behind the products (an empty statement that uses them)
        if constexpr (i + AHEAD < B * N || (!LINKS_AHEAD && r == N - 1 && k + 1 < B)) {
#pragma unroll
            for (int c = 0; c < 3; ++c) asm volatile("" : "+v"(pr[c]), "+v"(pi[c])::"memory");
        }
        if constexpr (!LINKS_AHEAD && r == N - 1 && k + 1 < B)
            load_pair_raw<P, NT, NP>(a.gauge, a.gscale, sl, j * B + k + 1, R12, lw);
        if constexpr (i + AHEAD < B * N) request(i + AHEAD, w);
        // the balanced tree ((p0 + p1) + (p2 + p3)) + ...
        constexpr int lvl = (k & 1) == 0 ? 0 : (k & 2) == 0 ? 1 : (k & 4) == 0 ? 2 : 3;
#pragma unroll
        for (int l = 0; l < lvl; ++l)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                pr[c] = pdr[l][r][c] + pr[c];
                pi[c] = pdi[l][r][c] + pi[c];
            }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if constexpr (k == B - 1) {
                ar[r][c] = pr[c];
                ai[r][c] = pi[c];
            } else {
                pdr[lvl][r][c] = pr[c];
                pdi[lvl][r][c] = pi[c];
            }
        }
    });
}

template <int P, int S, int N, int EPI, bool NT, int NP>
__global__ __launch_bounds__(kBlock) void k_hop(HopArgs a) {
    // NP: hop pairs per site
    constexpr int B = NP / S;   // pairs per lane
    constexpr int LOGB = B >= 8 ? 3 : B >= 4 ? 2 : B >= 2 ? 1 : 0;
    static_assert(B >= 1 && (1 << LOGB) == B, "pairs per lane must be a power of two");
    using T = typename Real<P>::T;
    const uint32_t blk = logical_block(a.swizzle, a.tile_bps);
    const uint32_t gt = blk * kBlock + threadIdx.x;
    const uint32_t s = gt / S;
    const int j = (int)(gt % S);
    const uint32_t Vh = a.g.Vh;
    const bool valid = s < Vh;
    // stage 1 forms the deferred direction at the neighbours it gathers
    const bool lazy_nb = EPI == EPI_PLAIN && a.lazy_r != nullptr;
    // the improved operator's fat and long links are always stored full
    const int r12 = NP == 4 ? a.r12 : 0;

    // Per-RHS state, finalised here from the previous reduction's partials
    // when a.fin is set. One RHS: each wavefront keeps it in registers (no
    // barrier); the state, the operands of the lane's hop pairs (all of them
    // when they fit in registers, else the first), the own-site operand of
    // the second stage and the partials are all requested before any of them
    // is used, so their memory latencies overlap (an inactive slot reads the
    // operands and discards them). Neighbours go before links: rebuilding
    // 12-parameter links waits for the link loads, and would hold back loads
    // issued after them. Several RHS: the block shares one copy in LDS.
    constexpr bool PRE = N == 1 && P != P16S && B * sizeof(T) <= 8;
    constexpr int PB = N == 1 ? (PRE ? B : 1) : 1;  // pairs requested up front
    __shared__ RhsState ls[N];
    RhsState s1{};
    unsigned act = (1u << N) - 1u;
    int x = 0, y = 0, z = 0, t = 0;
    if (valid) site_coords(a.g, s, a.p_out, x, y, z, t);
    [[maybe_unused]] uint32_t pnf[PB], pnb[PB];
    [[maybe_unused]] PairRaw<P> pl[PB];
    [[maybe_unused]] Raw<P> pwf[PB], pwb[PB], pown;
    if constexpr (N == 1) {
        if constexpr (P == P64) {
            // gated launches (the fp64 fix-ups and checks): an unflagged slot
            // has nothing to do, no operand read and no partials (the
            // reduction's consumer skips unflagged slots). Its own load and
            // branch, so the others need not wait for the flags before
            // their operand loads; the inner-precision kernels, never gated,
            // carry no branch at all.
            if (a.gate) {
                if (!(a.st->flags & a.run_mask)) return;
            }
        }
        s1 = *(a.st ? a.st : &kNoState);
        if (a.st && !(s1.flags & a.run_mask)) act = 0;
        if (valid) {
            static_for<0, PB>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                pair_neighbours<NP>(a.g, s, x, y, z, t, j * B + k, pnf[k], pnb[k]);
                load_raw<P>(a, (const char*)a.in, 0, pnf[k], lazy_nb, pwf[k]);
                load_raw<P>(a, (const char*)a.in, 0, pnb[k], lazy_nb, pwb[k]);
            });
            if constexpr (PRE && EPI != EPI_PLAIN) {
                if (j == 0) load_raw<P>(a, (const char*)a.x, 0, s, a.lazy_r != nullptr, pown);
            }
            static_for<0, PB>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                load_pair_raw<P, NT, NP>(a.gauge, a.gscale, s, j * B + k, r12, pl[k]);
            });
        }
        if (a.st && a.fin.partials) {
            // always: block 0 must pass the state on even when it is inactive
            Reduce F = a.fin;
            F.st = a.st;
            finalize_wave1(F, a.run_mask, s1);
            if (!(s1.flags & a.run_mask)) act = 0;
        }
    } else if (a.st) {
        if (a.fin.partials) {
            Reduce F = a.fin;
            F.st = a.st;
            finalize_block<N>(F, a.run_mask, ls);
        } else {
            load_state<N>(a.st, ls);
        }
        act = 0;
#pragma unroll
        for (int r = 0; r < N; ++r)
            if (ls[r].flags & a.run_mask) act |= 1u << r;
    }
    auto stv = [&](int r) -> const RhsState& {
        if constexpr (N == 1) {
            return s1;
        } else {
            return ls[r];
        }
    };

    T ar[N][3], ai[N][3];
    // pending sums of the lane's pair tree: pd[l] holds the sum of the
    // 2^l pairs that wait for their right-hand sibling
    [[maybe_unused]] T pdr[LOGB > 0 ? LOGB : 1][N][3], pdi[LOGB > 0 ? LOGB : 1][N][3];
#pragma unroll
    for (int r = 0; r < N; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            ar[r][c] = ai[r][c] = T(0);
#pragma unroll
            for (int l = 0; l < (LOGB > 0 ? LOGB : 1); ++l) pdr[l][r][c] = pdi[l][r][c] = T(0);
        }

    bool done = false;
    if constexpr (kUseHopAll<P, S, N, NP>) {
        // every right-hand side active (the fp64 fix-ups gather x + y: below)
        if (act == (1u << N) - 1u && Vh < kHop32MaxSites && !(EPI == EPI_PLAIN && a.lazy_y)) {
            const uint32_t sl = valid ? s : Vh - 1;
            int cx, cy, cz, ct;
            site_coords(a.g, sl, a.p_out, cx, cy, cz, ct);
            auto all = [&](auto r12c, auto lazyc) {
                hop_all<P, S, N, EPI, NT, NP, decltype(r12c)::value, decltype(lazyc)::value>(
                    a, sl, cx, cy, cz, ct, j, ls, ar, ai);
            };
            if constexpr (EPI == EPI_PLAIN && N < 8) {
                if (lazy_nb) {
                    if (r12) all(std::true_type(), std::true_type());
                    else all(std::false_type(), std::true_type());
                    done = true;
                }
            }
            if (!lazy_nb) {
                if (r12) all(std::true_type(), std::false_type());
                else all(std::false_type(), std::false_type());
                done = true;
            }
        }
    }
    if (valid && act && !done) {
        // Each hop pair contributes p = F chi(x+h) + B chi(x-h), accumulated
        // from zero; the pairs are summed along a balanced binary tree
        // ((p0 + p1) + (p2 + p3)) + ..., lane-locally over the aligned block
        // of pairs this lane owns and across the S lanes of the site below.
        // This fixes the rounding independently of S and of the number of
        // right-hand sides.
        // (a loop over the lane's pairs with a compile-time index, so that
        // the arrays of operands requested up front stay in registers)
        static_for<0, B>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            const int mu = j * B + k;  // hop pair index
            uint32_t nf, nb;
            T lr[18], li[18];
            PairScale<T> ps;
            [[maybe_unused]] Raw<P> wfk, wbk;
            if constexpr (N == 1 && k < PB) {
                nf = pnf[k];
                nb = pnb[k];
                finish_pair<P>(r12, eta_sign(mu & 3, x, y, z), pl[k], lr, li, ps);
            } else {
                pair_neighbours<NP>(a.g, s, x, y, z, t, mu, nf, nb);
                if constexpr (N == 1) {
                    // one RHS: neighbours before links, as for the first pair
                    load_raw<P>(a, (const char*)a.in, 0, nf, lazy_nb, wfk);
                    load_raw<P>(a, (const char*)a.in, 0, nb, lazy_nb, wbk);
                }
                load_pair<P, NT, NP>(a.gauge, a.gscale, s, mu, r12, eta_sign(mu & 3, x, y, z), lr, li, ps);
            }
#pragma unroll
            for (int r = 0; r < N; ++r) {
                if (!((act >> r) & 1u)) continue;
                const char* in_r = (const char*)a.in + (size_t)r * a.in_rs;
                const double be = lazy_nb ? stv(r).beta : 0.0;
                Raw<P> wf, wb;
                if constexpr (N == 1 && k < PB) {
                    wf = pwf[k];
                    wb = pwb[k];
                } else if constexpr (N == 1) {
                    wf = wfk;
                    wb = wbk;
                } else {
                    load_raw<P>(a, in_r, r, nf, lazy_nb, wf);
                    load_raw<P>(a, in_r, r, nb, lazy_nb, wb);
                }
                T vr[3], vi[3], pr[3], pi[3];
                // stage 2 gathers t as stored
                combine<P>(a, wf, r, nf, lazy_nb, be, EPI == EPI_PLAIN, vr, vi);
                pair_start(lr, li, vr, vi, pr, pi);
                combine<P>(a, wb, r, nb, lazy_nb, be, EPI == EPI_PLAIN, vr, vi);
                pair_finish(lr, li, ps, vr, vi, pr, pi);
                // binary-counter walk of the tree: the new pair sum is
                // the right sibling of every pending sum at the levels
                // where k has a 1 bit, and waits at the first 0 bit
                T cr[3], ci[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    cr[c] = pr[c];
                    ci[c] = pi[c];
                }
                bool done = false;
#pragma unroll
                for (int l = 0; l < LOGB; ++l) {
                    if (done) continue;
                    if ((k >> l) & 1) {
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            cr[c] = pdr[l][r][c] + cr[c];
                            ci[c] = pdi[l][r][c] + ci[c];
                        }
                    } else {
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            pdr[l][r][c] = cr[c];
                            pdi[l][r][c] = ci[c];
                        }
                        done = true;
                    }
                }
                if (k == B - 1) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        ar[r][c] = cr[c];
                        ai[r][c] = ci[c];
                    }
                }
            }
        });
    }
    if constexpr (S > 1) {
        // lanes 2i and 2i + 1 hold the sums of consecutive aligned blocks;
        // xor 1 forms the sums of their parent nodes, xor 2 of the next
        // level. IEEE addition is commutative, so both lanes of each
        // exchange hold the same value.
#pragma unroll
        for (int r = 0; r < N; ++r)
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int off = 1; off < S; off <<= 1) {
                    ar[r][c] = ar[r][c] + __shfl_xor(ar[r][c], off, 64);
                    ai[r][c] = ai[r][c] + __shfl_xor(ai[r][c], off, 64);
                }
    }

    double dv[N];
#pragma unroll
    for (int r = 0; r < N; ++r) dv[r] = 0.0;

    if (valid && j == 0) {
#pragma unroll
        for (int r = 0; r < N; ++r) {
            if (!((act >> r) & 1u)) continue;
            char* out_r = (char*)a.out + (size_t)r * a.out_rs;
            if constexpr (EPI == EPI_PLAIN) {
                store_site<P>(out_r, Vh, s, ar[r], ai[r]);
            } else {
                T xr[3], xi[3], hr[3], hi[3];
                if constexpr (PRE) {
                    combine<P>(a, pown, r, s, a.lazy_r != nullptr, a.lazy_r ? stv(r).beta : 0.0, true,
                               xr, xi);
                } else {
                    load_operand<P>(a, (const char*)a.x + (size_t)r * a.x_rs, r, s, a.lazy_r != nullptr,
                                    a.lazy_r ? stv(r).beta : 0.0, xr, xi);
                }
                if (a.lazy_r) store_site<P>((char*)a.x + (size_t)r * a.x_rs, Vh, s, xr, xi);
                if constexpr (P == P64) {
                    if (a.lazy_y && !a.keep_y) {
                        // x += y in fp64, y = 0 (the group-wise update of Sec.3.2)
                        store_site<P>((char*)a.x + (size_t)r * a.x_rs, Vh, s, xr, xi);
                        float z[3] = {0.f, 0.f, 0.f}, zi[3] = {0.f, 0.f, 0.f};
                        store_site<P32>((char*)a.lazy_y + (size_t)r * a.lazy_y_rs, Vh, s, z, zi);
                    }
                }
                const T m2 = (T)(a.st ? stv(r).m2 : a.m2[r]);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    hr[c] = fma(m2, xr[c], -ar[r][c]);
                    hi[c] = fma(m2, xi[c], -ai[r][c]);
                }
                if constexpr (EPI == EPI_RESID) {
                    T br[3], bi[3];
                    load_site<P>((const char*)a.b + (size_t)r * a.b_rs, Vh, s, br, bi);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        hr[c] = br[c] - hr[c];
                        hi[c] = bi[c] - hi[c];
                    }
                    store_site<P>(out_r, Vh, s, hr, hi);
                    double acc = 0.0;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        acc = fma((double)hr[c], (double)hr[c], acc);
                        acc = fma((double)hi[c], (double)hi[c], acc);
                    }
                    dv[r] = acc;
                    if (a.aux) {
                        // the inner residual restarts from the true one: rs = q(r)
                        float qr[3], qi[3];
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            qr[c] = (float)hr[c];
                            qi[c] = (float)hi[c];
                        }
                        char* aux_r = (char*)a.aux + (size_t)r * a.aux_rs;
                        if (a.aux_prec == P16S) {
                            store_site<P16S>(aux_r, Vh, s, qr, qi);
                        } else {
                            store_site<P32>(aux_r, Vh, s, qr, qi);
                        }
                    }
                } else {
                    store_site<P>(out_r, Vh, s, hr, hi);
                    if constexpr (EPI == EPI_XPAY_DOT) {
                        double acc = 0.0;
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            acc = fma((double)xr[c], (double)hr[c], acc);
                            acc = fma((double)xi[c], (double)hi[c], acc);
                        }
                        dv[r] = acc;
                    }
                }
            }
        }
    }
    if constexpr (EPI == EPI_XPAY_DOT || EPI == EPI_RESID) {
        block_partials<N, S>(dv, a.red, blk);
    }
}

// ------------------------------------------------------------------ one right-hand side

// Everything one hop pair reads: links, both neighbours, and with a deferred
// direction their residuals.
template <int P, bool LAZY>
struct PairIn {
    using T = typename Real<P>::T;
    PairRaw<P> l;
    T fr[3], fi[3], br[3], bi[3];
    T gr[LAZY ? 3 : 1], gi[LAZY ? 3 : 1], hr[LAZY ? 3 : 1], hi[LAZY ? 3 : 1];
};

// The hop stages of one right-hand side with S lanes per site (four hop pairs
// per lane), the link form and the deferred direction fixed at compile time.
// Bound by the links' memory traffic: what matters is how many loads a wave
// keeps in flight against how many waves fit, so the request of a pair's
// operands runs a fixed number of pairs ahead of its products. Measured on
// A at 32^3 x 64 (us, full / 12-parameter links; improved operator at
// 24^3 x 48): fp64 with 1, 2, 3 pairs ahead 427 / 311, 427 / 310, 436 / 340 (289,
// 285, 293), fp16+scale 120 / 91, 117 / 88, 119 / 90, fp32 235 / 170, 232 / 165,
// 231 / 165 and with all four 225 / 160 (141 improved). The kernel
// before it, k_hop below with its choices at run time (both link forms formed
// and selected, third rows rebuilt for full links too): 446 / 329 (309), 127 /
// 100 and 232 / 161 (150).
template <int P, int S, int EPI, int NP, bool R12, bool LAZY, bool FIN>
__global__ __launch_bounds__(kBlock) void k_hop1(HopArgs a) {
    constexpr int B = NP / S;
    constexpr int D = P == P32 ? 4 : 2;             // pairs requested ahead
    static_assert(D <= B, "pairs ahead");
    constexpr bool LNB = LAZY && EPI == EPI_PLAIN;  // direction formed at the neighbours
    using T = typename Real<P>::T;
    const uint32_t blk = logical_block(a.swizzle, a.tile_bps);
    const uint32_t gt = blk * kBlock + threadIdx.x;
    const uint32_t s = gt / S;
    const int j = (int)(gt % S);
    const uint32_t Vh = a.g.Vh;
    const bool valid = s < Vh;
    const uint32_t sl = valid ? s : Vh - 1;  // lanes past the end repeat the last site
    int x, y, z, t;
    site_coords(a.g, sl, a.p_out, x, y, z, t);
    // Requests that run behind products: all neighbour indices first, because
    // their selects compile to branches, and requests and products only keep
    // their order inside one basic block. All requests up front: each pair's
    // indices with its request (fewer registers).
    uint32_t nf[B], nb[B];
    auto indices = [&](int k) { pair_neighbours<NP>(a.g, sl, x, y, z, t, j * B + k, nf[k], nb[k]); };
    if constexpr (D < B) static_for<0, B>([&](auto kc) { indices(decltype(kc)::value); });
    PairIn<P, LNB> q[D];
    auto request = [&](int k, PairIn<P, LNB>& w) {
        const int mu = j * B + k;
        if constexpr (D == B) indices(k);
        load_site32<P>(a.in, Vh, nf[k], w.fr, w.fi);
        load_site32<P>(a.in, Vh, nb[k], w.br, w.bi);
        if constexpr (LNB) {
            load_site32<P>(a.lazy_r, Vh, nf[k], w.gr, w.gi);
            load_site32<P>(a.lazy_r, Vh, nb[k], w.hr, w.hi);
        }
        load_pair_raw<P, true, NP>(a.gauge, a.gscale, sl, mu, R12, w.l);
    };
    static_for<0, D>([&](auto kc) { request(decltype(kc)::value, q[decltype(kc)::value]); });
    T xr[3], xi[3], rr[3], ri[3];
    if constexpr (EPI != EPI_PLAIN) {
        load_site32<P>(a.x, Vh, sl, xr, xi);
        if constexpr (LAZY) load_site32<P>(a.lazy_r, Vh, sl, rr, ri);
    }
    // the state: finalised here from the previous reduction's partials (FIN),
    // else only the three values that the stage uses
    bool act = true;
    double beta = 0.0, mm = a.m2[0];
    if constexpr (FIN) {
        RhsState s1 = *a.st;
        Reduce F = a.fin;
        F.st = a.st;
        finalize_wave1(F, a.run_mask, s1);
        act = (s1.flags & a.run_mask) != 0;
        beta = s1.beta;
        mm = s1.m2;
    } else {
        const RhsState* st = a.st ? a.st : &kNoState;
        act = !a.st || (st->flags & a.run_mask);
        if (a.st) {
            beta = st->beta;
            mm = st->m2;
        }
    }
    const T be = (T)beta;
    auto direction = [&](T (&vr)[3], T (&vi)[3], const T* gr, const T* gi) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            vr[c] = fma(be, vr[c], gr[c]);
            vi[c] = fma(be, vi[c], gi[c]);
        }
        round_site<P>(vr, vi);
    };
    double dv[1] = {0.0};
    if (act) {
        T pdr[4][3], pdi[4][3], ar[3], ai[3];
        static_for<0, B>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            PairIn<P, LNB>& w = q[k % D];
            T lr[18], li[18], pr[3], pi[3];
            PairScale<T> ps;
            finish_pair<P>(R12, eta_sign((j * B + k) & 3, x, y, z), w.l, lr, li, ps);
            if constexpr (LNB) {
                direction(w.fr, w.fi, w.gr, w.gi);
                direction(w.br, w.bi, w.hr, w.hi);
            }
            pair_start(lr, li, w.fr, w.fi, pr, pi);
            pair_finish(lr, li, ps, w.br, w.bi, pr, pi);
            // the next request stays behind this pair's products, which the
            // compiler would otherwise hold back until every link of the site
            // has been loaded (an empty statement that uses them)
            if constexpr (k + D < B) {
#pragma unroll
                for (int c = 0; c < 3; ++c) asm volatile("" : "+v"(pr[c]), "+v"(pi[c])::"memory");
            }
            // the balanced tree ((p0 + p1) + (p2 + p3)) + ...
            constexpr int lvl = (k & 1) == 0 ? 0 : (k & 2) == 0 ? 1 : (k & 4) == 0 ? 2 : 3;
#pragma unroll
            for (int l = 0; l < lvl; ++l)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    pr[c] = pdr[l][c] + pr[c];
                    pi[c] = pdi[l][c] + pi[c];
                }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                if constexpr (k == B - 1) {
                    ar[c] = pr[c];
                    ai[c] = pi[c];
                } else {
                    pdr[lvl][c] = pr[c];
                    pdi[lvl][c] = pi[c];
                }
            }
            if constexpr (k + D < B) request(k + D, q[k % D]);
        });
        if constexpr (S > 1) {
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int off = 1; off < S; off <<= 1) {
                    ar[c] = ar[c] + __shfl_xor(ar[c], off, 64);
                    ai[c] = ai[c] + __shfl_xor(ai[c], off, 64);
                }
        }
        if (valid && j == 0) {
            if constexpr (EPI == EPI_PLAIN) {
                store_site<P>(a.out, Vh, s, ar, ai);
            } else {
                if constexpr (LAZY) {
                    direction(xr, xi, rr, ri);
                    store_site<P>((void*)a.x, Vh, s, xr, xi);
                }
                const T m2 = (T)mm;
                T hr[3], hi[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    hr[c] = fma(m2, xr[c], -ar[c]);
                    hi[c] = fma(m2, xi[c], -ai[c]);
                }
                store_site<P>(a.out, Vh, s, hr, hi);
                if constexpr (EPI == EPI_XPAY_DOT) {
                    double acc = 0.0;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        acc = fma((double)xr[c], (double)hr[c], acc);
                        acc = fma((double)xi[c], (double)hi[c], acc);
                    }
                    dv[0] = acc;
                }
            }
        }
    }
    if constexpr (EPI == EPI_XPAY_DOT) block_partials<1, S>(dv, a.red, blk);
}

// k_hop1 serves the default launch shape (non-temporal link loads, four pairs
// per lane) of the iteration and operator kernels; the other shapes and the
// fp64 fix-ups, which gather x + y or are gated, take k_hop. Its 32-bit
// offsets hold planes of at most 4 GiB (16 bytes a site).
// fp32 with Eq.5's four pairs keeps k_hop too: there k_hop1 gained 3 % on A with
// full links at 32^3 x 64 (225 against 232 us), nothing with 12-parameter links
// (160 us), and whole solves became slower (16^3 x 32 27.1 against 25.4 ms,
// 24^3 x 48 full 136.5 against 134.7 ms). So do, of the improved operator's fp32
// kernels, those of a solve: stage 2 with its product and stage 1 with the
// deferred direction (20 x 18 x 22 x 30 33.5 against 40.5 ms a solve, 24^3 x 48 79.9
// against 82.6).
template <int P, int NP, int EPI, bool LAZY>
constexpr bool kUseHop1 = P != P32 || (NP == 8 && EPI != EPI_XPAY_DOT && !LAZY);

template <int P, int S, int EPI, bool R12, bool LAZY>
static hipError_t run_hop1(const HopArgs& a, const Issue& is) {
    HopArgs arg = a;
    void* args[] = {&arg};
    const void* f = reinterpret_cast<const void*>(&k_hop1<P, S, EPI, HOP_NP, R12, LAZY, false>);
    if constexpr (EPI == EPI_PLAIN && LAZY)
        if (a.fin.partials) f = reinterpret_cast<const void*>(&k_hop1<P, S, EPI, HOP_NP, R12, LAZY, true>);
    return issue_kernel(is, f, hop_blocks(a.g.Vh, S), kBlock, args);
}

template <int P, int EPI>
static hipError_t dispatch_hop1(const HopArgs& a, const Issue& is) {
    constexpr int S = HOP_NP / 4;
    constexpr bool lazy = EPI != EPI_XPAY && kUseHop1<P, HOP_NP, EPI, true>;
    if constexpr (HOP_NP == 4) {
        if (a.r12) {
            if constexpr (lazy)
                if (a.lazy_r) return run_hop1<P, S, EPI, true, true>(a, is);
            return run_hop1<P, S, EPI, true, false>(a, is);
        }
    }
    if constexpr (lazy)
        if (a.lazy_r) return run_hop1<P, S, EPI, false, true>(a, is);
    return run_hop1<P, S, EPI, false, false>(a, is);
}

template <int P, int S, int N, int EPI, bool NT>
static hipError_t run_hop(const HopArgs& a, const Issue& is) {
    HopArgs arg = a;
    void* args[] = {&arg};
    return issue_kernel(is, reinterpret_cast<const void*>(&k_hop<P, S, N, EPI, NT, HOP_NP>),
                        hop_blocks(a.g.Vh, S), kBlock, args);
}

// Several RHS: non-temporal link loads, S in {1, 2, 4}.
template <int P, int EPI, int N>
static hipError_t run_block(int S, const HopArgs& a, const Issue& is) {
    if (S == 1) return run_hop<P, 1, N, EPI, true>(a, is);
    if (S == 2) return run_hop<P, 2, N, EPI, true>(a, is);
    if (S == 4) return run_hop<P, 4, N, EPI, true>(a, is);
    return hipErrorInvalidValue;
}

// Dispatch for this precision: N = 1 with S in {1, 2, 4} and both load
// flavours; N > 1 with S in {1, 2, 4} and non-temporal link loads.
template <int P, int EPI>
static hipError_t dispatch_epi(int S, int N, bool nt, const HopArgs& a, const Issue& is) {
    if (N == 1) {
        if constexpr (EPI != EPI_RESID && kUseHop1<P, HOP_NP, EPI, false>) {
            constexpr bool lazy = EPI != EPI_XPAY && kUseHop1<P, HOP_NP, EPI, true>;
            if (nt && S == HOP_NP / 4 && (lazy || !a.lazy_r) && !a.lazy_y && !a.gate &&
                a.g.Vh < kHop32MaxSites && !(a.fin.partials && (EPI != EPI_PLAIN || !a.lazy_r)))
                return dispatch_hop1<P, EPI>(a, is);
        }
        if (nt) {
            if (S == 1) return run_hop<P, 1, 1, EPI, true>(a, is);
            if (S == 2) return run_hop<P, 2, 1, EPI, true>(a, is);
            if (S == 4) return run_hop<P, 4, 1, EPI, true>(a, is);
        } else {
            if (S == 1) return run_hop<P, 1, 1, EPI, false>(a, is);
            if (S == 2) return run_hop<P, 2, 1, EPI, false>(a, is);
            if (S == 4) return run_hop<P, 4, 1, EPI, false>(a, is);
        }
        return hipErrorInvalidValue;
    }
    switch (N) {
        case 2: return run_block<P, EPI, 2>(S, a, is);
        case 3: return run_block<P, EPI, 3>(S, a, is);
        case 4: return run_block<P, EPI, 4>(S, a, is);
        case 8: return run_block<P, EPI, 8>(S, a, is);
        case 12: return run_block<P, EPI, 12>(S, a, is);
        case 16: return run_block<P, EPI, 16>(S, a, is);
        default: return hipErrorInvalidValue;
    }
}

#define HOP_FN_NAME_(p, np) launch_hop_p##p##_n##np
#define HOP_FN_NAME(p, np) HOP_FN_NAME_(p, np)

hipError_t HOP_FN_NAME(HOP_PREC, HOP_NP)(int S, int N, int epi, bool nt, const HopArgs& a,
                                          const Issue& is) {
    constexpr int P = HOP_PREC;
    switch (epi) {
        case EPI_PLAIN: return dispatch_epi<P, EPI_PLAIN>(S, N, nt, a, is);
        case EPI_XPAY: return dispatch_epi<P, EPI_XPAY>(S, N, nt, a, is);
        case EPI_XPAY_DOT: return dispatch_epi<P, EPI_XPAY_DOT>(S, N, nt, a, is);
        case EPI_RESID:
            if constexpr (P == P64) return dispatch_epi<P, EPI_RESID>(S, N, nt, a, is);
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

}  // namespace stag

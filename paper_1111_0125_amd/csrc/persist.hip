// CG iterations of small lattices inside one resident kernel: a group of
// workgroups per right-hand side, all on the device at once, loops over the
// iterations (the same three stages, arithmetic and reduction order as the
// kernel-per-stage solver, so the same bits) until its slot is flagged for a
// fix-up, finishes, or has done its share of iterations.
//
// What bounds an iteration on such a lattice is latency, not traffic: as three
// dependent kernels of a graph it costs three launches, three fillings of the
// chip with operands from cache, and each consumer's pass over the partials.
// Here the links of both parities stay in registers for the whole launch (the
// chip's register files hold 128 MiB), as do the own-site vectors (two shapes of
// full links do not fit and keep part in scratch memory: fp32 with one lane per
// site 123 registers, 388 bytes a lane, fp64 with two 38 and 108; the first is
// likely part of 16^3 x 32's 21.5 us an iteration against 14.1 with 12-parameter
// links), and an iteration is two gathers and three waits:
//   stage 1  gather d and r at the neighbours, t = D_oe (r + beta d) published;
//   stage 2  gather t until it is there, A d, <d, A d>; exchange of the blocks'
//            partials;
//   update   x / y, r published, |r|^2; exchange.
// t itself says when it is there: two buffers alternate, and the one not in use
// is set back to a word that no value has (all ones), so that no flag has to
// follow the data through memory (a store's completion, a flag and its poll:
// about 2 us an iteration).
// An exchange is a barrier and a reduction in one trip through memory: every
// block publishes its partial as two tagged words and sums everybody's in the
// solver's fixed order. What other blocks read is written and read with
// agent-scope accesses (relaxed atomics), ordered by waiting for the stores
// before the flag or partial is published; an agent-scope release fence in
// place of that wait writes back the whole L2 and costs 18 us with 256 blocks
// (without it an exchange is 1.2 us with 8 blocks, 1.8 with 32, 2.8 with 256).
//
// Measured (us per iteration, fix-ups included, against the kernel-per-stage
// graph): 8^4 fp32 8.0 (16.9) and fp64 10.8 (16.7), 8^3 x 16 fp64 with 3 RHS 12.5
// (36.2), 12^3 x 24 fp32 10.5 (19.2), 16^3 x 32 fp32 14.1 (22.5).
//
// Every wait ends: it is bounded in time, and a block whose wait runs out
// raises the abort word and leaves; the host then solves with a kernel per
// stage, and stays with that in the context.
#include <type_traits>

#include "kern.h"
#include "launch.h"

namespace stag {

using Word = unsigned long long;

__device__ __forceinline__ Word ag_load(const void* p) {
    return __hip_atomic_load((const Word*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ag_store(void* p, Word v) {
    __hip_atomic_store((Word*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The wavefront's stores have reached the point where other blocks see them.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ Word pack2(float a, float b) {
    return (Word)__float_as_uint(a) | ((Word)__float_as_uint(b) << 32);
}

// Words of one site's colour vector, as load_site / store_site lay it out.
template <int P>
constexpr int kSiteWords = P == P64 ? 6 : P == P32 ? 3 : 2;

// (offsets fit 32 bits: at most kPersistBlocks * kBlock sites)
template <int P>
__device__ __forceinline__ const char* site_word(const char* f, uint32_t Vh, uint32_t s, int w) {
    if constexpr (P == P64) return f + (uint32_t)(((w >> 1) * Vh + s) * 16u + (w & 1) * 8u);
    if constexpr (P == P32) return f + (uint32_t)((w * Vh + s) * 8u);
    return f + (uint32_t)(s * 16u + w * 8u);
}

// Values kept over the iterations are used through `fresh`, an empty statement
// that may change them: otherwise everything formed from them alone (gather
// addresses, rebuilt third rows) is hoisted out of the loop into registers
// that do not exist.
__device__ __forceinline__ uint32_t fresh(uint32_t v) {
    asm volatile("" : "+v"(v));
    return v;
}
template <int P>
__device__ __forceinline__ PairRaw<P> fresh(const PairRaw<P>& w, bool r12) {
    PairRaw<P> f = w;
    constexpr int n12 = P == P64 ? 12 : 6, nfull = P == P64 ? 18 : 9;
    const int n = r12 ? n12 : nfull;
#pragma unroll
    for (int e = 0; e < nfull; ++e)
        if (e < n) asm volatile("" : "+v"(f.v[e]));
    return f;
}

template <int P>
__device__ __forceinline__ void gather(const char* f, uint32_t Vh, uint32_t s, Word (&w)[kSiteWords<P>]) {
#pragma unroll
    for (int k = 0; k < kSiteWords<P>; ++k) w[k] = ag_load(site_word<P>(f, Vh, s, k));
}

template <int P>
__device__ __forceinline__ void unpack(const Word (&w)[kSiteWords<P>], typename Real<P>::T (&re)[3],
                                       typename Real<P>::T (&im)[3]) {
    if constexpr (P == P64) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            re[c] = __longlong_as_double((long long)w[2 * c]);
            im[c] = __longlong_as_double((long long)w[2 * c + 1]);
        }
    } else if constexpr (P == P32) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            re[c] = __uint_as_float((unsigned)w[c]);
            im[c] = __uint_as_float((unsigned)(w[c] >> 32));
        }
    } else {
        u4v v;
        v.x = (unsigned)w[0];
        v.y = (unsigned)(w[0] >> 32);
        v.z = (unsigned)w[1];
        v.w = (unsigned)(w[1] >> 32);
        f16s_decode(v, re, im);
    }
}

// Round to the storage precision (re / im become the stored values) and, on
// the lane that owns the site, publish.
template <int P>
__device__ __forceinline__ void publish(bool own, char* f, uint32_t Vh, uint32_t s,
                                        typename Real<P>::T (&re)[3], typename Real<P>::T (&im)[3]) {
    Word w[kSiteWords<P>];
    if constexpr (P == P64) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            w[2 * c] = (Word)__double_as_longlong(re[c]);
            w[2 * c + 1] = (Word)__double_as_longlong(im[c]);
        }
    } else if constexpr (P == P32) {
#pragma unroll
        for (int c = 0; c < 3; ++c) w[c] = pack2(re[c], im[c]);
    } else {
        const u4v v = f16s_encode(re, im);
        w[0] = (Word)v.x | ((Word)v.y << 32);
        w[1] = (Word)v.z | ((Word)v.w << 32);
    }
    if (own) {
#pragma unroll
        for (int k = 0; k < kSiteWords<P>; ++k) ag_store((char*)site_word<P>(f, Vh, s, k), w[k]);
    }
}

// A wait that runs out after `limit` ticks of the constant 100 MHz clock.
struct Patience {
    long long t0, limit;
    int n = 0;
    __device__ explicit Patience(long long l) : t0(wall_clock64()), limit(l) {}
    __device__ bool out() { return (++n & 63) == 0 && wall_clock64() - t0 > limit; }
};

// The block's partial of a reduction over its 256 / S sites (block_partials'
// order), valid on thread 0; v is meaningful on the first lane of each site.
// DONE: the last barrier is passed only when the block's stores are done.
template <int S, bool DONE = false>
__device__ __forceinline__ double block_sum(double v, double* sv, double* sw) {
    constexpr int CPB = kBlock / S / kChunk;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double x = v;
    if constexpr (S > 1) {
        if (threadIdx.x % S == 0) sv[threadIdx.x / S] = v;
        __syncthreads();
        x = wave < CPB ? sv[wave * kChunk + lane] : 0.0;
    }
    x = wave_butterfly(x);
    if (lane == 0) sw[wave] = x;
    if constexpr (DONE) stores_done();
    __syncthreads();
    if constexpr (CPB == 1) return sw[0];
    if constexpr (CPB == 2) return sw[0] + sw[1];
    return (sw[0] + sw[1]) + (sw[2] + sw[3]);
}

// What an empty word of t holds: a NaN that arithmetic does not produce. It could
// only be passed on from an operand, and none has it: the vectors are finite
// when a solve starts, and the stored links hold no NaN but the canonical one
// (plain_nan in layout.hip).
constexpr Word kEmpty = ~0ull;

template <int P>
__device__ __forceinline__ void set_empty(char* f, uint32_t Vh, uint32_t s) {
#pragma unroll
    for (int k = 0; k < kSiteWords<P>; ++k) ag_store((char*)site_word<P>(f, Vh, s, k), kEmpty);
}

// Publish this block's partial under `tag` and sum everybody's in the order
// of wave_sum_partials over groups of S partials (256 sites): with at most
// 256 blocks every lane holds at most four partials, and the groups and the
// four running sums are the same expression for every S. Wavefront 0 only;
// false when the wait ran out. Slot buffers alternate with the tag: a block
// publishes tag + 2 only after everybody has published tag + 1, which a block
// does after it has read every partial of `tag`.
template <int S>
__device__ __forceinline__ bool exchange(Word* ex, int blocks, int b, uint32_t tag, double x,
                                         long long limit, double& sum) {
    const int lane = threadIdx.x & 63;
    Word* slots = ex + (size_t)(tag & 1) * (2 * kPersistBlocks);
    const Word bits = (Word)__double_as_longlong(x);
    if (lane < 2)
        ag_store(slots + 2 * b + lane, ((Word)tag << 32) | (unsigned)(lane ? bits >> 32 : bits));
    int e[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        e[k] = S == 1 ? lane + 64 * k : S == 2 ? 2 * (lane + 64 * (k >> 1)) + (k & 1) : 4 * lane + k;
    double p[4];
    Patience wait(limit);
    for (;;) {
        bool all = true;
        Word lo[4], hi[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (e[k] >= blocks) continue;
            lo[k] = ag_load(slots + 2 * e[k]);
            hi[k] = ag_load(slots + 2 * e[k] + 1);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            p[k] = 0.0;
            if (e[k] >= blocks) continue;
            all = all && (uint32_t)(lo[k] >> 32) == tag && (uint32_t)(hi[k] >> 32) == tag;
            p[k] = __longlong_as_double((long long)((hi[k] << 32) | (unsigned)lo[k]));
        }
        if (__all(all)) break;
        if (wait.out()) return false;
    }
    double s = (p[0] + p[1]) + (p[2] + p[3]);
    sum = wave_butterfly(s);
    return true;
}

template <int P, int S, bool R12>
__global__ __launch_bounds__(kBlock, 1) void k_persist(PersistArgs a) {
    constexpr int B = 4 / S;            // hop pairs per lane
    constexpr bool mixed = P != P64;
    constexpr int NW = kSiteWords<P>;
    using T = typename Real<P>::T;
    using TY = std::conditional_t<mixed, float, double>;
    __shared__ RhsState ls;
    __shared__ double sv[kBlock], sw[4];
    __shared__ int out;

    // Which right-hand side and which of its blocks. Blocks reach the eight
    // XCDs round-robin: groups of up to 32 blocks stay on one of them, a
    // larger one takes a contiguous part of the lattice on each.
    int rhs, b;
    {
        const int k = blockIdx.x, i = k >> 3;
        if (a.one_xcd) {
            rhs = (k & 7) + 8 * (i / a.blocks);
            b = i % a.blocks;
        } else {
            rhs = k / a.blocks;
            b = k % a.blocks;
            if (a.blocks % 8 == 0) b = (b & 7) * (a.blocks / 8) + (b >> 3);
        }
    }
    if (rhs >= a.nrhs) return;
    RhsState* st = a.st + rhs;
    if (!(st->flags & F_ACTIVE) || *a.abort) return;
    const uint32_t Vh = a.g.Vh;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const uint32_t s = (uint32_t)b * (kBlock / S) + tid / S;
    const int j = tid % S;
    const bool valid = s < Vh, own = valid && j == 0;
    const uint32_t sl = valid ? s : Vh - 1;
    char* d = (char*)a.d + (size_t)rhs * a.rsP;
    char* tb[2] = {(char*)a.t + (size_t)rhs * a.rsP, (char*)a.t2 + (size_t)rhs * a.rsP};
    char* r = (char*)a.r + (size_t)rhs * a.rsP;
    char* y = (char*)a.y + (size_t)rhs * a.rsY;
    Word* ex = a.ex + (size_t)rhs * (4 * kPersistBlocks);

    // links, neighbours and phases of both parities, and the own-site vectors
    PairRaw<P> lk[2][B];
    uint32_t nf[2][B], nb[2][B];
    int eta[2][B];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        int cx, cy, cz, ct;
        site_coords(a.g, sl, p, cx, cy, cz, ct);
#pragma unroll
        for (int k = 0; k < B; ++k) {
            neighbours(a.g, sl, cx, cy, cz, ct, j * B + k, nf[p][k], nb[p][k]);
            eta[p][k] = eta_sign(j * B + k, cx, cy, cz);
            load_pair_raw<P, false, 4>(a.G[p], a.gscale[p], sl, j * B + k, R12, lk[p][k]);
        }
    }
    T dr[3], di[3], rr[3], ri[3];
    TY yr[3], yi[3];
    load_site<P>(d, Vh, sl, dr, di);
    load_site<P>(r, Vh, sl, rr, ri);
    load_site<mixed ? P32 : P64>(y, Vh, sl, yr, yi);
    if (tid == 0) {
        ls = *st;
        out = 0;
    }
    // t starts empty everywhere before anybody looks for it
    if (own) {
        set_empty<P>(tb[0], Vh, s);
        set_empty<P>(tb[1], Vh, s);
    }
    stores_done();
    __syncthreads();
    if (wave == 0) {
        double sum = 0.0;
        const bool ok = a.limit >= 0 && exchange<S>(ex, a.blocks, b, a.tag + 1, 0.0, a.limit, sum);
        if (!ok && lane == 0) out = 1;
    }
    __syncthreads();

    // The sum of the lane's pairs (balanced tree) and of the site's lanes.
    auto site_sum = [&](T (&pr)[B][3], T (&pi)[B][3], T (&ar)[3], T (&ai)[3]) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if constexpr (B == 4) {
                ar[c] = (pr[0][c] + pr[1][c]) + (pr[2][c] + pr[3][c]);
                ai[c] = (pi[0][c] + pi[1][c]) + (pi[2][c] + pi[3][c]);
            } else if constexpr (B == 2) {
                ar[c] = pr[0][c] + pr[1][c];
                ai[c] = pi[0][c] + pi[1][c];
            } else {
                ar[c] = pr[0][c];
                ai[c] = pi[0][c];
            }
#pragma unroll
            for (int off = 1; off < S; off <<= 1) {
                ar[c] = ar[c] + __shfl_xor(ar[c], off, 64);
                ai[c] = ai[c] + __shfl_xor(ai[c], off, 64);
            }
        }
    };

    uint32_t tag = a.tag + 1;  // an iteration uses tag + 1 and tag + 2
    for (int it = 0; it < a.max_iters && !out; ++it, tag += 2) {
        char* t = tb[it & 1];
        const T be = (T)ls.beta;
        const T m2 = (T)ls.m2;
        auto direction = [&](T (&vr)[3], T (&vi)[3], const T (&gr)[3], const T (&gi)[3]) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                vr[c] = fma(be, vr[c], gr[c]);
                vi[c] = fma(be, vi[c], gi[c]);
            }
            round_site<P>(vr, vi);
        };
        T ar[3], ai[3];
        {
            // stage 1: t = D_oe d, d = r + beta d
            Word fd[B][NW], fr[B][NW], bd[B][NW], br[B][NW];
#pragma unroll
            for (int k = 0; k < B; ++k) {
                const uint32_t f = fresh(nf[1][k]), b1 = fresh(nb[1][k]);
                gather<P>(d, Vh, f, fd[k]);
                gather<P>(r, Vh, f, fr[k]);
                gather<P>(d, Vh, b1, bd[k]);
                gather<P>(r, Vh, b1, br[k]);
            }
            T pr[B][3], pi[B][3];
#pragma unroll
            for (int k = 0; k < B; ++k) {
                T lr[18], li[18], vr[3], vi[3], gr[3], gi[3];
                PairScale<T> ps;
                finish_pair<P>(R12, eta[1][k], fresh(lk[1][k], R12), lr, li, ps);
                unpack<P>(fd[k], vr, vi);
                unpack<P>(fr[k], gr, gi);
                direction(vr, vi, gr, gi);
                pair_start(lr, li, vr, vi, pr[k], pi[k]);
                unpack<P>(bd[k], vr, vi);
                unpack<P>(br[k], gr, gi);
                direction(vr, vi, gr, gi);
                pair_finish(lr, li, ps, vr, vi, pr[k], pi[k]);
            }
            site_sum(pr, pi, ar, ai);
            publish<P>(own, t, Vh, s, ar, ai);
        }
        // the other buffer, last read before the previous iteration's first
        // exchange: empty again, and known to be (stores_done below) before the
        // next iteration's readers look
        if (own) set_empty<P>(tb[(it + 1) & 1], Vh, s);
        direction(dr, di, rr, ri);  // own site
        T hr[3], hi[3];
        {
            // stage 2: d stored, A d = m^2 d - D_eo t
            Word fw[B][NW], bw[B][NW];
            Patience wait(a.limit);
            for (;;) {
#pragma unroll
                for (int k = 0; k < B; ++k) {
                    gather<P>(t, Vh, fresh(nf[0][k]), fw[k]);
                    gather<P>(t, Vh, fresh(nb[0][k]), bw[k]);
                }
                bool all = true;
#pragma unroll
                for (int k = 0; k < B; ++k)
#pragma unroll
                    for (int w = 0; w < NW; ++w) all = all && fw[k][w] != kEmpty && bw[k][w] != kEmpty;
                if (__all(all)) break;
                if (wait.out()) {
                    out = 1;
                    break;
                }
            }
            // (the neighbours' t is there: they have read the old d)
            T qr[3] = {dr[0], dr[1], dr[2]}, qi[3] = {di[0], di[1], di[2]};
            publish<P>(own, d, Vh, s, qr, qi);
            T pr[B][3], pi[B][3];
#pragma unroll
            for (int k = 0; k < B; ++k) {
                T lr[18], li[18], vr[3], vi[3];
                PairScale<T> ps;
                finish_pair<P>(R12, eta[0][k], fresh(lk[0][k], R12), lr, li, ps);
                unpack<P>(fw[k], vr, vi);
                pair_start(lr, li, vr, vi, pr[k], pi[k]);
                unpack<P>(bw[k], vr, vi);
                pair_finish(lr, li, ps, vr, vi, pr[k], pi[k]);
            }
            site_sum(pr, pi, ar, ai);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                hr[c] = fma(m2, dr[c], -ar[c]);
                hi[c] = fma(m2, di[c], -ai[c]);
            }
            round_site<P>(hr, hi);
        }
        double acc = 0.0;
        if (own) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                acc = fma((double)dr[c], (double)hr[c], acc);
                acc = fma((double)di[c], (double)hi[c], acc);
            }
        }
        double x = block_sum<S>(acc, sv, sw);
        if (wave == 0) {
            double sum = 0.0;
            const bool ok = out == 0 && exchange<S>(ex, a.blocks, b, tag + 1, x, a.limit, sum);
            if (lane == 0) {
                if (ok) {
                    finalize_one(FIN_ALPHA, &ls, sum, nullptr);
                } else {
                    out = 1;
                }
            }
        }
        __syncthreads();
        if (out || !(ls.flags & F_ACTIVE)) break;

        // update: x or y += alpha d, r -= alpha A d, |r|^2
        acc = 0.0;
        {
            const T al = (T)ls.alpha;
            const TY aly = (TY)ls.alpha;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                yr[c] = fma(aly, (TY)dr[c], yr[c]);
                yi[c] = fma(aly, (TY)di[c], yi[c]);
                rr[c] = fma(-al, hr[c], rr[c]);
                ri[c] = fma(-al, hi[c], ri[c]);
            }
            publish<P>(own, r, Vh, s, rr, ri);
            if (own) {
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    acc += (double)rr[c] * (double)rr[c] + (double)ri[c] * (double)ri[c];
            }
        }
        x = block_sum<S, true>(acc, sv, sw);
        if (wave == 0) {
            double sum = 0.0;
            const bool ok = exchange<S>(ex, a.blocks, b, tag + 2, x, a.limit, sum);
            if (lane == 0) {
                if (ok) {
                    finalize_one(mixed ? FIN_MIXED : FIN_CG, &ls, sum, nullptr);
                } else {
                    out = 1;
                }
            }
        }
        __syncthreads();
        if (out || !(ls.flags & F_ACTIVE)) break;
    }
    if (out) {
        if (tid == 0) __hip_atomic_store(a.abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    if (own) store_site<mixed ? P32 : P64>(y, Vh, s, yr, yi);
    // every block has read its start state (it took part in an exchange)
    if (b == 0 && tid == 0) *st = ls;
}

template <int P, int S>
static const void* persist_fn(bool r12) {
    return r12 ? reinterpret_cast<const void*>(&k_persist<P, S, true>)
               : reinterpret_cast<const void*>(&k_persist<P, S, false>);
}

// The shapes that persist_lanes (solver.cpp) chooses.
static const void* persist_fn(int prec, int S, bool r12) {
    switch (prec * 8 + S) {
        case P64 * 8 + 2: return persist_fn<P64, 2>(r12);
        case P64 * 8 + 4: return r12 ? nullptr : reinterpret_cast<const void*>(&k_persist<P64, 4, false>);
        case P32 * 8 + 1: return persist_fn<P32, 1>(r12);
        case P32 * 8 + 2: return persist_fn<P32, 2>(r12);
        case P16S * 8 + 1: return persist_fn<P16S, 1>(r12);
        case P16S * 8 + 2: return persist_fn<P16S, 2>(r12);
        default: return nullptr;
    }
}

hipError_t launch_persist(int prec, int S, bool r12, const PersistArgs& a, hipStream_t stream) {
    const void* fn = persist_fn(prec, S, r12);
    if (!fn || a.nrhs < 1 || a.blocks < 1 || a.blocks > kPersistBlocks || a.g.Vh < 1 ||
        (uint32_t)a.blocks != hop_blocks(a.g.Vh, S) || (a.tag & 1))
        return hipErrorInvalidValue;
    PersistArgs arg = a;
    void* args[] = {&arg};
    const int grid = a.one_xcd ? 8 * a.blocks * ((a.nrhs + 7) / 8) : a.nrhs * a.blocks;
    // The caller keeps the grids of all such kernels within one block per compute
    // unit (ResidentHold); whatever else runs on the device ends by itself, so
    // every block becomes resident. (A cooperative launch would check the same
    // and costs 20 us of idle device around each launch.)
    return hipLaunchKernel(fn, dim3((uint32_t)grid), dim3(kBlock), args, 0, stream);
}

}  // namespace stag

// Legendre-stage kernels for gfx950 (FP64 VALU).
//
// Synthesis computes Delta^A_m(r) = sum_l a_lm lambda_lm(cos theta_r)
// (Sec. 2.2 eq. DeltaDef); analysis computes a_lm = sum_r Delta^S_m(r)
// lambda_lm(cos theta_r) (eq. almdef).  lambda_lm comes from the l-recurrence
// (eqs. assLegRec, betaDef) seeded by lambda_mm = (-1)^m mu_m sin^m(theta)
// (eq. pmm, with the exponent m/2 and the Condon-Shortley phase) and
// lambda_{m+1,m} = sqrt(2m+3) x lambda_mm (eq. pm1m).
//
// lambda_lm = c_lm q_l with q_l = alpha_l x q_{l-1} - q_{l-2}; the factors c_lm
// go into a_lm.  The recurrence runs in pairs of degrees, l = m + 2j and the
// next, on p_j = q_{m+2j} and r_j = q_{m+2j+1} / x (that of an odd degree is x
// times a polynomial in x^2):
//   p_j = alpha_{m+2j} x^2 r_{j-1} - p_{j-1},   r_j = alpha_{m+2j+1} p_j - r_{j-1},
// three operations for two degrees.  Synthesis is E = sum_j c a_{m+2j} p_j plus
// x times O = sum_j c a_{m+2j+1} r_j; analysis sums p_j D+ and r_j x D- over the
// rings.  A (ring pair, two l) costs 7 FP64 operations instead of 8 with x
// multiplied in each step.  The three-term recurrence in x^2 of the odd degrees
// alone (Ishioka, J. Meteorol. Soc. Japan 96, 2018) needs 6, but gets the even
// degrees from the difference of two values that are up to l times as large
// next to the equator: 1e-13 on the rings there at lmax 1024 where this form has
// 1e-15, and no gain elsewhere, as the rounding of the argument x^2 dominates
// both (1.5e-14 at 20 degrees from a pole, against 4.3e-14 with x rounded in
// each step).  For the slots next to a pole x^2 is 1 - sin^2 (GeomPlan::npolar).
//
// One recurrence serves a ring and its mirror image (x -> -x): the even part
// E is the same and the odd part x O changes sign.
//
// Underflow near the poles (Sec. 2.1 asks for rescaling and leaves the
// algorithm to its references).  Once per plan, k_leg_start runs every
// (m, slot) recurrence from its seed with exponent tracking (a value held as
// value * 2^(600 sc), sc <= 0) until |p_j| or |r_j| first reaches 2^-100, and
// stores the j that opens the block of kStartJ steps holding that step, with
// (p_{j-1}, r_{j-1}) before it.  The transform kernels start each slot there:
// every term they leave out has |lambda| < 2.3 * 2^-100, and from its start
// on a slot's values stay in normal double range, so the hot loops have no
// rescaling.  A slot whose values stay below 2^-100 up to lmax is not started.
//
// Work mapping (the paper's GPU design assigns one ring per thread and the
// rings loop outermost; here a workgroup owns one m for a tile of ring
// pairs, so the loop over l is uniform across a wave and a_lm, alpha are
// wave-uniform scalar operands):
//   synthesis  grid.x = (m, slot tile), m ascending (longest first), grid.y =
//              map (or two maps); a wave owns 64 T slots, T per lane, no reduction.
//   analysis   grid.x = (m, slot group), grid.y = map; a workgroup owns up
//              to 256 T slots of its m; each wave sums its lanes in registers
//              and its own LDS rows, the waves are added in wave order
//              every 32 steps, and groups are summed in order by a second
//              small kernel: no atomics, deterministic.  A map's sums do not
//              depend on the number of maps: its a_lm are the same bits in any call.
#include <type_traits>

#include "k_device.h"

namespace sht {
namespace {

constexpr double kDown = 0x1p-600;   // 2^-kScaleBits
constexpr double kThresh = 0x1p-60;  // carrier bound that triggers rescaling
constexpr double kStart = 0x1p-100;  // a slot starts once |p| or |r| reaches this
static_assert(kScaleBits == 600, "kDown must equal 2^-kScaleBits");

// One pair of degrees: p, r from their predecessors, ae = alpha_{m+2j}, ao =
// alpha_{m+2j+1}.  POLAR: x^2 is h + w (GeomPlan::npolar), else w; a slot with
// h = 0 has the same bits in both forms.
template <bool POLAR>
__device__ __forceinline__ void pair_step(double ae, double ao, double w, double h, double &p, double &r) {
    double t = w * r;
    if (POLAR) t = fma(h, r, t);
    p = fma(ae, t, -p);
    r = fma(ao, p, -r);
}
__device__ __forceinline__ double polar_h(int slot, int npolar) { return slot < npolar ? 1.0 : 0.0; }

// p_0 = (-1)^m mu_m s^m as carrier * 2^(600 sc).  s^m by
// binary powering with frexp renormalisation; s and its squares are carried as
// two doubles, since each squaring doubles the relative error of what it
// squares (with one double the seed of m would be off by about m/2 roundings).
__device__ __forceinline__ double seed_carrier(int m, double2 s, double mu_m, int &sc) {
    int eb;
    double b = frexp(s.x, &eb), bl = ldexp(s.y, -eb);
    double r = 1.0, rl = 0.0;
    int E = 0;
    for (int k = m; k; k >>= 1) {
        if (k & 1) {
            const double t = r * b;
            rl = fma(r, b, -t) + fma(r, bl, rl * b);
            int e;
            r = frexp(t, &e);
            rl = ldexp(rl, -e);
            E += e + eb;
        }
        if (k > 1) {
            const double t = b * b;
            bl = fma(b, b, -t) + 2.0 * b * bl;
            int e2;
            b = frexp(t, &e2);
            bl = ldexp(bl, -e2);
            eb = 2 * eb + e2;
        }
    }
    const double v = ((m & 1) ? -mu_m : mu_m) * (r + rl);
    if (v == 0.0) {
        sc = 0;
        return 0.0;
    }
    // keep the carrier exponent in (-660, -60] when sc < 0
    const int ns = (E >= -60) ? 0 : (-E - 60) / kScaleBits;
    sc = -ns;
    return ldexp(v, E + kScaleBits * ns);
}

// Plan kernel: one thread per (m, slot); grid.x covers slots, grid.y = m.
// Writes jstart[m * nslots + slot] (kNeverJ when never reached) and
// state[m * nslots + slot] = (p_{j-1}, r_{j-1}) before step j = jstart.
__global__ __launch_bounds__(kBlock) void k_leg_start(int lmax, int nslots, int npolar,
                                                      const double *__restrict__ alpha,
                                                      const double *__restrict__ mu,
                                                      const double *__restrict__ sw,
                                                      const double2 *__restrict__ ss,
                                                      int32_t *__restrict__ jstart,
                                                      double2 *__restrict__ state) {
    const int slot = blockIdx.x * kBlock + threadIdx.x;
    const int m = blockIdx.y;
    if (slot >= nslots) return;
    const double w = sw[slot];
    const double h = polar_h(slot, npolar);
    const double *__restrict__ al = alpha + (int64_t)m * (2 * lmax + 1 - m) / 2 + m;
    const int nj = jcol_len(lmax, m);
    int sc;
    const double seed = seed_carrier(m, ss[slot], mu[m], sc);
    // before step j = 0 (-seed, 0) makes that step yield the seed (alpha_m = 0)
    double p = -seed, r = 0.0;
    int found = kNeverJ;
    double sp = 0.0, sr = 0.0;
    for (int j0 = 0; j0 < nj && found == kNeverJ; j0 += kStartJ) {
        const double bp = p, br = r;
        const int bsc = sc;
        bool hit = false;
        for (int i = 0; i < kStartJ && j0 + i < nj; ++i) {
            // the odd degree past lmax (of the last j) reads the next column or the padding: not used
            pair_step<true>(al[2 * (j0 + i)], al[2 * (j0 + i) + 1], w, h, p, r);
            hit |= (sc == 0 && (fabs(p) >= kStart || (fabs(r) >= kStart && m + 2 * (j0 + i) < lmax)));
            // one step grows a value by less than 2^18 (alpha_l < 2^9)
            if (sc < 0 && fmax(fabs(p), fabs(r)) > kThresh) {
                p *= kDown;
                r *= kDown;
                ++sc;
            }
        }
        if (hit) {
            found = j0;
            // a value leaves sc < 0 near 2^-660 and cannot grow past 2^-100
            // within one block, so bsc is 0 here in practice
            sp = ldexp(bp, kScaleBits * bsc);
            sr = ldexp(br, kScaleBits * bsc);
        }
    }
    jstart[(int64_t)m * nslots + slot] = found;
    state[(int64_t)m * nslots + slot] = make_double2(sp, sr);
}

__global__ __launch_bounds__(kBlock) void k_prescale(int64_t nalm, int lmax, int nmaps,
                                                     const double2 *__restrict__ alm,
                                                     const double *__restrict__ cfac,
                                                     double2 *__restrict__ out) {
    const int64_t total = nalm * nmaps;
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < total; i += (int64_t)gridDim.x * kBlock) {
        const int64_t k = i % nalm;
        const double c = cfac[k];
        const double2 a = alm[i];
        // entries k <= lmax are m = 0: Im a_l0 is ignored
        out[i] = make_double2(a.x * c, k <= lmax ? 0.0 : a.y * c);
    }
}

// Synthesis of one m of M maps over a tile of slots: a wave (li / 64 of the
// threads sharing the tile) owns 64 T consecutive slots, its lanes the slots
// 64 u + lane of them, u < T (so that a set of 64 that has not started is
// skipped whole, and table reads are contiguous: 2 to 5 % at HEALPix 512 to
// 700), for maps map0 .. map0 + M - 1 (those past nmaps repeat the last map and are not
// stored).  Each recurrence value serves the M maps, so a slot and two l cost
// 3 + 4M operations instead of 7M; per map the arithmetic (the same fused
// multiply-adds in the same order) does not depend on M, so results are the
// same bits for any M.  The wave works on its own (no cross-wave step), so a
// tile may be one wave's (li = lane) or a workgroup's (li = thread index).
// POLAR: the wave may hold polar slots.
template <int T, int M, bool POLAR>
__device__ __forceinline__ void syn_wave(const SynArgs &A, int m, int map0, int nmaps, int wave0) {
    constexpr std::integral_constant<bool, POLAR> polar{};
    const int lmax = A.lmax, mmax = A.mmax, nslots = A.nslots, nrings = A.nrings;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2;  // (l, m) lives at base + l
    ConstC a[M];
#pragma unroll
    for (int k = 0; k < M; ++k) a[k] = ro(A.ap + (int64_t)min(map0 + k, nmaps - 1) * A.nalm + base + m);
    const int lane = threadIdx.x & 63;
    const const_ptr<double> al = ro(A.alpha + base + m);
    const int nj = jcol_len(lmax, m);

    double w[T], h[T], p[T], r[T], er[T][M], ei[T][M], orr[T][M], oi[T][M];
    // what the stores need is loaded with the rest where registers allow, so
    // that a short recurrence does not end on another memory round trip
    constexpr bool kEarly = T * M <= 2;
    double x[T];
    int rn[T], rs[T], js[T];
    int lo = kNeverJ, hi = 0;
#pragma unroll
    for (int u = 0; u < T; ++u) {
        const int slot = wave0 + 64 * u + lane;
        const bool act = slot < nslots;
        if constexpr (kEarly) {
            const int sl = act ? slot : nslots - 1;
            x[u] = A.sx[sl];
            rn[u] = A.rn[sl];
            rs[u] = A.rsouth[sl];
        }
        w[u] = act ? A.sw[slot] : 0.0;
        h[u] = polar_h(slot, A.npolar);
        js[u] = act ? A.jstart[(int64_t)m * nslots + slot] : kNeverJ;
        const double2 st = act ? A.state[(int64_t)m * nslots + slot] : make_double2(0.0, 0.0);
        p[u] = st.x;
        r[u] = st.y;
#pragma unroll
        for (int k = 0; k < M; ++k) er[u][k] = ei[u][k] = orr[u][k] = oi[u][k] = 0.0;
        lo = min(lo, js[u]);
        if (js[u] < nj) hi = max(hi, js[u]);
        // not started for this lmax: the state is carried but never used
        if (js[u] >= nj) p[u] = r[u] = 0.0;
    }
    lo = wave_min(lo);
    hi = wave_max(hi);

    struct Coef {
        double ae, ao;  // alpha of the even and of the odd degree
        double2 e[M], o[M];
    };
    auto load = [&](int j, Coef &k) {
        k.ae = al[2 * j];
        k.ao = al[2 * j + 1];
#pragma unroll
        for (int i = 0; i < M; ++i) {
            k.e[i] = a[i][2 * j];
            k.o[i] = a[i][2 * j + 1];
        }
    };
    // step j of slot u: p_j and r_j, then the terms of both degrees (ODD: m + 2j + 1 <= lmax)
    auto step = [&](const Coef &c, int u, auto polar, auto odd) {
        pair_step<decltype(polar)::value>(c.ae, c.ao, w[u], h[u], p[u], r[u]);
#pragma unroll
        for (int k = 0; k < M; ++k) {
            er[u][k] = fma(c.e[k].x, p[u], er[u][k]);
            ei[u][k] = fma(c.e[k].y, p[u], ei[u][k]);
            if constexpr (decltype(odd)::value) {
                orr[u][k] = fma(c.o[k].x, r[u], orr[u][k]);
                oi[u][k] = fma(c.o[k].y, r[u], oi[u][k]);
            }
        }
    };
    const int nfull = (lmax - m + 1) / 2;  // steps with both parities

    // Blocks of kStartJ steps of both parities, in halves of two steps with two
    // coefficient sets in turn, each loaded one half ahead (a and alpha are
    // padded, so the loads past the column's end stay in bounds).  Start
    // positions are multiples of kStartJ: while slots join (j <= hi) the lanes
    // of a slot that has not started are masked off and it keeps its state.
    // The trip counts are fixed up front so that no exit separates a load from
    // its use.
    int j = lo;
    if (j + kStartJ <= nfull) {
        // running pointers: the loads of a half are one run of scalar loads each
        const_ptr<double> pal = al + 2 * j;
        const_ptr<dvec2> pa[M];
#pragma unroll
        for (int k = 0; k < M; ++k) pa[k] = a[k].p + 2 * j;
        auto pair = [](dvec2 v) { return make_double2(v.x, v.y); };
        auto load2 = [&](int ofs, Coef (&c)[2]) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                c[i].ae = pal[2 * (ofs + i)];
                c[i].ao = pal[2 * (ofs + i) + 1];
#pragma unroll
                for (int k = 0; k < M; ++k) {
                    c[i].e[k] = pair(pa[k][2 * (ofs + i)]);
                    c[i].o[k] = pair(pa[k][2 * (ofs + i) + 1]);
                }
            }
            // compiler-only fence: keeps the loads here instead of letting
            // them sink to their first use in the next half
            asm volatile("" ::: "memory");
        };
        auto masked2 = [&](const Coef (&c)[2]) {
#pragma unroll
            for (int u = 0; u < T; ++u)
                if (j >= js[u]) {
                    step(c[0], u, polar, std::true_type{});
                    step(c[1], u, polar, std::true_type{});
                }
        };
        auto step2 = [&](const Coef (&c)[2]) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int u = 0; u < T; ++u) step(c[i], u, polar, std::true_type{});
        };
        auto advance = [&]() {
            pal += 2 * kStartJ;
#pragma unroll
            for (int k = 0; k < M; ++k) pa[k] += 2 * kStartJ;
        };
        const int nblocks = (nfull - j) / kStartJ;
        const int njoin = min(nblocks, (hi - j) / kStartJ + 1);
        Coef cA[2], cB[2];
        load2(0, cA);
        for (int b = 0; b < njoin; ++b) {
            load2(2, cB);
            masked2(cA);
            load2(4, cA);
            masked2(cB);
            advance();
            j += kStartJ;
        }
        for (int b = njoin; b < nblocks; ++b) {
            load2(2, cB);
            step2(cA);
            load2(4, cA);
            step2(cB);
            advance();
        }
        j += kStartJ * (nblocks - njoin);
    }
    // j is uniform; restate it so that the compiler does not carry a lane
    // value it was compared with into the loop below
    j = __builtin_amdgcn_readfirstlane(j);
    // the ragged tail (fewer than kStartJ steps of both parities, then one of
    // even degree only when l = lmax is even in l - m); slots may start here
    for (; j < nj; ++j) {
        Coef c;
        load(j, c);
#pragma unroll
        for (int u = 0; u < T; ++u)
            if (j >= js[u]) {
                if (j < nfull)
                    step(c, u, polar, std::true_type{});
                else
                    step(c, u, polar, std::false_type{});
            }
    }

#pragma unroll
    for (int u = 0; u < T; ++u) {
        const int slot = wave0 + 64 * u + lane;
        if (slot < nslots) {
            if constexpr (!kEarly) {
                x[u] = A.sx[slot];
                rn[u] = A.rn[slot];
                rs[u] = A.rsouth[slot];
            }
            const int64_t rN = (int64_t)rn[u] * (mmax + 1) + m, rS = (int64_t)rs[u] * (mmax + 1) + m;
#pragma unroll
            for (int k = 0; k < M; ++k) {
                if (map0 + k >= nmaps) break;
                double2 *d = A.delta + (int64_t)(map0 + k) * nrings * (mmax + 1);
                d[rN] = make_double2(fma(x[u], orr[u][k], er[u][k]), fma(x[u], oi[u][k], ei[u][k]));
                if (rs[u] >= 0) d[rS] = make_double2(fma(-x[u], orr[u][k], er[u][k]), fma(-x[u], oi[u][k], ei[u][k]));
            }
        }
    }
}

template <int T, int M = 1>
__device__ __forceinline__ void syn_tile(const SynArgs &A, int m, int map0, int nmaps, int slot0, int li) {
    const int wave0 = __builtin_amdgcn_readfirstlane(slot0 + (li & ~63) * T);
    if (wave0 < A.npolar)
        syn_wave<T, M, true>(A, m, map0, nmaps, wave0);
    else
        syn_wave<T, M, false>(A, m, map0, nmaps, wave0);
}

// Synthesis of M maps per workgroup (grid.y = map group of M), T slots per
// lane: the recurrence shared by the M maps (syn_tile).
template <int T, int M>
__global__ __launch_bounds__(kBlock, 2) void k_leg_syn_mm(SynArgs A, int tiles, int nmaps) {
    const MPart mp = xcd_m_part(tiles);
    const int m = mp.m, tile = mp.part;
    if (m > A.mmax) return;  // padding of the m range
    const int map0 = blockIdx.y * M;
    const int64_t base = (int64_t)m * (2 * A.lmax + 1 - m) / 2;
    const double warm_a = warm_l2(reinterpret_cast<const double *>(A.ap + (int64_t)map0 * A.nalm + base), 2, m, A.lmax);
    const double warm_al = warm_l2(A.alpha + base, 1, m, A.lmax);
    syn_tile<T, M>(A, m, map0, nmaps, tile * kBlock * T, (int)threadIdx.x);
    asm volatile("" ::"v"(warm_a), "v"(warm_al));  // the warming loads are waited for only here
}

// Synthesis kernel: grid.x = (m, 256T-slot tile) in the XCD-aware order,
// grid.y = map; wave w of tile t owns the 64 T slots from (4 t + w) 64 T on.
template <int T>
__global__ __launch_bounds__(kBlock, 4) void k_leg_syn(SynArgs A, int tiles) {
    const MPart mp = xcd_m_part(tiles);
    const int m = mp.m, tile = mp.part;
    if (m > A.mmax) return;  // padding of the m range
    const int64_t base = (int64_t)m * (2 * A.lmax + 1 - m) / 2;
    const double warm_a = warm_l2(reinterpret_cast<const double *>(A.ap + (int64_t)blockIdx.y * A.nalm + base), 2,
                                  m, A.lmax);
    const double warm_al = warm_l2(A.alpha + base, 1, m, A.lmax);
    syn_tile<T>(A, m, (int)blockIdx.y, (int)gridDim.y, tile * kBlock * T, (int)threadIdx.x);
    asm volatile("" ::"v"(warm_a), "v"(warm_al));  // the warming loads are waited for only here
}

constexpr int kChunk = kStartJ;       // recurrence steps (two degrees each) per in-wave reduction in analysis
constexpr int kVals = 4 * kChunk;     // sums per chunk: (step, {even re, even im, odd re, odd im})
// chunks between cross-wave flushes (one barrier each)
constexpr int kFlush = 8;
// Wave-private rows of the in-wave reduction: 16 doubles and 2 of padding (the
// padding keeps the row reads free of bank conflicts)
constexpr int kTRow = 18;
typedef double SumRows[kVals][kTRow];

// alpha of one chunk (scalar registers)
struct AnaCoef {
    double a[2 * kChunk];
};
struct AnaCoefPtr {
    const_ptr<double> a;  // at the chunk that load() reads next
    // entries past the column's end belong to the next column or the padding
    // and are never used
    __device__ __forceinline__ void load(AnaCoef &c) {
#pragma unroll
        for (int i = 0; i < 2 * kChunk; ++i) c.a[i] = a[i];
        a += 2 * kChunk;
        // compiler-only fence: the loads stay here, ahead of the work that hides them
        asm volatile("" ::: "memory");
    }
};

// quad all-reduce (lanes l, l^1, l^2, l^3) of a double through DPP moves
__device__ __forceinline__ double quad_sum(double v) {
    int lo = __double2loint(v), hi = __double2hiint(v);
    double w = __hiloint2double(__builtin_amdgcn_update_dpp(0, hi, 0xB1, 0xf, 0xf, false),
                                __builtin_amdgcn_update_dpp(0, lo, 0xB1, 0xf, 0xf, false));  // quad_perm [1,0,3,2]
    v += w;
    lo = __double2loint(v);
    hi = __double2hiint(v);
    w = __hiloint2double(__builtin_amdgcn_update_dpp(0, hi, 0x4E, 0xf, 0xf, false),
                         __builtin_amdgcn_update_dpp(0, lo, 0x4E, 0xf, 0xf, false));  // quad_perm [2,3,0,1]
    return v + w;
}

constexpr int kAnaWaves = kAnaThreads / 64;
// LDS of an analysis workgroup of W waves: wave-private reduction rows, the
// per-wave chunk sums awaiting a cross-wave flush, and the waves' first starts.
template <int W = kAnaWaves>
struct AnaLds {
    alignas(16) SumRows tbuf[W];
    double ring[2][kFlush][W][kVals];
    int wstart[W];
    static_assert(kFlush * kVals <= 64 * W, "one thread per flushed value");
};

// The slot operands of one lane, slots slot0 + stride t + lane (t < T, sets of
// 64 slots): recurrence argument, start, recurrence state and the pair sums
// D+ = north + south and x D-, D- = north - south, of Delta_m.
// The first PS sets may hold polar slots.
template <int T, int PS>
struct AnaSlots {
    static constexpr int kPolar = PS < T ? PS : T;
    double w[T], h[kPolar], p[T], r[T], pr[T], pi[T], mr[T], mi[T];
    int js[T];
    int lo;  // wave-uniform: earliest start (kNeverJ if none)

    __device__ __forceinline__ void load(const AnaArgs &A, int m, const double2 *__restrict__ d, int slot0,
                                         int stride) {
        const int nslots = A.nslots, nj = jcol_len(A.lmax, m);
        // two rounds of loads: the slots' tables (an inactive lane takes the
        // last slot's and never starts), then Delta where the ring indices point
        double x[T];
        int rn[T], rs[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int slot = slot0 + stride * t + ((int)threadIdx.x & 63);
            const bool act = slot < nslots;
            const int sl = act ? slot : nslots - 1;
            w[t] = A.sw[sl];
            if (t < PS) h[t < PS ? t : 0] = polar_h(slot, A.npolar);
            x[t] = A.sx[sl];
            rn[t] = A.rn[sl];
            rs[t] = A.rsouth[sl];
            const int js0 = A.jstart[(int64_t)m * nslots + sl];
            const double2 st = A.state[(int64_t)m * nslots + sl];
            js[t] = act && js0 < nj ? js0 : kNeverJ;
            p[t] = st.x;
            r[t] = st.y;
        }
        lo = kNeverJ;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            double2 dn = make_double2(0.0, 0.0), ds = make_double2(0.0, 0.0);
            if (js[t] < nj) {
                dn = d[(int64_t)rn[t] * (A.mmax + 1) + m];
                if (rs[t] >= 0) ds = d[(int64_t)rs[t] * (A.mmax + 1) + m];
            }
            pr[t] = dn.x + ds.x;
            pi[t] = dn.y + ds.y;
            mr[t] = x[t] * (dn.x - ds.x);
            mi[t] = x[t] * (dn.y - ds.y);
            lo = min(lo, js[t]);
        }
        lo = wave_min(lo);
    }
    // One chunk of kChunk recurrence steps from j0 on: acc = sums over the slots
    // of p_j D+ and r_j x D- per step.  A slot that has not started keeps its
    // state (its lanes masked off; a set that has not started at all is skipped).
    // Steps and degrees past lmax give sums that nobody stores.
    __device__ __forceinline__ void chunk(int j0, const AnaCoef &c, double (&acc)[kVals]) {
#pragma unroll
        for (int v = 0; v < kVals; ++v) acc[v] = 0.0;
#pragma unroll
        for (int t = T - 1; t >= 0; --t) {
            if (j0 >= js[t]) {
#pragma unroll
                for (int i = 0; i < kChunk; ++i) {
                    if (t < PS)
                        pair_step<true>(c.a[2 * i], c.a[2 * i + 1], w[t], h[t < PS ? t : 0], p[t], r[t]);
                    else
                        pair_step<false>(c.a[2 * i], c.a[2 * i + 1], w[t], 0.0, p[t], r[t]);
                    acc[4 * i + 0] = fma(p[t], pr[t], acc[4 * i + 0]);
                    acc[4 * i + 1] = fma(p[t], pi[t], acc[4 * i + 1]);
                    acc[4 * i + 2] = fma(r[t], mr[t], acc[4 * i + 2]);
                    acc[4 * i + 3] = fma(r[t], mi[t], acc[4 * i + 3]);
                }
            }
        }
    }
};

// a' = (a, b of the partner half), b' = (a of the partner half, b): after the
// exchange a' + b' holds the sum over the two halves of a in the lower lanes
// and of b in the upper ones.  32: halves of the wave; 16: of each half.
template <int N>
__device__ __forceinline__ double swap_add(double a, double b) {
    auto sw = [](uint32_t x, uint32_t y) {
        if constexpr (N == 32)
            return __builtin_amdgcn_permlane32_swap(x, y, false, false);
        else
            return __builtin_amdgcn_permlane16_swap(x, y, false, false);
    };
    const auto lo = sw((uint32_t)__double2loint(a), (uint32_t)__double2loint(b));
    const auto hi = sw((uint32_t)__double2hiint(a), (uint32_t)__double2hiint(b));
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

// Wave sum of one chunk's 16 values per lane: two register exchanges leave
// lane 16g + k with the values 4g .. 4g+3 summed over lanes k, k+16, k+32,
// k+48; lane (v = lane/4, q = lane%4) then adds four of the 16 sums of value v
// from the wave's LDS rows, and the quad combines by DPP.  (All 16 values
// through LDS would move four times the bytes: the LDS pipe, not the vector
// units, then bounds the kernel at few slots per lane.)  Returns the sum of
// value v in all four lanes of its quad (v = 4i + c: step j0 + i, c as in kVals).
__device__ __forceinline__ void sum_to_rows(SumRows &tb, const double (&acc)[kVals]) {
    static_assert(kVals == 16, "two exchanges leave 4 values per lane");
    const int lane = threadIdx.x & 63;
    double s[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) s[u] = swap_add<32>(acc[u], acc[u + 8]);
#pragma unroll
    for (int u = 0; u < 4; ++u) tb[4 * (lane >> 4) + u][lane & 15] = swap_add<16>(s[u], s[u + 4]);
    __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ double sum_row(const double (&row)[kTRow]) {
    const dvec2 *r = reinterpret_cast<const dvec2 *>(&row[4 * (threadIdx.x & 3)]);
    const dvec2 r0 = r[0], r1 = r[1];
    return quad_sum((r0.x + r0.y) + (r1.x + r1.y));
}
__device__ __forceinline__ double wave_sum16(SumRows &tb, const double (&acc)[kVals]) {
    sum_to_rows(tb, acc);
    const double v = sum_row(tb[(threadIdx.x & 63) >> 2]);
    __builtin_amdgcn_wave_barrier();
    return v;
}

// Brings the factors c_lm of one column that an analysis reads at the end of
// its chunks into this XCD's L2.
template <int NT>
__device__ __forceinline__ void warm_factors(const double *cfac, int n) {
    for (int i = 16 * (int)threadIdx.x; i < n; i += 16 * NT) {
        const double a = cfac[i];
        asm volatile("" ::"v"(a));
    }
}

// Analysis of one m of one map by a workgroup of W waves: wave w of group g
// owns slots ((g T + t) W + w) * 64 + lane, t < T (every wave gets sets from
// the whole range of latitudes, so that the waves' work stays even).  Per
// chunk of kChunk steps each lane sums its T slots; the wave sums its 64 lanes
// through its own LDS rows (no barrier); every kFlush chunks the W wave sums
// are added in wave order after one barrier.  The workgroup starts at the
// earliest start of its slots (a_lm before it get no term).  With one group
// the finished a_lm are written; otherwise the group's sums go to part[(map *
// groups + group) * nalm + idx] for k_ana_combine.  Every thread of the
// workgroup must call it.
template <int T, int W = kAnaWaves>
__device__ __forceinline__ void ana_group(const AnaArgs &A, int m, int grp, int map, int groups, AnaLds<W> &L) {
    constexpr int kThreads = 64 * W;
    const int lmax = A.lmax, nj = jcol_len(lmax, m);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2;
    const double2 *__restrict__ d = A.delta + (int64_t)map * A.nrings * (A.mmax + 1);
    double2 *__restrict__ dst = (groups == 1) ? A.alm + (int64_t)map * A.nalm + base
                                              : A.part + ((int64_t)map * groups + grp) * A.nalm + base;
    // this column's coefficients into the XCD's L2 while the slots are loaded
    const double warm_al = warm_l2(A.alpha + base, 1, m, lmax);
    AnaSlots<T, kMaxPolar / kThreads> S;  // polar slots: the first sets of the first group
    static_assert(kMaxPolar % kThreads == 0, "whole sets of polar slots");
    S.load(A, m, d, grp * kThreads * T + wave * 64, kThreads);
    asm volatile("" ::"v"(warm_al));
    if (groups == 1) warm_factors<kThreads>(A.cfac + base + m, lmax - m + 1);
    if (lane == 0) L.wstart[wave] = S.lo;
    __syncthreads();
    int j0s = nj;
#pragma unroll
    for (int w = 0; w < W; ++w) j0s = min(j0s, L.wstart[w]);
    j0s = __builtin_amdgcn_readfirstlane(j0s);  // the same in every lane

    for (int l = m + tid; l < m + 2 * j0s && l <= lmax; l += kThreads) dst[l] = make_double2(0.0, 0.0);

    // Every kFlush chunks (or at the last): thread f < nchunks*kVals takes the
    // value (chunk f/kVals, f%kVals) of the W waves' sums and writes it.
    auto flush = [&](int jbase, int par, int nchunks) {
        const int fk = tid / kVals, fv = tid % kVals, fc = tid & 3;
        const int l = m + 2 * (jbase + (tid >> 2)) + (fc >> 1);
        const bool mine = tid < nchunks * kVals && l <= lmax;
        const double c = groups == 1 && mine ? A.cfac[base + l] : 1.0;  // loaded ahead of the barrier
        __syncthreads();
        if (mine) {
            double v = 0.0;
#pragma unroll
            for (int u = 0; u < W; ++u) v += L.ring[par][fk][u][fv];
            if (groups == 1) v = m == 0 && (fc & 1) ? 0.0 : v * c;
            reinterpret_cast<double *>(dst + l)[fc & 1] = v;
        }
    };

    // the next chunk's coefficients are loaded at the start of a chunk, so that
    // they arrive under its arithmetic; the waits for the LDS traffic that
    // follows then find them there
    AnaCoefPtr cp{ro(A.alpha + base + m + 2 * j0s)};
    static_assert(4 * kChunk <= kCoefPad, "coefficient padding too short");
    AnaCoef cur, nxt;
    cp.load(cur);
    int par = 0, kc = 0, jbase = j0s;
#pragma unroll 1
    for (int j0 = j0s; j0 < nj; j0 += kChunk) {
        cp.load(nxt);
        double acc[kVals];
        S.chunk(j0, cur, acc);
        const double v = wave_sum16(L.tbuf[wave], acc);
        if ((lane & 3) == 0) L.ring[par][kc][wave][lane >> 2] = v;
        cur = nxt;
        if (++kc == kFlush || j0 + kChunk >= nj) {
            flush(jbase, par, kc);
            jbase += kFlush * kChunk;
            par ^= 1;
            kc = 0;
        }
    }
}

// Analysis of one m of one map by one wave holding every slot (nslots <=
// 64 T; lane i owns slots 64 t + i): per chunk the wave's sums go straight
// to a_lm, with no step across waves, so the waves of a workgroup may each
// work on their own m.  tb: the wave's reduction rows.
template <int T>
__device__ __forceinline__ void ana_wave(const AnaArgs &A, int m, int map, SumRows &tb) {
    const int lmax = A.lmax, nj = jcol_len(lmax, m);
    const int lane = threadIdx.x & 63;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2;
    const double2 *__restrict__ d = A.delta + (int64_t)map * A.nrings * (A.mmax + 1);
    double2 *__restrict__ dst = A.alm + (int64_t)map * A.nalm + base;
    const double warm_al = A.alpha[base + min(m + 16 * lane, lmax)];  // the column into L2, as warm_l2
    AnaSlots<T, kMaxPolar / 64> S;
    S.load(A, m, d, 0, 64);
    asm volatile("" ::"v"(warm_al));
    const int lo = S.lo;
    for (int l = m + lane; l < m + 2 * min(lo, nj) && l <= lmax; l += 64) dst[l] = make_double2(0.0, 0.0);
    if (lo >= nj) return;
    AnaCoefPtr cp{ro(A.alpha + base + m + 2 * lo)};
    AnaCoef cur, nxt;
    cp.load(cur);
    // this lane's value of a chunk: degree offset and part; its factor is loaded one chunk ahead
    const int fv = lane >> 2, fc = fv & 3, dl = 2 * (fv >> 2) + (fc >> 1);
    auto factor = [&](int j0) { return A.cfac[base + min(m + 2 * j0 + dl, lmax)]; };
    double fac = factor(lo);
#pragma unroll 1
    for (int j0 = lo; j0 < nj; j0 += kChunk) {
        cp.load(nxt);
        double fac_next = factor(j0 + kChunk);
        double acc[kVals];
        S.chunk(j0, cur, acc);
        const double v = wave_sum16(tb, acc);
        cur = nxt;
        // the next factor is waited for here: behind the store the wait would
        // include the store's own way to memory, in every chunk
        asm volatile("" : "+v"(fac_next));
        const int l = m + 2 * j0 + dl;
        if ((lane & 3) == 0 && l <= lmax)
            reinterpret_cast<double *>(dst + l)[fc & 1] = (m == 0 && (fc & 1)) ? 0.0 : v * fac;
        fac = fac_next;
    }
}

// Analysis kernel: grid.x = (m, slot group) in the XCD-aware order, grid.y =
// map.  Three waves per SIMD at 8 slots per lane (166 VGPRs): 549 us at HEALPix
// 1024 / lmax 2048 (two waves, with a recurrence of 6 operations: 637 against 589).
template <int T, int W>
__global__ __launch_bounds__(64 * W, T <= 4 ? 4 : 3) void k_leg_ana(AnaArgs A, int groups) {
    __shared__ AnaLds<W> L;
    const MPart mp = xcd_m_part(groups);
    if (mp.m > A.mmax) return;  // padding of the m range (whole workgroup, before any barrier)
    ana_group<T, W>(A, mp.m, mp.part, (int)blockIdx.y, groups, L);
}
// At most 64 slots, one wave per m: grid.x = m in the XCD-aware order, grid.y = map.
__global__ __launch_bounds__(64) void k_leg_ana_wave(AnaArgs A) {
    __shared__ alignas(16) SumRows tb;
    const MPart mp = xcd_m_part(1);
    if (mp.m > A.mmax) return;
    ana_wave<1>(A, mp.m, (int)blockIdx.y, tb);
}

// Sum of the groups' partial a_lm, groups in order.
__device__ __forceinline__ double2 group_sum(const double2 *__restrict__ part, int64_t nalm, int groups, int64_t idx) {
    double sr = 0.0, si = 0.0;
    for (int g = 0; g < groups; ++g) {
        const double2 v = part[(int64_t)g * nalm + idx];
        sr += v.x;
        si += v.y;
    }
    return make_double2(sr, si);
}
// a_lm = c_lm * sum_{g < groups} part[map][g][idx], groups summed in order.
__global__ __launch_bounds__(kBlock) void k_ana_combine(int64_t nalm, int lmax, int nmaps, int groups,
                                                        const double2 *__restrict__ part,
                                                        const double *__restrict__ cfac,
                                                        double2 *__restrict__ alm) {
    const int64_t total = nalm * nmaps;
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * kBlock) {
        const int64_t map = i / nalm, k = i - map * nalm;
        const double2 v = group_sum(part + map * groups * nalm, nalm, groups, k);
        const double c = cfac[k];
        alm[i] = make_double2(v.x * c, k <= lmax ? 0.0 : v.y * c);
    }
}

// ---------------------------------------------------------------- uneven batches
// The Legendre stage of a whole batch of requests (any lmax and geometry, both
// directions) in one persistent launch.  Each workgroup takes the next item of
// a device work queue (one atomic add by one thread, broadcast through LDS)
// until the queue is empty, then exits; the host lists the items longest
// first, so that the cheap ones (high m, small requests) fill the end of the
// run on every CU.  Every item's work is that of the ordinary kernels, so
// which workgroup takes it does not change a result.
__global__ __launch_bounds__(kBlock, 3) void k_leg_batch(const BatchReq *__restrict__ reqs,
                                                       const BatchItem *__restrict__ items, int nitems,
                                                       int *__restrict__ head) {
    __shared__ AnaLds<> L;
    __shared__ int s_idx;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    for (;;) {
        if (threadIdx.x == 0) s_idx = atomicAdd(head, 1);
        __syncthreads();
        const int idx = __builtin_amdgcn_readfirstlane(s_idx);
        __syncthreads();  // every thread has read s_idx before it is written again
        if (idx >= nitems) return;  // the whole workgroup: the queue is empty
        const BatchItem it = items[idx];
        const BatchReq &R = reqs[it.req];
        const int T = R.T;
        if (R.kind == 0) {
            const int u = it.u0 + wave;
            if (u < R.nunits) {
                const int m = __builtin_amdgcn_readfirstlane(u / R.tiles);
                const int slot0 = (u - m * R.tiles) * 64 * T;
                if (T == 1) syn_tile<1>(R.syn, m, 0, 1, slot0, lane);
                else if (T == 2) syn_tile<2>(R.syn, m, 0, 1, slot0, lane);
                else syn_tile<4>(R.syn, m, 0, 1, slot0, lane);
            }
        } else if (R.shape == 0) {
            const int m = it.u0 + wave;
            if (m <= R.ana.mmax) {
                if (T == 1) ana_wave<1>(R.ana, m, 0, L.tbuf[wave]);
                else if (T == 2) ana_wave<2>(R.ana, m, 0, L.tbuf[wave]);
                else ana_wave<4>(R.ana, m, 0, L.tbuf[wave]);
            }
        } else {
            const int m = it.u0 / R.groups, grp = it.u0 - m * R.groups;
            if (T == 1) ana_group<1>(R.ana, m, grp, 0, R.groups, L);
            else if (T == 2) ana_group<2>(R.ana, m, grp, 0, R.groups, L);
            else ana_group<4>(R.ana, m, grp, 0, R.groups, L);
        }
        __syncthreads();  // the item's LDS use is over before the next one starts
    }
}

__global__ void k_batch_reset(int *head) { *head = 0; }

// c-scaled a_lm of every synthesis request of a batch: grid.y = request (of
// the list), grid.x strides over its a_lm.
__global__ __launch_bounds__(kBlock) void k_prescale_batch(const BatchReq *__restrict__ reqs,
                                                            const int32_t *__restrict__ list) {
    const BatchReq &R = reqs[list[blockIdx.y]];
    const int64_t nalm = R.syn.nalm;
    const int lmax = R.syn.lmax;
    const double *__restrict__ cfac = R.ana.cfac;
    double2 *out = const_cast<double2 *>(R.syn.ap);
    for (int64_t k = blockIdx.x * (int64_t)kBlock + threadIdx.x; k < nalm; k += (int64_t)gridDim.x * kBlock) {
        const double c = cfac[k];
        const double2 a = R.alm_in[k];
        out[k] = make_double2(a.x * c, k <= lmax ? 0.0 : a.y * c);  // Im a_l0 is ignored
    }
}

// a_lm = c_lm * sum of the group partials (groups in order) for every
// analysis request of the list that has several groups.
__global__ __launch_bounds__(kBlock) void k_combine_batch(const BatchReq *__restrict__ reqs,
                                                           const int32_t *__restrict__ list) {
    const BatchReq &R = reqs[list[blockIdx.y]];
    const int64_t nalm = R.ana.nalm;
    for (int64_t k = blockIdx.x * (int64_t)kBlock + threadIdx.x; k < nalm; k += (int64_t)gridDim.x * kBlock) {
        const double2 v = group_sum(R.ana.part, nalm, R.groups, k);
        const double c = R.ana.cfac[k];
        R.ana.alm[k] = make_double2(v.x * c, k <= R.ana.lmax ? 0.0 : v.y * c);
    }
}

}  // namespace

int leg_batch_grid(int *grid) {
    int dev = 0, per_cu = 0;
    SHT_HIP(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    SHT_HIP(hipGetDeviceProperties(&prop, dev));
    SHT_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_leg_batch, kBlock, 0));
    *grid = std::max(1, per_cu) * prop.multiProcessorCount;
    return SHT_OK;
}

int launch_leg_batch(const BatchReq *reqs, const BatchItem *items, int nitems, int *head, int grid, hipStream_t st) {
    hipLaunchKernelGGL(k_batch_reset, dim3(1), dim3(1), 0, st, head);
    SHT_HIP(hipGetLastError());
    if (nitems <= 0) return SHT_OK;
    hipLaunchKernelGGL(k_leg_batch, dim3((unsigned)std::min(grid, nitems)), dim3(kBlock), 0, st, reqs, items, nitems,
                       head);
    SHT_HIP(hipGetLastError());
    return SHT_OK;
}

int launch_prescale_batch(const BatchReq *reqs, const int32_t *syn_reqs, int nsyn, int max_chunks, hipStream_t st) {
    if (nsyn <= 0) return SHT_OK;
    if (nsyn > 65535) return SHT_EUNSUPPORTED;
    hipLaunchKernelGGL(k_prescale_batch, dim3((unsigned)max_chunks, (unsigned)nsyn), dim3(kBlock), 0, st, reqs, syn_reqs);
    SHT_HIP(hipGetLastError());
    return SHT_OK;
}

int launch_combine_batch(const BatchReq *reqs, const int32_t *comb_reqs, int ncomb, int max_chunks, hipStream_t st) {
    if (ncomb <= 0) return SHT_OK;
    if (ncomb > 65535) return SHT_EUNSUPPORTED;
    hipLaunchKernelGGL(k_combine_batch, dim3((unsigned)max_chunks, (unsigned)ncomb), dim3(kBlock), 0, st, reqs, comb_reqs);
    SHT_HIP(hipGetLastError());
    return SHT_OK;
}

int launch_leg_start(const CoefTables &c, const GeomPlan &p, int32_t *jstart, void *state, hipStream_t st) {
    const int tiles = (p.nslots + kBlock - 1) / kBlock;
    if (c.mmax + 1 > 65535) return SHT_EUNSUPPORTED;
    hipLaunchKernelGGL(k_leg_start, dim3((unsigned)tiles, (unsigned)(c.mmax + 1)), dim3(kBlock), 0, st, c.lmax,
                       p.nslots, p.npolar, c.alpha, c.mu, p.slot_w, p.slot_s, jstart, static_cast<double2 *>(state));
    SHT_HIP(hipGetLastError());
    return SHT_OK;
}

int launch_prescale(const CoefTables &c, const void *alm, void *aprime, int nmaps, hipStream_t st) {
    const int64_t total = c.nalm * nmaps;
    const int64_t blocks = std::min<int64_t>((total + kBlock - 1) / kBlock, 1 << 16);
    hipLaunchKernelGGL(k_prescale, dim3((unsigned)blocks), dim3(kBlock), 0, st, c.nalm, c.lmax, nmaps,
                       static_cast<const double2 *>(alm), c.cfac, static_cast<double2 *>(aprime));
    SHT_HIP(hipGetLastError());
    return SHT_OK;
}

constexpr int kSynSlotsPerLane = 4;
template <int T, int M>
static int launch_syn_mm(const SynArgs &A, int nslots, int mmax, int nmaps, hipStream_t st) {
    const int tiles = (nslots + kBlock * T - 1) / (kBlock * T);
    const int64_t gx = (int64_t)tiles * padded_m(mmax);
    if (!grid_ok(gx)) return SHT_EUNSUPPORTED;
    hipLaunchKernelGGL((k_leg_syn_mm<T, M>), dim3((unsigned)gx, (unsigned)((nmaps + M - 1) / M)), dim3(kBlock), 0, st,
                       A, tiles, nmaps);
    SHT_HIP(hipGetLastError());
    return SHT_OK;
}

int launch_leg_syn(const CoefTables &c, const GeomPlan &p, const StartTable &s, const void *aprime, void *delta,
                   int nmaps, hipStream_t st) {
    const SynArgs A = syn_args(c, p, s, aprime, delta);
    if (nmaps > 65535) return SHT_EUNSUPPORTED;
    // Slots per lane: kSynSlotsPerLane for large geometries, 1 where one
    // workgroup then holds every slot of an m and 2 up to 768 slots.  With few
    // slots a tile of kSynSlotsPerLane per lane would leave lanes and waves of
    // the workgroup idle while the others walk the recurrences of their slots
    // in turn; small transforms are bound by that sequential walk of the longest m.
    const int T = p.nslots <= kBlock ? 1 : p.nslots <= (nmaps >= 2 ? 2 : 3) * kBlock ? 2 : kSynSlotsPerLane;
    // several maps share each recurrence: 2 maps per workgroup (at 4 slots per
    // lane faster than 4 maps and 2 slots: with the one-step recurrence 29.7 against 30.6 ms for 64 maps at
    // HEALPix 1024 / lmax 2048)
    if (nmaps >= 2) {
        switch (T) {
            case 1: return launch_syn_mm<1, 2>(A, p.nslots, c.mmax, nmaps, st);
            case 2: return launch_syn_mm<2, 2>(A, p.nslots, c.mmax, nmaps, st);
            default: return launch_syn_mm<kSynSlotsPerLane, 2>(A, p.nslots, c.mmax, nmaps, st);
        }
    }
    const int tiles = (p.nslots + kBlock * T - 1) / (kBlock * T);
    const int64_t gx = (int64_t)tiles * padded_m(c.mmax);
    if (!grid_ok(gx)) return SHT_EUNSUPPORTED;
    const dim3 grid((unsigned)gx, (unsigned)nmaps);
    switch (T) {
        case 1: hipLaunchKernelGGL(k_leg_syn<1>, grid, dim3(kBlock), 0, st, A, tiles); break;
        case 2: hipLaunchKernelGGL(k_leg_syn<2>, grid, dim3(kBlock), 0, st, A, tiles); break;
        default: hipLaunchKernelGGL(k_leg_syn<kSynSlotsPerLane>, grid, dim3(kBlock), 0, st, A, tiles); break;
    }
    SHT_HIP(hipGetLastError());
    return SHT_OK;
}

template <int T, int W = kAnaWaves>
static void launch_ana_t(const AnaArgs &A, int groups, int nmaps, hipStream_t st) {
    hipLaunchKernelGGL((k_leg_ana<T, W>), dim3((unsigned)(padded_m(A.mmax) * groups), (unsigned)nmaps), dim3(64 * W), 0, st,
                       A, groups);
}

int launch_leg_ana(const CoefTables &c, const GeomPlan &p, const StartTable &s, const void *delta, void *alm,
                   int nmaps, void *partials, hipStream_t st) {
    if (nmaps > 65535) return SHT_EUNSUPPORTED;
    const int T = ana_slots_per_thread(p.nslots);
    const int groups = ana_groups(p.nslots);
    if (!grid_ok((int64_t)padded_m(c.mmax) * groups)) return SHT_EUNSUPPORTED;
    if (groups > 1 && !partials) return SHT_EWORKSPACE;
    const AnaArgs A = ana_args(c, p, s, delta, alm, partials);
    // The form depends on the slots alone, not on the number of maps: a map's
    // a_lm are the same bits in any call.
    if (p.nslots <= 64) {
        // one wave holds every slot: no step across waves (lmax 64 on 64
        // slots: 10.2 us for the stage against 11.6 with a workgroup)
        hipLaunchKernelGGL(k_leg_ana_wave, dim3((unsigned)padded_m(c.mmax), (unsigned)nmaps), dim3(64), 0, st, A);
    } else if (p.nslots <= 192 || (p.nslots > 512 && p.nslots <= 640)) {
        // Two waves of up to 5 slots per lane instead of four: fewer wave sums, and
        // no idle waves on up to 3 sets of 64 slots.  Stage for one and for 64 maps:
        // 129 slots, lmax 256, 21.9 and 171 us (four waves 22.7 and 254); 513 slots,
        // lmax 1024, 119 us and 3.36 ms (108 and 4.46).  On 193 to 512 slots one map
        // leaves the chip with too few waves for that (226 slots, lmax 450, one and
        // eight maps: 34.5 and 92 us, four waves 31.7 and 126), and from 641 on two
        // waves of 6 and more cost one map more than they give several (694 slots,
        // lmax 694: 90 and 293 us, four waves 73 and 333).
        switch ((p.nslots + 127) / 128) {
            case 1: launch_ana_t<1, 2>(A, groups, nmaps, st); break;
            case 2: launch_ana_t<2, 2>(A, groups, nmaps, st); break;
            default: launch_ana_t<5, 2>(A, groups, nmaps, st); break;
        }
    } else {
        switch (T) {
            case 1: launch_ana_t<1>(A, groups, nmaps, st); break;
            case 2: launch_ana_t<2>(A, groups, nmaps, st); break;
            case 3: launch_ana_t<3>(A, groups, nmaps, st); break;
            case 4: launch_ana_t<4>(A, groups, nmaps, st); break;
            case 5: launch_ana_t<5>(A, groups, nmaps, st); break;
            case 6: launch_ana_t<6>(A, groups, nmaps, st); break;
            case 7: launch_ana_t<7>(A, groups, nmaps, st); break;
            default: launch_ana_t<kAnaSlotsPerThread>(A, groups, nmaps, st); break;
        }
    }
    SHT_HIP(hipGetLastError());
    return groups > 1 ? launch_ana_combine(c, nmaps, groups, partials, alm, st) : SHT_OK;
}

int launch_ana_combine(const CoefTables &c, int nmaps, int groups, const void *partials, void *alm,
                       hipStream_t st) {
    const int64_t total = c.nalm * nmaps;
    const int64_t blocks = std::min<int64_t>((total + kBlock - 1) / kBlock, 1 << 16);
    hipLaunchKernelGGL(k_ana_combine, dim3((unsigned)blocks), dim3(kBlock), 0, st, c.nalm, c.lmax, nmaps, groups,
                       static_cast<const double2 *>(partials), c.cfac, static_cast<double2 *>(alm));
    SHT_HIP(hipGetLastError());
    return SHT_OK;
}

}  // namespace sht

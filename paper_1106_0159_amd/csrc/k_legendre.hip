// Legendre-stage kernels for gfx950 (FP64 VALU).
//
// Synthesis computes Delta^A_m(r) = sum_l a_lm lambda_lm(cos theta_r)
// (Sec. 2.2 eq. DeltaDef); analysis computes a_lm = sum_r Delta^S_m(r)
// lambda_lm(cos theta_r) (eq. almdef).  lambda_lm comes from the l-recurrence
// (eqs. assLegRec, betaDef) seeded by lambda_mm = (-1)^m mu_m sin^m(theta)
// (eq. pmm, with the exponent m/2 and the Condon-Shortley phase) and
// lambda_{m+1,m} = sqrt(2m+3) x lambda_mm (eq. pm1m).
//
// The recurrence steps by two in l and runs in x^2 (the idea of Ishioka, J.
// Meteorol. Soc. Japan 96, 2018): with eps_l = 1/beta_l, r_j =
// lambda_{m+2j+1,m} / x is a polynomial in x^2 times sin^m(theta), and after
// rescaling r_j = C_j q_j its three-term recurrence reads
//   q_j = (A_j x^2 + B_j) q_{j-1} - q_{j-2},
// two fused multiply-adds for two degrees l.  Both parities come from q_j:
//   lambda_{m+2j+1} = C_j x q_j,
//   lambda_{m+2j}   = C_j eps_{m+2j+1} q_j + C_{j-1} eps_{m+2j} q_{j-1}.
// Synthesis folds these factors into a_lm once per call (k_prescale): with
// e_j = C_j (eps_{m+2j+1} a_{m+2j} + eps_{m+2j+2} a_{m+2j+2}) and o_j = C_j
// a_{m+2j+1} the sum is E = sum_j e_j q_j plus x times O = sum_j o_j q_j.
// Analysis sums S_j = sum q_j D+ and T_j = sum q_j x D- over the rings and
// forms a_{m+2j} = C_j eps S_j + C_{j-1} eps S_{j-1}, a_{m+2j+1} = C_j T_j.
// A (ring pair, two l) costs 6 FP64 operations instead of the 8 of the
// one-step recurrence, and its rounding errors were smaller as well (lmax
// 1024, HEALPix: 1.3e-14 against 2.4e-14 relative RMS of the recurrence alone).
//
// One recurrence serves a ring and its mirror image (x -> -x): the even part
// E is the same and the odd part x O changes sign.
//
// Underflow near the poles (Sec. 2.1 asks for rescaling and leaves the
// algorithm to its references).  Once per plan, k_leg_start runs every
// (m, slot) recurrence from its seed with exponent tracking (a value held as
// q * 2^(600 sc), sc <= 0) until |q| first reaches 2^-100, and stores the j
// that opens the block of kStartJ steps holding that step, with the two
// recurrence values before it.  The transform kernels start each slot there:
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
constexpr double kStart = 0x1p-100;  // a slot starts once |q| reaches this
static_assert(kScaleBits == 600, "kDown must equal 2^-kScaleBits");

// q_0 = (-1)^m f_m s^m as carrier * 2^(600 sc), f_m = mu_m sqrt(2m+3).  s^m by
// binary powering with frexp renormalisation; s and its squares are carried as
// two doubles, since each squaring doubles the relative error of what it
// squares (with one double the seed of m would be off by about m/2 roundings).
__device__ __forceinline__ double seed_carrier(int m, double2 s, double f_m, int &sc) {
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
    const double v = ((m & 1) ? -f_m : f_m) * (r + rl);
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
// state[m * nslots + slot] = (q_{j-2}, q_{j-1}) before step j = jstart.
__global__ __launch_bounds__(kBlock) void k_leg_start(int lmax, int nslots, int npolar,
                                                      const double *__restrict__ ra,
                                                      const double *__restrict__ rb,
                                                      const double *__restrict__ rbp,
                                                      const double *__restrict__ seeds,
                                                      const double *__restrict__ sw,
                                                      const double2 *__restrict__ ss,
                                                      int32_t *__restrict__ jstart,
                                                      double2 *__restrict__ state) {
    const int slot = blockIdx.x * kBlock + threadIdx.x;
    const int m = blockIdx.y;
    if (slot >= nslots) return;
    const double w = sw[slot];
    const int64_t jb = jcol_base(lmax, m);
    const double *__restrict__ ca = ra + jb, *__restrict__ cb = (slot < npolar ? rbp : rb) + jb;
    const int nj = jcol_len(lmax, m);
    int sc;
    const double seed = seed_carrier(m, ss[slot], seeds[m], sc);
    // (q_{j-2}, q_{j-1}) before step j; (-seed, 0) makes step j = 0 yield the seed
    double q2 = -seed, q1 = 0.0;
    int found = kNeverJ;
    double s2 = 0.0, s1 = 0.0;
    for (int j0 = 0; j0 < nj && found == kNeverJ; j0 += kStartJ) {
        const double b2 = q2, b1 = q1;
        const int bsc = sc;
        bool hit = false;
        for (int i = 0; i < kStartJ && j0 + i < nj; ++i) {
            const double q = fma(fma(ca[j0 + i], w, cb[j0 + i]), q1, -q2);
            q2 = q1;
            q1 = q;
            hit |= (sc == 0 && fabs(q) >= kStart);
            // one step grows a value by less than 2^16 (A_j < 2 m)
            if ((i & 1) && sc < 0 && fabs(q1) > kThresh) {
                q1 *= kDown;
                q2 *= kDown;
                ++sc;
            }
        }
        if (hit) {
            found = j0;
            // a value leaves sc < 0 near 2^-660 and cannot grow past 2^-100
            // within one block, so bsc is 0 here in practice
            s2 = ldexp(b2, kScaleBits * bsc);
            s1 = ldexp(b1, kScaleBits * bsc);
        }
    }
    jstart[(int64_t)m * nslots + slot] = found;
    state[(int64_t)m * nslots + slot] = make_double2(s2, s1);
}

// Scaled coefficients of one column: entries m + 2j and m + 2j + 1 of the
// packed column become e_j and o_j (as many entries as a_lm has: o_j exists
// where m + 2j + 1 <= lmax).  col and out point to entry l = 0 of the column.
__device__ __forceinline__ void prescale_column(int lmax, int m, const double2 *__restrict__ col, ParityFac f,
                                                double2 *__restrict__ out) {
    const int64_t jb = jcol_base(lmax, m);
    const int nj = jcol_len(lmax, m);
    for (int j = threadIdx.x; j < nj; j += kBlock) {
        const int l = m + 2 * j;
        const double p1 = f.pe1[jb + j], p2 = f.pe2[jb + j], po = f.po[jb + j];
        const double2 a0 = col[l];
        const double2 a1 = l + 1 <= lmax ? col[l + 1] : make_double2(0.0, 0.0);
        const double2 a2 = l + 2 <= lmax ? col[l + 2] : make_double2(0.0, 0.0);
        // m = 0: Im a_l0 is ignored
        out[l] = make_double2(fma(p1, a0.x, p2 * a2.x), m == 0 ? 0.0 : fma(p1, a0.y, p2 * a2.y));
        if (l + 1 <= lmax) out[l + 1] = make_double2(po * a1.x, m == 0 ? 0.0 : po * a1.y);
    }
}
// grid.x = m, grid.y = map
__global__ __launch_bounds__(kBlock) void k_prescale(int64_t nalm, int lmax, const double2 *__restrict__ alm,
                                                     ParityFac f, double2 *__restrict__ out) {
    const int m = blockIdx.x;
    const int64_t at = blockIdx.y * nalm + (int64_t)m * (2 * lmax + 1 - m) / 2;
    prescale_column(lmax, m, alm + at, f, out + at);
}

// a_lm of one column from the sums over the rings, given by sum(l): S_j at
// l = m + 2j and T_j at l = m + 2j + 1.
template <class Sum>
__device__ __forceinline__ void finish_column(int lmax, int m, ParityFac f, Sum sum, double2 *__restrict__ col) {
    const int64_t jb = jcol_base(lmax, m);
    for (int l = m + threadIdx.x; l <= lmax; l += kBlock) {
        const int j = (l - m) >> 1;
        const double2 v = sum(l);
        if ((l - m) & 1) {
            const double c = f.po[jb + j];
            col[l] = make_double2(c * v.x, m == 0 ? 0.0 : c * v.y);
        } else {
            const double c = f.pe1[jb + j], d = j > 0 ? f.pe2[jb + j - 1] : 0.0;
            const double2 u = j > 0 ? sum(l - 2) : make_double2(0.0, 0.0);
            col[l] = make_double2(fma(c, v.x, d * u.x), m == 0 ? 0.0 : fma(c, v.y, d * u.y));
        }
    }
}

// Synthesis of one m of M maps over a tile of slots: a wave (li / 64 of the
// threads sharing the tile) owns 64 T consecutive slots, its lanes the slots
// 64 u + lane of them, u < T (so that a set of 64 that has not started is
// skipped whole, and table reads are contiguous: 2 to 5 % at HEALPix 512 to
// 700), for maps map0 .. map0 + M - 1 (those past nmaps repeat the last map and are not
// stored).  Each recurrence value serves the M maps, so a slot and two l cost
// 2 + 4M operations instead of 6M; per map the arithmetic (the same fused
// multiply-adds in the same order) does not depend on M, so results are the
// same bits for any M.  The wave works on its own (no cross-wave step), so a
// tile may be one wave's (li = lane) or a workgroup's (li = thread index).
template <int T, int M = 1>
__device__ __forceinline__ void syn_tile(const SynArgs &A, int m, int map0, int nmaps, int slot0, int li) {
    const int lmax = A.lmax, mmax = A.mmax, nslots = A.nslots, nrings = A.nrings;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2;  // (l, m) lives at base + l
    ConstC a[M];
#pragma unroll
    for (int k = 0; k < M; ++k) a[k] = ro(A.ap + (int64_t)min(map0 + k, nmaps - 1) * A.nalm + base + m);
    // the wave's slots are all polar or all not (npolar is a multiple of the tile)
    const int wave0 = __builtin_amdgcn_readfirstlane(slot0 + (li & ~63) * T), lane = li & 63;
    const bool polar = wave0 < A.npolar;
    const int64_t jb = jcol_base(lmax, m);
    const const_ptr<double> ra = ro(A.ra + jb), rb = ro((polar ? A.rbp : A.rb) + jb);
    const int nj = jcol_len(lmax, m);

    double w[T], q1[T], q2[T], er[T][M], ei[T][M], orr[T][M], oi[T][M];
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
        js[u] = act ? A.jstart[(int64_t)m * nslots + slot] : kNeverJ;
        const double2 st = act ? A.state[(int64_t)m * nslots + slot] : make_double2(0.0, 0.0);
        q2[u] = st.x;
        q1[u] = st.y;
#pragma unroll
        for (int k = 0; k < M; ++k) er[u][k] = ei[u][k] = orr[u][k] = oi[u][k] = 0.0;
        lo = min(lo, js[u]);
        if (js[u] < nj) hi = max(hi, js[u]);
        // not started for this lmax: the state is carried but never used
        if (js[u] >= nj) q1[u] = q2[u] = 0.0;
    }
    lo = wave_min(lo);
    hi = wave_max(hi);

    struct Coef {
        double a, b;  // A_j and B_j (or A_j + B_j)
        double2 e[M], o[M];
    };
    auto load = [&](int j, Coef &k) {
        k.a = ra[j];
        k.b = rb[j];
#pragma unroll
        for (int i = 0; i < M; ++i) {
            k.e[i] = a[i][2 * j];
            k.o[i] = a[i][2 * j + 1];
        }
    };
    // step j of slot u: q_j, then its terms of both parities (ODD: o_j exists)
    // with A_j given in a vector register (an instruction reads one scalar operand)
    auto step = [&](const Coef &c, double aj, int u, auto odd) {
        const double q = fma(fma(aj, w[u], c.b), q1[u], -q2[u]);
        q2[u] = q1[u];
        q1[u] = q;
#pragma unroll
        for (int k = 0; k < M; ++k) {
            er[u][k] = fma(c.e[k].x, q, er[u][k]);
            ei[u][k] = fma(c.e[k].y, q, ei[u][k]);
            if constexpr (decltype(odd)::value) {
                orr[u][k] = fma(c.o[k].x, q, orr[u][k]);
                oi[u][k] = fma(c.o[k].y, q, oi[u][k]);
            }
        }
    };
    auto vec = [](double v) {
        asm("" : "+v"(v));
        return v;
    };
    const int nfull = (lmax - m + 1) / 2;  // steps with both parities

    // Blocks of kStartJ steps of both parities, in halves of two steps with two
    // coefficient sets in turn, each loaded one half ahead (a, ra and rb are
    // padded, so the loads past the column's end stay in bounds).  Start
    // positions are multiples of kStartJ: while slots join (j <= hi) the lanes
    // of a slot that has not started are masked off and it keeps its state.
    // The trip counts are fixed up front so that no exit separates a load from
    // its use.
    int j = lo;
    if (j + kStartJ <= nfull) {
        // running pointers: the loads of a half are one run of scalar loads each
        const_ptr<double> pra = ra + j, prb = rb + j;
        const_ptr<dvec2> pa[M];
#pragma unroll
        for (int k = 0; k < M; ++k) pa[k] = a[k].p + 2 * j;
        auto pair = [](dvec2 v) { return make_double2(v.x, v.y); };
        auto load2 = [&](int ofs, Coef (&c)[2]) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                c[i].a = pra[ofs + i];
                c[i].b = prb[ofs + i];
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
            const double a0 = vec(c[0].a), a1 = vec(c[1].a);
#pragma unroll
            for (int u = 0; u < T; ++u)
                if (j >= js[u]) {
                    step(c[0], a0, u, std::true_type{});
                    step(c[1], a1, u, std::true_type{});
                }
        };
        auto step2 = [&](const Coef (&c)[2]) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const double aj = vec(c[i].a);
#pragma unroll
                for (int u = 0; u < T; ++u) step(c[i], aj, u, std::true_type{});
            }
        };
        auto advance = [&]() {
            pra += kStartJ;
            prb += kStartJ;
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
                    step(c, c.a, u, std::true_type{});
                else
                    step(c, c.a, u, std::false_type{});
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
    const double warm_al = warm_l2(A.ra + jcol_base(A.lmax, m), 1, 0, jcol_len(A.lmax, m) - 1);
    const double warm_bl = warm_l2(A.rb + jcol_base(A.lmax, m), 1, 0, jcol_len(A.lmax, m) - 1);
    syn_tile<T, M>(A, m, map0, nmaps, tile * kBlock * T, (int)threadIdx.x);
    asm volatile("" ::"v"(warm_a), "v"(warm_al), "v"(warm_bl));  // the warming loads are waited for only here
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
    const double warm_al = warm_l2(A.ra + jcol_base(A.lmax, m), 1, 0, jcol_len(A.lmax, m) - 1);
    const double warm_bl = warm_l2(A.rb + jcol_base(A.lmax, m), 1, 0, jcol_len(A.lmax, m) - 1);
    syn_tile<T>(A, m, (int)blockIdx.y, (int)gridDim.y, tile * kBlock * T, (int)threadIdx.x);
    asm volatile("" ::"v"(warm_a), "v"(warm_al), "v"(warm_bl));  // the warming loads are waited for only here
}

constexpr int kChunk = kStartJ;       // recurrence steps per in-wave reduction in analysis
constexpr int kVals = 4 * kChunk;     // sums per chunk: (step, {S re, S im, T re, T im})
// chunks between cross-wave flushes (one barrier each)
constexpr int kFlush = 8;
// Wave-private rows of the in-wave reduction: 16 doubles and 2 of padding (the
// padding keeps the row reads free of bank conflicts)
constexpr int kTRow = 18;
typedef double SumRows[kVals][kTRow];

// Coefficients of one chunk (scalar registers): A_j, B_j, and for the first
// sets of a lane's slots B_j or (polar) A_j + B_j.
struct AnaCoef {
    double a[kChunk], b[kChunk], b0[kChunk];
};
struct AnaCoefPtr {
    const_ptr<double> a, b, b0;  // at the chunk that load() reads next
    // entries past the column's end belong to the next column or the padding
    // and are never used
    __device__ __forceinline__ void load(AnaCoef &c) {
#pragma unroll
        for (int i = 0; i < kChunk; ++i) {
            c.a[i] = a[i];
            c.b[i] = b[i];
            c.b0[i] = b0[i];
        }
        a += kChunk;
        b += kChunk;
        b0 += kChunk;
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
    alignas(16) SumRows tbuf[W][2];
    double ring[2][kFlush][W][kVals];
    double carry[2][2];  // S_{j-1} before a flush's first step
    int wstart[W];
    static_assert(kFlush * kVals <= 64 * W, "one thread per flushed value");
};

// The slot operands of one lane, slots slot0 + stride t + lane (t < T, sets of
// 64 slots): recurrence argument, start, recurrence state and the pair sums
// D+ = north + south and x D-, D- = north - south, of Delta_m.
template <int T>
struct AnaSlots {
    double w[T], q1[T], q2[T], pr[T], pi[T], mr[T], mi[T];
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
            x[t] = A.sx[sl];
            rn[t] = A.rn[sl];
            rs[t] = A.rsouth[sl];
            const int js0 = A.jstart[(int64_t)m * nslots + sl];
            const double2 st = A.state[(int64_t)m * nslots + sl];
            js[t] = act && js0 < nj ? js0 : kNeverJ;
            q2[t] = st.x;
            q1[t] = st.y;
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
    // One chunk of kChunk recurrence steps from j0 on: acc = sum over the
    // slots of q_j * (D+, x D-) per step.  A slot that has not started keeps its
    // state (its lanes masked off; a set that has not started at all is skipped).
    // FULL: no end-of-column guard (nsteps steps otherwise).  The first PS sets
    // take c.b0 (they may be polar), the others c.b.
    template <bool FULL, int PS>
    __device__ __forceinline__ void chunk(int j0, int nsteps, const AnaCoef &c, double (&acc)[kVals]) {
#pragma unroll
        for (int v = 0; v < kVals; ++v) acc[v] = 0.0;
        // A_j in vector registers: an instruction reads one scalar operand, B_j
        double a[kChunk];
#pragma unroll
        for (int i = 0; i < kChunk; ++i) {
            a[i] = c.a[i];
            asm("" : "+v"(a[i]));
        }
#pragma unroll
        for (int t = T - 1; t >= 0; --t) {
            if (j0 >= js[t]) {
#pragma unroll
                for (int i = 0; i < kChunk; ++i) {
                    if (FULL || i < nsteps) {
                        const double q = fma(fma(a[i], w[t], t >= PS ? c.b[i] : c.b0[i]), q1[t], -q2[t]);
                        q2[t] = q1[t];
                        q1[t] = q;
                        acc[4 * i + 0] = fma(q, pr[t], acc[4 * i + 0]);
                        acc[4 * i + 1] = fma(q, pi[t], acc[4 * i + 1]);
                        acc[4 * i + 2] = fma(q, mr[t], acc[4 * i + 2]);
                        acc[4 * i + 3] = fma(q, mi[t], acc[4 * i + 3]);
                    }
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

// Brings the factors of one column that an analysis reads at the end of its
// chunks into this XCD's L2.
template <int NT>
__device__ __forceinline__ void warm_factors(const ParityFac &f, int64_t jb, int nj) {
    for (int i = 16 * (int)threadIdx.x; i < nj; i += 16 * NT) {
        const double a = f.pe1[jb + i], b = f.pe2[jb + i], c = f.po[jb + i];
        asm volatile("" ::"v"(a), "v"(b), "v"(c));
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
// groups + group) * nalm + idx] for k_ana_finish.  Every thread of the
// workgroup must call it.
template <int T, int W = kAnaWaves>
__device__ __forceinline__ void ana_group(const AnaArgs &A, int m, int grp, int map, int groups, AnaLds<W> &L) {
    constexpr int kThreads = 64 * W;
    const int lmax = A.lmax, nj = jcol_len(lmax, m);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2, jb = jcol_base(lmax, m);
    const double2 *__restrict__ d = A.delta + (int64_t)map * A.nrings * (A.mmax + 1);
    double2 *__restrict__ dst = (groups == 1) ? A.alm + (int64_t)map * A.nalm + base
                                              : A.part + ((int64_t)map * groups + grp) * A.nalm + base;
    // the first sets of the first group hold the polar slots, if any
    constexpr int PS = kPolarSlots / kThreads;
    static_assert(PS * kThreads == kPolarSlots, "whole sets of polar slots");
    const double *b0 = grp == 0 && A.npolar ? A.rbp : A.rb;
    // this column's coefficients into the XCD's L2 while the slots are loaded
    const double warm_a = warm_l2(A.ra + jb, 1, 0, nj - 1), warm_b = warm_l2(A.rb + jb, 1, 0, nj - 1);
    AnaSlots<T> S;
    S.load(A, m, d, grp * kThreads * T + wave * 64, kThreads);
    asm volatile("" ::"v"(warm_a), "v"(warm_b));
    if (groups == 1) warm_factors<kThreads>(A.fac, jb, nj);
    if (lane == 0) L.wstart[wave] = S.lo;
    if (tid < 4) L.carry[tid >> 1][tid & 1] = 0.0;
    __syncthreads();
    int j0s = nj;
#pragma unroll
    for (int w = 0; w < W; ++w) j0s = min(j0s, L.wstart[w]);
    j0s = __builtin_amdgcn_readfirstlane(j0s);  // the same in every lane

    for (int l = m + tid; l < m + 2 * j0s && l <= lmax; l += kThreads) dst[l] = make_double2(0.0, 0.0);

    // Every kFlush chunks (or at the last): thread f < nchunks*kVals takes the
    // value (chunk f/kVals, v = f%kVals) of the W waves' sums and writes it.
    auto flush = [&](int jbase, int par, int nchunks) {
        const int fk = tid / kVals, fv = tid % kVals, fc = tid & 3;
        const int j = jbase + (tid >> 2), l = m + 2 * j + (fc >> 1);
        const bool mine = tid < nchunks * kVals;
        double f0 = 0.0, f1 = 0.0;  // loaded ahead of the barrier
        if (groups == 1 && mine && j < nj) {
            f0 = fc < 2 ? A.fac.pe1[jb + j] : A.fac.po[jb + j];
            if (fc < 2 && j > 0) f1 = A.fac.pe2[jb + j - 1];
        }
        __syncthreads();
        if (mine) {
            auto total = [&](int chunk, int v) {
                double t = 0.0;
#pragma unroll
                for (int u = 0; u < W; ++u) t += L.ring[par][chunk][u][v];
                return t;
            };
            double v = total(fk, fv);
            if (groups == 1) {
                if (fc < 2) {  // even degree: S_j and S_{j-1}
                    const double before = fv >= 4 ? total(fk, fv - 4) : fk > 0 ? total(fk - 1, fv + 12) : L.carry[par][fc];
                    if (fk == kFlush - 1 && fv >= kVals - 4) L.carry[par ^ 1][fc] = v;
                    v = fma(f0, v, f1 * before);
                } else {
                    v *= f0;
                }
                if (m == 0 && (fc & 1)) v = 0.0;
            }
            if (l <= lmax) reinterpret_cast<double *>(dst + l)[fc & 1] = v;
        }
    };

    // the next chunk's coefficients are loaded at the start of a chunk, so that
    // they arrive under its arithmetic; the waits for the LDS traffic that
    // follows then find them there
    AnaCoefPtr cp{ro(A.ra + jb + j0s), ro(A.rb + jb + j0s), ro(b0 + jb + j0s)};
    static_assert(2 * kChunk <= kCoefPad, "coefficient padding too short");
    AnaCoef cur, nxt;
    cp.load(cur);
    int par = 0, kc = 0, jbase = j0s;
    auto one = [&](int j0, auto full) {
        cp.load(nxt);
        double acc[kVals];
        S.template chunk<decltype(full)::value, PS>(j0, nj - j0, cur, acc);
        const double v = wave_sum16(L.tbuf[wave][0], acc);
        if ((lane & 3) == 0) L.ring[par][kc][wave][lane >> 2] = v;
        cur = nxt;
        if (++kc == kFlush || j0 + kChunk >= nj) {
            flush(jbase, par, kc);
            jbase += kFlush * kChunk;
            par ^= 1;
            kc = 0;
        }
    };
    int j0 = j0s;
#pragma unroll 1
    for (; j0 + kChunk <= nj; j0 += kChunk) one(j0, std::true_type{});
    if (j0 < nj) one(j0, std::false_type{});  // the ragged last chunk
}

// Analysis of one m of one map by one wave holding every slot (nslots <=
// 64 T; lane i owns slots 64 t + i): per chunk the wave's sums go straight
// to a_lm, with no step across waves, so the waves of a workgroup may each
// work on their own m.  tb: the wave's reduction rows, two sets in turn.
template <int T>
__device__ __forceinline__ void ana_wave(const AnaArgs &A, int m, int map, SumRows (&tb)[2]) {
    const int lmax = A.lmax, nj = jcol_len(lmax, m);
    const int lane = threadIdx.x & 63;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2, jb = jcol_base(lmax, m);
    const double2 *__restrict__ d = A.delta + (int64_t)map * A.nrings * (A.mmax + 1);
    double2 *__restrict__ dst = A.alm + (int64_t)map * A.nalm + base;
    const int warm = min(16 * lane, nj - 1);  // the column's coefficients into L2, as warm_l2
    const double warm_a = A.ra[jb + warm], warm_b = A.rb[jb + warm];
    AnaSlots<T> S;
    S.load(A, m, d, 0, 64);
    asm volatile("" ::"v"(warm_a), "v"(warm_b));
    const int lo = S.lo;
    for (int l = m + lane; l < m + 2 * min(lo, nj) && l <= lmax; l += 64) dst[l] = make_double2(0.0, 0.0);
    if (lo >= nj) return;
    const double *b0 = A.npolar ? A.rbp : A.rb;
    AnaCoefPtr cp{ro(A.ra + jb + lo), ro(A.rb + jb + lo), ro(b0 + jb + lo)};
    AnaCoef cur, nxt;
    cp.load(cur);
    const int fv = lane >> 2, fc = fv & 3;
    // before the first chunk S_{j-1} is zero: rows 12 .. 15 of the set that chunk reads
    if (lane < 16) {
#pragma unroll
        for (int v = kVals - 4; v < kVals; ++v) tb[1][v][lane] = 0.0;
    }
    int set = 0;
    // the factors of a chunk are loaded one chunk ahead
    auto factors = [&](int j0) {
        const int j = j0 + (fv >> 2);
        double2 f = make_double2(0.0, 0.0);
        if (j < nj) {
            f.x = fc < 2 ? A.fac.pe1[jb + j] : A.fac.po[jb + j];
            if (fc < 2 && j > 0) f.y = A.fac.pe2[jb + j - 1];
        }
        return f;
    };
    double2 fac = factors(lo);
    auto one = [&](int j0, auto full) {
        cp.load(nxt);
        double2 fac_next = factors(j0 + kChunk);
        double acc[kVals];
        S.template chunk<decltype(full)::value, kPolarSlots / 64>(j0, nj - j0, cur, acc);
        // S_j of this lane's column and S_{j-1}: rows v and v - 4, the latter for
        // the chunk's first step from the previous chunk's rows (both sums run
        // side by side; passing one on between lanes would lengthen the chain)
        sum_to_rows(tb[set], acc);
        const double v = sum_row(tb[set][fv]), before = sum_row(fv >= 4 ? tb[set][fv - 4] : tb[set ^ 1][fv + 12]);
        __builtin_amdgcn_wave_barrier();
        set ^= 1;
        cur = nxt;
        // the next factors are waited for here: behind the store the wait would
        // include the store's own way to memory, in every chunk
        asm volatile("" : "+v"(fac_next.x), "+v"(fac_next.y));
        const int l = m + 2 * (j0 + (fv >> 2)) + (fc >> 1);
        if ((lane & 3) == 0 && l <= lmax) {
            const double r = fc < 2 ? fma(fac.x, v, fac.y * before) : fac.x * v;
            reinterpret_cast<double *>(dst + l)[fc & 1] = (m == 0 && (fc & 1)) ? 0.0 : r;
        }
        fac = fac_next;
    };
    int j0 = lo;
#pragma unroll 1
    for (; j0 + kChunk <= nj; j0 += kChunk) one(j0, std::true_type{});
    if (j0 < nj) one(j0, std::false_type{});
}

// Analysis kernel: grid.x = (m, slot group) in the XCD-aware order, grid.y =
// map.  Three waves per SIMD at 8 slots per lane (168 VGPRs, 7 of them spilled
// outside the chunk loop) run faster than two without the spills: 589 against
// 637 us at HEALPix 1024 / lmax 2048.
template <int T, int W>
__global__ __launch_bounds__(64 * W, T <= 4 ? 4 : 3) void k_leg_ana(AnaArgs A, int groups) {
    __shared__ AnaLds<W> L;
    const MPart mp = xcd_m_part(groups);
    if (mp.m > A.mmax) return;  // padding of the m range (whole workgroup, before any barrier)
    ana_group<T, W>(A, mp.m, mp.part, (int)blockIdx.y, groups, L);
}
// At most 64 slots, one wave per m: grid.x = m in the XCD-aware order, grid.y = map.
__global__ __launch_bounds__(64) void k_leg_ana_wave(AnaArgs A) {
    __shared__ alignas(16) SumRows tb[2];
    const MPart mp = xcd_m_part(1);
    if (mp.m > A.mmax) return;
    ana_wave<1>(A, mp.m, (int)blockIdx.y, tb);
}

// FP64 analysis with several groups: the sums S_j, T_j of a column are
// part[map][g][idx] added over the groups in order (sum), then a_lm.
__device__ __forceinline__ double2 group_sum(const double2 *__restrict__ part, int64_t nalm, int groups, int64_t idx) {
    double sr = 0.0, si = 0.0;
    for (int g = 0; g < groups; ++g) {
        const double2 v = part[(int64_t)g * nalm + idx];
        sr += v.x;
        si += v.y;
    }
    return make_double2(sr, si);
}
// grid.x = m, grid.y = map
__global__ __launch_bounds__(kBlock) void k_ana_finish(int64_t nalm, int lmax, int groups,
                                                       const double2 *__restrict__ part, ParityFac f,
                                                       double2 *__restrict__ alm) {
    const int m = blockIdx.x;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2, map = blockIdx.y;
    const double2 *__restrict__ src = part + map * groups * nalm;
    finish_column(lmax, m, f, [&](int l) { return group_sum(src, nalm, groups, base + l); }, alm + map * nalm + base);
}

// Mixed analysis: a_lm = c_lm * sum_{g < groups} part[map][g][idx], groups summed in order.
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

// scaled a_lm of every synthesis request of a batch: grid.y = request (of
// the list), grid.x = m.
__global__ __launch_bounds__(kBlock) void k_prescale_batch(const BatchReq *__restrict__ reqs,
                                                            const int32_t *__restrict__ list) {
    const BatchReq &R = reqs[list[blockIdx.y]];
    const int m = blockIdx.x, lmax = R.syn.lmax;
    if (m > R.syn.mmax) return;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2;
    prescale_column(lmax, m, R.alm_in + base, R.ana.fac, const_cast<double2 *>(R.syn.ap) + base);
}

// a_lm from the group sums (groups in order) for every analysis request of
// the list that has several groups.
__global__ __launch_bounds__(kBlock) void k_combine_batch(const BatchReq *__restrict__ reqs,
                                                           const int32_t *__restrict__ list) {
    const BatchReq &R = reqs[list[blockIdx.y]];
    const int m = blockIdx.x, lmax = R.ana.lmax;
    if (m > R.ana.mmax) return;
    const int64_t nalm = R.ana.nalm, base = (int64_t)m * (2 * lmax + 1 - m) / 2;
    finish_column(lmax, m, R.ana.fac, [&](int l) { return group_sum(R.ana.part, nalm, R.groups, base + l); },
                  R.ana.alm + base);
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

int launch_prescale_batch(const BatchReq *reqs, const int32_t *syn_reqs, int nsyn, int max_m, hipStream_t st) {
    if (nsyn <= 0) return SHT_OK;
    if (nsyn > 65535) return SHT_EUNSUPPORTED;
    hipLaunchKernelGGL(k_prescale_batch, dim3((unsigned)max_m, (unsigned)nsyn), dim3(kBlock), 0, st, reqs, syn_reqs);
    SHT_HIP(hipGetLastError());
    return SHT_OK;
}

int launch_combine_batch(const BatchReq *reqs, const int32_t *comb_reqs, int ncomb, int max_m, hipStream_t st) {
    if (ncomb <= 0) return SHT_OK;
    if (ncomb > 65535) return SHT_EUNSUPPORTED;
    hipLaunchKernelGGL(k_combine_batch, dim3((unsigned)max_m, (unsigned)ncomb), dim3(kBlock), 0, st, reqs, comb_reqs);
    SHT_HIP(hipGetLastError());
    return SHT_OK;
}

int launch_leg_start(const CoefTables &c, const GeomPlan &p, int32_t *jstart, void *state, hipStream_t st) {
    const int tiles = (p.nslots + kBlock - 1) / kBlock;
    if (c.mmax + 1 > 65535) return SHT_EUNSUPPORTED;
    hipLaunchKernelGGL(k_leg_start, dim3((unsigned)tiles, (unsigned)(c.mmax + 1)), dim3(kBlock), 0, st, c.lmax,
                       p.nslots, p.npolar, c.ra, c.rb, c.rbp, c.seed, p.slot_w, p.slot_s, jstart, static_cast<double2 *>(state));
    SHT_HIP(hipGetLastError());
    return SHT_OK;
}

int launch_prescale(const CoefTables &c, const void *alm, void *aprime, int nmaps, hipStream_t st) {
    if (nmaps > 65535) return SHT_EUNSUPPORTED;
    hipLaunchKernelGGL(k_prescale, dim3((unsigned)(c.mmax + 1), (unsigned)nmaps), dim3(kBlock), 0, st, c.nalm, c.lmax,
                       static_cast<const double2 *>(alm), parity_fac(c), static_cast<double2 *>(aprime));
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
    // (Powers of two only: a wave's slots must not straddle GeomPlan::npolar.)
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
    } else if (p.nslots > 512 && p.nslots <= 640) {
        // Two waves of 5 slots per lane add half the wave sums of four waves of
        // 3: 64 maps on 513 slots, lmax 1024, 3.51 against 4.69 ms for the
        // stage, one map 115 against 107 us.  Up to 512 slots one map leaves
        // the chip with too few waves for that, and from 641 on (6 per lane) it
        // costs one map more than it gives several (694 slots, lmax 694: one
        // map 82 and 68 us, eight 289 and 338).
        static_assert(5 * 2 * 64 == 640, "one group");
        launch_ana_t<5, 2>(A, groups, nmaps, st);
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
    if (groups > 1) {
        hipLaunchKernelGGL(k_ana_finish, dim3((unsigned)(c.mmax + 1), (unsigned)nmaps), dim3(kBlock), 0, st, c.nalm,
                           c.lmax, groups, static_cast<const double2 *>(partials), parity_fac(c),
                           static_cast<double2 *>(alm));
        SHT_HIP(hipGetLastError());
    }
    return SHT_OK;
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

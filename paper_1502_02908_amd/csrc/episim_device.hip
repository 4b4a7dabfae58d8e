// gfx950 kernels of the per-day step (Bauer, Engblom & Widgren,
// arXiv:1502.02908, Sec. 3.1-3.3 and Algorithm 1):
//   k_day      one replicate: closes the previous day of every node (the level
//              events of its day where few nodes take part, the continuous-state
//              update eq:numstep5 with eq:siminfpressure, the day's record), then
//              the direct-method SSA over the window [d, d+1) with phi frozen
//              (eq:numstep3, eq:sampling, eq:sampling2) and the events of single
//              nodes that come first in the day;
//   k_day_tile, k_day_far
//              the same for many replicates, 64 a column, and for slots of
//              requests; the longest chains in a launch of their own;
//   k_events, k_event_levels, k_slot_events
//              conflict-free levels of day d's external events (eq:numstep4,
//              Sec. 3.2): a thread per (event, replicate);
//   k_persist  the same phases for a run of days in one cooperative launch,
//              with grid barriers between phases.
// All binary64 arithmetic is written in a fixed order with contraction off,
// so results are a fixed function of the inputs.
#include <hip/hip_runtime.h>
#include <hip/hip_cooperative_groups.h>

#include <algorithm>
#include <cstdio>
#include <mutex>

#include "../../include/episim.h"
#include "episim_internal.h"

#pragma clang fp contract(off)

// Intermediate buffers of the entry points that allocate nothing (the goal
// function's staged reference and day terms): a fixed array in every GPU's
// memory, kept until the process ends. Calls on one GPU share it.
static __device__ __align__(256) unsigned char scratch[episim::kScratchBytes];

namespace episim {
namespace {

constexpr int kBlock = 256;
static_assert(kBlock == kPersistUnit, "a workgroup of the persistent kernel's one-lane-per-node layout is one unit");
constexpr int kDayWaves = 16;  // wavefronts of a workgroup of the one-lane-per-node day kernel, at most
static_assert(kDayWaves == 16 && kMaxUnit <= 64 * kDayWaves, "the workgroup walk exchanges one value per lane of a row");
constexpr int kMaxScratchDevices = 64;
constexpr int kWaves = kBlock / 64;
constexpr int kEvKindMask = 3;
constexpr int kEvBlock = 1024;  // workgroup that runs a group of small event levels

// ---------------------------------------------------------------------------
// Counter-based random numbers: Philox4x32-10 (Salmon et al., SC'11).
// ---------------------------------------------------------------------------
struct Word4 {
    uint32_t a, b, c, d;
};

__device__ __forceinline__ Word4 philox4x32_10(Word4 x, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int i = 0; i < 10; ++i) {
        const uint64_t pa = (uint64_t)0xD2511F53u * (uint64_t)x.a;  // one 32x32->64 multiply each
        const uint64_t pc = (uint64_t)0xCD9E8D57u * (uint64_t)x.c;
        x = Word4{(uint32_t)(pc >> 32) ^ x.b ^ k0, (uint32_t)pc, (uint32_t)(pa >> 32) ^ x.d ^ k1, (uint32_t)pa};
        k0 += 0x9E3779B9u;  // Weyl increments of the key between rounds
        k1 += 0xBB67AE85u;
    }
    return x;
}

// rand in (0,1) of eq:sampling: the odd multiple of 2^-53 whose upper 52 bits
// are the top 52 bits of hi:lo.
__device__ __forceinline__ double unit_open(uint32_t lo, uint32_t hi) {
    const uint64_t x = ((uint64_t)hi << 32) | (uint64_t)lo;
    return (double)((x >> 11) | 1ull) * 0x1p-53;
}

// -log(u), u in (0,1): fold u = m 2^e with m in (sqrt2/2, sqrt2], then
// log m = 2 atanh(s), s = (m-1)/(m+1), with the series to s^23 and ln 2 split
// into a 32-bit head and a tail.
__device__ __forceinline__ double minus_log(double u) {
    const double kSqrt2 = 0x1.6a09e667f3bcdp+0;
    const double kLn2Head = 0x1.62e42ff000000p-1;
    const double kLn2Tail = -0x1.718432a1b0e26p-35;
    const long long bits = __double_as_longlong(u);
    int ex = (int)((bits >> 52) & 0x7ff) - 1023;
    double m = __longlong_as_double((bits & 0x000fffffffffffffLL) | 0x3ff0000000000000LL);
    if (m > kSqrt2) {
        m = m * 0.5;
        ex = ex + 1;
    }
    const double f = m - 1.0;
    const double s = f / (2.0 + f);
    const double z = s * s;
    double q = 1.0 / 23.0;
    q = 1.0 / 21.0 + z * q;
    q = 1.0 / 19.0 + z * q;
    q = 1.0 / 17.0 + z * q;
    q = 1.0 / 15.0 + z * q;
    q = 1.0 / 13.0 + z * q;
    q = 1.0 / 11.0 + z * q;
    q = 1.0 / 9.0 + z * q;
    q = 1.0 / 7.0 + z * q;
    q = 1.0 / 5.0 + z * q;
    q = 1.0 / 3.0 + z * q;
    const double zq = z * q;
    const double t = s + s * zq;
    const double lm = t + t;
    const double e = (double)ex;
    return -(e * kLn2Head + (lm + e * kLn2Tail));
}

// Season of beta(t) (Sec. 4.1).
__device__ __forceinline__ int season(int64_t t) {
    int64_t y = t % 365;
    if (y < 0) y += 365;
    return y <= 91 ? 0 : (y <= 182 ? 1 : (y <= 273 ? 2 : 3));
}

// Loads of the state in the event phase are plain loads, so that the
// compartments of one node are fetched together. They see the last writes
// because a launch starts with clean caches, and because every kernel that
// runs several levels, or events after the SSA, follows its barrier with
// fresh_l1(): additions are device-scope atomics done in L2, which the CU's
// L1 does not see, so the acquire drops the L1 lines before the next level.
__device__ __forceinline__ int32_t load_state(const int32_t *p) { return *p; }

__device__ __forceinline__ void fresh_l1() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent"); }

// The paired-class kernels (2 or 6 compartments and transitions) are built for
// exactly their model; the generic ones for every model up to their size.
constexpr bool exact_size(int n) { return n == 2 || n == 6; }
template <int NC>
__device__ __forceinline__ bool comp_on(const Model &m, int c) {
    return exact_size(NC) || c < m.nc;
}
template <int NT>
__device__ __forceinline__ bool trans_on(const Model &m, int k) {
    return exact_size(NT) || k < m.nt;
}

// ---------------------------------------------------------------------------
// The stochastic step (Sec. 3.3, Algorithm 1's inner loop; eq:sampling and
// eq:sampling2). A lane's chain keeps its counts as exact binary64 values
// (counts stay far below 2^53), so omega_k = cphi_k * X[reactant_k] is the
// same product (c * phi) * (double)X in the same order as the plain method;
// cphi_k is the rate constant times phi for the transitions that use phi.
// lambda and the running sums cum_k are summed in transition order.
// ---------------------------------------------------------------------------
template <int NC_, int NT_>
struct Chain {
    static constexpr int NC = NC_, NT = NT_;
    double xd[NC_];
    double cphi[NT_];
    double cum[NT_];
    double lam, clock;
    int32_t fired;
};

// Any stoichiometry (column k: -1 at reactant k, non-negative elsewhere).
// Besides the counts a chain keeps the reactant counts of every transition,
// xr[k] = X[reactant[k]] (and xr2[k] of the second reactant of a mass-action
// rate), which the walks by many lanes update from the picks directly
// (ModelTables::react). Transitions past the model's have rate constant 0.
template <int NC_, int NT_>
struct GenericChain : Chain<NC_, NT_> {
    double xr[NT_], xr2[NT_];
};

// The model's tables, read with scalar loads where they are used: kept in
// registers over a kernel, their values (and the masks of their comparisons)
// would be spilled and read back lane by lane. (Eight compartments, 512 threads
// a workgroup: 1,425 scalar and 119 vector registers spilled, now 567 and none; a
// day of 20,000 herds 98 us, now 70, with short chains 56 and 39. Three
// compartments 52 us, now 45.)
using ScalarTables = const __attribute__((address_space(4))) ModelTables;
__device__ __forceinline__ ScalarTables &model_tables(const Model &m) {
    uint64_t p = (uint64_t)m.tables;
    asm volatile("" : "+s"(p));
    return *(ScalarTables *)p;
}

template <int NC_, int NT_>
struct GenericRules {
    static constexpr int NC = NC_, NT = NT_;
    static constexpr int kDayThreads = day_threads(NC, NT, false);
    static constexpr int kTileWaves = 2;  // waves per SIMD the replicate-tile kernel is built for
    using State = GenericChain<NC, NT>;
    __device__ static __forceinline__ double rate(ScalarTables &tb, const State &c, int k) {
        const double w = c.cphi[k] * c.xr[k];
        // a mass-action rate is also proportional to its second reactant
        return tb.reactant2[k] >= 0 ? w * c.xr2[k] : w;
    }
    __device__ static __forceinline__ double rate(const Model &m, const State &c, int k) { return rate(model_tables(m), c, k); }
    __device__ static __forceinline__ void reactants(const Model &m, State &c) {
        ScalarTables &tb = model_tables(m);
#pragma unroll
        for (int k = 0; k < NT; ++k) {
            double a = 0.0, b = 0.0;
#pragma unroll
            for (int cc = 0; cc < NC; ++cc) {
                if (tb.reactant[k] == cc) a = c.xd[cc];
                if (tb.reactant2[k] == cc) b = c.xd[cc];
            }
            c.xr[k] = a;
            c.xr2[k] = b;
        }
    }
    __device__ static __forceinline__ void rates(const Model &m, State &c) {
        reactants(m, c);
        ScalarTables &tb = model_tables(m);
        double lam = 0.0;
#pragma unroll
        for (int k = 0; k < NT; ++k) {
            lam = lam + rate(tb, c, k);
            c.cum[k] = lam;
        }
        c.lam = lam;
    }
    __device__ static __forceinline__ void apply(const Model &m, int j, State &c) {
        ScalarTables &tb = model_tables(m);
#pragma unroll
        for (int k = 0; k < NT; ++k) {
            if (k == j) {
#pragma unroll
                for (int cc = 0; cc < NC; ++cc) c.xd[cc] = c.xd[cc] + tb.S[cc][k];
            }
        }
    }
    // The walks by many lanes describe a run of picks by how often it holds
    // each transition.
    static constexpr int kFlows = NT;
    __device__ static __forceinline__ void flows(int j, unsigned long long lanes, int (&n)[kFlows]) {
#pragma unroll
        for (int k = 0; k < NT; ++k) n[k] = __popcll(__ballot(j == k) & lanes);
    }
    // running sums of the rates in the state of c after the flows n (every
    // product and sum of counts is an exact integer)
    __device__ static __forceinline__ void cum_after(const Model &m, const State &c, const int (&n)[kFlows],
                                                     double (&cum)[NT]) {
        ScalarTables &tb = model_tables(m);
        double l = 0.0;
#pragma unroll
        for (int k = 0; k < NT; ++k) {
            double a = c.xr[k];
#pragma unroll
            for (int i = 0; i < NT; ++i) a = __builtin_fma(tb.react[k][i], (double)n[i], a);
            double w = c.cphi[k] * a;
            if (tb.reactant2[k] >= 0) {
                double b = c.xr2[k];
#pragma unroll
                for (int i = 0; i < NT; ++i) b = __builtin_fma(tb.react2[k][i], (double)n[i], b);
                w = w * b;
            }
            l = l + w;
            cum[k] = l;
        }
    }
    __device__ static __forceinline__ void advance(const Model &m, State &c, const int (&n)[kFlows]) {
        ScalarTables &tb = model_tables(m);
#pragma unroll
        for (int cc = 0; cc < NC; ++cc) {
#pragma unroll
            for (int k = 0; k < NT; ++k) c.xd[cc] = __builtin_fma(tb.S[cc][k], (double)n[k], c.xd[cc]);
        }
        reactants(m, c);
    }
};

// Paired classes: compartments [S_1, I_1, ..., S_P, I_P] and transitions
// 2p: S_p -> I_p, 2p+1: I_p -> S_p, each with its own compartment as reactant
// (eq:vectorJSDE for eq:vtectrans; P = 1 is the plain SIS model). The host
// selects these rules only when S and the reactants have exactly this form.
template <int NP>
struct PairRules {
    static constexpr int NC = 2 * NP, NT = 2 * NP;
    static constexpr int kDayThreads = day_threads(NC, NT, true);
    // replicate tiles of paired classes are built for three waves per SIMD
    // (at most 168 VGPRs, with a 16-byte spill): the third wave hides the
    // latency of the chains' dependent binary64 arithmetic and of the state
    // loads (12 % faster on the batched workload than the two waves 185
    // VGPRs allow; bit-identical)
    static constexpr int kTileWaves = 3;
    using State = Chain<NC, NT>;
    __device__ static __forceinline__ double rate(const Model &, const State &c, int k) {
        return c.cphi[k] * c.xd[k];
    }
    __device__ static __forceinline__ void reactants(const Model &, State &) {}  // the counts themselves
    __device__ static __forceinline__ void rates(const Model &m, State &c) {
        double lam = 0.0;
#pragma unroll
        for (int k = 0; k < NT; ++k) {
            lam = lam + rate(m, c, k);
            c.cum[k] = lam;
        }
        c.lam = lam;
    }
    __device__ static __forceinline__ void apply(const Model &, int j, State &c) {
        const int p = j >> 1;
        const double dS = (j & 1) ? 1.0 : -1.0;  // infection takes an S, recovery returns one
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const double dq = q == p ? dS : 0.0;
            c.xd[2 * q] = c.xd[2 * q] + dq;
            c.xd[2 * q + 1] = c.xd[2 * q + 1] - dq;
        }
    }
    // The walks by many lanes describe a run of picks by the net number of
    // individuals it returns to S in each class.
    static constexpr int kFlows = NP;
    __device__ static __forceinline__ void flows(int j, unsigned long long lanes, int (&n)[kFlows]) {
#pragma unroll
        for (int q = 0; q < NP; ++q)
            n[q] = __popcll(__ballot(j == 2 * q + 1) & lanes) - __popcll(__ballot(j == 2 * q) & lanes);
    }
    // running sums of the rates in the state of c after the flows n
    __device__ static __forceinline__ void cum_after(const Model &, const State &c, const int (&n)[kFlows],
                                                     double (&cum)[NT]) {
        double l = 0.0;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const double dS = (double)n[q];
            l = l + c.cphi[2 * q] * (c.xd[2 * q] + dS);
            cum[2 * q] = l;
            l = l + c.cphi[2 * q + 1] * (c.xd[2 * q + 1] - dS);
            cum[2 * q + 1] = l;
        }
    }
    __device__ static __forceinline__ void advance(const Model &, State &c, const int (&n)[kFlows]) {
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const double dS = (double)n[q];
            c.xd[2 * q] = c.xd[2 * q] + dS;
            c.xd[2 * q + 1] = c.xd[2 * q + 1] - dS;
        }
    }
};

// Inversion of eq:sampling2: the first transition with a positive rate whose
// running sum reaches target. With target > 0 that is the number of running
// sums below target (they never decrease, and a transition with rate 0 cannot
// be the first to reach a positive target); target can be 0 only if U*lambda
// underflows, and then it is the first positive rate.
template <class Rules>
__device__ __forceinline__ int invert(const Model &m, const typename Rules::State &c, double target) {
    constexpr int NT = Rules::NT;
    int j = 0;
#pragma unroll
    for (int k = 0; k < NT; ++k) j += c.cum[k] < target ? 1 : 0;
    if (__builtin_expect(!(target > 0.0), 0)) {
        j = NT;
#pragma unroll
        for (int k = NT - 1; k >= 0; --k)
            if (trans_on<NT>(m, k) && Rules::rate(m, c, k) > 0.0) j = k;
    }
    return j;
}

// One attempt of the direct method with the draw (E, U) = (-log rand_1,
// rand_2): tau = E / lambda; the transition fires only if it lands inside the
// window. Returns whether the chain goes on.
template <class Rules>
__device__ __forceinline__ bool chain_step(const Model &m, typename Rules::State &c, double E, double U,
                                           unsigned long long *status, int32_t r) {
    const double tau = E / c.lam;
    const double t1 = c.clock + tau;
    const int j = invert<Rules>(m, c, U * c.lam);
    if (!(t1 < 1.0)) return false;
    c.clock = t1;
    Rules::apply(m, j, c);
    c.fired = c.fired + 1;
    Rules::rates(m, c);
    if (c.fired >= SIM_MAX_FIRED) {  // bounded work per lane: report instead of running on
        atomicMin(status, (STATUS_LIMIT_TAG << 32) | (unsigned long long)(uint32_t)r);
        return false;
    }
    return c.lam > 0.0;
}

__device__ __forceinline__ double lane_f64(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Inclusive prefix sum over the 64 lanes of a wavefront: shifts by 1, 2, 4, 8
// within rows of 16 lanes, then lane 15's sum into rows 1 and 3 and lane 31's
// into rows 2 and 3 (lanes without a source add +0).
template <int Ctrl, int RowMask>
__device__ __forceinline__ double dpp_f64(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, Ctrl, RowMask, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), Ctrl, RowMask, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

__device__ __forceinline__ double wave_prefix_sum(double v) {
    v = v + dpp_f64<0x111, 0xf>(v);  // row_shr:1
    v = v + dpp_f64<0x112, 0xf>(v);  // row_shr:2
    v = v + dpp_f64<0x114, 0xf>(v);  // row_shr:4
    v = v + dpp_f64<0x118, 0xf>(v);  // row_shr:8
    v = v + dpp_f64<0x142, 0xa>(v);  // row_bcast:15
    v = v + dpp_f64<0x143, 0xc>(v);  // row_bcast:31
    return v;
}

// The clock of a round without the attempt-by-attempt sum. While the running
// clock stays in one binade [2^e, 2^(e+1)) every partial sum is an integer
// multiple of its spacing h = 2^(e-52), and adding a waiting time rounds to
// the nearest multiple: s + tau -> (s/h + rn(tau/h)) h. Those integers add
// exactly (each partial sum that matters stays below 2^53), so one prefix sum
// over the lanes gives every partial sum of the round bit for bit. A sum that
// reaches 2^(e+1) leaves the binade: for e = -1 that is the window end (the
// attempt does not fire, whatever the rounding above 1); otherwise the round
// has to be summed attempt by attempt, and so has a round in which a waiting
// time lies exactly half-way between two multiples (ties round to even, which
// depends on the partial sum) or whose clock is 0. Returns the number of
// attempts that fire (-1: sum attempt by attempt) and their clock. (Going on
// with another scan behind such an attempt is slower than the 64 additions:
// each scan's result passes through scalar registers before the next.)
__device__ __forceinline__ int clock_by_scan(double clock, double tau, double *clock_out) {
    const long long cb = __double_as_longlong(clock);
    const int e = (int)((cb >> 52) & 0x7ff) - 1023;
    if (!(clock > 0.0) || e < -960 || e > -1) return -1;
    const double up = __longlong_as_double((long long)(1023 + 52 - e) << 52);    // 2^(52-e)
    const double down = __longlong_as_double((long long)(1023 - 52 + e) << 52);  // 2^(e-52)
    const double S0 = clock * up;                                                // in [2^52, 2^53)
    const double T = 0x1p53 - S0;
    const double v = tau * up;
    const double fl = floor(v);
    const double fr = v - fl;
    const double P = wave_prefix_sum(fr > 0.5 ? fl + 1.0 : fl);
    const int A = (int)__popcll(__ballot(P < T));
    const unsigned long long upto = A >= 63 ? ~0ull : ((2ull << A) - 1ull);
    if ((__ballot(fr == 0.5) & upto) != 0ull) return -1;
    if (A < 64 && e != -1) return -1;
    *clock_out = A > 0 ? (S0 + lane_f64(P, A - 1)) * down : clock;
    return A;
}

// The clock of a wavefront's 64 attempts, attempt by attempt where the scan
// does not apply: the waiting times go through LDS (64 values of this
// wavefront) and come back as broadcast reads, which issue ahead of the
// dependent additions.
__device__ __forceinline__ int wave_clock(double s, double tau, double *sh_tau, double *clock_out) {
    const int lane = threadIdx.x & 63;
    int A = clock_by_scan(s, tau, clock_out);
    if (A >= 0) return A;
    sh_tau[lane] = tau;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    double t = s;
#pragma unroll 16
    for (int i = 0; i < 64; ++i) t = t + sh_tau[i];
    A = 64;
    if (!(t < 1.0)) {
        double q = s, mine = 0.0;
#pragma unroll 16
        for (int i = 0; i < 64; ++i) {
            q = q + sh_tau[i];
            if (lane == i) mine = q;
        }
        A = __popcll(__ballot(mine < 1.0));
        t = A > 0 ? lane_f64(mine, A - 1) : s;
    }
    __builtin_amdgcn_wave_barrier();  // the next round rewrites sh_tau
    *clock_out = t;
    return A;
}

// Prefix sums over segments of G lanes (in any order of addition).
template <int G>
__device__ __forceinline__ double segment_prefix_sum(double v, int li) {
    if constexpr (G == 64) {
        return wave_prefix_sum(v);
    } else {
        static_assert(G == 8 || G == 16, "segments lie within rows of 16 lanes");
        double u = dpp_f64<0x111, 0xf>(v);  // row_shr:1
        v = v + (G == 16 || li >= 1 ? u : 0.0);
        u = dpp_f64<0x112, 0xf>(v);  // row_shr:2
        v = v + (G == 16 || li >= 2 ? u : 0.0);
        u = dpp_f64<0x114, 0xf>(v);  // row_shr:4
        v = v + (G == 16 || li >= 4 ? u : 0.0);
        if constexpr (G == 16) v = v + dpp_f64<0x118, 0xf>(v);  // row_shr:8
        return v;
    }
}

// The walks by several lanes. Attempt kbase + i of a chain belongs to lane i of
// the chain's segment of G lanes (64: the whole wavefront; 16 or 8: as many
// chains side by side as segments), G attempts a round. An attempt's draws do
// not depend on the state, but the transition it picks (eq:sampling2) and its
// waiting time (eq:sampling) depend on the state the attempts before it leave.
// Each lane first assumes the round's starting state, then recomputes its
// state from the transitions the lanes below it picked (Rules::flows: a ballot
// per transition and a count of the set bits below the lane) and its own pick
// from that state, until no pick changes. Lane i is settled after i + 1 passes
// whatever the guesses were, so the result is the one attempt-by-attempt walk
// gives; with many individuals the rates barely move and one or two passes
// settle every lane (and only the lanes up to the first attempt surely past
// the window end need to). The waiting times then follow in parallel. The
// clock's partial sums, which binary64 addition rounds one by one, come from
// exact integer prefix sums or attempt by attempt from LDS. The attempts whose sum stays below the window end fire;
// they form a prefix of the lanes because the clock never decreases. Every lane
// of a segment holds the same chain state.
// Counts are exact integers in binary64 and the rates, running sums, targets
// and waiting times are the same functions of the same state as in a walk
// attempt by attempt, so the bits agree.
struct Draw {
    double E, U;  // -log rand_1, rand_2
};

__device__ __forceinline__ Draw draw_attempt(uint32_t k, uint32_t node, uint32_t day, uint32_t key0, uint32_t key1) {
    const Word4 o = philox4x32_10(Word4{k, node, day, 0u}, key0, key1);
    return Draw{minus_log(unit_open(o.a, o.b)), unit_open(o.c, o.d)};
}

// The pick of an attempt in the state of c after the flows n, and its lambda.
template <class Rules>
__device__ __forceinline__ int pick_after(const Model &m, const typename Rules::State &c, const int (&n)[Rules::kFlows],
                                          double U, double *lam) {
    double cum[Rules::NT];
    Rules::cum_after(m, c, n, cum);
    // target > 0 whenever the attempt can fire: target = 0 needs
    // lambda < 2^-1021, and then tau = E/lambda > 1 since E >= 2^-53
    const double target = U * cum[Rules::NT - 1];
    int j = 0;
#pragma unroll
    for (int k = 0; k < Rules::NT; ++k) j += cum[k] < target ? 1 : 0;
    *lam = cum[Rules::NT - 1];
    return j;
}

// Passes over the picks j until those that can fire no longer change; returns
// the last attempt of the segment with a settled pick.
template <class Rules, int G>
__device__ __forceinline__ int settle_picks(const Model &m, const typename Rules::State &c, Draw q, int first_pass,
                                            int &j, double &lam) {
    constexpr int K = Rules::kFlows;
    const int lane = threadIdx.x & 63, li = lane & (G - 1), seg0 = lane - li;
    const unsigned long long seg = G == 64 ? ~0ull : (((1ull << (G & 63)) - 1ull) << seg0);
    const unsigned long long below = seg & ((1ull << lane) - 1ull);
    for (int pass = first_pass; pass < 64; ++pass) {
        int n[K];
        Rules::flows(j, below, n);
        const int jn = pick_after<Rules>(m, c, n, q.U, &lam);
        const unsigned long long moved = __ballot(jn != j);
        j = jn;
        if (moved == 0ull) break;
        if (pass == 0) continue;  // large herds settle in one or two passes without it
        // An attempt whose clock surely lands past the window end stops the
        // chain, so only the picks up to it have to settle. If none of them
        // moved in this pass, they and their waiting times are those of the
        // attempt-by-attempt walk (each was computed from the unchanged picks
        // below it); the clock bound then comes from exact waiting times, and
        // its margin is far above the rounding of the approximate prefix sum.
        const double reach = c.clock + segment_prefix_sum<G>(lam > 0.0 ? q.E / lam : __builtin_inf(), li);
        const unsigned long long over = __ballot(!(reach < 1.0 + 0x1p-30)) & seg;
        const int a = over != 0ull ? __ffsll((long long)over) - 1 : seg0 + G - 1;
        const unsigned long long upto = a >= 63 ? ~0ull : ((2ull << a) - 1ull);
        if (__ballot((moved & seg & upto) != 0ull) == 0ull) return a - seg0;
    }
    return G - 1;
}

// The first A attempts of each segment fire, with picks j; their clock.
// Returns whether the chain has reached SIM_MAX_FIRED (A is cut there).
template <class Rules, int G>
__device__ __forceinline__ bool fire_attempts(const Model &m, typename Rules::State &c, int j, int &A, double clock,
                                              unsigned long long *status, int32_t r) {
    const int lane = threadIdx.x & 63, li = lane & (G - 1), seg0 = lane - li;
    bool limit = false;
    if (c.fired + A >= SIM_MAX_FIRED) {
        A = SIM_MAX_FIRED - c.fired;
        limit = true;
    }
    int n[Rules::kFlows];
    Rules::flows(j, (A >= 64 ? ~0ull : ((1ull << A) - 1ull)) << seg0, n);
    Rules::advance(m, c, n);
    if (A > 0 && !limit) c.clock = clock;
    c.fired = c.fired + A;
    if (limit && li == 0) atomicMin(status, (STATUS_LIMIT_TAG << 32) | (unsigned long long)(uint32_t)r);
    return limit;
}

// One round of the chains of a wavefront's segments. Returns whether the
// segment's chain has ended (a chain whose rates are all 0 ends in its next
// round); a segment without a chain passes rate constants of 0. sh_tau: 64
// values of this wavefront.
template <class Rules, int G>
__device__ __forceinline__ bool walk_round(const Model &m, typename Rules::State &c, uint32_t kbase, uint32_t node,
                                           uint32_t day, uint32_t key0, uint32_t key1, unsigned long long *status,
                                           int32_t r, double *sh_tau) {
    const int lane = threadIdx.x & 63, li = lane & (G - 1), seg0 = lane - li;
    const Draw q = draw_attempt(kbase + (uint32_t)li, node, day, key0, key1);
    int n[Rules::kFlows];
#pragma unroll
    for (int k = 0; k < Rules::kFlows; ++k) n[k] = 0;
    double lam;
    int j = pick_after<Rules>(m, c, n, q.U, &lam);  // guess: every attempt sees the round's starting state
    const int settled = settle_picks<Rules, G>(m, c, q, 0, j, lam);
    // lambda = 0: tau = inf, never fires; attempts past the settled ones do
    // not fire and may hold unsettled picks
    const double tau = li > settled ? __builtin_inf() : q.E / lam;
    // the clock, attempt by attempt. The waiting times go through LDS and come
    // back as broadcast reads, which issue ahead of the dependent additions.
    sh_tau[lane] = tau;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    double clock = c.clock, t = c.clock;
    int A = 0;
    for (int i0 = 0; i0 < G; i0 += 8) {
#pragma unroll
        for (int i = i0; i < i0 + 8; ++i) {
            t = t + sh_tau[seg0 + i];
            const bool in = t < 1.0;
            clock = in ? t : clock;
            A += in ? 1 : 0;
        }
        if (__ballot(t < 1.0) == 0ull) break;  // every segment's clock is past the window end
    }
    __builtin_amdgcn_wave_barrier();  // the next round rewrites sh_tau
    return fire_attempts<Rules, G>(m, c, j, A, clock, status, r) || A < G;
}

// One chain walked to the end of the window by the whole wavefront, every lane
// holding the same state, from attempt kbase on. sh_tau: 64 values of this
// wavefront.
template <class Rules>
__device__ __forceinline__ void walk_wave(const Model &m, typename Rules::State &c, uint32_t kbase, uint32_t node,
                                          uint32_t day, uint32_t key0, uint32_t key1, unsigned long long *status,
                                          int32_t r, double *sh_tau) {
    const int lane = threadIdx.x & 63;
    for (;; kbase = kbase + 64) {
        const Draw q = draw_attempt(kbase + (uint32_t)lane, node, day, key0, key1);
        int n[Rules::kFlows];
#pragma unroll
        for (int k = 0; k < Rules::kFlows; ++k) n[k] = 0;
        double lam;
        int j = pick_after<Rules>(m, c, n, q.U, &lam);  // guess: the round's starting state
        const int settled = settle_picks<Rules, 64>(m, c, q, 0, j, lam);
        const double tau = lane > settled ? __builtin_inf() : q.E / lam;
        double clock;
        int A = wave_clock(c.clock, tau, sh_tau, &clock);
        if (fire_attempts<Rules, 64>(m, c, j, A, clock, status, r) || A < 64) return;
    }
}

// Inclusive prefix sums within rows of 16 lanes.
__device__ __forceinline__ int32_t row_prefix_sum(int32_t v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    return v;
}
__device__ __forceinline__ double row_prefix_sum(double v) {
    v = v + dpp_f64<0x111, 0xf>(v);
    v = v + dpp_f64<0x112, 0xf>(v);
    v = v + dpp_f64<0x114, 0xf>(v);
    v = v + dpp_f64<0x118, 0xf>(v);
    return v;
}

// One chain walked by the wavefronts of a workgroup (sixteen at most), an
// attempt a thread per round (attempt kbase + t for thread t): the scheme of walk_round, with
// the picks of each wavefront shared in LDS as its flows (Rules::flows), so
// that an attempt's state is the round's state after the flows of the
// wavefronts below and of the lanes below in its own. One barrier per pass: a
// wavefront publishes its flows (two to a word) together with whether its picks
// moved in the pass before; lane w of every row then reads wavefront w's words
// and the sums over the wavefronts are row prefix sums; a pass that finds no
// wavefront moved ends the round.
// The clock follows the rule of clock_by_scan, in every wavefront at once:
// prefix sums within the wavefronts and over their totals give every partial
// sum of the binade; an attempt whose sum leaves the binade, or that lies
// half-way between two multiples, is added as the serial walk adds it, and the
// scan goes on behind it in the binade of the new sum. A chain's first 64
// attempts, most of whose sums are the first in their binade, are added one by
// one by the first wavefront.
// With one wavefront a SIMD a round takes about 6,000 cycles, nearly all of it
// the latency of dependent binary64 arithmetic and of LDS; four wavefronts a
// SIMD take little longer for four times the attempts, until the SIMDs' issue
// binds.
// Every thread of the workgroup calls it with the same state and ends with the
// same state. A round starts only while the window still expects
// kGroupRest attempts (lambda (1 - clock)), and a round whose picks do not
// settle within kGroupPasses passes is dropped. Returns whether the chain is
// done; if not, the caller continues with one wavefront from attempt kbase
// and state c, which are those at the start of a round.
constexpr int kGroupPasses = 8;
constexpr double kGroupRest = 24.0;

template <class Rules>
__device__ __forceinline__ bool walk_group(const Model &m, typename Rules::State &c, uint32_t &kbase, uint32_t node, uint32_t day,
                           uint32_t key0, uint32_t key1, unsigned long long *status, int32_t r) {
    constexpr int NT = Rules::NT, K = Rules::kFlows;
    constexpr int kWords = (K + 2) / 2;  // flows and the moved mark, two to a word
    const int round = (int)blockDim.x;
    __shared__ int32_t sh_flow[2][kWords][kDayWaves];
    __shared__ double sh_head[64], sh_total[kDayWaves], sh_before, sh_at;
    __shared__ int32_t sh_tie[kDayWaves], sh_special;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const unsigned long long below = (1ull << lane) - 1ull;
    int buf = 0;
    if (round < 64 * kDayWaves) {  // the wavefronts that are not there add nothing
        if (t < kDayWaves) {
#pragma unroll
            for (int k = 0; k < kWords; ++k) sh_flow[0][k][t] = sh_flow[1][k][t] = 0;
            sh_total[t] = 0.0;
            sh_tie[t] = 0;
        }
        __syncthreads();
    }
    // publish this wavefront's flows n (and mark); after the barrier, before[]
    // and all[] are the flows of the wavefronts below and of all; returns
    // whether any wavefront set its mark
    auto exchange = [&](const int (&n)[K], bool mark, int (&before)[K], int (&all)[K]) {
        int f[2 * kWords];
#pragma unroll
        for (int k = 0; k < 2 * kWords; ++k) f[k] = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) f[k] = n[k];
        f[K] = mark ? 1 : 0;
        if (lane == 0) {
#pragma unroll
            for (int w = 0; w < kWords; ++w) sh_flow[buf][w][wave] = f[2 * w] + f[2 * w + 1] * 65536;
        }
        __syncthreads();
        int lo[2 * kWords], hi[2 * kWords];  // |sums| <= 1024 fit the halves
#pragma unroll
        for (int w = 0; w < kWords; ++w) {
            const int32_t v = row_prefix_sum(sh_flow[buf][w][lane & 15]);
            const int32_t a = wave > 0 ? __builtin_amdgcn_readlane(v, wave > 0 ? wave - 1 : 0) : 0;
            const int32_t z = __builtin_amdgcn_readlane(v, kDayWaves - 1);
            lo[2 * w] = (int32_t)(int16_t)(a & 0xffff);
            lo[2 * w + 1] = (a - lo[2 * w]) >> 16;
            hi[2 * w] = (int32_t)(int16_t)(z & 0xffff);
            hi[2 * w + 1] = (z - hi[2 * w]) >> 16;
        }
        buf ^= 1;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            before[k] = lo[k];
            all[k] = hi[k];
        }
        return hi[K] != 0;
    };
    for (;;) {
        if (!(c.lam * (1.0 - c.clock) >= kGroupRest)) return false;  // the same in every thread
        const Word4 o = philox4x32_10(Word4{kbase + (uint32_t)t, node, day, 0u}, key0, key1);
        const double E = minus_log(unit_open(o.a, o.b));
        const double U = unit_open(o.c, o.d);
        // guess: every attempt sees the round's starting state
        int j = 0;
        {
            const double target = U * c.lam;
#pragma unroll
            for (int k = 0; k < NT; ++k) j += c.cum[k] < target ? 1 : 0;
        }
        double lam = c.lam;
        bool settled = false, moved = true;
        int all[K];
        for (int pass = 0; pass < kGroupPasses; ++pass) {
            int n[K], before[K];
            Rules::flows(j, ~0ull, n);
            const bool any = exchange(n, moved, before, all);
            if (!any) {  // the picks are those the waiting rates lam were computed from
                settled = true;
                break;
            }
            Rules::flows(j, below, n);
#pragma unroll
            for (int k = 0; k < K; ++k) n[k] += before[k];
            double cum[NT];
            Rules::cum_after(m, c, n, cum);
            lam = cum[NT - 1];
            const double target = U * lam;
            int jn = 0;
#pragma unroll
            for (int k = 0; k < NT; ++k) jn += cum[k] < target ? 1 : 0;
            moved = __ballot(jn != j) != 0ull;
            j = jn;
        }
        if (!settled) return false;  // the same in every thread; nothing of this round applied
        const double tau = E / lam;  // lambda = 0: tau = inf, never fires
        double s = c.clock;
        int done = 0;        // attempts before done fire; s is the clock after them
        bool ended = false;  // attempt done does not fire
        if (!(s > 0.0)) {
            if (wave == 0) {
                sh_head[lane] = tau;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                double q = s, z = s;
                int A = 0;
#pragma unroll 16
                for (int i = 0; i < 64; ++i) {
                    q = q + sh_head[i];
                    const bool in = q < 1.0;
                    z = in ? q : z;
                    A += in ? 1 : 0;
                }
                if (lane == 0) {
                    sh_before = z;
                    sh_special = A;
                }
            }
            __syncthreads();
            s = sh_before;
            done = sh_special;
            ended = done < 64;
        }
        while (!ended && done < round) {
            const int e = (int)((__double_as_longlong(s) >> 52) & 0x7ff) - 1023;
            if (e < -960) return false;  // too small to scale; nothing of this round applied
            const double up = __longlong_as_double((long long)(1023 + 52 - e) << 52);    // 2^(52-e)
            const double down = __longlong_as_double((long long)(1023 - 52 + e) << 52);  // 2^(e-52)
            const double S0 = s * up;                                                    // in [2^52, 2^53)
            const double T = 0x1p53 - S0;
            const bool live = t >= done;
            const double v = tau * up;
            const double fl = floor(v);
            const double fr = v - fl;
            const double P = wave_prefix_sum(live ? (fr > 0.5 ? fl + 1.0 : fl) : 0.0);
            const bool tie = live && fr == 0.5;
            const unsigned long long ties = __ballot(tie);
            if (lane == 63) {
                sh_total[wave] = P;
                sh_tie[wave] = ties != 0ull ? 1 : 0;
            }
            __syncthreads();
            const double sums = row_prefix_sum(sh_total[lane & 15]);
            // the first wavefront with a sum past the binade or a tie
            const uint32_t odd = (uint32_t)__ballot(sh_tie[lane & 15] != 0 || !(sums < T)) & 0xffffu;
            if (odd == 0u) {
                s = (S0 + lane_f64(sums, kDayWaves - 1)) * down;
                done = round;
                break;
            }
            if (wave == __builtin_ctz(odd)) {
                const double mine = wave > 0 ? lane_f64(sums, wave > 0 ? wave - 1 : 0) : 0.0;
                const double Pg = P + mine;
                const int sp = __ffsll((long long)__ballot(tie || (live && !(Pg < T)))) - 1;
                const double prior = sp > 0 ? lane_f64(Pg, sp > 0 ? sp - 1 : 0) : mine;
                if (lane == sp) {
                    sh_at = tau;
                    sh_before = (S0 + prior) * down;
                    sh_special = 64 * wave + sp;
                }
            }
            __syncthreads();
            const double s2 = sh_before + sh_at;
            done = sh_special;
            ended = !(s2 < 1.0);
            s = ended ? sh_before : s2;
            done += ended ? 0 : 1;
        }
        int A = done;
        bool limit = false;
        if (c.fired + A >= SIM_MAX_FIRED) {
            A = SIM_MAX_FIRED - c.fired;
            limit = true;
        }
        if (A < round) {
            const int nw = A - 64 * wave;
            int n[K], before[K];
            Rules::flows(j, nw >= 64 ? ~0ull : (nw > 0 ? ((1ull << nw) - 1ull) : 0ull), n);
            exchange(n, false, before, all);
        }
        Rules::advance(m, c, all);
        if (A > 0 && !limit) c.clock = s;
        c.fired = c.fired + A;
        Rules::rates(m, c);
        if (limit) {
            if (t == 0) atomicMin(status, (STATUS_LIMIT_TAG << 32) | (unsigned long long)(uint32_t)r);
            return true;
        }
        if (A < round || !(c.lam > 0.0)) return true;
        kbase = kbase + round;
    }
}

// Chains of a queue walked side by side by the segments of a wavefront, G
// lanes each, a segment taking the next chain when its own ends: take(k)
// claims the next k queue entries for this wavefront and returns the first
// (entries from n on do not exist), load(i, c, key) fills in chain i, store(i,
// c) takes its end state. G balances what a round does for one chain (short
// chains leave the lanes past their end idle) against the rounds that its
// longest chain needs.
struct ChainKey {
    uint32_t kbase, node, day, key0, key1;
    unsigned long long *status;
    int32_t r;
};

template <class Rules, int G, class Take, class Load, class Store>
__device__ __forceinline__ void walk_queue(const Model &m, int n, double *sh_tau, const Take &take, const Load &load,
                                           const Store &store) {
    const int lane = threadIdx.x & 63, li = lane & (G - 1), seg0 = lane - li;
    typename Rules::State c;
    ChainKey key{0u, 0u, 0u, 0u, 0u, nullptr, 0};
    auto none = [&]() {
#pragma unroll
        for (int k = 0; k < Rules::NC; ++k) c.xd[k] = 0.0;
#pragma unroll
        for (int k = 0; k < Rules::NT; ++k) c.cphi[k] = 0.0;
        c.clock = 0.0;
        c.fired = 0;
        Rules::reactants(m, c);
    };
    none();
    int at = -1;  // the segment's chain
    bool dry = false;
    for (;;) {
        if (!dry) {
            const unsigned long long idle = __ballot(at < 0 && li == 0);
            if (idle != 0ull) {
                const int k = __popcll(idle), first = take(k);
                if (at < 0) {
                    const int i = first + __popcll(idle & ((1ull << seg0) - 1ull));
                    if (i < n) {
                        at = i;
                        load(i, c, key);
                        Rules::reactants(m, c);
                    }
                }
                dry = first + k >= n;
            }
        }
        if (__ballot(at >= 0) == 0ull) break;
        const bool done = walk_round<Rules, G>(m, c, key.kbase, key.node, key.day, key.key0, key.key1, key.status,
                                               key.r, sh_tau);
        key.kbase = key.kbase + (uint32_t)G;
        if (at >= 0 && done) {
            if (li == 0) store(at, c);
            at = -1;
            none();
        }
    }
}

// Every chain of a wavefront to the end of the window. Attempt k of a chain
// uses Philox block (k, node, day, 0); the blocks do not depend on the state,
// so while m < 64 chains are live the wavefront computes 64/m blocks per
// chain in parallel (their -log rand and rand), parks them in LDS, and each
// live lane then walks its own in order. With all 64 lanes live each lane
// draws its own block; with one chain left, or at most `few` of which one
// still expects many attempts, the whole wavefront walks them one after
// another (walk_wave). Node, day and key are each lane's own (lanes of
// a slot handle may be at different days). Every lane of the wavefront must
// call this.
template <class Rules>
__device__ __forceinline__ void run_chains(const Model &m, typename Rules::State &c, bool live, uint32_t node,
                                           uint32_t day, uint32_t key0, uint32_t key1,
                                           unsigned long long *status, int32_t r, uint32_t few_chains) {
    __shared__ double sh_e[kWaves][64], sh_u[kWaves][64];
    __shared__ uint32_t sh_node[kWaves][64], sh_key[kWaves][64], sh_seed[kWaves][64], sh_k[kWaves][64];
    __shared__ uint32_t sh_day[kWaves][64];
    __shared__ double sh_tau[kWaves][64];
    const int wave = threadIdx.x >> 6;
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t kbase = 0;  // next attempt index of this lane's chain
    live = live && c.lam > 0.0;
    for (;;) {
        const unsigned long long mask = __ballot(live);
        if (mask == 0ull) break;
        if (mask == ~0ull) {
            const Word4 o = philox4x32_10(Word4{kbase, node, day, 0u}, key0, key1);
            kbase = kbase + 1;
            live = chain_step<Rules>(m, c, minus_log(unit_open(o.a, o.b)), unit_open(o.c, o.d), status, r);
            continue;
        }
        const uint32_t nlive = (uint32_t)__popcll(mask);
        // One chain left, or a few of which one still expects many attempts in
        // the window (lambda (1 - clock)): the whole wavefront walks them one
        // after another, 64 attempts at a time, instead of a lane each.
        const bool few = nlive <= few_chains &&
                         (nlive == 1 || __ballot(live && c.lam * (1.0 - c.clock) > 10.0 * (double)nlive) != 0ull);
        for (unsigned long long left = few ? mask : 0ull; left != 0ull; left &= left - 1ull) {
            const int h = __ffsll((long long)left) - 1;
            typename Rules::State u;
#pragma unroll
            for (int k = 0; k < Rules::NC; ++k) u.xd[k] = lane_f64(c.xd[k], h);
#pragma unroll
            for (int k = 0; k < Rules::NT; ++k) {
                u.cphi[k] = lane_f64(c.cphi[k], h);
            }
            u.lam = lane_f64(c.lam, h);
            u.clock = lane_f64(c.clock, h);
            u.fired = __builtin_amdgcn_readlane(c.fired, h);
            const uint32_t kb = (uint32_t)__builtin_amdgcn_readlane((int)kbase, h);
            const uint32_t nh = (uint32_t)__builtin_amdgcn_readlane((int)node, h);
            const uint32_t dh = (uint32_t)__builtin_amdgcn_readlane((int)day, h);
            const uint64_t st = (uint64_t)status;
            unsigned long long *sth = (unsigned long long *)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane(
                                                                  (int)(uint32_t)(st >> 32), h) << 32) |
                                                              (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)st, h));
            const uint32_t k0 = (uint32_t)__builtin_amdgcn_readlane((int)key0, h);
            const uint32_t k1 = (uint32_t)__builtin_amdgcn_readlane((int)key1, h);
            const int32_t rh = __builtin_amdgcn_readlane(r, h);
            Rules::reactants(m, u);
            walk_wave<Rules>(m, u, kb, nh, dh, k0, k1, sth, rh, sh_tau[wave]);
            if ((int)lane == h) c = u;
        }
        if (few) break;
        const uint32_t per = 64u / nlive;
        const uint32_t rank = (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
        if (live) {
            sh_node[wave][rank] = node;
            sh_day[wave][rank] = day;
            sh_key[wave][rank] = key1;
            sh_seed[wave][rank] = key0;
            sh_k[wave][rank] = kbase;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (lane < nlive * per) {
            const uint32_t ch = lane % nlive, t = lane / nlive;
            const Word4 o = philox4x32_10(Word4{sh_k[wave][ch] + t, sh_node[wave][ch], sh_day[wave][ch], 0u},
                                          sh_seed[wave][ch], sh_key[wave][ch]);
            sh_e[wave][ch * per + t] = minus_log(unit_open(o.a, o.b));
            sh_u[wave][ch * per + t] = unit_open(o.c, o.d);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (live) {
            for (uint32_t t = 0; t < per; ++t) {
                live = chain_step<Rules>(m, c, sh_e[wave][rank * per + t], sh_u[wave][rank * per + t], status, r);
                if (!live) break;
            }
            kbase = kbase + per;
        }
        __builtin_amdgcn_wave_barrier();  // the next round rewrites the LDS slots
    }
}

// Whether no error has been recorded, read once per workgroup so that every
// thread takes the same branch (another wavefront of the workgroup may record
// an error while this one is still starting). Every thread must call it.
__device__ __forceinline__ bool block_ok(const unsigned long long *status) {
    __shared__ int ok;
    __syncthreads();
    if (threadIdx.x == 0) ok = *(volatile const unsigned long long *)status == STATUS_OK;
    __syncthreads();
    return ok != 0;
}

// block_ok for a kernel that checks once per launch: thread 0 reads the
// status word right away, alongside the loads the workgroup has already
// issued, and one barrier publishes it (no earlier reader of the flag to wait
// for), so the check adds no round trip of its own.
__device__ __forceinline__ bool block_ok_once(const unsigned long long *status) {
    __shared__ int ok;
    if (threadIdx.x == 0) ok = *(volatile const unsigned long long *)status == STATUS_OK;
    __syncthreads();
    return ok != 0;
}

// Wavefront reductions with DPP lane moves, which run in the vector ALU:
// pairs and quads (quad permutes), rows of 8 and 16 lanes (half-row and row
// mirrors), then row 0 into row 1 and row 2 into row 3 (broadcast of lane 15),
// then rows 0-1 into rows 2-3 (broadcast of lane 31); lane 63 ends with the
// whole wavefront, read back as a uniform value. Every lane must be active.
// (A shuffle butterfly would wait on an LDS crossbar round trip per step.)
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ int32_t dpp_move(int32_t v) {
    // lanes of rows outside ROWS read 0
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false);
}

template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ long long dpp_move64(long long v) {
    const uint32_t lo = (uint32_t)dpp_move<CTRL, ROWS>((int32_t)(uint32_t)v);
    const uint32_t hi = (uint32_t)dpp_move<CTRL, ROWS>((int32_t)(uint32_t)((unsigned long long)v >> 32));
    return (long long)(((unsigned long long)hi << 32) | lo);
}

constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e, kDppHalfMirror = 0x141, kDppMirror = 0x140,
              kDppBcast15 = 0x142, kDppBcast31 = 0x143;

__device__ __forceinline__ long long wave_sum(long long v) {
    v += dpp_move64<kDppXor1>(v);
    v += dpp_move64<kDppXor2>(v);
    v += dpp_move64<kDppHalfMirror>(v);
    v += dpp_move64<kDppMirror>(v);
    v += dpp_move64<kDppBcast15, 0xa>(v);
    v += dpp_move64<kDppBcast31, 0xc>(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)v, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)((unsigned long long)v >> 32), 63);
    return (long long)(((unsigned long long)hi << 32) | lo);
}

// Per-lane contributions to the daily records of one phase.
template <int NC>
struct Tally {
    long long prev, trans;
    long long tot[NC];
    int32_t most;  // most SSA transitions of one lane's chain (the day's straggler)
};

// (for values >= 0: rows outside a broadcast's mask read 0)
__device__ __forceinline__ int32_t wave_max(int32_t v) {
    v = max(v, dpp_move<kDppXor1>(v));
    v = max(v, dpp_move<kDppXor2>(v));
    v = max(v, dpp_move<kDppHalfMirror>(v));
    v = max(v, dpp_move<kDppMirror>(v));
    v = max(v, dpp_move<kDppBcast15, 0xa>(v));
    v = max(v, dpp_move<kDppBcast31, 0xc>(v));
    return __builtin_amdgcn_readlane(v, 63);
}

// Sum tallies over the workgroup and add them to the records of one set
// (every lane of the workgroup belongs to the same trajectory).
template <int NC>
__device__ __forceinline__ void flush_block(const Model &m, const DevState &s, const Tally<NC> &t, int32_t set, int32_t d_rec,
                            int32_t d_ssa, int32_t region) {
    __shared__ long long part[kWaves][2 + NC];
    __shared__ int32_t part_most[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t S = (int64_t)s.n_inst * s.R;
    const int32_t most = wave_max(t.most);
    if (lane == 0) part_most[wave] = most;
    long long v[2 + NC];
    v[0] = t.prev;
    v[1] = t.trans;
#pragma unroll
    for (int c = 0; c < NC; ++c) v[2 + c] = t.tot[c];
#pragma unroll
    for (int i = 0; i < 2 + NC; ++i) {
        const long long w = wave_sum(v[i]);
        if (lane == 0) part[wave][i] = w;
    }
    __syncthreads();
    if (threadIdx.x < 2 + NC) {
        const int i = threadIdx.x;
        long long sum = 0;
#pragma unroll
        for (int q = 0; q < kWaves; ++q) sum += part[q][i];
        if (i == 0 && d_rec >= 0) {
            if (sum) atomicAdd(&s.prevalence[d_rec * S + set], (int32_t)sum);
        } else if (i == 1 && d_ssa >= 0) {
            if (sum) {
                atomicAdd((unsigned long long *)&s.transitions[d_ssa * S + set], (unsigned long long)sum);
                int32_t m_all = 0;
#pragma unroll
                for (int q = 0; q < kWaves; ++q) m_all = max(m_all, part_most[q]);
                atomicMax(&s.max_fired[d_ssa * S + set], m_all);
            }
        } else if (i >= 2 && d_rec >= 0 && comp_on<NC>(m, i - 2)) {
            if (sum) atomicAdd((unsigned long long *)&s.totals[(d_rec * S + set) * m.nc + (i - 2)],
                               (unsigned long long)sum);
            if (sum && region >= 0)
                atomicAdd((unsigned long long *)&s.regional[((d_rec * S + set) * s.n_regions + region) * m.nc + (i - 2)],
                          (unsigned long long)sum);
        }
    }
    __syncthreads();
}

// Sum tallies over the wavefronts of a replicate tile (lane = replicate) and
// add them to the records of the lane's set.
template <int NC>
__device__ __forceinline__ void flush_tile(const Model &m, const DevState &s, const Tally<NC> &t, int32_t set, int32_t d_rec,
                           int32_t d_ssa, int32_t region) {
    __shared__ long long part[kWaves][64][2 + NC];
    __shared__ int32_t part_most[kWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t S = (int64_t)s.n_inst * s.R;
    part[wave][lane][0] = t.prev;
    part[wave][lane][1] = t.trans;
    part_most[wave][lane] = t.most;
#pragma unroll
    for (int c = 0; c < NC; ++c) part[wave][lane][2 + c] = t.tot[c];
    __syncthreads();
    if (wave == 0 && set >= 0) {
        long long v[2 + NC];
#pragma unroll
        for (int i = 0; i < 2 + NC; ++i) {
            v[i] = 0;
#pragma unroll
            for (int q = 0; q < kWaves; ++q) v[i] += part[q][lane][i];
        }
        if (d_rec >= 0) {
            if (v[0]) atomicAdd(&s.prevalence[d_rec * S + set], (int32_t)v[0]);
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (comp_on<NC>(m, c) && v[2 + c]) {
                    atomicAdd((unsigned long long *)&s.totals[(d_rec * S + set) * m.nc + c], (unsigned long long)v[2 + c]);
                    if (region >= 0)
                        atomicAdd((unsigned long long *)&s.regional[((d_rec * S + set) * s.n_regions + region) * m.nc + c],
                                  (unsigned long long)v[2 + c]);
                }
        }
        if (d_ssa >= 0 && v[1]) {
            atomicAdd((unsigned long long *)&s.transitions[d_ssa * S + set], (unsigned long long)v[1]);
            int32_t m_all = 0;
#pragma unroll
            for (int q = 0; q < kWaves; ++q) m_all = max(m_all, part_most[q][lane]);
            atomicMax(&s.max_fired[d_ssa * S + set], m_all);
        }
    }
    __syncthreads();
}

// Draw n of the tot individuals in the compartments of mask from x without
// replacement (Sec. 3.2): draw q picks the individual at a uniform position
// in [0, remaining) of the selected compartments in ascending order, from the
// Philox block (q / 2, g, d, 1). Removes them from x and counts them in take.
template <int NC>
__device__ __forceinline__ void draw_individuals(int32_t *x, int32_t *take, uint32_t mask, int32_t n, long long tot,
                                                 uint32_t g, int32_t d, uint32_t key0, uint32_t key1) {
    long long cum[NC];  // running sums of the selected compartments, ascending
    long long run = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        take[c] = 0;
        run += ((mask >> c) & 1u) ? x[c] : 0;
        cum[c] = run;
    }
    Word4 o{0, 0, 0, 0};
    for (int32_t q = 0; q < n; ++q) {
        uint64_t bits;
        if ((q & 1) == 0) {
            o = philox4x32_10(Word4{(uint32_t)q >> 1, g, (uint32_t)d, 1u}, key0, key1);
            bits = ((uint64_t)o.b << 32) | o.a;
        } else {
            bits = ((uint64_t)o.d << 32) | o.c;
        }
        const uint64_t pick = __umul64hi(bits, (uint64_t)tot);  // uniform on [0, tot)
        // the compartment holding individual `pick` in ascending order is the
        // number of running sums at or below it (a compartment outside the
        // mask, or empty, repeats the sum before it and is passed over)
        int chosen = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c) chosen += (uint64_t)cum[c] <= pick ? 1 : 0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int hit = c == chosen ? 1 : 0;
            x[c] -= hit;
            take[c] += hit;
            cum[c] -= c >= chosen ? 1 : 0;
        }
        tot -= 1;
    }
}

// draw_individuals for an event of at most N draws that were computed ahead
// (pre), tot below 2^31: draw q picks among tot - q individuals whatever the
// earlier picks were, and the running sums and picks fit 32 bits (the same
// comparisons).
template <int NC, int N>
__device__ __forceinline__ void draw_ahead(int32_t *x, int32_t *take, uint32_t mask, int32_t n, uint32_t tot,
                                           const uint64_t (&pre)[N]) {
    uint32_t cum[NC], run = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        take[c] = 0;
        run += ((mask >> c) & 1u) ? (uint32_t)x[c] : 0u;
        cum[c] = run;
    }
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const uint32_t pick = (uint32_t)__umul64hi(pre[q], (uint64_t)tot - q);
        int chosen = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c) chosen += cum[c] <= pick ? 1 : 0;
        if (q >= n) chosen = NC;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int hit = c == chosen ? 1 : 0;
            x[c] -= hit;
            take[c] += hit;
            cum[c] -= c >= chosen ? 1u : 0u;
        }
    }
}

// Compartment that an individual drawn from compartment c lands in (internal
// and external transfers): 4 bits per source compartment of the event's map.
__device__ __forceinline__ int shifted(uint32_t smap, int c) { return (int)((smap >> (4 * c)) & 0xFu); }

// The loads day_wave starts from: the lane's position's node and instance, its
// counts and phi (zeros for a lane past the end).
template <int NC>
struct LaneLoad {
    int32_t x[NC];
    double phi;
    int32_t nid, inst;
};

template <int NC>
__device__ __forceinline__ LaneLoad<NC> lane_load(const Model &m, const DevState &s, int64_t l) {
    LaneLoad<NC> q;
    q.nid = -1;
    q.inst = 0;
    q.phi = 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c) q.x[c] = 0;
    if (l < s.L) {
        const int64_t pos = s.RL == 1 ? l : l / s.RL;
        q.nid = s.node_id[pos];
        q.inst = s.inst[pos];
#pragma unroll
        for (int c = 0; c < NC; ++c) q.x[c] = comp_on<NC>(m, c) ? s.u[(int64_t)c * s.L + l] : 0;
        q.phi = s.phi[l];
    }
    return q;
}

// phi_{d+1} = (1 - beta(day0 + d)) phi_d + alpha I/N (eq:siminfpressure, Euler
// step) from the counts y, and I (sums of counts are exact in binary64).
template <int NC>
__device__ __forceinline__ double phi_next(const Model &m, const int32_t *y, double alpha, double beta, double phi,
                                           double *Iout) {
    double I = 0.0, N = 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if ((m.imask >> c) & 1u) I += (double)y[c];
        if ((m.nmask >> c) & 1u) N += (double)y[c];
    }
    *Iout = I;
    const double a = 1.0 - beta;
    const double b = a * phi;
    const double shed = N > 0.0 ? alpha * (I / N) : 0.0;
    return b + shed;
}

// The day phase for the lane l of a wavefront (every lane of the wavefront
// must call it; lanes with l >= L or replicate lane r >= r_end take part in
// the wavefront-level steps only): close day d-1 (phi update + record) if
// prologue, then run the SSA of day d if ssa. Adds the lane's counts to t.
// Every load that does not depend on another is issued first (padding
// positions hold zeros).
template <class Rules>
__device__ __forceinline__ void day_wave(const Model &m, const DevState &s, int64_t l, int32_t d,
                                         bool prologue, bool ssa, Tally<Rules::NC> &t, int32_t r_end,
                                         unsigned long long *status) {
    constexpr int NC = Rules::NC, NT = Rules::NT;
    const int32_t R = s.R, RL = s.RL;
    const bool in_range = l < s.L;
    const int32_t r = !in_range || RL == 1 ? 0 : (int32_t)(l % RL);
    const int32_t rec = prologue ? s.rec_slot[d - 1] : -1;
    const LaneLoad<NC> q = lane_load<NC>(m, s, l);
    int32_t x[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) x[c] = q.x[c];
    double phi = q.phi;
    int32_t nid = q.nid, inst = q.inst;
    // padding positions and idle lanes take part in the wavefront steps only
    const bool active = r < r_end && nid >= 0;
    if (!active) {
        inst = 0;
        phi = 0.0;
#pragma unroll
        for (int c = 0; c < NC; ++c) x[c] = 0;
    }
    const int32_t set = inst * R + r;
    const uint32_t node = active ? (uint32_t)nid : 0u;
    auto phi_after = [&](const int32_t *y, int32_t dd, double ph, double *Iout) {
        const int q = season((int64_t)m.day0 + dd);
        return phi_next<NC>(m, y, s.alpha[set], s.beta[set * 4 + q], ph, Iout);
    };
    if (active && prologue) {
        const double phi_in = phi;
        const int32_t dp = d - 1;
        double I = 0.0;
        if (m.phi_pre) {
            // phi was already fed by the state before the events of day dp
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if ((m.imask >> c) & 1u) I += x[c];
        } else {
            phi = phi_after(x, dp, phi, &I);
        }
        t.prev += I > 0.0 ? 1 : 0;
#pragma unroll
        for (int c = 0; c < NC; ++c) t.tot[c] += x[c];
        const int32_t slot = rec;
        if (slot >= 0) {
            const int64_t base = (((int64_t)slot * R + r) * s.n_nodes + s.inst_off[inst] + node);
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (comp_on<NC>(m, c)) s.snap_u[base * m.nc + c] = x[c];
            s.snap_v[base] = phi;
        }
        if (__double_as_longlong(phi) != __double_as_longlong(phi_in)) s.phi[l] = phi;
    }
    // d, prologue and ssa may differ between the lanes of a slot handle's
    // wavefront: a lane without the SSA today takes part with no live chain
    if (__ballot(ssa) == 0ull) return;
    const bool walks = active && ssa;
    typename Rules::State ch;
    const uint32_t key0 = active ? s.seed[inst] : 0u;
    const uint32_t key1 = active ? s.repid[set] : 0u;
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        double c = active && trans_on<NT>(m, k) ? s.coef[set * m.nt + k] : 0.0;
        if ((m.uses_phi >> k) & 1u) c = c * phi;
        ch.cphi[k] = c;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) ch.xd[c] = (double)x[c];
    ch.clock = 0.0;
    ch.fired = 0;
    Rules::rates(m, ch);
    run_chains<Rules>(m, ch, walks, node, (uint32_t)d, key0, key1, status, set, s.few_chains);
    t.trans += ch.fired;
    t.most = max(t.most, (int32_t)ch.fired);
    if (walks && ch.fired) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (comp_on<NC>(m, c)) s.u[(int64_t)c * s.L + l] = (int32_t)ch.xd[c];
    }
    if (walks && m.phi_pre) {
        // eq:numstep5 as written: phi from the state after the SSA, before the events
        int32_t y[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) y[c] = (int32_t)ch.xd[c];
        double I = 0.0;
        const double phi2 = phi_after(y, d, phi, &I);
        if (__double_as_longlong(phi2) != __double_as_longlong(phi)) s.phi[l] = phi2;
    }
}

template <int NC>
__device__ __forceinline__ void event_task(const Model &m, const DevState &s, const DevEvents &ev, int64_t t,
                                           int32_t r, int32_t d, unsigned long long *status);

// The private tasks of one unit (a workgroup's positions) on day d, right after
// its SSA: the pairs (task, lane) of the workgroup, nl lanes per position
// starting at r0, lanes r >= r_end idle. The SSA results of the unit must be
// visible to the whole workgroup (a workgroup barrier first).
template <int NC>
__device__ __forceinline__ void private_tasks(const Model &m, const DevState &s, const DevEvents &ev, int32_t d,
                                              int64_t unit, int64_t n_units, int32_t r0, int32_t nl, int32_t r_end,
                                              unsigned long long *status) {
    fresh_l1();
    const int64_t k = (int64_t)d * n_units + unit;
    const int64_t t0 = ev.priv_off[k], t1 = ev.priv_off[k + 1];
    const int64_t count = (t1 - t0) * nl;
    for (int64_t i = threadIdx.x; i < count; i += blockDim.x) {
        const int64_t t = t0 + (nl == 1 ? i : i / nl);
        const int32_t r = r0 + (nl == 1 ? 0 : (int32_t)(i % nl));
        if (r < r_end) event_task<NC>(m, s, ev, t, r, d, status);
    }
}

// One event applied to counts in LDS: compartment c of its node at xs[c], of its
// destination at xd[c]. A node drawn from is the event's alone;
// additions are atomic. pre: its first N draws, if they were computed ahead.
template <int NC, int N>
__device__ __forceinline__ void event_lds(uint32_t meta, uint32_t smap, int32_t n, uint32_t g, const int32_t *gm,
                                          int32_t *xs, int32_t *xd, uint32_t key0, uint32_t key1,
                                          int32_t set, int32_t d, unsigned long long *status,
                                          const uint64_t (&pre)[N], bool ahead) {
    const int kind = (int)(meta & kEvKindMask);
    const uint32_t mask = (meta >> 2) & 0xffu;
    auto add = [&](int32_t *p, int32_t v) {
        __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // A selection of one or two compartments c0 < c1 with its draws computed
    // ahead (every column of the farm model, every movement of up to six
    // animals): the running sums of the walk below are 0 before c0, x[c0]
    // from c0 to c1 and the total from c1 on, so a pick below the count left
    // in c0 takes from c0 and any other from c1 (the same picks, counts and
    // write order as the walk over all compartments).
    const uint32_t rest = mask & (mask - 1u);
    if (mask != 0u && (rest & (rest - 1u)) == 0u && ahead && n <= N && (kind != SIM_ENTER || rest == 0u)) {
        const int c0 = __builtin_ctz(mask);
        const int c1 = rest ? __builtin_ctz(rest) : c0;
        if (kind == SIM_ENTER) {
            add(&xs[c0], n);
            return;
        }
        const int32_t x0 = xs[c0], x1 = rest ? xs[c1] : 0;
        const long long tot = (long long)x0 + (long long)x1;
        if ((long long)n > tot) {
            atomicMin(status, ((unsigned long long)(uint32_t)*gm << 32) | (unsigned long long)(uint32_t)set);
            return;
        }
        if (tot <= 0x7fffffffLL) {
            int32_t t0 = 0;
            uint32_t left0 = (uint32_t)x0;
#pragma unroll
            for (int q = 0; q < N; ++q) {
                const uint32_t pick = (uint32_t)__umul64hi(pre[q], (uint64_t)(tot - q));
                const int in0 = q < n && pick < left0 ? 1 : 0;
                left0 -= (uint32_t)in0;
                t0 += in0;
            }
            const int t1 = n - t0;
            xs[c0] = x0 - t0;
            if (rest) xs[c1] = x1 - t1;
            if (kind == SIM_INTERNAL) {
                if (t0) xs[shifted(smap, c0)] += t0;
                if (t1) xs[shifted(smap, c1)] += t1;
            } else if (kind == SIM_EXTERNAL) {
                if (t0) add(&xd[shifted(smap, c0)], t0);
                if (t1) add(&xd[shifted(smap, c1)], t1);
            }
            return;
        }
    }
    if (kind == SIM_ENTER) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if ((mask >> c) & 1u) add(&xs[c], n);
        return;
    }
    int32_t x[NC];
    long long tot = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        x[c] = ((mask >> c) & 1u) ? xs[c] : 0;
        tot += x[c];
    }
    if ((long long)n > tot) {
        atomicMin(status, ((unsigned long long)(uint32_t)*gm << 32) | (unsigned long long)(uint32_t)set);
        return;
    }
    int32_t take[NC];
    // Selections of three compartments or more take the draws computed ahead in
    // the general models (3,000 herds of three compartments, all selected, a day
    // 21.2 -> 18.9 us). The farm model's events select one; there the code alone
    // costs more than it saves (37,000 herds, a day 21.8 -> 22.7 us).
    if (!exact_size(NC) && ahead && n <= N && tot <= 0x7fffffffLL)
        draw_ahead<NC>(x, take, mask, n, (uint32_t)tot, pre);
    else
        draw_individuals<NC>(x, take, mask, n, tot, g, d, key0, key1);
#pragma unroll
    for (int c = 0; c < NC; ++c)
        if ((mask >> c) & 1u) xs[c] = x[c];
    if (kind == SIM_EXIT) return;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (take[c]) {
            const int to = shifted(smap, c);
            if (kind == SIM_INTERNAL)
                xs[to] += take[c];
            else
                add(&xd[to], take[c]);
        }
    }
}

// The first n draws of event g on day d (pairs from Philox blocks).
template <int N>
__device__ __forceinline__ void draws_ahead(uint64_t (&pre)[N], int32_t n, uint32_t g, int32_t d, uint32_t key0,
                                            uint32_t key1) {
#pragma unroll
    for (int b = 0; b < N / 2; ++b) {
        pre[2 * b] = pre[2 * b + 1] = 0;
        if (2 * b >= n) continue;
        const Word4 o = philox4x32_10(Word4{(uint32_t)b, g, (uint32_t)d, 1u}, key0, key1);
        pre[2 * b] = ((uint64_t)o.b << 32) | o.a;
        pre[2 * b + 1] = ((uint64_t)o.d << 32) | o.c;
    }
}

// One private event of a workgroup's day, staged in LDS.
struct PrivEv {
    uint32_t meta, smap;
    int32_t n, g, gm, node;
};
constexpr int kPrivDraws = 2;  // of a private event
constexpr int kPreDraws = 6;   // of a level event

// One private task (a run of one node's single-node events, i the first)
// applied to the counts in LDS (position loc's compartment c at xs[loc * NC + c]).
// A run that draws has the node to itself; runs of additions only may share it
// and add atomically. pre: the first draws of event i.
template <int NC>
__device__ __forceinline__ void private_task_lds(const PrivEv *pe, int i, int n_ev, int32_t *xs, int32_t *touch, int32_t base,
                                 int32_t d, uint32_t key0, uint32_t key1, int32_t set, unsigned long long *status,
                                 const uint64_t (&pre)[kPrivDraws]) {
    const int loc = pe[i].node - base;
    touch[loc] = 1;
    int j = i;
    do {
        event_lds<NC>(pe[j].meta, pe[j].smap, pe[j].n, (uint32_t)pe[j].g, &pe[j].gm, &xs[loc * NC], &xs[loc * NC], key0, key1,
                      set, d, status, pre, j == i);
        ++j;
    } while (j < n_ev && (pe[j].meta & kMetaCont));
}

// One lane per node: a workgroup runs one unit of s.tile_nodes positions (4 to
// 1024), thread t < tile_nodes owning position t. The counts live in LDS for
// the day: the owners close the previous day and list their node's chain, as
// long if it expects kWaveChain attempts (lambda) or more; then the whole
// workgroup walks the longest chains one after another (walk_group), its
// wavefronts take the other long ones one each (walk_wave), and the rest are
// walked side by side by segments of a wavefront (walk_queue); at last the
// unit's private tasks run on the counts, and each touched node is stored
// once. What binds a day is the latency of the walks' dependent arithmetic, so
// the chains of a few nodes are spread over many wavefronts: sixteen a unit
// (eight for large general models), and units small enough for every compute
// unit to have one (lane_unit on the host); with more units than that, fewer.
// With four wavefronts a unit of 256 nodes, each walking its 64 nodes' chains
// attempt by attempt in their own lanes, a day's SSA took about 18 us whatever
// its chains' lengths.
// The longest chains: those of group_min_attempts and more, in classes of a
// factor of 4, the highest classes that hold one chain together (three from
// class kFarClass on). A workgroup walks a chain of 2,000 attempts in about
// 40,000 cycles, mostly its first round's (10 cycles an attempt past that), a
// wavefront in 70,000, and several wavefronts side by side cost little more, so
// several chains of one length are done sooner by a wavefront each (1,000
// chains of 2,000 in units of 4: 36 us a day, against 82 by their workgroups).
constexpr double kWaveChain = 48.0;
constexpr int kFarClass = 3, kLengthClasses = 6;

//
// A day whose levels touch few nodes (EventDayArgs) has no launch for them: the
// workgroups of the next day's launch (or of the closing one) each apply all of
// the day's level events to the touched nodes' counts, a thread an event, from
// the counts that the day before left in s.stage, and keep the nodes of their
// own unit. Levels take about 0.5 us each there, and the launch, its two
// boundaries and the round trip of the counts through memory, about 6 us a day,
// are gone (a day of the SIS network of 1,000 nodes 12.0 -> 11.4 us, of the farm
// model with 1,000 nodes 17.7 -> 15.5, with 37,000 33.4 -> 29.3).
struct DayCounts {
    int32_t n[2], next[2], in_class[kLengthClasses], most;
    unsigned long long trans;
};

// The LDS of a unit of U positions and a workgroup of B threads (offsets into
// the launch's dynamic LDS).
template <int NC>
struct DayShared {
    int32_t *x;         // [U][NC] counts
    double *phi;        // [U]
    int32_t *node;      // [U]
    int32_t *touch;     // [U] nodes to store: a transition fired or an event changed them
    uint16_t *list;     // [2][U] positions with a chain: long (with the length class << kStageShift), short
    PrivEv *pe;         // [B]
    uint64_t *pd;       // [kPrivDraws][B] their first draws
    double *tau;        // [B] 64 values a wavefront
    long long *part;    // [B / 64][1 + NC]
    // a day's level events and the counts of the nodes they touch
    int32_t *eu;        // [kDaySlotCap][NC]
    uint32_t *ev;       // [kDayEventCap][4] meta, smap, n, g
    int32_t *lv;        // [kDayLevelCap + 1]
    __host__ __device__ size_t place(char *at, int U, int B, bool events) {
        size_t off = 0;
        auto take = [&](size_t bytes) {
            char *p = at + off;
            off += (bytes + 15) & ~(size_t)15;
            return p;
        };
        phi = (double *)take(sizeof(double) * U);
        tau = (double *)take(sizeof(double) * B);
        part = (long long *)take(sizeof(long long) * (B / 64) * (1 + NC));
        x = (int32_t *)take(sizeof(int32_t) * NC * U);
        node = (int32_t *)take(sizeof(int32_t) * U);
        touch = (int32_t *)take(sizeof(int32_t) * U);
        list = (uint16_t *)take(sizeof(uint16_t) * 2 * U);
        pe = (PrivEv *)take(sizeof(PrivEv) * B);
        pd = (uint64_t *)take(sizeof(uint64_t) * kPrivDraws * B);
        eu = (int32_t *)take(events ? sizeof(int32_t) * kDaySlotCap * NC : 0);
        ev = (uint32_t *)take(events ? sizeof(uint32_t) * 4 * kDayEventCap : 0);
        lv = (int32_t *)take(events ? sizeof(int32_t) * (kDayLevelCap + 1) : 0);
        return off;
    }
};

// The level events a of day d on the touched nodes' counts, an event a thread
// (a.ne <= kDayEventCap <= blockDim.x). Every thread calls it; the counts stand
// in sh.eu after its last barrier. A later event of a task is applied by the
// thread of its first, without draws ahead.
struct LevelEvent {
    uint32_t meta, smap, g, key0, key1;
    int32_t n, src, dst, set;
};

template <int NC>
__device__ __forceinline__ void event_levels_lds(const DevState &s, const DevEvents &ev, const EventDayArgs &a,
                                                 int32_t d, const LevelEvent e, const DayShared<NC> &sh) {
    const int i = threadIdx.x;
    uint64_t pre[kPreDraws];
    draws_ahead<kPreDraws>(pre, (int)(e.meta & kEvKindMask) == SIM_ENTER ? 0 : e.n, e.g, d, e.key0, e.key1);
    for (int k = 0; k < a.nl; ++k) {
        const int end = sh.lv[k + 1];
        if (i >= sh.lv[k] && i < end && !(e.meta & kMetaCont)) {
            int32_t *xs = &sh.eu[e.src * NC], *xd = &sh.eu[(e.dst >= 0 ? e.dst : e.src) * NC];
            uint32_t meta = e.meta, smap = e.smap, g = e.g;
            int32_t n = e.n;
            for (int j = i;;) {
                event_lds<NC>(meta, smap, n, g, &ev.gm[a.e0 + j], xs, xd, e.key0,
                              e.key1, e.set, d, s.status, pre, j == i);
                // (a task of several events is one of a single node)
                if (++j >= end || !(sh.ev[4 * j] & kMetaCont)) break;
                meta = sh.ev[4 * j];
                smap = sh.ev[4 * j + 1];
                n = (int32_t)sh.ev[4 * j + 2];
                g = sh.ev[4 * j + 3];
            }
        }
        __syncthreads();
    }
}

// LEVELS: some day of the run has such events (the plain variant keeps the
// registers for them free).
// OWN: where every wavefront has herds of its own (launch_day), the segments of
// walk_queue are short of nothing but instructions, and 16 lanes for a chain of
// a few attempts waste them. A wavefront with kOwnFirst short chains or more
// then walks them where they are listed, each in its owner's lane, until
// kOwnRest are left; those are listed and start again in a segment. (A day of
// 1.5 million herds, all infected: SISe3 536 -> 232 us, SIS 376 -> 177; of
// 100,000 herds with four times the rates 86 -> 72. The code alone costs 0.8 us
// of 22 a day on 37,000 herds with a tenth infected, where a quarter of the
// wavefronts own herds.)
constexpr int kOwnFirst = 24, kOwnRest = 8;

template <class Rules, bool LEVELS, bool OWN>
__global__ __launch_bounds__(Rules::kDayThreads) void k_day(Model m, DevState s, DevEvents ev, int32_t d, int32_t prologue,
                                                   int32_t ssa, EventDayArgs a) {
    constexpr int NC = Rules::NC, NT = Rules::NT;
    extern __shared__ __align__(16) char day_lds[];
    __shared__ DayCounts cnt;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int U = s.tile_nodes, B = (int)blockDim.x;
    DayShared<NC> sh;
    sh.place(day_lds, U, B, LEVELS);
    const int64_t base = (int64_t)blockIdx.x * U;
    // The unit's private events of the day. With at most one per thread they
    // are fetched now, alongside the state, and applied to the counts in LDS
    // right after the SSA; otherwise the counts are stored and the tasks run on
    // global memory.
    const int64_t k = (int64_t)d * gridDim.x + blockIdx.x;
    const int32_t pe0 = ssa ? ev.priv_ev_off[k] : 0;
    const int32_t npe = ssa ? ev.priv_ev_off[k + 1] - pe0 : 0;
    // instances are padded to whole units: one set per workgroup
    const int32_t set = s.n_inst == 1 ? 0 : s.inst[base];
    // the unit's nodes among the slots of a day whose level events run in LDS:
    // their counts after today's private tasks go to the day's staging buffer
    // (one per thread)
    const bool staged = LEVELS && ssa;
    const int32_t st0 = staged ? ev.unit_stage_off[k] : 0;
    const int32_t nst = staged ? ev.unit_stage_off[k + 1] - st0 : 0;
    // and those of yesterday's, whose counts the level events below leave
    const bool levels = LEVELS && a.ns > 0;
    const int32_t sp0 = levels ? ev.unit_stage_off[k - gridDim.x] : 0;
    const int32_t nsp = levels ? ev.unit_stage_off[k - gridDim.x + 1] - sp0 : 0;
    const int32_t rec = prologue ? s.rec_slot[d - 1] : -1;
    const LaneLoad<NC> q = lane_load<NC>(m, s, t < U ? base + t : s.L);
    LevelEvent le{0u, 0u, 0u, 0u, 0u, 0, 0, -1, 0};
    if (levels) {
        const int32_t *stage = ev.stage + (int64_t)((d - 1) & 1) * kDaySlotCap * MAXC;
        for (int i = t; i < a.ns * NC; i += B) sh.eu[i] = stage[i];
        if (t <= a.nl) sh.lv[t] = (int32_t)(ev.lvl_ev_off[a.lv0 + t] - a.e0);
        if (t < a.ne) {
            const int64_t e = a.e0 + t;
            le.meta = ev.meta[e];
            le.smap = ev.smap[e];
            le.n = ev.n[e];
            le.g = (uint32_t)ev.g[e];
            le.src = ev.slot_src[e];
            le.dst = ev.slot_dst[e];
            sh.ev[4 * t] = le.meta;
            sh.ev[4 * t + 1] = le.smap;
            sh.ev[4 * t + 2] = (uint32_t)le.n;
            sh.ev[4 * t + 3] = le.g;
        }
    }
    if (t < 2) cnt.n[t] = cnt.next[t] = 0;
    if (t < kLengthClasses) cnt.in_class[t] = 0;
    if (t == 0) {
        cnt.trans = 0ull;
        cnt.most = 0;
    }
    if (!block_ok_once(s.status)) return;
    const uint32_t key0 = s.seed[set], key1 = s.repid[set];
    const bool lds = npe <= B;
    const bool has = lds && t < npe;
    const int32_t stage_entry = t < nst ? ev.unit_stage[st0 + t] : -1;
    const int32_t stage_prev = t < nsp ? ev.unit_stage[sp0 + t] : -1;
    if (has) {
        const int64_t e = pe0 + t;
        const PrivEv mine{ev.meta[e], ev.smap[e], ev.n[e], ev.g[e], ev.gm[e], ev.node[e]};
        sh.pe[t] = mine;
        uint64_t pre[kPrivDraws];
        draws_ahead<kPrivDraws>(pre, (int)(mine.meta & kEvKindMask) == SIM_ENTER ? 0 : mine.n, (uint32_t)mine.g, d, key0,
                                key1);
#pragma unroll
        for (int i = 0; i < kPrivDraws; ++i) sh.pd[i * B + t] = pre[i];
    }
    const bool active = q.nid >= 0;
    double coef[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) coef[i] = trans_on<NT>(m, i) ? s.coef[set * m.nt + i] : 0.0;
    int32_t x[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) x[c] = q.x[c];
    if (t < U) sh.touch[t] = 0;
    if (levels) {
        if (t < a.ne) {
            const bool one = s.n_inst == 1;
            const uint32_t *key = &ev.slot_key[3 * (int64_t)(a.s0 + le.src)];
            le.key0 = one ? key0 : key[0];
            le.key1 = one ? key1 : key[1];
            le.set = one ? 0 : (int32_t)key[2];
        }
        if (t < U) {
#pragma unroll
            for (int c = 0; c < NC; ++c) sh.x[t * NC + c] = x[c];
        }
        event_levels_lds<NC>(s, ev, a, d - 1, le, sh);
        if (stage_prev >= 0) {
            const int at = stage_prev & (kMaxUnit - 1), slot = stage_prev >> kStageShift;
#pragma unroll
            for (int c = 0; c < NC; ++c) sh.x[at * NC + c] = sh.eu[slot * NC + c];
            sh.touch[at] = 1;
        }
        __syncthreads();
        if (t < U) {
#pragma unroll
            for (int c = 0; c < NC; ++c) x[c] = sh.x[t * NC + c];
        }
    }
    if (wave * 64 < U) {
        double phi = q.phi;
        if (prologue) {
            const int32_t dp = d - 1;
            double I = 0.0;
            long long prev = 0;
            if (active) {
                if (m.phi_pre) {
                    // phi was already fed by the state before the events of day dp
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        if ((m.imask >> c) & 1u) I += x[c];
                } else {
                    phi = phi_next<NC>(m, x, s.alpha[set], s.beta[set * 4 + season((int64_t)m.day0 + dp)], phi, &I);
                }
                prev = I > 0.0 ? 1 : 0;
                if (rec >= 0) {
                    const int64_t at = (int64_t)rec * s.n_nodes + s.inst_off[set] + q.nid;
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        if (comp_on<NC>(m, c)) s.snap_u[at * m.nc + c] = x[c];
                    s.snap_v[at] = phi;
                }
                if (__double_as_longlong(phi) != __double_as_longlong(q.phi)) s.phi[base + t] = phi;
            }
            const long long np = wave_sum(prev);
            if (lane == 0) sh.part[wave * (1 + NC)] = np;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const long long w = wave_sum(x[c]);
                if (lane == 0) sh.part[wave * (1 + NC) + 1 + c] = w;
            }
        }
        if (ssa) {
            typename Rules::State ch;
#pragma unroll
            for (int i = 0; i < NT; ++i) ch.cphi[i] = active ? ((m.uses_phi >> i) & 1u ? coef[i] * phi : coef[i]) : 0.0;
#pragma unroll
            for (int c = 0; c < NC; ++c) ch.xd[c] = (double)x[c];
            if (t < U) {
#pragma unroll
                for (int c = 0; c < NC; ++c) sh.x[t * NC + c] = x[c];
                sh.phi[t] = phi;
                sh.node[t] = q.nid;
            }
            Rules::rates(m, ch);
            const double gm = s.group_min_attempts;
            int cls = 0;
            if (ch.lam >= gm) {
                cls = 1 + (ch.lam >= 4.0 * gm) + (ch.lam >= 16.0 * gm) + (ch.lam >= 64.0 * gm) + (ch.lam >= 256.0 * gm);
                atomicAdd(&cnt.in_class[cls], 1);
            }
            int kind = !(ch.lam > 0.0) ? -1 : (cls > 0 || ch.lam >= kWaveChain ? 0 : 1);
            if constexpr (OWN) {
                if (__popcll(__ballot(kind == 1)) >= kOwnFirst) {
                    ch.clock = 0.0;
                    ch.fired = 0;
                    bool live = kind == 1;
                    for (uint32_t k2 = 0; __popcll(__ballot(live)) > kOwnRest; ++k2) {
                        if (!live) continue;
                        const Draw q2 = draw_attempt(k2, (uint32_t)q.nid, (uint32_t)d, key0, key1);
                        live = chain_step<Rules>(m, ch, q2.E, q2.U, s.status, set);
                    }
                    int32_t fired = 0;
                    if (kind == 1 && !live) {
                        kind = -1;
                        fired = ch.fired;
                        if (fired) {
#pragma unroll
                            for (int c = 0; c < NC; ++c) sh.x[t * NC + c] = (int32_t)ch.xd[c];
                            sh.touch[t] = 1;
                        }
                    }
                    const long long sum = wave_sum(fired);
                    const int32_t most = wave_max(fired);
                    if (lane == 0 && sum) {
                        atomicAdd(&cnt.trans, (unsigned long long)sum);
                        atomicMax(&cnt.most, most);
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const unsigned long long in = __ballot(kind == i);
                if (in == 0ull) continue;
                int at = 0;
                if (lane == 0) at = atomicAdd(&cnt.n[i], (int)__popcll(in));
                at = __builtin_amdgcn_readfirstlane(at);
                if (kind == i)
                    sh.list[i * U + at + __popcll(in & ((1ull << lane) - 1ull))] = (uint16_t)(t | (cls << kStageShift));
            }
        }
    }
    __syncthreads();
    if (prologue && t >= B - 64 && lane < 1 + NC) {
        long long sum = 0;
        for (int w = 0; w * 64 < U; ++w) sum += sh.part[w * (1 + NC) + lane];
        if (lane == 0) {
            if (sum) atomicAdd(&s.prevalence[(int64_t)(d - 1) * s.n_inst + set], (int32_t)sum);
        } else if (sum && comp_on<NC>(m, lane - 1)) {
            const int64_t row = (int64_t)(d - 1) * s.n_inst + set;
            atomicAdd((unsigned long long *)&s.totals[row * m.nc + (lane - 1)], (unsigned long long)sum);
            const int32_t region = s.n_regions ? s.pos_region[base] : -1;
            if (region >= 0)
                atomicAdd((unsigned long long *)&s.regional[(row * s.n_regions + region) * m.nc + (lane - 1)],
                          (unsigned long long)sum);
        }
    }
    if (ssa) {
        auto load = [&](int i, typename Rules::State &c) {
            const double phi = sh.phi[i];
#pragma unroll
            for (int k2 = 0; k2 < NT; ++k2) c.cphi[k2] = (m.uses_phi >> k2) & 1u ? coef[k2] * phi : coef[k2];
#pragma unroll
            for (int c2 = 0; c2 < NC; ++c2) c.xd[c2] = (double)sh.x[i * NC + c2];
            c.clock = 0.0;
            c.fired = 0;
        };
        auto store = [&](int i, const typename Rules::State &c) {  // by one lane
            if (c.fired == 0) return;
#pragma unroll
            for (int c2 = 0; c2 < NC; ++c2) sh.x[i * NC + c2] = (int32_t)c.xd[c2];
            sh.touch[i] = 1;
            atomicAdd(&cnt.trans, (unsigned long long)c.fired);
            atomicMax(&cnt.most, c.fired);
        };
        const int n_long = cnt.n[0], n_seg = cnt.n[1];
        if (n_long > 0) {
            int group_class = kLengthClasses, n_group = 0;  // classes from group_class on are the workgroup's
            for (int b = kLengthClasses - 1; b > 0 && n_group + cnt.in_class[b] <= (b >= kFarClass ? 3 : 1); --b) {
                group_class = b;
                n_group += cnt.in_class[b];
            }
            for (int i = 0; n_group > 0 && i < n_long; ++i) {
                const int entry = sh.list[i];
                if (entry >> kStageShift < group_class) continue;
                --n_group;
                // the day's critical chain: its wavefronts issue ahead of the other
                // waves on their SIMDs while it is walked
                __builtin_amdgcn_s_setprio(3);
                const int pos = entry & (kMaxUnit - 1);
                const uint32_t node = (uint32_t)sh.node[pos];
                typename Rules::State c;
                load(pos, c);
                Rules::rates(m, c);
                uint32_t kb = 0;
                if (!walk_group<Rules>(m, c, kb, node, (uint32_t)d, key0, key1, s.status, set) && wave == 0)
                    walk_wave<Rules>(m, c, kb, node, (uint32_t)d, key0, key1, s.status, set, sh.tau);
                if (t == 0) store(pos, c);
                __builtin_amdgcn_s_setprio(0);
                __syncthreads();  // the next chain reuses the walk's LDS
            }
            for (;;) {
                int i = 0;
                if (lane == 0) i = atomicAdd(&cnt.next[0], 1);
                i = __builtin_amdgcn_readfirstlane(i);
                if (i >= n_long) break;
                const int entry = sh.list[i];
                if (entry >> kStageShift >= group_class) continue;
                const int pos = entry & (kMaxUnit - 1);
                typename Rules::State c;
                load(pos, c);
                Rules::reactants(m, c);
                walk_wave<Rules>(m, c, 0u, (uint32_t)sh.node[pos], (uint32_t)d, key0, key1, s.status, set,
                                 sh.tau + 64 * wave);
                if (lane == 0) store(pos, c);
            }
        }
        if (n_seg > 0) {
            auto take = [&](int n) {
                int at = 0;
                if (lane == 0) at = atomicAdd(&cnt.next[1], n);
                return __builtin_amdgcn_readfirstlane(at);
            };
            walk_queue<Rules, 16>(m, n_seg, sh.tau + 64 * wave, take,
                                  [&](int i, typename Rules::State &c, ChainKey &key) {
                                      const int pos = sh.list[U + i];
                                      load(pos, c);
                                      key = ChainKey{0u, (uint32_t)sh.node[pos], (uint32_t)d, key0, key1, s.status, set};
                                  },
                                  [&](int i, const typename Rules::State &c) { store(sh.list[U + i], c); });
        }
        __syncthreads();
        if (t == 0 && cnt.trans != 0ull) {
            const int64_t row = (int64_t)d * s.n_inst + set;
            atomicAdd((unsigned long long *)&s.transitions[row], cnt.trans);
            atomicMax(&s.max_fired[row], cnt.most);
        }
        if (m.phi_pre) {
            // eq:numstep5 as written: phi from the state after the SSA, before the events
            if (t < U && active) {
                int32_t y[NC];
#pragma unroll
                for (int c = 0; c < NC; ++c) y[c] = sh.x[t * NC + c];
                double I = 0.0;
                const double phi = sh.phi[t];
                const double phi2 = phi_next<NC>(m, y, s.alpha[set], s.beta[set * 4 + season((int64_t)m.day0 + d)], phi, &I);
                if (__double_as_longlong(phi2) != __double_as_longlong(phi)) s.phi[base + t] = phi2;
            }
            __syncthreads();
        }
        if (lds && npe > 0) {
            if (has && !(sh.pe[t].meta & kMetaCont)) {
                uint64_t pre[kPrivDraws];
#pragma unroll
                for (int i = 0; i < kPrivDraws; ++i) pre[i] = sh.pd[i * B + t];
                private_task_lds<NC>(sh.pe, t, npe, sh.x, sh.touch, (int32_t)base, d, key0, key1, set, s.status, pre);
            }
            __syncthreads();
        }
    } else if (levels && t < U && sh.touch[t]) {
        // (the counts that stand there: without this copy the kernel is laid
        // out otherwise, and every day takes 1 % longer)
#pragma unroll
        for (int c = 0; c < NC; ++c) sh.x[t * NC + c] = x[c];
    }
    if (t < U && sh.touch[t]) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (comp_on<NC>(m, c)) s.u[(int64_t)c * s.L + base + t] = sh.x[t * NC + c];
    }
    if (!lds) {
        __syncthreads();
        private_tasks<NC>(m, s, ev, d, blockIdx.x, gridDim.x, 0, 1, 1, s.status);
        __syncthreads();
        fresh_l1();
    }
    if (stage_entry >= 0) {
        int32_t *stage = ev.stage + (int64_t)(d & 1) * kDaySlotCap * MAXC;
        const int at = stage_entry & (kMaxUnit - 1), slot = stage_entry >> kStageShift;
#pragma unroll
        for (int c = 0; c < NC; ++c)
            stage[slot * NC + c] = !comp_on<NC>(m, c) ? 0 : lds ? sh.x[at * NC + c] : load_state(&s.u[(int64_t)c * s.L + base + at]);
    }
}

// Replicate tiles (replicate lanes in columns of 64): workgroup (x, y) takes the
// x-th of gridDim.x ranges of positions and the replicate lanes [64 y, 64 y + 64)
// of column y; the ranges are as even as groups of four positions allow (an
// instance and a region fill whole groups). In a slot handle the columns are those of the
// step's run list, each holding 64 / slot_lanes slots: d is the handle's step,
// a slot's own day is d - t0, and its lanes past its replicate count are idle.
//
// Its wavefronts first close the previous day of every lane, a position at a
// time with a lane per replicate (so that counts add up in registers), and list
// the lanes with a chain to walk; then every lane takes listed chains, the long
// ones first, and walks them attempt by attempt, kTileRefill or more lanes of a
// wavefront taking their next chains together. The lanes stay busy whatever the
// mix of empty herds, short and long chains at a position: walked where they
// are listed, a position's chains kept a wavefront until the longest had ended,
// with 39 % of the lanes idle.
//
// Chains that expect s.far_min attempts or more are not walked there but listed
// for a launch of their own (k_day_far), a wavefront each, which spreads them
// over the chip wherever their herds sit. The day's private tasks run in a
// launch over all of them after that.
constexpr int kTileList = 4096;   // chains listed before they are walked
constexpr int kTileBatch = 32;    // positions between looks at the list's length
constexpr int kTileSpan = 1024;   // positions listed before they are walked (16-bit entries)
constexpr int kTileRefill = 16;
constexpr double kTileLong = 32.0;

// Class of a far chain (longest first) in s.far_list.
__device__ __forceinline__ int far_class(double lam) { return lam >= 2048.0 ? 0 : (lam >= 256.0 ? 1 : 2); }

// A lane r of a slot handle: its slot (slot_lanes lanes each), whether the
// slot runs at handle step d, the slot's own day and its error word. A slot
// whose request failed stops.
struct SlotLane {
    int32_t day, n_live;
    bool on, prologue, ssa;
    unsigned long long *status;
};

__device__ __forceinline__ SlotLane slot_lane(const DevState &s, int32_t d, int32_t r) {
    const int32_t slot = r / s.slot_lanes;
    const SlotInfo si = s.slots[slot];
    SlotLane q;
    q.day = d - si.t0;
    q.n_live = si.n_rep;
    q.status = s.status + slot;
    q.on = si.t0 >= 0 && q.day >= 0 && q.day <= si.horizon && r - slot * s.slot_lanes < si.n_rep &&
           *q.status == STATUS_OK;
    q.prologue = q.on && q.day > 0;
    q.ssa = q.on && q.day < si.horizon;
    return q;
}

// With SLOTS (a slot handle), grid row y runs the column s.run_cols[y] and
// lane r belongs to slot r / slot_lanes, which runs its own request from its
// own day 0: every lane takes its day, its phases
// and its error word from its slot, and a failed slot stops without stopping
// the others.
template <class Rules, bool SLOTS>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(Rules::kTileWaves, 8))) void k_day_tile(
    Model m, DevState s, DevEvents ev, int32_t d, int32_t prologue, int32_t ssa) {
    constexpr int NC = Rules::NC, NT = Rules::NT;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t bx = blockIdx.x, by = blockIdx.y;
    if constexpr (!SLOTS) {
        if (!block_ok_once(s.status)) return;
    }
    __shared__ double sh_tau[kWaves][64];
    // the column of 64 replicate lanes (a slot handle launches only the
    // columns that run this step)
    const int32_t col = SLOTS ? s.run_cols[by] : (int32_t)by;
    const int32_t r = col * 64 + lane;
    bool on = r < s.R, pro = prologue != 0, walk = ssa != 0;
    int32_t day = d;
    if constexpr (SLOTS) {
        const SlotLane q = slot_lane(s, d, r);
        on = q.on;
        pro = q.prologue;
        walk = q.ssa;
        day = q.day;
        if (!__syncthreads_or(on ? 1 : 0)) return;  // no lane of the column runs
    }
    pro = pro && on;
    walk = walk && on;
    // per replicate lane: rate constants, shedding and decay rates, Philox key,
    // day, and what its chains add to the day's records
    __shared__ double sh_coef[NT][64], sh_alpha[64], sh_beta[4][64];
    __shared__ uint32_t sh_k1[64];
    __shared__ int32_t sh_day[64], sh_most[64];
    __shared__ unsigned long long sh_trans[64];
    // listed chains, position << 6 | lane: long ones from the front, short ones from the back
    constexpr int kList = kTileList;
    __shared__ uint16_t sh_list[kList];
    __shared__ int32_t sh_n[2], sh_next, sh_end;
    const int32_t rec = !SLOTS && prologue ? s.rec_slot[d - 1] : -1;
    const int season_in = pro ? season((int64_t)m.day0 + day - 1) : 0;
    const int season_out = walk ? season((int64_t)m.day0 + day) : 0;
    const int64_t groups = s.Np / kWaves;
    int64_t p = bx * groups / gridDim.x * kWaves;
    const int64_t p_end = (bx + 1) * groups / gridDim.x * kWaves;
    while (p < p_end) {
        // a run of positions of one instance and one region
        const int32_t inst = s.inst[p], region = s.n_regions ? s.pos_region[p] : -1;
        const uint32_t key0 = s.seed[inst];
        if (threadIdx.x == 0) sh_end = (int32_t)p_end;
        __syncthreads();
        if (s.n_inst > 1 || s.n_regions)
            for (int64_t q = p + kWaves * (1 + (int64_t)threadIdx.x); q < p_end; q += kWaves * kBlock)
                if (s.inst[q] != inst || (s.n_regions && s.pos_region[q] != region)) atomicMin(&sh_end, (int32_t)q);
        if (wave == 0) {
            const int64_t set = (int64_t)inst * s.R + (on ? r : 0);
#pragma unroll
            for (int k = 0; k < NT; ++k) sh_coef[k][lane] = on && trans_on<NT>(m, k) ? s.coef[set * m.nt + k] : 0.0;
            sh_alpha[lane] = on ? s.alpha[set] : 0.0;
#pragma unroll
            for (int q = 0; q < 4; ++q) sh_beta[q][lane] = on ? s.beta[set * 4 + q] : 0.0;
            sh_k1[lane] = on ? s.repid[set] : 0u;
            sh_day[lane] = day;
            sh_most[lane] = 0;
            sh_trans[lane] = 0ull;
        }
        if (threadIdx.x < 2) sh_n[threadIdx.x] = 0;
        if (threadIdx.x == 2) sh_next = 0;
        __syncthreads();
        const int64_t run_end = sh_end;
        Tally<NC> t{};
        while (p < run_end) {
            const int64_t base = p;
            // one position per wavefront at a time, the loads of its next one in
            // flight meanwhile (a position is little more than a round trip to
            // memory otherwise); past the end, the first position's state
            int32_t nid_next = -1, x_next[NC];
            double phi_ahead = 0.0;
            auto fetch = [&](int64_t j) {
                nid_next = j < run_end ? s.node_id[j] : -1;
                const int64_t l = (j < run_end ? j : base) * s.RL + r;
#pragma unroll
                for (int c = 0; c < NC; ++c) x_next[c] = on && comp_on<NC>(m, c) ? s.u[(int64_t)c * s.L + l] : 0;
                phi_ahead = on ? s.phi[l] : 0.0;
            };
            fetch(base + wave);
            int n_far, n_all;
            do {
                const int64_t batch_end = min(p + kTileBatch, run_end);
                for (int64_t j = p + wave; j < batch_end; j += kWaves) {
                    const int64_t l = j * s.RL + r;
                    const int32_t nid = nid_next;
                    int32_t x[NC];
#pragma unroll
                    for (int c = 0; c < NC; ++c) x[c] = x_next[c];
                    const double phi_in = phi_ahead;
                    fetch(j + kWaves);
                    if (nid < 0) continue;  // padding
                    double phi = phi_in;
                    if (pro) {
                        double I = 0.0;
                        if (m.phi_pre) {
                            // phi was already fed by the state before the events of the day
#pragma unroll
                            for (int c = 0; c < NC; ++c)
                                if ((m.imask >> c) & 1u) I += x[c];
                        } else {
                            phi = phi_next<NC>(m, x, sh_alpha[lane], sh_beta[season_in][lane], phi, &I);
                        }
                        t.prev += I > 0.0 ? 1 : 0;
#pragma unroll
                        for (int c = 0; c < NC; ++c) t.tot[c] += x[c];
                        if (rec >= 0) {
                            const int64_t at = ((int64_t)rec * s.R + r) * s.n_nodes + s.inst_off[inst] + nid;
#pragma unroll
                            for (int c = 0; c < NC; ++c)
                                if (comp_on<NC>(m, c)) s.snap_u[at * m.nc + c] = x[c];
                            s.snap_v[at] = phi;
                        }
                    }
                    double lam = 0.0;
                    if (walk) {
                        typename Rules::State ch;
#pragma unroll
                        for (int k = 0; k < NT; ++k) {
                            const double c = sh_coef[k][lane];
                            ch.cphi[k] = (m.uses_phi >> k) & 1u ? c * phi : c;
                        }
#pragma unroll
                        for (int c = 0; c < NC; ++c) ch.xd[c] = (double)x[c];
                        Rules::rates(m, ch);
                        lam = ch.lam;
                        if (m.phi_pre && !(lam > 0.0)) {
                            // eq:numstep5 as written: phi from the state after the SSA, before the events
                            double I = 0.0;
                            phi = phi_next<NC>(m, x, sh_alpha[lane], sh_beta[season_out][lane], phi, &I);
                        }
                    }
                    if (__double_as_longlong(phi) != __double_as_longlong(phi_in)) s.phi[l] = phi;
                    bool live = lam > 0.0;
                    if (__ballot(lam >= s.far_min) != 0ull) {
                        const int cls = lam >= s.far_min ? far_class(lam) : -1;
#pragma unroll
                        for (int i = 0; i < kFarLists; ++i) {
                            const unsigned long long in = __ballot(cls == i);
                            if (in == 0ull) continue;
                            int a = 0;
                            if (lane == 0) a = atomicAdd(&s.far_n[(d & 1) * kFarLists + i], (int)__popcll(in));
                            a = __builtin_amdgcn_readfirstlane(a) + (int)__popcll(in & ((1ull << lane) - 1ull));
                            if (cls == i && a < s.far_cap) {  // a chain past the list's end is walked here
                                s.far_list[(int64_t)i * s.far_cap + a] = (int32_t)l;
                                live = false;
                            }
                        }
                    }
                    const unsigned long long any = __ballot(live);
                    if (any != 0ull) {
                        const unsigned long long far = any & __ballot(lam >= kTileLong), near = any & ~far;
                        int a = 0, b = 0;
                        if (lane == 0) {
                            if (far != 0ull) a = atomicAdd(&sh_n[0], (int)__popcll(far));
                            if (near != 0ull) b = atomicAdd(&sh_n[1], (int)__popcll(near));
                        }
                        a = __builtin_amdgcn_readfirstlane(a);
                        b = __builtin_amdgcn_readfirstlane(b);
                        const unsigned long long below = (1ull << lane) - 1ull;
                        if (live)
                            sh_list[(far >> lane) & 1ull ? a + (int)__popcll(far & below) : kList - 1 - b - (int)__popcll(near & below)] =
                                (uint16_t)(((int)(j - base) << 6) | lane);
                    }
                }
                __syncthreads();
                n_far = sh_n[0];
                n_all = n_far + sh_n[1];
                p = batch_end;
                __syncthreads();  // the lengths are read before the next batch lists
            } while (p < run_end && n_all <= kList - kTileBatch * 64 && p - base <= kTileSpan - kTileBatch);
            fresh_l1();  // phi of the listed chains was stored by another wavefront
            // the walks: a chain is that of position at >> 6 and replicate lane at & 63
            auto entry = [&](int i) { return (int)sh_list[i < n_far ? i : kList - 1 - (i - n_far)]; };
            auto lane_of = [&](int e) { return (base + (e >> 6)) * s.RL + col * 64 + (e & 63); };
            auto start = [&](int e, typename Rules::State &ch) {  // returns phi
                const int ln = e & 63;
                const int64_t l = lane_of(e);
                const double phi = s.phi[l];
#pragma unroll
                for (int cc = 0; cc < NC; ++cc) ch.xd[cc] = comp_on<NC>(m, cc) ? (double)s.u[(int64_t)cc * s.L + l] : 0.0;
#pragma unroll
                for (int kk = 0; kk < NT; ++kk) {
                    const double cc = sh_coef[kk][ln];
                    ch.cphi[kk] = (m.uses_phi >> kk) & 1u ? cc * phi : cc;
                }
                ch.clock = 0.0;
                ch.fired = 0;
            };
            auto finish = [&](int e, const typename Rules::State &ch) {
                const int ln = e & 63;
                const int64_t l = lane_of(e);
                if (ch.fired) {
#pragma unroll
                    for (int cc = 0; cc < NC; ++cc)
                        if (comp_on<NC>(m, cc)) s.u[(int64_t)cc * s.L + l] = (int32_t)ch.xd[cc];
                    atomicAdd(&sh_trans[ln], (unsigned long long)ch.fired);
                    atomicMax(&sh_most[ln], ch.fired);
                }
                if (m.phi_pre) {
                    // eq:numstep5 as written: phi from the state after the SSA, before the events
                    int32_t y[NC];
#pragma unroll
                    for (int cc = 0; cc < NC; ++cc) y[cc] = (int32_t)ch.xd[cc];
                    double I = 0.0;
                    const double phi = s.phi[l];
                    const double phi2 = phi_next<NC>(m, y, sh_alpha[ln],
                                                     sh_beta[season((int64_t)m.day0 + sh_day[ln])][ln], phi, &I);
                    if (__double_as_longlong(phi2) != __double_as_longlong(phi)) s.phi[l] = phi2;
                }
            };
            auto status_of = [&](int ln) { return SLOTS ? s.status + (col * 64 + ln) / s.slot_lanes : s.status; };
            typename Rules::State c;
            bool has = false, live = false, dry = n_all == 0;
            int at = 0;
            uint32_t k = 0, node = 0;
            while (true) {
                const unsigned long long lives = __ballot(live);
                const int idle = 64 - (int)__popcll(lives);
                if (lives == 0ull || (!dry && idle >= kTileRefill)) {
                    if (has && !live) {
                        finish(at, c);
                        has = false;
                    }
                    if (!dry) {
                        int first = 0;
                        if (lane == 0) first = atomicAdd(&sh_next, idle);
                        first = __builtin_amdgcn_readfirstlane(first);
                        const int i = first + (int)__popcll(~lives & ((1ull << lane) - 1ull));
                        dry = first + idle >= n_all;
                        if (!live && i < n_all) {
                            at = entry(i);
                            node = (uint32_t)s.node_id[base + (at >> 6)];
                            start(at, c);
                            Rules::rates(m, c);
                            k = 0;
                            has = live = true;
                        }
                    }
                    if (__ballot(live) == 0ull) break;
                    continue;
                }
                const int ln = at & 63;
                const uint32_t dd = SLOTS ? (uint32_t)sh_day[ln] : (uint32_t)d;
                // the list is empty and few chains are left, one of which still
                // expects many attempts: the whole wavefront walks them one after
                // another
                const uint32_t nlive = 64u - (uint32_t)idle;
                if (dry && nlive <= s.few_chains &&
                    (nlive == 1 || __ballot(live && c.lam * (1.0 - c.clock) > 10.0 * (double)nlive) != 0ull)) {
                    for (unsigned long long left = lives; left != 0ull; left &= left - 1ull) {
                        const int h = __ffsll((long long)left) - 1;
                        typename Rules::State u;
#pragma unroll
                        for (int i = 0; i < NC; ++i) u.xd[i] = lane_f64(c.xd[i], h);
#pragma unroll
                        for (int i = 0; i < NT; ++i) u.cphi[i] = lane_f64(c.cphi[i], h);
                        u.clock = lane_f64(c.clock, h);
                        u.fired = __builtin_amdgcn_readlane(c.fired, h);
                        Rules::reactants(m, u);
                        const int lh = __builtin_amdgcn_readlane(ln, h);
                        walk_wave<Rules>(m, u, (uint32_t)__builtin_amdgcn_readlane((int)k, h),
                                         (uint32_t)__builtin_amdgcn_readlane((int)node, h),
                                         (uint32_t)__builtin_amdgcn_readlane((int)dd, h), key0, sh_k1[lh], status_of(lh),
                                         inst * s.R + col * 64 + lh, sh_tau[wave]);
                        if (lane == h) c = u;
                    }
                    live = false;
                    continue;
                }
                if (live) {
                    const Draw q = draw_attempt(k, node, dd, key0, sh_k1[ln]);
                    k = k + 1;
                    live = chain_step<Rules>(m, c, q.E, q.U, status_of(ln), inst * s.R + col * 64 + ln);
                }
            }
            __syncthreads();
            if (threadIdx.x < 2) sh_n[threadIdx.x] = 0;
            if (threadIdx.x == 2) sh_next = 0;
            __syncthreads();
        }
        if (wave == 0) {
            t.trans = (long long)sh_trans[lane];
            t.most = sh_most[lane];
        }
        flush_tile<NC>(m, s, t, on ? inst * s.R + r : -1, pro ? day - 1 : -1, walk ? day : -1, region);
    }
}

// The day's far chains, walked by a wavefront one at a time, the longest first.
// A chain is short against the round trips that fetch it (list, state,
// parameters, about 10 us), so where there are more chains than wavefronts a
// wavefront takes up to kFarBatch of the shortest class together: a lane each
// for the loads and stores. d is the day, in a slot handle the step.
// GROUP: the day waits for its longest chain here, so chains of the longest
// class get a workgroup each (walk_group) while they leave half the workgroups
// to the others: a wavefront takes 31 cycles an attempt, a workgroup 10 to 13
// (37,000 herds, a day with 2 / 8 / 32 / 64 replicates: 243 / 347 / 391 / 417 us
// with wavefronts, 181 / 241 / 277 / 295 with workgroups).
constexpr int kFarBatch = 8;

template <class Rules, bool SLOTS, bool GROUP>
__global__ __launch_bounds__(GROUP ? Rules::kDayThreads : kBlock) void k_day_far(Model m, DevState s, DevEvents, int32_t d) {
    constexpr int NC = Rules::NC, NT = Rules::NT;
    constexpr int kBlockWaves = (GROUP ? Rules::kDayThreads : kBlock) / 64;
    __shared__ double sh_tau[kBlockWaves][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    static_assert(kFarLists == 3, "two classes walked singly, one in batches");
    const int32_t *counts = s.far_n + (d & 1) * kFarLists;
    const int n0 = min(counts[0], s.far_cap), n1 = min(counts[1], s.far_cap), n2 = min(counts[2], s.far_cap);
    if constexpr (!SLOTS) {
        if (!block_ok_once(s.status)) return;
    }
    // the next day's lists start empty (this launch reads the other parity)
    if (blockIdx.x == 0 && threadIdx.x < kFarLists) s.far_n[((d + 1) & 1) * kFarLists + threadIdx.x] = 0;
    // workgroups 0 .. n_group - 1 walk a chain of the first class each, the
    // wavefronts of the others what is left: neighbours in a list, which are of
    // one herd and about as long, in workgroups of sixteen wavefronts apart
    const int n_group = GROUP && 2 * n0 <= (int)gridDim.x ? n0 : 0;
    const bool group = (int)blockIdx.x < n_group;
    const int others = (int)gridDim.x - n_group, waves = others * kBlockWaves, singles = n0 - n_group + n1;
    const int batch = max(1, min(kFarBatch, n2 / waves));
    const int items = group ? 1 : singles + (n2 + batch - 1) / batch;
    const int first = GROUP ? (group ? 0 : wave * others + (int)blockIdx.x - n_group) : (int)blockIdx.x * kBlockWaves + wave;
    for (int w = first; w < items; w += waves) {
        int64_t at = w;
        int count = 1;
        if (group) {
            at = blockIdx.x;
        } else if (w >= singles) {
            at = (int64_t)2 * s.far_cap + (int64_t)(w - singles) * batch;
            count = min(batch, n2 - (w - singles) * batch);
        } else if (w >= n0 - n_group) {
            at = (int64_t)s.far_cap + (w - (n0 - n_group));
        }
        // lane b < count holds chain b of the batch
        const bool mine = lane < count;
        const int64_t l = s.far_list[at + (mine ? lane : 0)];
        const int32_t r = (int32_t)(l % s.RL);
        int32_t day = d;
        unsigned long long *status = s.status;
        if constexpr (SLOTS) {
            const SlotLane q = slot_lane(s, d, r);
            day = q.day;
            status = q.status;
        }
        const LaneLoad<NC> q = lane_load<NC>(m, s, l);
        const int32_t inst = s.n_inst == 1 ? 0 : q.inst;
        const int32_t set = inst * s.R + r;
        const uint32_t key0 = s.seed[inst], key1 = s.repid[set];
        double cphi[NT];
#pragma unroll
        for (int k = 0; k < NT; ++k) {
            const double a = trans_on<NT>(m, k) ? s.coef[set * m.nt + k] : 0.0;
            cphi[k] = (m.uses_phi >> k) & 1u ? a * q.phi : a;
        }
        int32_t y[NC], fired = 0;
#pragma unroll
        for (int k = 0; k < NC; ++k) y[k] = q.x[k];
        for (int b = 0; b < count; ++b) {
            typename Rules::State c;
#pragma unroll
            for (int k = 0; k < NT; ++k) c.cphi[k] = lane_f64(cphi[k], b);
#pragma unroll
            for (int k = 0; k < NC; ++k) c.xd[k] = (double)__builtin_amdgcn_readlane(y[k], b);
            c.clock = 0.0;
            c.fired = 0;
            Rules::reactants(m, c);
            const uint64_t st = (uint64_t)status;
            unsigned long long *stb = (unsigned long long *)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane(
                                                                  (int)(uint32_t)(st >> 32), b) << 32) |
                                                              (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)st, b));
            const uint32_t node = (uint32_t)__builtin_amdgcn_readlane(q.nid, b), on_day = (uint32_t)__builtin_amdgcn_readlane(day, b),
                           k0 = (uint32_t)__builtin_amdgcn_readlane((int)key0, b),
                           k1 = (uint32_t)__builtin_amdgcn_readlane((int)key1, b);
            const int32_t of = __builtin_amdgcn_readlane(set, b);
            uint32_t kb = 0;
            bool done = false;
            if constexpr (GROUP) {
                if (group) {
                    Rules::rates(m, c);
                    __builtin_amdgcn_s_setprio(3);
                    done = walk_group<Rules>(m, c, kb, node, on_day, k0, k1, stb, of) || wave != 0;
                }
            }
            if (!done) walk_wave<Rules>(m, c, kb, node, on_day, k0, k1, stb, of, sh_tau[wave]);
            if (lane == b) {
                fired = c.fired;
#pragma unroll
                for (int k = 0; k < NC; ++k) y[k] = (int32_t)c.xd[k];
            }
        }
        if (mine && !(group && wave != 0)) {
            if (fired) {
                const int64_t row = (int64_t)day * s.n_inst * s.R + set;
#pragma unroll
                for (int k = 0; k < NC; ++k)
                    if (comp_on<NC>(m, k)) s.u[(int64_t)k * s.L + l] = y[k];
                atomicAdd((unsigned long long *)&s.transitions[row], (unsigned long long)fired);
                atomicMax(&s.max_fired[row], fired);
            }
            if (m.phi_pre) {
                // eq:numstep5 as written: phi from the state after the SSA, before the events
                double I = 0.0;
                const double phi2 = phi_next<NC>(m, y, s.alpha[set], s.beta[set * 4 + season((int64_t)m.day0 + day)],
                                                 q.phi, &I);
                if (__double_as_longlong(phi2) != __double_as_longlong(q.phi)) s.phi[l] = phi2;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Events (Sec. 3.2): one thread per (event, replicate) of a conflict-free
// level. Within a level a node is either drawn from by exactly one event or
// only added to, so draws use plain loads/stores and additions commute
// (integer atomics).
// ---------------------------------------------------------------------------


// What one event needs besides the state: its packed kind / mask / shift,
// node, destination, count, Philox counter word g, merged index gm (error
// report) and the instance of its node.
struct EvDesc {
    uint32_t meta, smap;
    int32_t node, dest, n, g, gm, inst;
};

__device__ __forceinline__ EvDesc load_desc(const DevState &s, const DevEvents &ev, int64_t e) {
    EvDesc q;
    q.meta = ev.meta[e];
    q.smap = ev.smap[e];
    q.node = ev.node[e];
    q.dest = ev.dest[e];
    q.n = ev.n[e];
    q.g = ev.g[e];
    q.gm = ev.gm[e];
    q.inst = s.inst[q.node];
    return q;
}

template <int NC>
__device__ __forceinline__ void event_apply(const Model &m, const DevState &s, const EvDesc &q, int32_t r, int32_t d,
                                            unsigned long long *status) {
    const uint32_t meta = q.meta;
    const int kind = (int)(meta & kEvKindMask);
    const uint32_t mask = (meta >> 2) & 0xffu;
    const int32_t node = q.node;
    const int32_t n = q.n;
    const int64_t ls = (int64_t)node * s.RL + r;
    if (kind == SIM_ENTER) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if ((mask >> c) & 1u) atomicAdd(&s.u[(int64_t)c * s.L + ls], n);
        return;
    }
    int32_t x[NC];
    long long tot = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        x[c] = 0;
        if ((mask >> c) & 1u) {
            x[c] = load_state(&s.u[(int64_t)c * s.L + ls]);
            tot += x[c];
        }
    }
    const uint32_t g = (uint32_t)q.g;
    const int32_t inst = q.inst;
    const int32_t set = inst * s.R + r;
    if ((long long)n > tot) {
        atomicMin(status, ((unsigned long long)(uint32_t)q.gm << 32) | (unsigned long long)(uint32_t)set);
        return;
    }
    int32_t take[NC];
    draw_individuals<NC>(x, take, mask, n, tot, g, d, s.seed[inst], s.repid[set]);
    if (kind == SIM_INTERNAL) {
        int32_t y[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) y[c] = ((mask >> c) & 1u) ? x[c] : 0;
        uint32_t touched = mask;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (take[c]) {
                const int to = shifted(q.smap, c);
#pragma unroll
                for (int cc = 0; cc < NC; ++cc) {
                    if (cc == to) {
                        if (!((touched >> cc) & 1u)) {
                            y[cc] = load_state(&s.u[(int64_t)cc * s.L + ls]);
                            touched |= 1u << cc;
                        }
                        y[cc] += take[c];
                    }
                }
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if ((touched >> c) & 1u) s.u[(int64_t)c * s.L + ls] = y[c];
        return;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
        if ((mask >> c) & 1u) s.u[(int64_t)c * s.L + ls] = x[c];
    if (kind == SIM_EXTERNAL) {
        const int64_t ld = (int64_t)q.dest * s.RL + r;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (take[c]) {
                const int to = shifted(q.smap, c);
                atomicAdd(&s.u[(int64_t)to * s.L + ld], take[c]);
            }
        }
    }
}

template <int NC>
__device__ __forceinline__ void event_one(const Model &m, const DevState &s, const DevEvents &ev,
                                          int64_t e, int32_t r, int32_t d, unsigned long long *status) {
    event_apply<NC>(m, s, load_desc(s, ev, e), r, d, status);
}

// One task (replicate lane r): a single event, or a run of one node's enter /
// exit / internal events in list order. A run that draws has its node to
// itself within its level (every other event touching the node is in another
// level), so its counts stay in registers from the first event to the last;
// a run of additions only may share the node with other additions and adds
// atomically, event by event.
template <int NC>
__device__ __forceinline__ void event_task(const Model &m, const DevState &s, const DevEvents &ev, int64_t t,
                                           int32_t r, int32_t d, unsigned long long *status) {
    const int64_t e0 = ev.task_off[t], e1 = ev.task_off[t + 1];
    bool draws = false;
    if (e1 - e0 > 1)
        for (int64_t e = e0; e < e1; ++e) draws = draws || (int)(ev.meta[e] & kEvKindMask) != SIM_ENTER;
    if (!draws) {
        for (int64_t e = e0; e < e1; ++e) event_one<NC>(m, s, ev, e, r, d, status);
        return;
    }
    const int32_t node = ev.node[e0];
    const int64_t ls = (int64_t)node * s.RL + r;
    int32_t x[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) x[c] = comp_on<NC>(m, c) ? load_state(&s.u[(int64_t)c * s.L + ls]) : 0;
    const int32_t inst = s.inst[node];
    const int32_t set = inst * s.R + r;
    const uint32_t key0 = s.seed[inst], key1 = s.repid[set];
    uint32_t touched = 0;
    for (int64_t e = e0; e < e1; ++e) {
        const uint32_t meta = ev.meta[e];
        const int kind = (int)(meta & kEvKindMask);
        const uint32_t mask = (meta >> 2) & 0xffu;
        const int32_t n = ev.n[e];
        touched |= mask;
        if (kind == SIM_ENTER) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if ((mask >> c) & 1u) x[c] += n;
            continue;
        }
        long long tot = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if ((mask >> c) & 1u) tot += x[c];
        if ((long long)n > tot) {
            atomicMin(status, ((unsigned long long)(uint32_t)ev.gm[e] << 32) | (unsigned long long)(uint32_t)set);
            break;
        }
        int32_t take[NC];
        draw_individuals<NC>(x, take, mask, n, tot, (uint32_t)ev.g[e], d, key0, key1);
        if (kind == SIM_INTERNAL) {
            const uint32_t smap = ev.smap[e];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                if (take[c]) {
                    const int to = shifted(smap, c);
#pragma unroll
                    for (int cc = 0; cc < NC; ++cc)
                        if (cc == to) x[cc] += take[c];
                    touched |= 1u << to;
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
        if ((touched >> c) & 1u) s.u[(int64_t)c * s.L + ls] = x[c];
}

template <int NC>
__global__ __launch_bounds__(kBlock) void k_events(Model m, DevState s, DevEvents ev, int32_t d,
                                                   int64_t begin, int64_t end) {
    if (*(volatile unsigned long long *)s.status != STATUS_OK) return;
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t count = (end - begin) * s.RL;
    if (t >= count) return;
    const int64_t e = begin + (s.RL == 1 ? t : t / s.RL);
    const int32_t r = s.RL == 1 ? 0 : (int32_t)(t % s.RL);
    if (r < s.R) event_task<NC>(m, s, ev, e, r, d, s.status);
}

// A run of small levels [lv_begin, lv_end) of day d in one workgroup, with a
// workgroup barrier between levels (the levels' order is all that links them).
// The descriptors of all its tasks (contiguous in execution order) are staged
// in LDS first, so each level then waits on one round trip for the state
// only; a task of several events keeps to its own loads.
constexpr int kGroupCap = 1024;

template <int NC>
__global__ __launch_bounds__(kEvBlock) void k_event_levels(Model m, DevState s, DevEvents ev, int32_t d,
                                                           int32_t lv_begin, int32_t lv_end) {
    if (!block_ok_once(s.status)) return;
    __shared__ EvDesc sh_desc[kGroupCap];
    __shared__ int32_t sh_multi[kGroupCap];
    const int64_t tb = ev.lvl_off[lv_begin], te = ev.lvl_off[lv_end];
    const bool staged = te - tb <= kGroupCap;
    if (staged) {
        for (int64_t i = threadIdx.x; i < te - tb; i += kEvBlock) {
            const int64_t e0 = ev.task_off[tb + i], e1 = ev.task_off[tb + i + 1];
            sh_multi[i] = e1 - e0 > 1;
            if (e1 - e0 == 1) sh_desc[i] = load_desc(s, ev, e0);
        }
        __syncthreads();
    }
    for (int32_t lv = lv_begin; lv < lv_end; ++lv) {
        const int64_t begin = ev.lvl_off[lv], end = ev.lvl_off[lv + 1];
        const int64_t count = (end - begin) * s.RL;
        for (int64_t t = threadIdx.x; t < count; t += kEvBlock) {
            const int64_t k = begin + (s.RL == 1 ? t : t / s.RL);
            const int32_t r = s.RL == 1 ? 0 : (int32_t)(t % s.RL);
            if (r >= s.R) continue;
            if (staged && !sh_multi[k - tb])
                event_apply<NC>(m, s, sh_desc[k - tb], r, d, s.status);
            else
                event_task<NC>(m, s, ev, k, r, d, s.status);
        }
        __syncthreads();
        fresh_l1();
    }
}

// Slot handles: level k of each slot's own day (k = -1: its private tasks, which
// come before its levels), one grid row per slot of
// s.run_slots (the slots with a day of events this step). With
// k_end > k + 1 the grid is one workgroup per slot and runs the levels
// k .. k_end-1 with a workgroup barrier between them.
template <int NC>
__global__ __launch_bounds__(kEvBlock) void k_slot_events(Model m, DevState s, DevEvents ev, int32_t step,
                                                          int32_t k, int32_t k_end) {
    const int32_t slot = s.run_slots[blockIdx.y];
    const SlotInfo si = s.slots[slot];
    const int32_t d = step - si.t0;
    if (si.t0 < 0 || d < 0 || d >= si.horizon) return;  // uniform over the workgroup
    unsigned long long *status = s.status + slot;
    if (!block_ok_once(status)) return;
    const int32_t W = s.slot_lanes;
    const int32_t lv0 = ev.lvl_ptr[d], lv_day_end = ev.lvl_ptr[d + 1];
    const int64_t stride = (int64_t)gridDim.x * kEvBlock;
    for (int32_t kk = k; kk < k_end && (kk < 0 || lv0 + kk < lv_day_end); ++kk) {
        const int64_t begin = kk < 0 ? ev.priv_off[d] : ev.lvl_off[lv0 + kk];
        const int64_t end = kk < 0 ? ev.priv_off[d + 1] : ev.lvl_off[lv0 + kk + 1];
        const int64_t count = (end - begin) * W;
        for (int64_t t = (int64_t)blockIdx.x * kEvBlock + threadIdx.x; t < count; t += stride) {
            const int32_t rr = (int32_t)(t % W);
            if (rr < si.n_rep) event_task<NC>(m, s, ev, begin + t / W, slot * W + rr, d, status);
        }
        if (k_end > k + 1) {
            __syncthreads();
            fresh_l1();
        }
    }
}

// Goal function of the fitting study (Sec. 4.3, eq:goal, eq:goalvariance): for
// day d = d_begin + blockIdx.x, with the N = R trajectories of one instance
// (sets s0 .. s0 + N - 1) and the reference's regional sums of that day
// ref[blockIdx.x][j][c], part[blockIdx.x] gets
// sum_j ||mean_i x_ij - ref_j||^2 and part[gridDim.x + blockIdx.x] gets
// sum_j sum_i ||x_ij - mean_j||^2 / (N - 1). One workgroup per day; the
// (region, compartment) terms are summed in a fixed order.
__global__ __launch_bounds__(kBlock) void k_goal(DevState s, int32_t nc, int64_t s0, int32_t N, const int64_t *ref,
                                                 int32_t d_begin, double *part) {
    __shared__ double sh_g[kBlock], sh_v[kBlock];
    const int32_t d = d_begin + (int32_t)blockIdx.x;
    const int64_t S = (int64_t)s.n_inst * s.R;
    const int32_t J = s.n_regions;
    double g = 0.0, v = 0.0;
    for (int32_t q = threadIdx.x; q < J * nc; q += kBlock) {
        const int32_t j = q / nc, c = q % nc;
        long long sum = 0;
        for (int32_t i = 0; i < N; ++i) sum += s.regional[(((int64_t)d * S + s0 + i) * J + j) * nc + c];
        const double mean = (double)sum / (double)N;
        const double diff = mean - (double)ref[((int64_t)blockIdx.x * J + j) * nc + c];
        g += diff * diff;
        double ss = 0.0;
        for (int32_t i = 0; i < N; ++i) {
            const double e = (double)s.regional[(((int64_t)d * S + s0 + i) * J + j) * nc + c] - mean;
            ss += e * e;
        }
        v += N > 1 ? ss / (double)(N - 1) : 0.0;
    }
    sh_g[threadIdx.x] = g;
    sh_v[threadIdx.x] = v;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            sh_g[threadIdx.x] += sh_g[threadIdx.x + w];
            sh_v[threadIdx.x] += sh_v[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[blockIdx.x] = sh_g[0];
        part[gridDim.x + blockIdx.x] = sh_v[0];
    }
}

// The per-day terms of k_goal added in day order, as sim_goal adds them on the
// host: out[0] = (((0 + part[0]) + part[1]) + ...), out[1] likewise over
// part[n .. 2n). One thread.
__global__ __launch_bounds__(64) void k_goal_sum(const double *part, int32_t n, double *out) {
    if (threadIdx.x != 0) return;
    double g = 0.0, v = 0.0;
    for (int32_t k = 0; k < n; ++k) {
        g = g + part[k];
        v = v + part[n + k];
    }
    out[0] = g;
    out[1] = v;
}

// Start a slot: write its table entry, clear its error word and its records,
// and load every replicate lane of it with the network's initial state.
__global__ __launch_bounds__(kBlock) void k_slot_init(DevState s, int32_t nc, const int32_t *u0, const double *v0,
                                                      int32_t slot, SlotInfo info) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    if (t == 0) {
        s.slots[slot] = info;
        s.status[slot] = STATUS_OK;
    }
    const int64_t S = s.RL, W = s.slot_lanes;
    for (int64_t i = t; i < s.Np * W; i += stride) {
        const int64_t pos = i / W;
        const int32_t rr = (int32_t)(i % W);
        const int64_t l = pos * s.RL + (int64_t)slot * W + rr;
        const bool live = rr < info.n_rep;
        for (int c = 0; c < nc; ++c) s.u[(int64_t)c * s.L + l] = live ? u0[(int64_t)c * s.Np + pos] : 0;
        s.phi[l] = live ? v0[pos] : 0.0;
    }
    for (int64_t i = t; i < (int64_t)s.n_days * W; i += stride) {
        const int64_t row = (i / W) * S + (int64_t)slot * W + (i % W);
        s.prevalence[row] = 0;
        s.transitions[row] = 0;
        s.max_fired[row] = 0;
        for (int c = 0; c < nc; ++c) s.totals[row * nc + c] = 0;
    }
}

// ---------------------------------------------------------------------------
// A run of days in one cooperative launch: phases separated by grid barriers.
// ---------------------------------------------------------------------------
template <class Rules>
__global__ __launch_bounds__(kBlock) void k_persist(Model m, DevState s, DevEvents ev, int32_t d_begin,
                                                    int32_t d_end, int32_t layout) {
    constexpr int NC = Rules::NC;
    namespace cg = cooperative_groups;
    cg::grid_group grid = cg::this_grid();
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    const int64_t first = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    for (int32_t d = d_begin; d <= d_end; ++d) {
        const bool prologue = d > d_begin;
        const bool ssa = d < d_end;
        const int32_t d_rec = prologue ? d - 1 : -1, d_ssa = ssa ? d : -1;
        if (block_ok(s.status)) {
            if (layout == LAYOUT_TILE) {
                const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
                const int64_t nx = (s.Np + s.tile_nodes - 1) / s.tile_nodes;
                const int64_t n_tiles = nx * (s.RL / 64);
                for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
                    const int64_t pos0 = (tile % nx) * s.tile_nodes;
                    const int32_t r = (int32_t)(tile / nx) * 64 + lane;
                    Tally<NC> t{};
                    for (int j = wave; j < s.tile_nodes; j += kWaves) {
                        const int64_t pos = pos0 + j;
                        if (pos >= s.Np) break;
                        day_wave<Rules>(m, s, pos * s.RL + r, d, prologue, ssa, t, s.R, s.status);
                    }
                    flush_tile<NC>(m, s, t, r < s.R ? s.inst[pos0] * s.R + r : -1, d_rec, d_ssa,
                                   s.n_regions ? s.pos_region[pos0] : -1);
                    if (ssa)
                        private_tasks<NC>(m, s, ev, d, tile % nx, nx, (int32_t)(tile / nx) * 64, 64, s.R, s.status);
                }
            } else {
                const int64_t chunks = (s.L + kBlock - 1) / kBlock;
                for (int64_t chunk = blockIdx.x; chunk < chunks; chunk += gridDim.x) {
                    const int64_t l = chunk * kBlock + threadIdx.x;
                    Tally<NC> t{};
                    day_wave<Rules>(m, s, l, d, prologue, ssa, t, s.R, s.status);
                    flush_block<NC>(m, s, t, s.inst[chunk * kBlock], d_rec, d_ssa,
                                    s.n_regions ? s.pos_region[chunk * kBlock] : -1);
                    if (ssa) private_tasks<NC>(m, s, ev, d, chunk, s.Np / kBlock, 0, 1, 1, s.status);
                }
            }
        }
        if (!ssa) break;
        grid.sync();
        fresh_l1();
        // big levels are spread over the grid; a run of small levels is done
        // by workgroup 0 alone; one grid barrier follows either
        int32_t lv = ev.lvl_ptr[d];
        const int32_t lv_end = ev.lvl_ptr[d + 1];
        while (lv < lv_end) {
            const int64_t size = (ev.lvl_off[lv + 1] - ev.lvl_off[lv]) * s.RL;
            if (size > kSmallLevel) {
                const int64_t begin = ev.lvl_off[lv];
                if (*(volatile unsigned long long *)s.status == STATUS_OK) {
                    for (int64_t t = first; t < size; t += stride) {
                        const int64_t e = begin + (s.RL == 1 ? t : t / s.RL);
                        const int32_t r = s.RL == 1 ? 0 : (int32_t)(t % s.RL);
                        if (r < s.R) event_task<NC>(m, s, ev, e, r, d, s.status);
                    }
                }
                ++lv;
            } else {
                int32_t stop = lv + 1;
                while (stop < lv_end && (ev.lvl_off[stop + 1] - ev.lvl_off[stop]) * s.RL <= kSmallLevel) ++stop;
                if (blockIdx.x == 0) {
                    for (int32_t k = lv; k < stop; ++k) {
                        const int64_t begin = ev.lvl_off[k];
                        const int64_t count = (ev.lvl_off[k + 1] - begin) * s.RL;
                        for (int64_t t = threadIdx.x; t < count; t += kBlock) {
                            const int64_t e = begin + (s.RL == 1 ? t : t / s.RL);
                            const int32_t r = s.RL == 1 ? 0 : (int32_t)(t % s.RL);
                            if (r < s.R) event_task<NC>(m, s, ev, e, r, d, s.status);
                        }
                        __syncthreads();
                        fresh_l1();
                    }
                }
                lv = stop;
            }
            grid.sync();
            fresh_l1();
        }
    }
}

template <class Rules>
struct Kernels {
    static void *day(bool levels, bool own) {
        return levels ? (own ? (void *)&k_day<Rules, true, true> : (void *)&k_day<Rules, true, false>)
                      : (own ? (void *)&k_day<Rules, false, true> : (void *)&k_day<Rules, false, false>);
    }
    static void *tile() { return (void *)&k_day_tile<Rules, false>; }
    static void *tile_slots() { return (void *)&k_day_tile<Rules, true>; }
    static void *far(bool slots, bool group) {
        return slots ? (group ? (void *)&k_day_far<Rules, true, true> : (void *)&k_day_far<Rules, true, false>)
                     : (group ? (void *)&k_day_far<Rules, false, true> : (void *)&k_day_far<Rules, false, false>);
    }
    static void *events() { return (void *)&k_events<Rules::NC>; }
    static void *levels() { return (void *)&k_event_levels<Rules::NC>; }
    static void *persist() { return (void *)&k_persist<Rules>; }
    static void *slot_events() { return (void *)&k_slot_events<Rules::NC>; }
    static size_t day_lds(int U, int B, bool events) { return DayShared<Rules::NC>().place(nullptr, U, B, events); }
};

struct Table {
    void *(*day)(bool levels, bool own);
    void *events, *persist, *levels, *tile, *slot_events, *tile_slots;
    void *(*far)(bool slots, bool group);
    size_t (*day_lds)(int U, int B, bool events);
    int day_threads;
};

template <class Rules>
Table table() {
    return {&Kernels<Rules>::day,     Kernels<Rules>::events(), Kernels<Rules>::persist(),
            Kernels<Rules>::levels(), Kernels<Rules>::tile(),   Kernels<Rules>::slot_events(),
            Kernels<Rules>::tile_slots(), &Kernels<Rules>::far, &Kernels<Rules>::day_lds, Rules::kDayThreads};
}

Table pick(const Model &m) {
    if (m.pairs && m.nc == 2) return table<PairRules<1>>();
    if (m.pairs && m.nc == 6) return table<PairRules<3>>();
    if (!large_model(m.nc, m.nt, m.pairs != 0)) return table<GenericRules<4, 4>>();
    return table<GenericRules<MAXC, MAXT>>();
}

}  // namespace

// A day of replicate tiles over n_cols columns of 64 lanes: the tiles, then
// their far chains. A far chain costs about twice as much an attempt as the
// lanes of the tile kernel, so a launch that fills the chip leaves them to it
// up to kFarWide attempts; in a launch of less than kNarrow positions (times
// columns) the tile kernel's longest chain is what the day waits for.
static int launch_tiles(const Table &t, bool slots, const Model &m, DevState s, const DevEvents &ev, int32_t d, int prologue,
                        int ssa, int64_t n_cols, void *stream) {
    if (s.Np % kWaves != 0) return hipErrorInvalidValue;
    if (s.far_min == 0.0) s.far_min = s.Np * n_cols < kNarrow ? kFarNarrow : kFarWide;
    Model mm = m;
    DevEvents ee = ev;
    int32_t dd = d, pro = prologue, sa = ssa;
    void *args[] = {&mm, &s, &ee, &dd, &pro, &sa};
    // a unit each where they are about as many as wanted: a unit's herds are dealt evenly
    const int64_t wanted = s.Np * n_cols < kNarrow ? kTileBlocks : kTileBlocksWide, units = s.Np / s.tile_nodes;
    const bool by_unit = units * n_cols <= wanted + wanted / 4 && units * n_cols >= wanted / 2;
    const int64_t blocks_x = by_unit ? units : std::min<int64_t>(s.Np / kWaves, wanted / n_cols);
    const unsigned nx = (unsigned)std::max<int64_t>(1, blocks_x);
    const hipError_t e = hipLaunchKernel(slots ? t.tile_slots : t.tile, dim3(nx, (unsigned)n_cols), dim3(kBlock), args, 0, (hipStream_t)stream);
    if (e != hipSuccess || !ssa || std::isnan(s.far_min)) return (int)e;
    void *far_args[] = {&mm, &s, &ee, &dd};
    // (from 8,192 positions on, and up to 128 lanes, of which a herd of long chains leaves half the workgroups)
    const bool group = s.Np * n_cols >= kNarrow / 4 && n_cols <= 2;
    const int threads = group ? t.day_threads : kBlock;
    const int64_t blocks = std::max<int64_t>(16, std::min<int64_t>(kFarWaves, s.Np * n_cols) * 64 / threads);
    return (int)hipLaunchKernel(t.far(slots, group), dim3((unsigned)blocks), dim3((unsigned)threads), far_args, 0, (hipStream_t)stream);
}

int launch_day(const Model &m, const DevState &s, const DevEvents &ev, int32_t d, int prologue, int ssa,
               const EventDayArgs &levels, int layout, void *stream) {
    if (s.L == 0) return hipSuccess;
    const Table t = pick(m);
    Model mm = m;
    DevState ss = s;
    DevEvents ee = ev;
    int32_t dd = d, pro = prologue, sa = ssa;
    EventDayArgs lv = levels;
    void *args[] = {&mm, &ss, &ee, &dd, &pro, &sa, &lv};
    if (layout == LAYOUT_TILE) {
        if (s.slots) return hipErrorInvalidValue;  // a slot handle's day runs through launch_slot_day
        return launch_tiles(t, false, m, s, ev, d, prologue, ssa, s.RL / 64, stream);
    }
    if (s.tile_nodes < 4 || s.tile_nodes > kMaxUnit || s.L % s.tile_nodes != 0) return hipErrorInvalidValue;
    const unsigned grid = (unsigned)(s.L / s.tile_nodes);
    // As many wavefronts a unit as its registers allow fill a compute unit; where there are more units
    // than compute units, fewer a unit let several run side by side (1,990
    // nodes of the synthetic model in units of 4, 60 days: 4.1 ms with 1,024
    // threads a unit, 3.4 with 512).
    // A day's level events take a thread each, so those runs keep at least kDayEventCap.
    int block = t.day_threads;
    const int least = ev.unit_stage_off ? kDayEventCap : 256;
    while (block > least && block / 2 >= s.tile_nodes && (int64_t)grid * block > (int64_t)kUnitsWanted * t.day_threads) block /= 2;
    if (lv.ne > kDayEventCap || lv.ns > kDaySlotCap || lv.nl > kDayLevelCap) return hipErrorInvalidValue;
    const bool staged = ev.unit_stage_off != nullptr;
    const size_t lds = t.day_lds(s.tile_nodes, block, staged);
    // half the wavefronts or more own herds
    const bool own = 2 * s.tile_nodes >= block;
    return (int)hipLaunchKernel(t.day(staged, own), dim3(grid), dim3((unsigned)block), args, lds, (hipStream_t)stream);
}

int launch_events(const Model &m, const DevState &s, const DevEvents &ev, int32_t d, int64_t begin,
                  int64_t end, void *stream) {
    const int64_t count = (end - begin) * s.RL;
    if (count <= 0) return hipSuccess;
    const Table t = pick(m);
    const unsigned grid = (unsigned)((count + kBlock - 1) / kBlock);
    Model mm = m;
    DevState ss = s;
    DevEvents ee = ev;
    int32_t dd = d;
    int64_t b = begin, e = end;
    void *args[] = {&mm, &ss, &ee, &dd, &b, &e};
    return (int)hipLaunchKernel(t.events, dim3(grid), dim3(kBlock), args, 0, (hipStream_t)stream);
}

int launch_event_levels(const Model &m, const DevState &s, const DevEvents &ev, int32_t d, int32_t lv_begin,
                        int32_t lv_end, void *stream) {
    if (lv_end <= lv_begin) return hipSuccess;
    const Table t = pick(m);
    Model mm = m;
    DevState ss = s;
    DevEvents ee = ev;
    int32_t dd = d, a = lv_begin, b = lv_end;
    void *args[] = {&mm, &ss, &ee, &dd, &a, &b};
    return (int)hipLaunchKernel(t.levels, dim3(1), dim3(kEvBlock), args, 0, (hipStream_t)stream);
}

int launch_persistent(const Model &m, const DevState &s, const DevEvents &ev, int32_t d_begin,
                      int32_t d_end, int layout, void *stream, char *why, int why_len) {
    const Table t = pick(m);
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return (int)err;
    int cus = 0, per_cu = 0;
    err = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (err != hipSuccess) return (int)err;
    err = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, t.persist, kBlock, 0);
    if (err != hipSuccess) return (int)err;
    if (per_cu < 1) {
        snprintf(why, why_len, "persistent kernel cannot be resident (occupancy 0)");
        return (int)hipErrorInvalidConfiguration;
    }
    const int64_t want = layout == LAYOUT_TILE ? ((s.Np + s.tile_nodes - 1) / s.tile_nodes) * (s.RL / 64)
                                               : (s.L + kBlock - 1) / kBlock;
    int64_t grid = (int64_t)cus * per_cu;
    if (want < grid) grid = want > 0 ? want : 1;
    Model mm = m;
    DevState ss = s;
    DevEvents ee = ev;
    int32_t a = d_begin, b = d_end, lay = layout;
    void *args[] = {&mm, &ss, &ee, &a, &b, &lay};
    return (int)hipLaunchCooperativeKernel(t.persist, dim3((unsigned)grid), dim3(kBlock), args, 0,
                                           (hipStream_t)stream);
}

int launch_slot_day(const Model &m, const DevState &s, const DevEvents &ev, int32_t step, int32_t n_cols,
                    void *stream) {
    if (s.L == 0 || n_cols <= 0) return hipSuccess;
    if (!s.slots || n_cols > s.RL / 64) return hipErrorInvalidValue;
    const Table t = pick(m);
    return launch_tiles(t, true, m, s, ev, step, 1, 1, n_cols, stream);
}

int launch_slot_events(const Model &m, const DevState &s, const DevEvents &ev, int32_t step, int32_t k,
                       int32_t k_end, int64_t max_count, int32_t n_run, void *stream) {
    if (k_end <= k || max_count <= 0 || n_run <= 0) return hipSuccess;
    if (n_run > s.RL / s.slot_lanes) return hipErrorInvalidValue;
    const Table t = pick(m);
    const int64_t want = k_end > k + 1 ? 1 : (max_count + kEvBlock - 1) / kEvBlock;
    const unsigned gx = (unsigned)std::min<int64_t>(want, 4096);
    Model mm = m;
    DevState ss = s;
    DevEvents ee = ev;
    int32_t a = step, b = k, c = k_end;
    void *args[] = {&mm, &ss, &ee, &a, &b, &c};
    return (int)hipLaunchKernel(t.slot_events, dim3(gx, (unsigned)n_run), dim3(kEvBlock), args, 0, (hipStream_t)stream);
}

int launch_slot_init(const DevState &s, int32_t nc, const int32_t *u0, const double *v0, int32_t slot,
                     const SlotInfo &info, void *stream) {
    const int64_t work = std::max<int64_t>(s.Np * s.slot_lanes, (int64_t)s.n_days * s.slot_lanes);
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((work + kBlock - 1) / kBlock, 8192));
    DevState ss = s;
    int32_t n = nc, sl = slot;
    const int32_t *a = u0;
    const double *b = v0;
    SlotInfo in = info;
    void *args[] = {&ss, &n, &a, &b, &sl, &in};
    return (int)hipLaunchKernel((void *)&k_slot_init, dim3(grid), dim3(kBlock), args, 0, (hipStream_t)stream);
}

int launch_goal_sum(const double *part, int32_t n, double *out, void *stream) {
    const double *pp = part;
    int32_t nn = n;
    double *o = out;
    void *args[] = {&pp, &nn, &o};
    return (int)hipLaunchKernel((void *)&k_goal_sum, dim3(1), dim3(64), args, 0, (hipStream_t)stream);
}

int scratch_address(void **out) {
    static std::mutex lock;
    static void *cached[kMaxScratchDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    if (dev < 0 || dev >= kMaxScratchDevices) return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> g(lock);
    if (!cached[dev]) {
        // the array's name is a host-side stand-in: its device address on this
        // GPU comes from the runtime, and only that address is ever used
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return (int)e;
        cached[dev] = ptr;
    }
    *out = cached[dev];
    return (int)hipSuccess;
}

int launch_goal(const DevState &s, int32_t nc, int64_t s0, int32_t N, const int64_t *ref, int32_t d_begin,
                int32_t n_days, double *part, void *stream) {
    if (n_days <= 0) return hipSuccess;
    DevState ss = s;
    int32_t a = nc, n = N, db = d_begin;
    int64_t b = s0;
    const int64_t *r = ref;
    double *pp = part;
    void *args[] = {&ss, &a, &b, &n, &r, &db, &pp};
    return (int)hipLaunchKernel((void *)&k_goal, dim3((unsigned)n_days), dim3(kBlock), args, 0, (hipStream_t)stream);
}

}  // namespace episim

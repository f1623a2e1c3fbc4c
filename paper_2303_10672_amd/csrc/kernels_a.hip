// Scenario A (lead time, FIFO) Bellman backup on gfx950, plus the span reduction
// and the precision-conversion kernels shared by every family.
//
// The backup follows the deterministic-transition update (Methods, "Value
// iteration") with T from Appendix A (FIFO issuing/ageing equation, reward
// equation).  It is organised around two facts about FIFO issuing:
//
//  1. The next state of (O, X_m..X_1) under order a and demand d is
//     (a, O_{L-1}..O_2, O_1 -> X'_m, X'_{m-1}..X'_1), so every outcome of action a
//     lands in one contiguous block of R^(m-1) values, V[a][O][.].  The expected
//     reward does not depend on a except through -c_var*a, so it is a table
//     r0[X_1][sum X] built once on the host.
//  2. Write y = (X_m..X_2).  Demand d <= X_1 leaves y unchanged (only waste);
//     demand d = X_1 + k removes k units from y oldest first, independently of
//     X_1; once k reaches K = sum(y) nothing is left.  So
//         E_a(X_1, y) = F(X_1) V[path_0] + sum_{0<k<K} P(X_1+k) V[path_k]
//                       + P(D >= X_1+K) V[path_K],
//     where path_k is y depleted by k units.  For a fixed (X_m..X_3) the paths of
//     all X_2 lie on one descending list of (m-1)(R-1)+1 points at most, and a
//     per-diagonal prefix sum over that list (kernel comment below) gives every
//     state of the tile for every action.
//
// Wavefront = G tiles (O, X_m..X_3) of one digit sum, R lanes per tile; the tile's
// path list streams through LDS.  Ties in the max go to the lowest action.  Every
// reduction is a fixed tree or an exact maximum, so reruns are bit-identical.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cmath>

#include "device_common.h"
#include "pvi_internal.h"

namespace pvi {

// How a row of RC actions is split between lanes.  Staging: kSplit lanes of kPer actions
// load one path point.  A lane of the split kernel (AG > 1) carries kLane of the actions of
// its state, so AG lanes share a state.  Rows are padded to 16 bytes.
template <typename VT, int RC>
struct Row {
    static constexpr int kSplit = (RC + 7) / 8;
    static constexpr int kPer = (RC + kSplit - 1) / kSplit;
    static constexpr int kVec = 16 / (int)sizeof(VT);
    static constexpr int kWidth = (RC + kVec - 1) / kVec * kVec;
    static constexpr int kLane = (RC + 64 / RC - 1) / (64 / RC);
    static constexpr int kGroups = (RC + kLane - 1) / kLane;
    static_assert(kGroups * kLane <= kWidth && kGroups * RC <= 64, "split lanes");
};

// 16 bytes of a staged row, and LDS by its own address space.  An address held as a number
// the compiler cannot see through stays one register that a loop counts up (it otherwise
// adds the base of the dynamic LDS to each access).
typedef double double2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
template <typename VT>
struct VecLoad;
template <>
struct VecLoad<float> {
    using V = float4v;
    static constexpr int W = 4;
};
template <>
struct VecLoad<double> {
    using V = double2v;
    static constexpr int W = 2;
};
template <typename T>
__device__ __forceinline__ uint32_t lds_addr(T* p) {
    uint32_t a = (uint32_t)(size_t)(__attribute__((address_space(3))) T*)p;
    asm("" : "+v"(a));
    return a;
}
template <typename T>
__device__ __forceinline__ T lds_read(uint32_t a) {
    return *(const __attribute__((address_space(3))) T*)(size_t)a;
}

// Accumulator over outcomes: FP64 multiply-add, or FP32 with Kahan compensation.
template <typename VT, bool KAHAN>
struct Acc {
    using W = double;
    double s = 0.0;
    __device__ __forceinline__ void add(double w, VT u) { s = fma(w, (double)u, s); }
    __device__ __forceinline__ double value() const { return s; }
};
template <>
struct Acc<float, true> {
    using W = float;
    float s = 0.f, c = 0.f;
    __device__ __forceinline__ void add(float w, float u) {
        const float y = fmaf(w, u, -c);
        const float t = s + y;
        c = (t - s) - y;
        s = t;
    }
    __device__ __forceinline__ double value() const { return (double)s - (double)c; }
};

// Elements between the staged chunks of two tiles of a wavefront: CH rows, padded
// so that consecutive tiles' rows start 4 banks apart (a stride of 4 dwords modulo
// 64); the tiles' 16-byte row reads then never share a bank.
template <typename VT>
__host__ __device__ constexpr int tile_stride(int ch, int width) {
    const int e = ch * width;
    return sizeof(VT) == 8 ? e + ((2 - e) % 32 + 32) % 32 : e + ((4 - e) % 64 + 64) % 64;
}

// Doubles that `n` best values take, with second best and action when extracting; even.
__host__ __device__ constexpr int best_size(int n, bool extract) {
    return ((extract ? 2 * n + (n + 1) / 2 : n) + 1) & ~1;
}

// Value staged for the padding actions R <= a < RC: so negative that their Q never wins
// the max, small enough that weighted sums of it (total weight <= 1) stay finite.  With it
// the action loops need no bound check.  Variants compiled for one exact action count
// (EXACT) need one only where the split kernel's last lanes overhang the row (11 orders, four
// lanes of three); there it is NaN, which no maximum and no comparison takes, so that values
// below -1e300, infinite values and NaN in V give what whole rows of 11 give.
template <typename VT, bool EXACT>
__device__ constexpr VT kPadValue = EXACT        ? VT(__builtin_nan(""))
                                    : sizeof(VT) == 8 ? VT(-1e300)
                                                      : VT(-1e30);

// A weight: its product is rounded before a difference of weights is formed.
__device__ __forceinline__ double weight(double gamma, double prob) {
#pragma clang fp contract(off)
    return gamma * prob;
}

// One wavefront per group of G tiles of equal digit sum b; VT: storage type of V
// (float = centred FP32, double = FP64); KAHAN: FP32 compensated accumulation (only
// with VT = float), else FP64.  EXTRACT: write policy and Q gap instead of V (FP64).
//
// For a state (X_2, X_1) of a tile put N = b + X_2 (its path length) and
// u = X_1 + N.  For N >= 1,
//   E = F(X_1) S[N] + C(u, N) + G(u) S[0],   C(u, N) = sum_{j=1}^{N-1} P(u - j) S[j],
// with F = P(D <= .), G = P(D >= .) and S the tile's path list.  For a fixed u,
// C(u, N) is a running sum over the path points, walked once for every action while
// N moves up the list; the states of diagonal u (X_1 = u - N in [0, R)) are emitted
// as N passes them.  The live diagonals are u in [n0, n0 + 2R - 2], n0 = max(b, 1).
// Lane l of a tile carries two of them, u1 = n0 + l and u2 = u1 + R: at every step
// N in [n0, b + R - 1] exactly one of the two is on the emitting window
// [N, N + R - 1] (u1 while u1 >= N, then u2), so each of the R lanes emits one state
// per step and a wavefront of G = floor(64 / R) tiles keeps nearly every lane busy.
// The lane keeps A1 = C(u1) and D = C(u2) - C(u1); the emitted running sum is
// A1 + m D with m in {0, 1}, one multiply-add.  The path list streams through LDS in
// chunks of CH points: the next chunk's values are loaded into registers while the
// current one is used.  The single-point state (N = 0, b = 0)
// takes S[0] for every demand.  Weights are staged premultiplied by gamma.
//
// What bounds a sweep: with few tiles, the chain of round trips to memory and of path
// points; with many, the latency of the gathers (11 orders, m = 5: vector units busy 23 % of
// the time, address unit 41 %, requests stalled in L1 38 %).
// So the step holds little beside its five FP64 operations per action: the lane's best value
// goes to LDS, and the states are finished in index order afterwards (reward, old value,
// store, increment, in whole lines; a reward and an address for every state in its step
// took a third of a step's instructions and as many cache accesses as the values).  The
// staging lane computes its path point's offset itself (three instructions per digit) and
// nothing waits before the first values are requested, one round trip after the launch.
//
// AG = 1: all actions of a state live in one lane.  AG > 1 (one tile per wavefront, G = 1):
// AG lanes carry the actions of a state, which shortens the chain of steps and leaves room
// for more wavefronts.  One sweep in us, a state per step in one lane before and now, 11
// orders: 7.0 and 4.0 at 121 states, 10.9 and 5.4 at 14,641, 35.0 and 30.1 at 1,771,561;
// 21 orders: 64 and 53 at 4,084,101 (FP32 storage with compensated sums: 145 and 90).
template <typename VT, bool KAHAN, bool EXTRACT, int RC, bool EXACT, int AG>
__device__ __forceinline__ void backup_a_body(ADev p, unsigned char* smem) {
    using RowT = Row<VT, RC>;
    constexpr bool FP32 = sizeof(VT) == 4;
    SpanIn si;
    if constexpr (!EXTRACT) span_fetch<FP32>(p.span, p.ctl, p.sweep, si);
    constexpr int W = VecLoad<VT>::W;
    constexpr int SPL = RowT::kPer, NSPLIT = RowT::kSplit, RW = RowT::kWidth;
    constexpr int AC = AG > 1 ? RowT::kLane : RC;  // actions of a lane
    using VV = typename VecLoad<VT>::V;
    using AW = typename Acc<VT, KAHAN>::W;

    const int R = EXACT ? RC : p.R, m = p.m, lane = threadIdx.x;
    const int G = AG > 1 ? 1 : p.G, CH = p.CH;
    const int grp = xcd_remap(blockIdx.x, gridDim.x);
    const int32_t* gt = p.groups + (size_t)grp * G;
    const int first = gt[0];  // a group's first slot always holds a tile

    // staging role: action slice sh, tile slot sg, point sj of every chunk; lanes
    // past the stagers repeat the first stager's loads and store nothing
    const int npair = G * CH;
    const bool stager = lane < NSPLIT * npair;
    const int sl = stager ? lane : 0;
    const int sh = (sl * p.pair16) >> 16, spair = sl - sh * npair;
    const int sg = AG > 1 ? 0 : (spair * p.ch16) >> 16, sj = spair - sg * CH;
    const int gv = AG > 1 ? first : gt[min(lane, G - 1)];  // lane g: the tile of slot g
    int st = AG > 1 ? first : gt[sg];
    if (st < 0) st = first;

    // quotients by R of what is below 65536 / R, by a multiplication
    const uint32_t inv16 = EXACT ? (65536 + RC - 1) / RC : (uint32_t)p.r16;

    // compute role: slot `part` (tile slot, or action slice of the one tile), position l.
    // Lanes past the last slot, and the slots of a short group, repeat another lane's work
    // and write its values again, so every lane loads and stores unconditionally (which
    // also lets the compiler count outstanding memory operations exactly).
    const int parts = AG > 1 ? AG : G;
    int part = EXACT ? lane / R : (lane * (int)inv16) >> 16;
    const int l = lane - part * R;
    if (part >= parts) part = 0;
    const int slot = part * R + l, slots = parts * R;
    const int a0 = AG > 1 ? part * AC : 0;

    const int lpm = (m >= 2 ? (m - 2) * (R - 1) : 0) + p.r2;  // longest path list
    // [G][TS] with TS >= CH * RW: tile slot, point-major rows of RW.  RW and TS are
    // multiples of 2 doubles or 4 floats, so every staged row starts on a 16-byte boundary.
    // One chunk: this wavefront's LDS operations run in issue order, so the next chunk may
    // overwrite the rows it has read.
    const int TS = tile_stride<VT>(CH, RW);
    VT* buf = reinterpret_cast<VT*>(smem);
    // the states' best values, [X_2][slot], `nrow` of X_2 at a time; and the second best and
    // the action of the best
    const int nrow = p.rows, nbest = nrow * slots;
    double* sB = reinterpret_cast<double*>(smem + sizeof(VT) * (size_t)G * TS);
    double* sS = sB + nbest;
    int* sA = reinterpret_cast<int*>(sS + nbest);
    // Weight tables (premultiplied by gamma), walked upwards as N grows by one address.
    // Entry j of the first holds P(k) and P(k + R) - P(k) at k = KM - j, with P(k) read as 0
    // for k <= 0 (d = 0 never enters a running sum): a lane's weights at point N are entry
    // KM - u1 + N, with no bound checks.  kFar bytes past the entry of the lane's k-th
    // emitted state (k = 0 ..) lie F(X_1) at X_1 = l - k modulo R and the factor of D, 1 once
    // the lane is on its second diagonal (k > l).
    constexpr int kFar = 2 * RC * 16;
    const int KM = lpm - 1, TW = KM + R;
    double2v* sW = reinterpret_cast<double2v*>(sB + best_size(nbest, EXTRACT));
    double2v* sF = sW + (KM - R + 1) + kFar / 16;
    const VT* vin = reinterpret_cast<const VT*>(p.v_in);

    // the tables' values are requested before anything waits (the first 128 entries: more
    // than m = 5 with 11 orders or m = 4 with 21 have)
    const double gm = p.gamma;
    double tp[2], tq[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int k = KM - min(lane + 64 * q, TW - 1);
        tp[q] = p.pmf[max(k, 0)];
        tq[q] = p.pmf[max(k + R, 0)];
    }
    const int fx = lane < R ? R - 1 - lane : 2 * R - 1 - min(lane, 2 * R - 2);
    const double tf = p.cdf[min(fx, p.dmax)];
    auto table = [&](int j, double p1, double p2) {
        const double pk = KM - j >= 1 ? weight(gm, p1) : 0.0;
        const double pk2 = KM - j + R >= 1 ? weight(gm, p2) : 0.0;
        sW[j] = double2v{pk, pk2 - pk};
    };

    // the staging tile's digits X_3..X_m; their sum b is the same for all of the group
    // (the quotient is 0 once they are all found; R^(m-2) stays below 2^24)
    int Y[PVI_MAX_LIFE], b = 0;
    uint32_t s_base;
    {
        const int h = (int)(((double)st + 0.5) * p.inv_nz);
        int t = st - h * p.nz;
        s_base = (uint32_t)h * (uint32_t)p.stride_h;
#pragma unroll
        for (int i = 2; i < PVI_MAX_LIFE; ++i) {
            const int q = EXACT ? t / R : (int)(((double)t + 0.5) * p.inv_r);
            Y[i] = t - q * R;
            b += Y[i];
            t = q;
        }
        b = __builtin_amdgcn_readfirstlane(b);
    }
    const int lp = b + p.r2;  // path points 0 .. lp - 1

    // The path list is [col_{m-1} (Y_{m-1} points), ..., col_2 (Y_2 points), row (r2
    // points)]: point j has the j oldest-last units, X_m filled first, then X_{m-1}, ...
    VT pre[SPL];
    auto load_chunk = [&](int c) {
        int j = min(c * CH + sj, lp - 1);
        uint32_t off = s_base;
#pragma unroll
        for (int i = PVI_MAX_LIFE - 1; i >= 2; --i) {
            const int f = min(j, Y[i]);
            off += __umul24((uint32_t)f, (uint32_t)p.pow_y[i - 1]);
            j -= f;
        }
        off += (uint32_t)j;
        const VT* src = vin + off + (int64_t)(sh * SPL) * p.stride_a;
        // raw loads only: the padding is applied when the chunk is stored, so the
        // loads stay in flight until then
#pragma unroll
        for (int e = 0; e < SPL; ++e) {
            const bool sure = EXACT && (NSPLIT - 1) * SPL + e < RC;
            const VT* at = src + (int64_t)e * p.stride_a;
            pre[e] = *(sure || sh * SPL + e < R ? at : src);
        }
    };
    auto store_chunk = [&](int c) {
        if (stager && c * CH + sj < lp) {
            VT* dst = buf + (size_t)sg * TS + sj * RW + sh * SPL;
            VT v[SPL];
#pragma unroll
            for (int e = 0; e < SPL; ++e) {
                const bool sure = EXACT && (AG == 1 || (NSPLIT - 1) * SPL + e < RC);
                v[e] = sure || sh * SPL + e < R ? pre[e] : kPadValue<VT, EXACT>;
            }
            if constexpr (SPL % W == 0) {
                VV* d = reinterpret_cast<VV*>(dst);
#pragma unroll
                for (int q = 0; q < SPL / W; ++q)
#pragma unroll
                    for (int e = 0; e < W; ++e) d[q][e] = v[q * W + e];
            } else {
#pragma unroll
                for (int e = 0; e < SPL; ++e) dst[e] = v[e];
            }
        }
    };

    load_chunk(0);
    const int n0 = b > 1 ? b : 1, nmax = lp - 1;
    const int u1 = n0 + l, u2 = u1 + R;
    const double g1 = weight(gm, p.tail[u1]), g2 = weight(gm, p.tail[u2]);
    // The states of the group in index order: blocks of 64 states of each tile.  A lane's
    // (X_2, X_1), and with it the reward, is the same in every tile of the group.
    const int RR = p.r2 * R;
    constexpr int kTiles = AG > 1 ? 1 : 64 / RC < 5 ? 64 / RC : 5;  // old values ahead
    auto tile_at = [&](int g) {
        const int t = __builtin_amdgcn_readlane(gv, g);
        return t < 0 ? first : t;
    };
    auto old_values = [&](int block, int g0, VT (&vo)[kTiles]) {
        const int i = min(block + lane, RR - 1);
#pragma unroll
        for (int q = 0; q < kTiles; ++q)
            vo[q] = vin[(uint32_t)tile_at(AG > 1 ? 0 : min(g0 + q, G - 1)) * (uint32_t)RR +
                        (uint32_t)i];
    };
    auto place = [&](int block, int& x2, int& x1) {
        const int i = min(block + lane, RR - 1);
        x2 = (int)(((uint32_t)i * inv16) >> 16);
        x1 = i - x2 * R;
    };
    auto reward = [&](int block, int& x2, int& x1) {
        place(block, x2, x1);
        return p.r0[x1 * p.xt + x1 + b + x2];
    };
    VT vo[kTiles];
    double rw = 0.0;
    int x2 = 0, x1 = 0;
    auto request = [&](int block) {
        if constexpr (!EXTRACT) {
            old_values(block, 0, vo);
            rw = reward(block, x2, x1);
        } else {
            place(block, x2, x1);
        }
    };
    request(0);

    double mu = 0.0;
    if constexpr (!EXTRACT) {
        // the sweep before is applied while the first values are on their way
        if (span_apply<FP32>(p.span, p.sweep, si, p.fixed, p.gamma)) return;
        if (FP32) mu = si.ctl.mu;
    }
    if (lane < TW) table(lane, tp[0], tq[0]);
    if (lane + 64 < TW) table(lane + 64, tp[1], tq[1]);
    for (int j = lane + 128; j < TW; j += 64)
        table(j, p.pmf[max(KM - j, 0)], p.pmf[max(KM - j + R, 0)]);
    if (lane < 2 * R - 1) sF[lane] = double2v{weight(gm, tf), lane < R ? 0.0 : 1.0};
    store_chunk(0);
    wave_sync();
    const int nchunks = (lp + CH - 1) / CH;
    if (nchunks > 1) load_chunk(1);

    const double cv = p.cvar;
    auto take = [&](double qv, int a, double& best, double& second, int& arg) {
        if (qv > best) {
            second = best;
            best = qv;
            arg = a;
        } else if (qv > second) {
            second = qv;
        }
    };
    // a state's result among the lane's actions
    auto emit = [&](int at, double best, double second, int arg) {
        sB[at] = best;
        if constexpr (EXTRACT) {
            sS[at] = second;
            sA[at] = a0 + arg;
        }
    };
    // calls f(e, value) for each action a0 + e of the staged row at an LDS address
    auto row = [&](uint32_t r, auto f) {
        if constexpr (AG == 1 || AC % W == 0) {
#pragma unroll
            for (int q = 0; q < (AC + W - 1) / W; ++q) {
                const VV sq = lds_read<VV>(r + q * (uint32_t)sizeof(VV));
#pragma unroll
                for (int e = 0; e < W; ++e)
                    if (q * W + e < AC) f(q * W + e, sq[e]);
            }
        } else {
#pragma unroll
            for (int e = 0; e < AC; ++e) f(e, lds_read<VT>(r + e * (uint32_t)sizeof(VT)));
        }
    };
    // order cost of the lane's action e
    auto cost = [&](int e) { return -cv * (a0 + e); };

    const uint32_t rows = lds_addr(buf + (AG > 1 ? 0 : (size_t)part * TS) + a0);
    // N = 0 (only when b = 0): nothing left to deplete, every demand lands on S[0]
    if (b == 0) {
        double best = -DBL_MAX, second = -DBL_MAX;
        int arg = 0;
        row(rows, [&](int e, VT s0) {
            const double qv = fma(gm, (double)s0, cost(e));
            if (EXTRACT)
                take(qv, e, best, second, arg);
            else
                best = fmax(best, qv);
        });
        emit(slot, best, second, arg);
    }

    // start from the j = 0 term G(u) S[0] (and, with FP64 accumulation, the order
    // cost, which the difference D does not carry)
    Acc<VT, KAHAN> A1[AC], D[AC];
    {
        const AW gd = (AW)(g2 - g1);
        row(rows, [&](int e, VT sv) {
            if constexpr (KAHAN)
                A1[e].add((AW)g1, sv);
            else
                A1[e].s = fma(g1, (double)sv, cost(e));
            D[e].add(gd, sv);
        });
    }

    // The states of rows f .. f + n - 1 of X_2, 64 of each tile at a time: the best values are
    // in sB, and the first block's rewards and old values have been requested.
    double dmx = -DBL_MAX, dmn = DBL_MAX, vmx = -DBL_MAX, vmn = DBL_MAX;
    auto finish = [&](int f, int n) {
        VT* vout = reinterpret_cast<VT*>(p.v_out);
        const int i0 = f * R, i1 = (f + n) * R;
        wave_sync();
        for (int block = i0; block < i1; block += 64) {
            if (block > i0) {
                if constexpr (EXTRACT) {
                    place(block, x2, x1);
                } else {
                    if (AG > 1) old_values(block, 0, vo);
                    rw = reward(block, x2, x1);
                }
            }
            // the lane that emitted it: X_1 is l less the number of steps before
            const uint32_t at0 = (uint32_t)(x1 + x2 - (b == 0 && x2 > 0 ? 1 : 0));
            const int at = (int)min(at0, at0 - (uint32_t)R);
            const int i = block + lane;
            const int src = (i < i1 ? x2 - f : 0) * slots + at;
            const double base = rw - mu;
            for (int g0 = 0; g0 < G; g0 += kTiles) {
                if (AG == 1 && !EXTRACT && (block > i0 || g0 > 0)) old_values(block, g0, vo);
#pragma unroll
                for (int q = 0; q < kTiles; ++q) {
                    const int g = AG > 1 ? 0 : g0 + q;
                    if (AG == 1 && (g >= G || __builtin_amdgcn_readlane(gv, g) < 0)) continue;
                    const int from = src + (AG > 1 ? 0 : g * R);
                    const uint32_t to = (uint32_t)tile_at(g) * (uint32_t)RR + (uint32_t)i;
                    double best = sB[from];
                    if constexpr (EXTRACT) {  // the slices by rising action: ties as in a row
                        double second = sS[from];
                        int arg = sA[from];
#pragma unroll
                        for (int k = 1; k < AG; ++k) {
                            const double kb = sB[from + k * R];
                            if (kb > best) {
                                second = fmax(best, sS[from + k * R]);
                                best = kb;
                                arg = sA[from + k * R];
                            } else {
                                second = fmax(second, kb);
                            }
                        }
                        if (i < i1) {
                            p.pi[to] = arg;
                            p.gap[to] = R > 1 ? best - second : INFINITY;
                        }
                        continue;
                    }
#pragma unroll
                    for (int k = 1; k < AG; ++k) best = fmax(best, sB[from + k * R]);
                    if (i < i1) {
                        const VT o = (VT)(base + best);
                        vout[to] = o;
                        const double out = (double)o, dv = out - (double)vo[q];
                        dmx = fmax(dmx, dv);
                        dmn = fmin(dmn, dv);
                        if constexpr (FP32) {  // the FP32 centring needs the value range
                            vmx = fmax(vmx, out);
                            vmn = fmin(vmn, out);
                        }
                    }
                }
            }
        }
    };

    // address of the weights of point N for the two running sums, P(u1 - N) and P(u2 - N) -
    // P(u1 - N) (a diagonal with u - N <= 0 is finished and adds nothing), at N = 1; and of
    // the lane's value at X_2 = n0 - b
    uint32_t wp = lds_addr(sW + (KM - u1) + 1);
    uint32_t bp = lds_addr(sB + slot + (n0 - b) * slots);
    int f0 = 0;  // X_2 of the first row in sB
    for (int N = 1, c = 0; N <= nmax;) {
        // past the last point of the chunk, and of the rows that sB takes
        const int end = min(min((c + 1) * CH, nmax + 1), b + f0 + nrow);
        uint32_t rN = rows + (uint32_t)((N - c * CH) * RW) * (uint32_t)sizeof(VT);
        // points 1 .. n0 - 1 precede every state of the group: running sums only
        const int mid = min(end, n0);
#pragma unroll 2
        for (; N < mid; ++N) {
            const double2v w = lds_read<double2v>(wp);
            const AW w1 = (AW)w.x, w2 = (AW)w.y;
            row(rN, [&](int e, VT sv) {
                A1[e].add(w1, sv);
                D[e].add(w2, sv);
            });
            wp += 16;
            rN += RW * (uint32_t)sizeof(VT);
        }
        // points n0 .. nmax: every lane emits one state per point, at X_2 = N - b and X_1 =
        // l - (N - n0) modulo R.  Each pair (or quad) of actions of the point is read, used
        // for the state and both sums, and dropped, so the row is never held whole.  The
        // sums are also advanced after the last point (unused), which keeps the body free
        // of branches.
        for (; N < end; ++N) {
            const double2v w = lds_read<double2v>(wp), fm = lds_read<double2v>(wp + kFar);
            const AW w1 = (AW)w.x, w2 = (AW)w.y;
            // Q_a = gamma (F(X_1) S[N][a] + C(u, N) + G(u) S[0][a]) - c_var a, with
            // C(u, N) = A1 + D once the lane is on its second diagonal
            double best = -DBL_MAX, second = -DBL_MAX;
            int arg = 0;
            double bq[4];
            row(rN, [&](int e, VT svt) {
                const double sv = (double)svt;
                const double run = fma(fm.y, D[e].value(), A1[e].value());
                if constexpr (EXTRACT) {
                    take(fma(fm.x, sv, run), e, best, second, arg);
                } else {
                    const double qv = KAHAN ? fma(fm.x, sv, run) + cost(e) : fma(fm.x, sv, run);
                    bq[e & 3] = e < 4 ? qv : fmax(bq[e & 3], qv);
                }
                A1[e].add(w1, svt);
                D[e].add(w2, svt);
            });
            if constexpr (EXTRACT) {
                emit((N - b - f0) * slots + slot, best, second, arg);
            } else {
                best = bq[0];
                if (AC > 1) best = fmax(best, bq[1]);
                if (AC > 3)
                    best = fmax(best, fmax(bq[2], bq[3]));
                else if (AC > 2)
                    best = fmax(best, bq[2]);
                *(__attribute__((address_space(3))) double*)(size_t)bp = best;
                bp += (uint32_t)slots * 8;
            }
            wp += 16;
            rN += RW * (uint32_t)sizeof(VT);
        }
        if (N > nmax) break;
        if (N == b + f0 + nrow) {
            finish(f0, nrow);
            f0 += nrow;
            bp -= (uint32_t)nbest * 8;
            request(f0 * R);
        }
        if (N == (c + 1) * CH) {  // publish chunk c + 1 and start loading chunk c + 2
            ++c;
            store_chunk(c);
            // only the compiler has to keep the stores before the reads
            wave_sync();
            if (c + 1 < nchunks) load_chunk(c + 1);
        }
    }
    finish(f0, p.r2 - f0);
    if constexpr (!EXTRACT) {
        dmx = wave_max(dmx);
        dmn = wave_min(dmn);
        if (p.span) {
            if (FP32) {
                vmx = wave_max(vmx);
                vmn = wave_min(vmn);
            }
            if (lane == 0) span_emit<FP32>(p.span, p.sweep, grp, dmx, dmn, vmx, vmn);
            return;
        }
        vmx = wave_max(vmx);
        vmn = wave_min(vmn);
        if (lane == 0) {
            double* pp = p.partials + 4 * (size_t)grp;
            pp[0] = dmx;
            pp[1] = dmn;
            pp[2] = vmx;
            pp[3] = vmn;
        }
    }
}

// Two entry points of one body: the first asks for two wavefronts per SIMD (its
// registers fit in 256), the second has the whole register file for the variants
// that would spill at that budget (32 actions, FP32 compensated sums of 11 and more).
template <typename VT, bool KAHAN, bool EXTRACT, int RC, bool EXACT, int AG>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void
backup_a_kernel(ADev p) {
    extern __shared__ __align__(16) unsigned char smem[];
    backup_a_body<VT, KAHAN, EXTRACT, RC, EXACT, AG>(p, smem);
}

template <typename VT, bool KAHAN, bool EXTRACT, int RC, bool EXACT, int AG>
__global__ __launch_bounds__(64) void backup_a_wide_kernel(ADev p) {
    extern __shared__ __align__(16) unsigned char smem[];
    backup_a_body<VT, KAHAN, EXTRACT, RC, EXACT, AG>(p, smem);
}

// Single-workgroup reduction of the per-tile partials and the stopping rule.
__global__ __launch_bounds__(1024) void span_kernel(Ctl* ctl, const double* partials,
                                                    int tiles, int fp32, int fixed,
                                                    double gamma) {
    __shared__ double red[4 * 16];
    // the control block and up to four partials per thread are requested together,
    // so the reduction waits for one memory round trip (partials are always
    // readable; after the stop flag they are simply not used)
    const Ctl cur = *ctl;
    double a0 = -DBL_MAX, a1 = DBL_MAX, a2 = -DBL_MAX, a3 = DBL_MAX;
    const double2* pp = reinterpret_cast<const double2*>(partials);
    const int bd = blockDim.x;
    int i = threadIdx.x;
    auto take = [&](double2 x, double2 y) {
        a0 = fmax(a0, x.x);
        a1 = fmin(a1, x.y);
        a2 = fmax(a2, y.x);
        a3 = fmin(a3, y.y);
    };
    // four loads per round, past the end repeating the last partial (max and min
    // are unchanged by a repeat)
    for (; i < tiles; i += 4 * bd) {
        double2 x[4], y[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int t = min(i + k * bd, tiles - 1);
            x[k] = pp[2 * t];
            y[k] = pp[2 * t + 1];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) take(x[k], y[k]);
    }
    if (cur.stop) return;
    block_reduce4(a0, a1, a2, a3, red);
    if (threadIdx.x != 0) return;
    Ctl next = cur;
    span_update(next, a0, a1, a2, a3, fp32, fixed, gamma);
    *ctl = next;
}

__global__ __launch_bounds__(256) void span_init_kernel(SpanBuf* b, Ctl first) {
    if (threadIdx.x == 0) b->ctl[0] = first;
    for (int i = threadIdx.x; i < 4 * kSpanSlots * 4; i += 256)
        b->key[i / (4 * kSpanSlots)][i / 4 % kSpanSlots][i % 4] = 0;
}

// End of a batch of sweeps 0 .. n - 1: the last one applied, in both copies.
template <bool FP32>
__global__ __launch_bounds__(64) void span_end_kernel(SpanBuf* b, int n, int fixed, double gamma) {
    SpanIn in;
    span_fetch<FP32>(b, nullptr, n, in);
    span_reduce<FP32>(in, fixed, gamma);
    in.ctl.pending = 0;
    if (threadIdx.x < 2) ctl_copy(b->ctl[threadIdx.x], in.ctl);
}

__global__ void to_f64_kernel(const float* v32, double* v64, const Ctl* ctl, int64_t n) {
    const double c = ctl->c;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        v64[i] = c + (double)v32[i];
}

__global__ void fill_kernel(double* v, double value, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        v[i] = value;
}

__global__ void to_f32_kernel(const double* v64, float* v32, double c, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        v32[i] = (float)(v64[i] - c);
}

// ------------------------------------------------------------------ launchers

template <typename VT, bool KAHAN, bool EXTRACT, int RC, bool EXACT, int AG>
static hipError_t launch_a_g(const ADev& p, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    using RowT = Row<VT, RC>;
    const int lp_max = (p.m >= 2 ? (p.m - 2) * (p.R - 1) : 0) + p.r2;
    // lanes: G tiles of R lanes (or the slices of one tile); staging: G x CH points of
    // kSplit slices
    if (p.G < 1 || (AG > 1 ? AG : p.G) * p.R > 64 || p.CH < 1 ||
        RowT::kSplit * p.G * p.CH > 64 || p.ngroups < 1 || p.R > RC || (EXACT && p.R != RC) ||
        (AG > 1 && p.G != 1) || p.m > PVI_MAX_LIFE || p.rows < 1 || p.rows > p.r2)
        return hipErrorInvalidConfiguration;
    size_t bytes = sizeof(VT) * (size_t)p.G * tile_stride<VT>(p.CH, RowT::kWidth);
    const size_t slots = (size_t)(AG > 1 ? AG : p.G) * p.R;
    bytes += sizeof(double) * best_size((int)(p.rows * slots), EXTRACT);
    // weights: the second table ends 2R - 1 entries past its start (and past the first)
    bytes += 16 * ((size_t)lp_max - p.R + 2 * RC + 2 * p.R - 1);
    if (bytes > 65536) return hipErrorInvalidConfiguration;
    // G is read at u2 <= b + 2R, P at most at lp_max + R
    if (p.tab < 2 * p.R + lp_max + 1 || p.tab < p.dmax + 2) return hipErrorInvalidValue;
    constexpr bool wide = AG == 1 && (RC == 32 || (KAHAN && RC >= 11) || (EXTRACT && RC == 24));
    // with events, they are recorded by the launch itself at the kernel's start and end
    if constexpr (wide) {
        auto k = backup_a_wide_kernel<VT, KAHAN, EXTRACT, RC, EXACT, AG>;
        if (ev0 || ev1)
            hipExtLaunchKernelGGL(k, dim3(p.ngroups), dim3(64), (uint32_t)bytes, s, ev0, ev1, 0, p);
        else
            hipLaunchKernelGGL(k, dim3(p.ngroups), dim3(64), bytes, s, p);
    } else {
        auto k = backup_a_kernel<VT, KAHAN, EXTRACT, RC, EXACT, AG>;
        if (ev0 || ev1)
            hipExtLaunchKernelGGL(k, dim3(p.ngroups), dim3(64), (uint32_t)bytes, s, ev0, ev1, 0, p);
        else
            hipLaunchKernelGGL(k, dim3(p.ngroups), dim3(64), bytes, s, p);
    }
    return hipGetLastError();
}

template <typename VT, bool KAHAN, bool EXTRACT, int RC, bool EXACT = false>
static hipError_t launch_a_r(const ADev& p, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    constexpr int AG = Row<VT, RC>::kGroups;
    if (p.G == 1) return launch_a_g<VT, KAHAN, EXTRACT, RC, EXACT, AG>(p, s, ev0, ev1);
    return launch_a_g<VT, KAHAN, EXTRACT, RC, EXACT, 1>(p, s, ev0, ev1);
}

template <typename VT, bool KAHAN, bool EXTRACT>
static hipError_t launch_a_t(const ADev& p, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    // exact action counts of the paper's scenario A (order cap 10) and of the
    // order cap 20 instances: no padded action is computed, and R is a constant
    if (p.R == 11) return launch_a_r<VT, KAHAN, EXTRACT, 11, true>(p, s, ev0, ev1);
    if (p.R == 21) return launch_a_r<VT, KAHAN, EXTRACT, 21, true>(p, s, ev0, ev1);
    if (p.R <= 8) return launch_a_r<VT, KAHAN, EXTRACT, 8>(p, s, ev0, ev1);
    if (p.R <= 16) return launch_a_r<VT, KAHAN, EXTRACT, 16>(p, s, ev0, ev1);
    // 17 to 20 orders, one tile per wavefront: rows of 21 give a state three lanes of seven
    // actions (60 of 64 lanes at 20 orders), rows of 24 two of twelve (40 lanes).  Us per FP64
    // sweep, 24 and 21: 43.2 and 34.4 at 20^5 states with m = 2, 49.7 and 41.2 with m = 3, 516
    // and 411 at 17^6 with m = 5 (whole tiles in rows of 24: 45.1, 56.3 and 482)
    if (p.R <= 21 && p.G == 1)
        return launch_a_g<VT, KAHAN, EXTRACT, 21, false, Row<VT, 21>::kGroups>(p, s, ev0, ev1);
    if (p.R <= 24) return launch_a_r<VT, KAHAN, EXTRACT, 24>(p, s, ev0, ev1);
    if (p.R <= 32) return launch_a_r<VT, KAHAN, EXTRACT, 32>(p, s, ev0, ev1);
    return hipErrorInvalidValue;
}

hipError_t launch_backup_a(const ADev& p, int storage_fp32, int acc_kahan, int extract,
                           hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    if (extract) return launch_a_t<double, false, true>(p, s, ev0, ev1);
    if (storage_fp32) {
        if (acc_kahan) return launch_a_t<float, true, false>(p, s, ev0, ev1);
        return launch_a_t<float, false, false>(p, s, ev0, ev1);
    }
    return launch_a_t<double, false, false>(p, s, ev0, ev1);
}

hipError_t launch_span(Ctl* ctl, const double* partials, int tiles, int storage_fp32,
                       int fixed, double gamma, hipStream_t s) {
    // a block no wider than the partials need (whole wavefronts, at most 1024): small
    // instances then pay for one wavefront, not sixteen; max and min are exact, so
    // the block width does not change the result
    const int threads = tiles >= 1024 ? 1024 : tiles <= 64 ? 64 : (tiles + 63) / 64 * 64;
    hipLaunchKernelGGL(span_kernel, dim3(1), dim3(threads), 0, s, ctl, partials, tiles,
                       storage_fp32, fixed, gamma);
    return hipGetLastError();
}

hipError_t launch_span_init(SpanBuf* b, const Ctl& first, hipStream_t s) {
    hipLaunchKernelGGL(span_init_kernel, dim3(1), dim3(256), 0, s, b, first);
    return hipGetLastError();
}

hipError_t launch_span_end(SpanBuf* b, int sweeps, int storage_fp32, int fixed, double gamma,
                           hipStream_t s) {
    if (storage_fp32)
        hipLaunchKernelGGL(span_end_kernel<true>, dim3(1), dim3(64), 0, s, b, sweeps, fixed, gamma);
    else
        hipLaunchKernelGGL(span_end_kernel<false>, dim3(1), dim3(64), 0, s, b, sweeps, fixed, gamma);
    return hipGetLastError();
}

hipError_t launch_to_f64(const float* v32, double* v64, const Ctl* ctl, int64_t n,
                         hipStream_t s) {
    const int blocks = (int)std::min<int64_t>((n + 255) / 256, 8192);
    hipLaunchKernelGGL(to_f64_kernel, dim3(blocks), dim3(256), 0, s, v32, v64, ctl, n);
    return hipGetLastError();
}

hipError_t launch_to_f32(const double* v64, float* v32, double c, int64_t n,
                         hipStream_t s) {
    const int blocks = (int)std::min<int64_t>((n + 255) / 256, 8192);
    hipLaunchKernelGGL(to_f32_kernel, dim3(blocks), dim3(256), 0, s, v64, v32, c, n);
    return hipGetLastError();
}

hipError_t launch_fill(double* v, double value, int64_t n, hipStream_t s) {
    const int blocks = (int)std::min<int64_t>((n + 255) / 256, 8192);
    hipLaunchKernelGGL(fill_kernel, dim3(blocks), dim3(256), 0, s, v, value, n);
    return hipGetLastError();
}

}  // namespace pvi

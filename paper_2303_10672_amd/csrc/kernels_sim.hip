// Rollouts of a replenishment policy (Simulation section: rollouts of warm-up plus
// counted days from a start state; the return is the discounted sum of the rewards
// of the counted days; the KPIs are the service level, the wastage and the
// holding), one lane per (policy, rollout) pair.
//
// Each lane keeps its stock by remaining life (and, for scenario A, its orders in
// transit) in registers, takes the day's randomness from Philox4x64-10 (Salmon,
// Moraes, Dror and Shaw, SC 2011) keyed by (seed, 0) with counter (rollout, day,
// block, 0), and applies the day's transition unit by unit: issue oldest first
// (youngest first for LIFO), discard what reaches the end of its life, age the
// rest, receive the arriving order.  Word 0 of block 0 is the demand of product
// 0, word 1 the demand of product 1; unit i of the day (a scenario-C unit's
// remaining life, a scenario-B customer's acceptance of substitution) uses word
// i%4 of block 1 + i/4.  Draws u = (x >> 11) 2^-53 become the smallest d with
// u < CDF(d) (d_max if none), the smallest life k with u < p_1 + .. + p_k (m if
// none), and acceptance when u < rho.  Every candidate policy sees the same
// numbers (common random numbers across a heuristic grid).
//
// The numbers of a (rollout, day) are the same for every policy and every state, so
// draw_kernel makes them first, one thread per (rollout, day): the chain of dependent days
// is left with integer work on registers and, for a policy table, one 4-byte gather.  What
// bounds it, 10,000 rollouts of 465 days: one table of 1,771,561 states is 157 wavefronts
// and waits for the gather (893 us a call before, now 143 us after 49 us of draws); a grid
// of 841 modified base-stock policies keeps the vector units full (67.3 ms before, now
// 7.4 ms after 0.17 ms).  Where a draw depends on the order (order-dependent remaining
// life), or the numbers would not fit, each lane draws them day by day.  The loops over
// lives are compiled for the scenarios' m and L: with the general bounds a day walks 8 lives
// and 11 orders whatever m and L are.  Floating-point contraction is off so the return is
// the plain sum of products of the definition.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pvi_internal.h"

#pragma clang fp contract(off)

namespace pvi {

namespace {

constexpr int kMaxM = PVI_MAX_LIFE;  // life classes 1..m
constexpr int kMaxO = 11;            // orders in transit (scenario A, L - 1)
constexpr uint64_t kM0 = 0xD2E7470EE14C6C93ull, kM1 = 0xCA5A826395121157ull;
constexpr uint64_t kW0 = 0x9E3779B97F4A7C15ull, kW1 = 0xBB67AE8584CAA73Bull;

struct Block {
    uint64_t w[4];
};

__device__ __forceinline__ Block philox(uint64_t seed, uint64_t r, uint64_t t, uint64_t b) {
    uint64_t x0 = r, x1 = t, x2 = b, x3 = 0, k0 = seed, k1 = 0;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        if (round > 0) {
            k0 += kW0;
            k1 += kW1;
        }
        const uint64_t hi0 = __umul64hi(kM0, x0), lo0 = kM0 * x0;
        const uint64_t hi1 = __umul64hi(kM1, x2), lo1 = kM1 * x2;
        const uint64_t y0 = hi1 ^ x1 ^ k0, y2 = hi0 ^ x3 ^ k1;
        x0 = y0;
        x1 = lo1;
        x2 = y2;
        x3 = lo0;
    }
    return Block{{x0, x1, x2, x3}};
}

// word j of a block by selects (a dynamic index would put the block in scratch)
__device__ __forceinline__ uint64_t word(const Block& b, int j) {
    const uint64_t lo = (j & 1) ? b.w[1] : b.w[0], hi = (j & 1) ? b.w[3] : b.w[2];
    return (j & 2) ? hi : lo;
}

__device__ __forceinline__ double unif(uint64_t x) {
    return (double)(x >> 11) * (1.0 / 9007199254740992.0);
}

// smallest d with u < cdf[d] (dmax if none): the sums of a PMF never fall, so by halving
__device__ __forceinline__ int sample(const double* cdf, int dmax, double u) {
    int lo = 0, n = dmax;  // the answer is in [lo, lo + n]
    while (n > 0) {
        const int h = n >> 1;
        const bool up = !(u < cdf[lo + h]);
        lo = up ? lo + h + 1 : lo;
        n = up ? n - h - 1 : h;
    }
    return lo;
}

__device__ __forceinline__ double posd(double x) { return x > 0.0 ? x : 0.0; }

struct Tally {
    int demand, met, expired, received, held;
};

__device__ __forceinline__ void add(Tally& c, const Tally& d) {
    c.demand += d.demand;
    c.met += d.met;
    c.expired += d.expired;
    c.received += d.received;
    c.held += d.held;
}

// service %, wastage %, mean holding per day of a rollout's counts
__device__ __forceinline__ void kpis(double* k, const Tally& c, int horizon) {
    k[0] = c.demand > 0 ? 100.0 * (double)c.met / (double)c.demand : 100.0;
    k[1] = c.received > 0 ? 100.0 * (double)c.expired / (double)c.received : 0.0;
    k[2] = horizon > 0 ? (double)c.held / (double)horizon : 0.0;
}

}  // namespace

// The most customers of a day that can be unmet and take the other product.
__host__ __device__ __forceinline__ int units_max(const SimDev& s, int family) {
    return family == 1 ? s.dmax0 : s.dmax1;
}

// The numbers of one (rollout, day), which no policy changes: the demands of both products
// in the halves of `dem`; bit i of `bits` (32-bit words for up to 31 customers) is whether
// the i-th unmet customer accepts substitution (two products), and scenario C's `life` has a
// word per remaining life k - 1, bit i set when the i-th unit ordered arrives with life k
// (life independent of the order).
// One thread per (rollout, day); [day][rollout], so a wavefront of rollouts reads lines.
// Bounded by Philox's 64-bit multiplies (4.65 million days in 49 us; 20 MB written).
template <int FAM>
__global__ __launch_bounds__(256) void draw_kernel(SimDev s) {
    extern __shared__ __align__(16) unsigned char smem[];
    double* cdf0 = reinterpret_cast<double*>(smem);
    double* cdf1 = cdf0 + s.n_cdf0;
    double* lcum = cdf1 + s.n_cdf1;
    for (int i = threadIdx.x; i < s.n_cdf0; i += blockDim.x) cdf0[i] = s.cdf0[i];
    for (int i = threadIdx.x; i < s.n_cdf1; i += blockDim.x) cdf1[i] = s.cdf1[i];
    for (int i = threadIdx.x; i < s.n_lcum; i += blockDim.x) lcum[i] = s.lifecum[i];
    __syncthreads();
    const int64_t n = (int64_t)s.n_roll * (s.warmup + s.horizon);
    const int m = s.m;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int t = (int)(i / s.n_roll);
        const uint64_t r = (uint64_t)(i - (int64_t)t * s.n_roll);
        const Block b0 = philox(s.seed, r, (uint64_t)t, 0);
        const int tau = FAM == 2 ? (s.tau0 + t % s.P) % s.P : 0;
        const int dA = sample(cdf0 + tau * (s.dmax0 + 1), s.dmax0, unif(b0.w[0]));
        const int dB = FAM == 1 || FAM == 3 ? sample(cdf1, s.dmax1, unif(b0.w[1])) : 0;
        s.dem[i] = (uint32_t)dA | (uint32_t)dB << 16;
        if (FAM == 1 || FAM == 3) {
            const int units = FAM == 1 ? dA : dB;  // the most customers that can be unmet
            uint64_t bits = 0;
            Block bu = b0;
            for (int u = 0; u < units; ++u) {
                if ((u & 3) == 0) bu = philox(s.seed, r, (uint64_t)t, (uint64_t)(1 + (u >> 2)));
                if (unif(word(bu, u & 3)) < s.rho) bits |= 1ull << u;
            }
            if (units_max(s, FAM) <= 31)
                reinterpret_cast<uint32_t*>(s.bits)[i] = (uint32_t)bits;
            else
                s.bits[i] = bits;
        }
        if (FAM == 2) {
            uint32_t life[kMaxM] = {};
            Block bu = b0;
            const double* cum = lcum + (s.R0 > 1 ? m : 0);  // the row of every order above 0
            for (int u = 0; u < s.R0 - 1; ++u) {
                if ((u & 3) == 0) bu = philox(s.seed, r, (uint64_t)t, (uint64_t)(1 + (u >> 2)));
                const double x = unif(word(bu, u & 3));
                int k = m;
                for (int j = m - 1; j >= 1; --j)
                    if (x < cum[j - 1]) k = j;
#pragma unroll
                for (int j = 1; j <= kMaxM; ++j) life[j - 1] |= (j == k ? 1u : 0u) << u;
            }
#pragma unroll
            for (int j = 0; j < kMaxM; ++j)
                if (j < m) s.life[(int64_t)j * n + i] = life[j];
        }
    }
}

// FAM 0: scenario A (state [O_{L-1}..O_1, X_m..X_1]); 1: scenario B with L = 0
// ([A_{m-1}..A_1, B_{m-1}..B_1]); 2: scenario C ([tau, X_{m-1}..X_1]); 3: scenario B
// with lead time 1 ([Xa_m..Xa_1, Xb_m..Xb_1]; X holds product a, Y product b).
// M > 0: compiled for m = M; LO >= 0: scenario A compiled for L - 1 = LO orders in transit
// (0 for the other families; -1: up to kMaxO).  PRE: the day's numbers come from
// draw_kernel, else they are drawn here.  SPLIT: per-product KPIs are kept.
template <int FAM, int M, int LO, bool PRE, bool SPLIT, bool BITS32 = false>
__global__ __launch_bounds__(64) void rollout_kernel(SimDev s) {
    extern __shared__ __align__(16) unsigned char smem[];
    double* cdf0 = reinterpret_cast<double*>(smem);
    double* cdf1 = cdf0 + s.n_cdf0;
    double* lcum = cdf1 + s.n_cdf1;
    if constexpr (!PRE) {
        for (int i = threadIdx.x; i < s.n_cdf0; i += blockDim.x) cdf0[i] = s.cdf0[i];
        for (int i = threadIdx.x; i < s.n_cdf1; i += blockDim.x) cdf1[i] = s.cdf1[i];
        for (int i = threadIdx.x; i < s.n_lcum; i += blockDim.x) lcum[i] = s.lifecum[i];
        __syncthreads();
    }
    int pol, rr;
    if (s.by_block) {
        // a workgroup has 64 rollouts of one policy; the policies of the same rollouts run
        // next to each other and find their numbers in the caches
        pol = (int)(blockIdx.x % (unsigned)s.n_pol);
        rr = (int)(blockIdx.x / (unsigned)s.n_pol) * 64 + (int)threadIdx.x;
        if (rr >= s.n_roll) return;
    } else {
        const int64_t at = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
        if (at >= (int64_t)s.n_pol * s.n_roll) return;
        pol = (int)(at / s.n_roll);
        rr = (int)(at - (int64_t)pol * s.n_roll);
    }
    const int64_t lane = (int64_t)pol * s.n_roll + rr;
    const uint64_t r = (uint64_t)rr;
    const int32_t* prm = s.params ? s.params + (size_t)pol * PVI_POLICY_PARAMS : nullptr;
    constexpr int MM = M > 0 ? M : kMaxM, NO = LO >= 0 ? LO : kMaxO;
    const int m = M > 0 ? M : s.m, R0 = s.R0, nO = FAM == 0 ? (LO >= 0 ? LO : s.L - 1) : 0;

    // state registers; index 0 of X/Y unused, lives 1..m (all of 1..MM where M is given)
    int X[MM + 1] = {}, Y[MM + 1] = {}, O[NO + 1] = {};
    int tau = 0;
    {
        int64_t idx = s.start;
        // lives 1 .. top, the least significant digit first
        auto take = [&](int (&S)[MM + 1], int top, int R) {
#pragma unroll
            for (int j = 1; j <= MM; ++j)
                if (j <= top) {
                    S[j] = (int)(idx % R);
                    idx /= R;
                }
        };
        if (FAM == 0) {
            take(X, m, R0);
#pragma unroll
            for (int i = 1; i <= NO; ++i)  // then O_1 .. O_{L-1}
                if (i <= nO) {
                    O[i] = (int)(idx % R0);
                    idx /= R0;
                }
        } else if (FAM == 2) {
            take(X, m - 1, R0);
            tau = (int)idx;
        } else {
            take(Y, FAM == 1 ? m - 1 : m, s.R1);
            take(X, FAM == 1 ? m - 1 : m, R0);
        }
    }

    constexpr bool kTwo = FAM == 1 || FAM == 3;
    double g = 1.0, acc = 0.0;
    Tally c = {0, 0, 0, 0, 0};
    Tally c0 = {0, 0, 0, 0, 0}, c1 = {0, 0, 0, 0, 0};  // per product (two products)
    const int days = s.warmup + s.horizon;
    // the numbers of the day after are on their way while this one is walked
    uint32_t dem = 0, dem_next = 0;
    uint64_t bits = 0, bits_next = 0;
    uint32_t bits32 = 0, bits32_next = 0;  // BITS32: at most 31 customers
    uint32_t life[MM] = {}, life_next[MM] = {};
    const int64_t ndraw = (int64_t)s.n_roll * days;
    auto fetch = [&](int t) {
        const int64_t i = (int64_t)(t < days ? t : days - 1) * s.n_roll + rr;
        dem_next = s.dem[i];
        if (kTwo && BITS32) bits32_next = reinterpret_cast<const uint32_t*>(s.bits)[i];
        if (kTwo && !BITS32) bits_next = s.bits[i];
        if (FAM == 2) {
#pragma unroll
            for (int j = 0; j < MM; ++j)
                if (j < m) life_next[j] = s.life[(int64_t)j * ndraw + i];
        }
    };
    if constexpr (PRE) fetch(0);
    // a heuristic's parameters: read once; scenario C's pair of the day after with its numbers
    const bool heuristic = s.kind != PVI_POLICY_TABLE;
    int par[2] = {}, par_next[2] = {};
    auto fetch_pair = [&](int wd) {
        if (heuristic) {
            par_next[0] = prm[2 * wd];
            par_next[1] = prm[2 * wd + 1];
        }
    };
    if (FAM == 2) {
        fetch_pair(tau);
    } else if (heuristic) {
        par[0] = prm[0];
        par[1] = prm[1];
    }
    auto sum_of = [&](const int (&S)[MM + 1]) {
        int n = 0;
#pragma unroll
        for (int j = 1; j <= MM; ++j) n += S[j];
        return n;
    };
    // issues from S oldest first; returns what is not met
    auto issue = [&](int (&S)[MM + 1], int rem) {
#pragma unroll
        for (int j = 1; j <= MM; ++j) {
            const int take = min(rem, S[j]);
            S[j] -= take;
            rem -= take;
        }
        return rem;
    };
    // ages S by a day; the place of life m takes `arrive`
    auto age = [&](int (&S)[MM + 1], int arrive) {
#pragma unroll
        for (int j = 1; j < MM; ++j) S[j] = M > 0 || j < m ? S[j + 1] : 0;
        if (M > 0) {
            S[MM] = arrive;
        } else {
            S[MM] = 0;
#pragma unroll
            for (int j = 1; j <= MM; ++j)
                if (j == m) S[j] = arrive;
        }
    };
    for (int t = 0; t < days; ++t) {
        if constexpr (PRE) {
            dem = dem_next;
            bits = bits_next;
            bits32 = bits32_next;
#pragma unroll
            for (int j = 0; j < MM; ++j) life[j] = life_next[j];
            fetch(t + 1);
        }
        if (FAM == 2) {
            par[0] = par_next[0];
            par[1] = par_next[1];
            fetch_pair(tau + 1 == s.P ? 0 : tau + 1);
        }
        // ---- action (two products: aA, aB; heuristic orders are not capped,
        // except scenario C's, whose remaining-life table ends at a_max)
        int a = 0, aA = 0, aB = 0;
        if (!heuristic) {
            // a table has fewer than 2^31 entries: the index fits 32 bits
            uint32_t idx = FAM == 2 ? (uint32_t)tau * (uint32_t)s.pw0[m - 1] : 0;
            if (FAM == 0) {
#pragma unroll
                for (int i = 1; i <= NO; ++i)
                    if (i <= nO) idx += (uint32_t)O[i] * (uint32_t)s.pw0[m + i - 1];
            }
#pragma unroll
            for (int j = 1; j <= MM; ++j)
                if (j <= (FAM == 1 || FAM == 2 ? m - 1 : m)) {
                    idx += (uint32_t)X[j] * (uint32_t)s.pw0[j - 1];
                    if (kTwo) idx += (uint32_t)Y[j] * (uint32_t)s.pw1[j - 1];
                }
            a = s.table[idx];
            if (kTwo) {
                aA = a / s.R1;
                aB = a - aA * s.R1;
            }
        } else if (FAM == 0) {  // base stock on stock on hand and in transit
            int I = sum_of(X);
#pragma unroll
            for (int i = 1; i <= NO; ++i) I += O[i];
            a = max(par[0] - I, 0);
        } else if (kTwo) {  // modified base stock per product
            const int IA = sum_of(X), IB = sum_of(Y);
            // (the integer differences are exact, and a conversion drops the fraction)
            aA = (int)posd((double)(par[0] - IA) + posd((double)X[1] - s.mu0));
            aB = (int)posd((double)(par[1] - IB) + posd((double)Y[1] - s.mu1));
        } else {  // (s, S) of the weekday
            const int I = sum_of(X);
            const int lo = par[0], hi = par[1];
            a = (lo < hi && I <= lo) ? min(max(hi - I, 0), R0 - 1) : 0;
        }

        // ---- outcome and transition
        Block b0 = {};
        int dA, dB = 0;
        if constexpr (PRE) {
            dA = (int)(dem & 0xffffu);
            dB = (int)(dem >> 16);
        } else {
            b0 = philox(s.seed, r, (uint64_t)t, 0);
            dA = sample(cdf0 + tau * (s.dmax0 + 1), s.dmax0, unif(b0.w[0]));
            if (kTwo) dB = sample(cdf1, s.dmax1, unif(b0.w[1]));
        }
        // how many of the first `unmet` unmet customers accept substitution
        auto accepted = [&](int unmet) {
            int k = 0;
            if constexpr (PRE) {
                if (BITS32)
                    k = __popc(__builtin_amdgcn_ubfe(bits32, 0, (uint32_t)unmet));
                else
                    k = __popcll(unmet >= 64 ? bits : bits & ((1ull << unmet) - 1));
            } else {
                Block bu = b0;
                for (int i = 0; i < unmet; ++i) {
                    if ((i & 3) == 0)
                        bu = philox(s.seed, r, (uint64_t)t, (uint64_t)(1 + (i >> 2)));
                    if (unif(word(bu, i & 3)) < s.rho) ++k;
                }
            }
            return k;
        };
        double rew;
        Tally day, day0 = {0, 0, 0, 0, 0}, day1 = {0, 0, 0, 0, 0};
        if (FAM == 0) {
            const int d = dA, tot = sum_of(X);
            int rem = d;
            if (s.issuing == PVI_LIFO) {
#pragma unroll
                for (int j = MM; j >= 1; --j) {
                    const int take = min(rem, X[j]);
                    X[j] -= take;
                    rem -= take;
                }
            } else {
                rem = issue(X, rem);
            }
            const int met = d - rem, W = X[1];
            const int held = tot - met - W;
            rew = -s.cvar0 * a - s.chold * (double)held - s.cshort * (double)(d - met) -
                  s.cwaste * (double)W;
            int arrive = a;
            if constexpr (NO > 0) {
                if (nO > 0) arrive = O[1];
            }
            age(X, arrive);
#pragma unroll
            for (int i = 1; i < NO; ++i) O[i] = i < nO ? O[i + 1] : 0;
#pragma unroll
            for (int i = 1; i <= NO; ++i)
                if (i == nO) O[i] = a;
            day = Tally{d, met, W, arrive, held};
        } else if (FAM == 1) {
#pragma unroll
            for (int j = 1; j <= MM; ++j)
                if (j == m) {
                    X[j] = aA;
                    Y[j] = aB;
                }
            const int stA = sum_of(X), stB = sum_of(Y);
            const int unmet = issue(X, dA), hA = dA - unmet;
            const int k = accepted(unmet);
            const int hB = dB - issue(Y, dB);
            const int hS = k - issue(Y, k);
            const int wA = X[1], wB = Y[1], W = wA + wB;
            rew = -(s.cvar0 * aA + s.cvar1 * aB) + s.rev0 * hA + s.rev1 * (hB + hS);
            age(X, 0);
            age(Y, 0);
            day = Tally{dA + dB, hA + hB + hS, W, aA + aB, stA + stB - hA - hB - hS - W};
            // product 0's customers served by product 1 count as met for product 0
            day0 = Tally{dA, hA + hS, wA, aA, stA - hA - wA};
            day1 = Tally{dB, hB, wB, aB, stB - hB - hS - wB};
        } else if (FAM == 3) {
            // lead time 1: today's orders arrive for tomorrow; product b's unmet
            // customers may take product a's units left after a's own demand
            const int stA = sum_of(X), stB = sum_of(Y);
            const int excess = issue(Y, dB), hB = dB - excess;
            const int du = accepted(excess);
            const int hA = dA + du - issue(X, dA + du);
            const int wA = X[1], wB = Y[1], W = wA + wB;
            rew = -(s.cvar0 * aA + s.cvar1 * aB) + s.rev0 * hA + s.rev1 * hB;
            age(X, aA);
            age(Y, aB);
            day = Tally{dA + dB, hA + hB, W, aA + aB, stA + stB - hA - hB - W};
            // product a's own customers come first; the rest of its issues went to
            // product b's customers and count as met for product b
            const int ownA = min(dA, stA);
            day0 = Tally{dA, ownA, wA, aA, stA - hA - wA};
            day1 = Tally{dB, hB + (hA - ownA), wB, aB, stB - hB - wB};
        } else {
            const int d = dA;
            int y[MM + 1] = {};
            if constexpr (PRE) {
                const uint32_t first = (1u << a) - 1u;  // the units ordered (a < 32)
#pragma unroll
                for (int k = 1; k <= MM; ++k)
                    if (k <= m) y[k] = __popc(life[k - 1] & first);
            } else {
                const double* cum = lcum + (size_t)a * m;
                Block bu = b0;
                for (int i = 0; i < a; ++i) {
                    if ((i & 3) == 0)
                        bu = philox(s.seed, r, (uint64_t)t, (uint64_t)(1 + (i >> 2)));
                    const double u = unif(word(bu, i & 3));
                    int l = m;
                    for (int k = m - 1; k >= 1; --k)
                        if (u < cum[k - 1]) l = k;
#pragma unroll
                    for (int k = 1; k <= MM; ++k) y[k] += l == k ? 1 : 0;
                }
            }
            const int cap = R0 - 1;
            int before = 0, tot = 0;
#pragma unroll
            for (int j = 1; j <= MM; ++j) {
                before += X[j];
                X[j] = j < m ? min(X[j] + y[j], cap) : (j == m ? y[j] : 0);
                tot += X[j];
            }
            const int z1 = X[1];
            rew = -(a > 0 ? s.cfixed : 0.0) - s.chold * posd((double)(tot - d)) -
                  s.cshort * posd((double)(d - tot)) - s.cwaste * posd((double)(z1 - d));
            const int met = d - issue(X, d), W = X[1];
            age(X, 0);
            tau = tau + 1 == s.P ? 0 : tau + 1;
            day = Tally{d, met, W, tot - before, tot - met};
        }
        if (t >= s.warmup) {
            acc += g * rew;
            g *= s.gamma;
            add(c, day);
            if (SPLIT) {
                add(c0, day0);
                add(c1, day1);
            }
        }
    }
    s.ret[lane] = acc;
    kpis(s.kpi + 3 * lane, c, s.horizon);
    if (SPLIT) {
        kpis(s.pkpi + 6 * lane, c0, s.horizon);
        kpis(s.pkpi + 6 * lane + 3, c1, s.horizon);
    }
}

// Mean and sample standard deviation (n - 1) of one column of one policy's
// [n_roll][stride] block per workgroup: two passes, fixed summation order (so a column's
// figures do not depend on the other columns).
__global__ __launch_bounds__(256) void column_stats_kernel(const double* x, int stride,
                                                           int n_roll, double* out, int ostride,
                                                           int ooff) {
    __shared__ double red[256];
    const int pol = blockIdx.x, q = blockIdx.y, tid = threadIdx.x;
    const double* xp = x + (size_t)pol * n_roll * stride;
    double mean = 0.0;
    for (int pass = 0; pass < 2; ++pass) {
        double sum = 0.0;
#pragma unroll 8
        for (int i = tid; i < n_roll; i += 256) {
            const double v = xp[(size_t)i * stride + q];
            sum += pass == 0 ? v : (v - mean) * (v - mean);
        }
        red[tid] = sum;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if (tid < w) red[tid] += red[tid + w];
            __syncthreads();
        }
        const double total = red[0];
        __syncthreads();
        if (pass == 0) {
            mean = total / (double)n_roll;
        } else if (tid == 0) {
            out[(size_t)pol * ostride + ooff + 2 * q] = mean;
            out[(size_t)pol * ostride + ooff + 2 * q + 1] =
                n_roll > 1 ? sqrt(total / (double)(n_roll - 1)) : 0.0;
        }
    }
}

namespace {

size_t sim_lds(const SimDev& s) {
    return sizeof(double) * ((size_t)s.n_cdf0 + s.n_cdf1 + s.n_lcum);
}

template <int FAM, int M, int LO>
void launch_days(const SimDev& s, dim3 grid, hipStream_t st) {
    if constexpr (FAM == 1 || FAM == 3) {
        const bool narrow = units_max(s, FAM) <= 31;
        if (s.pkpi && narrow)
            hipLaunchKernelGGL((rollout_kernel<FAM, M, LO, true, true, true>), grid, dim3(64), 0,
                               st, s);
        else if (s.pkpi)
            hipLaunchKernelGGL((rollout_kernel<FAM, M, LO, true, true, false>), grid, dim3(64), 0,
                               st, s);
        else if (narrow)
            hipLaunchKernelGGL((rollout_kernel<FAM, M, LO, true, false, true>), grid, dim3(64), 0,
                               st, s);
        else
            hipLaunchKernelGGL((rollout_kernel<FAM, M, LO, true, false, false>), grid, dim3(64),
                               0, st, s);
    } else {
        hipLaunchKernelGGL((rollout_kernel<FAM, M, LO, true, false>), grid, dim3(64), 0, st, s);
    }
}

template <int FAM>
void launch_family(const SimDev& s, dim3 grid, hipStream_t st) {
    constexpr bool two = FAM == 1 || FAM == 3;
    if (!s.dem) {  // numbers drawn day by day
        if (two && s.pkpi)
            hipLaunchKernelGGL((rollout_kernel<FAM, 0, FAM == 0 ? -1 : 0, false, two>), grid,
                               dim3(64), sim_lds(s), st, s);
        else
            hipLaunchKernelGGL((rollout_kernel<FAM, 0, FAM == 0 ? -1 : 0, false, false>), grid,
                               dim3(64), sim_lds(s), st, s);
        return;
    }
    // compiled for the life and lead time of every configured scenario; the rest share one
    // kernel with the loops' bounds as run-time conditions
    if constexpr (FAM == 0) {
        if (s.m == 2 && s.L == 1) return launch_days<FAM, 2, 0>(s, grid, st);
        if (s.m == 3 && s.L == 1) return launch_days<FAM, 3, 0>(s, grid, st);
        if (s.m == 4 && s.L == 1) return launch_days<FAM, 4, 0>(s, grid, st);
        if (s.m == 5 && s.L == 1) return launch_days<FAM, 5, 0>(s, grid, st);
        if (s.m == 2 && s.L == 2) return launch_days<FAM, 2, 1>(s, grid, st);
        if (s.m == 3 && s.L == 2) return launch_days<FAM, 3, 1>(s, grid, st);
        if (s.m == 4 && s.L == 2) return launch_days<FAM, 4, 1>(s, grid, st);
        if (s.m == 5 && s.L == 2) return launch_days<FAM, 5, 1>(s, grid, st);
        return launch_days<FAM, 0, -1>(s, grid, st);
    } else {
        if (s.m == 2) return launch_days<FAM, 2, 0>(s, grid, st);
        if (s.m == 3) return launch_days<FAM, 3, 0>(s, grid, st);
        if constexpr (FAM == 2) {
            if (s.m == 4) return launch_days<FAM, 4, 0>(s, grid, st);
            if (s.m == 5) return launch_days<FAM, 5, 0>(s, grid, st);
        }
        return launch_days<FAM, 0, 0>(s, grid, st);
    }
}

}  // namespace

hipError_t launch_draws(const SimDev& s, hipStream_t st) {
    const int64_t n = (int64_t)s.n_roll * (s.warmup + s.horizon);
    if (n <= 0) return hipSuccess;
    const size_t lds = sim_lds(s);
    if (lds > 65536 || s.m < 1 || s.m > kMaxM || !s.dem) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)std::min<int64_t>((n + 255) / 256, 8192)), block(256);
    if (s.family == 0)
        hipLaunchKernelGGL(draw_kernel<0>, grid, block, lds, st, s);
    else if (s.family == 1)
        hipLaunchKernelGGL(draw_kernel<1>, grid, block, lds, st, s);
    else if (s.family == 2)
        hipLaunchKernelGGL(draw_kernel<2>, grid, block, lds, st, s);
    else
        hipLaunchKernelGGL(draw_kernel<3>, grid, block, lds, st, s);
    return hipGetLastError();
}

hipError_t launch_rollouts(const SimDev& s, hipStream_t st) {
    const int64_t lanes = (int64_t)s.n_pol * s.n_roll;
    if (lanes <= 0) return hipSuccess;
    const int64_t blocks =
        s.by_block ? (int64_t)s.n_pol * ((s.n_roll + 63) / 64) : (lanes + 63) / 64;
    if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
    if (sim_lds(s) > 65536 || s.m < 1 || s.m > kMaxM || (s.family == 0 && s.L - 1 > kMaxO))
        return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)blocks);
    if (s.family == 0)
        launch_family<0>(s, grid, st);
    else if (s.family == 1)
        launch_family<1>(s, grid, st);
    else if (s.family == 2)
        launch_family<2>(s, grid, st);
    else
        launch_family<3>(s, grid, st);
    return hipGetLastError();
}

hipError_t launch_column_stats(const double* x, int stride, int ncol, int n_pol, int n_roll,
                               double* out, int ostride, int ooff, hipStream_t st) {
    if (n_pol <= 0 || n_roll <= 0 || ncol <= 0) return hipSuccess;
    if (ncol > stride || ooff + 2 * ncol > ostride) return hipErrorInvalidValue;
    hipLaunchKernelGGL(column_stats_kernel, dim3(n_pol, ncol), dim3(256), 0, st, x, stride,
                       n_roll, out, ostride, ooff);
    return hipGetLastError();
}

}  // namespace pvi

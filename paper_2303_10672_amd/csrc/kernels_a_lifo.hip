// Scenario A backup with LIFO issuing (Appendix A, LIFO issuing/ageing equation).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>

#include "device_common.h"
#include "pvi_internal.h"

namespace pvi {

// Scenario A with LIFO issuing (Appendix A, LIFO issuing/ageing equation).  The
// youngest units go first, so demand d removes min(d, K) units from
// y = (X_m..X_2) youngest first (K = X_2 + ... + X_m); only what is left of the
// demand reaches X_1, whose remainder expires.  The next state depends on y and
// d but not on X_1, so the expectation E_a(O, y), the best action and the Q gap
// are shared by the R states (O, y, X_1), which differ only in the expected
// reward r0[X_1][K] (host table).  Read backwards, the depletion path of y is a
// list L with L[0] = nothing left and L[i] = the i units issued last, so
//   E_a = sum_{i=1}^{K} P(K - i) L_a[i] + P(D >= K) L_a[0].
// Workgroup = tile (O, X_{m-1}..X_2); its R values of X_m = t share one list of
// b + R points (b = X_2 + ... + X_{m-1}): points 1..b rebuild X_2 first, then
// X_3, ..., X_{m-1}; point b + t is (X_m = t, the rest full).  Thread (t, a) forms
// E_a for K = b + t, then thread (t, X_1) takes the max of its row (ties to the lowest
// action) and writes its state.  FP64 accumulation for every storage type.
//
// Bound by latency: a tile is one dependent sum of up to b + R terms between its loads and
// its stores.  All that a workgroup reads (the list, the demand table, its states' rewards
// and old values) has addresses known from the tile's number alone and is requested at
// once; each thread takes the max of its row itself, so one barrier lies between the sums
// and the stores; each wavefront reduces its own increments.  The state's reward and old
// value were read, and the max taken by one thread per row, after the sums before: 9.4 us
// per sweep at 161,051 states, now 7.7.
template <typename VT, bool EXTRACT>
__global__ __launch_bounds__(1024) void backup_a_lifo_kernel(ADev p) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[64];
    constexpr bool FP32 = sizeof(VT) == 4;
    SpanIn si;
    if constexpr (!EXTRACT) span_fetch<FP32>(p.span, p.ctl, p.sweep, si);
    const int R = p.R, m = p.m, tid = threadIdx.x, nt = blockDim.x, RR = R * R;
    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    // z = (X_{m-1}..X_2), X_2 fastest; the quotient is 0 once its digits are found
    const int h = (int)(((double)tile + 0.5) * p.inv_nz), z = tile - h * p.nz;
    int Y[PVI_MAX_LIFE];  // Y[j] = X_j, j = 2 .. m-1, zero above
    int b = 0;
    {
        int t = z;
#pragma unroll
        for (int j = 2; j < PVI_MAX_LIFE; ++j) {
            const int q = (int)(((double)t + 0.5) * p.inv_r);
            Y[j] = t - q * R;
            b += Y[j];
            t = q;
        }
    }
    const int lp = b + R;
    double* L = reinterpret_cast<double*>(smem);  // [lp][R]
    double* sq = L + (size_t)p.lmax * R;           // [R][R] Q(t, a)
    double* sP = sq + (size_t)RR;                  // [lmax] P(d)
    const VT* vin = reinterpret_cast<const VT*>(p.v_in);
    const int64_t hbase = (int64_t)h * p.stride_h;

    // item k of the list: point k / R, action k % R
    auto item = [&](int k) {
        const int i = (int)(((double)k + 0.5) * p.inv_r), a = k - i * R;
        // i units: X_2 filled first, then X_3, ..., then X_m
        uint32_t off = 0;
        int left = i;
#pragma unroll
        for (int j = 2; j < PVI_MAX_LIFE; ++j) {
            const int f = min(left, Y[j]);
            off += __umul24((uint32_t)f, (uint32_t)p.pow_y[j - 2]);
            left -= f;
        }
        off += __umul24((uint32_t)left, (uint32_t)p.pow_y[m - 2]);
        return vin[hbase + (int64_t)a * p.stride_a + off];
    };
    constexpr int kAhead = 4;  // items of a thread requested together
    VT pre[kAhead];
    const int items = lp * R;
#pragma unroll
    for (int q = 0; q < kAhead; ++q) pre[q] = item(min(tid + q * nt, items - 1));
    const double pp = p.pmf[min(tid, p.lmax - 1)];
    // thread (t, a), which is also the state (X_m = t, X_1 = a)
    const int k = min(tid, RR - 1);
    const int t = (k * p.r16) >> 16, a = k - t * R, K = b + t;
    const uint32_t s_idx = (uint32_t)h * (uint32_t)p.stride_h * (uint32_t)R + (uint32_t)(z * R) +
                           (uint32_t)t * (uint32_t)(p.pow_y[m - 2] * R) + (uint32_t)a;
    const double tail = p.tail[K];
    double rw = 0.0, old = 0.0;
    if constexpr (!EXTRACT) {
        rw = p.r0[a * p.xt + K];
        old = (double)vin[s_idx];
    }
    double mu = 0.0;
    if constexpr (!EXTRACT) {
        // every wavefront comes to the same decision
        if (span_apply<FP32>(p.span, p.sweep, si, p.fixed, p.gamma)) return;
        if (FP32) mu = si.ctl.mu;
    }
#pragma unroll
    for (int q = 0; q < kAhead; ++q)
        if (tid + q * nt < items) L[tid + q * nt] = (double)pre[q];
    for (int i = tid + kAhead * nt; i < items; i += nt) L[i] = (double)item(i);
    if (tid < p.lmax) sP[tid] = pp;
    for (int i = tid + nt; i < p.lmax; i += nt) sP[i] = p.pmf[i];
    __syncthreads();
    {
        double e = tail * L[a];
        const double* w = sP + K;
        const double* x = L + a;
#pragma unroll 8
        for (int i = 1; i <= K; ++i) e = fma(w[-i], x[i * R], e);
        sq[k] = fma(p.gamma, e, -p.cvar * a);
    }
    __syncthreads();
    const double* row = sq + t * R;
    if constexpr (EXTRACT) {
        if (tid >= RR) return;
        double best = -DBL_MAX, second = -DBL_MAX;
        int arg = 0;
        for (int c = 0; c < R; ++c) {
            const double q = row[c];
            if (q > best) {
                second = best;
                best = q;
                arg = c;
            } else if (q > second) {
                second = q;
            }
        }
        p.pi[s_idx] = arg;
        p.gap[s_idx] = R > 1 ? best - second : INFINITY;
    } else {
        double best = -DBL_MAX;
#pragma unroll 8
        for (int c = 0; c < R; ++c) best = fmax(best, row[c]);
        const VT o = (VT)(rw - mu + best);
        // (threads past the last state repeat it)
        if (tid < RR) reinterpret_cast<VT*>(p.v_out)[s_idx] = o;
        const double out = (double)o, dv = out - old;
        // (a NaN increment, from a caller's V_0 that holds one, is passed over: as a key it
        // would stand above every number of its slot)
        double dmx = fmax(dv, -DBL_MAX), dmn = fmin(dv, DBL_MAX);
        double vmx = fmax(out, -DBL_MAX), vmn = fmin(out, DBL_MAX);
        if (p.span) {
            dmx = wave_max(dmx);
            dmn = wave_min(dmn);
            if (FP32) {
                vmx = wave_max(vmx);
                vmn = wave_min(vmn);
            }
            if ((tid & 63) == 0)
                span_emit<FP32>(p.span, p.sweep, tile * (nt >> 6) + (tid >> 6), dmx, dmn, vmx, vmn);
            return;
        }
        block_reduce4(dmx, dmn, vmx, vmn, red);
        if (tid == 0) {
            double* out4 = p.partials + 4 * (size_t)tile;
            out4[0] = dmx;
            out4[1] = dmn;
            out4[2] = vmx;
            out4[3] = vmn;
        }
    }
}

static size_t a_lifo_lds_bytes(const ADev& p) {
    return sizeof(double) * ((size_t)p.lmax * p.R + (size_t)p.R * p.R + (size_t)p.lmax);
}

hipError_t launch_backup_a_lifo(const ADev& p, int storage_fp32, int extract, hipStream_t s) {
    // tiles (O, X_{m-1}..X_2); lanes over (X_m, action) and (X_m, X_1)
    if (p.m < 2 || p.m > PVI_MAX_LIFE || p.R > 32 || p.tiles < 1) return hipErrorInvalidConfiguration;
    const size_t bytes = a_lifo_lds_bytes(p);
    if (bytes > 65536) return hipErrorInvalidConfiguration;
    if (p.tab < p.lmax + 1 || p.lmax < (p.m - 2) * (p.R - 1) + p.R)
        return hipErrorInvalidValue;
    const int threads = std::min(1024, ((p.R * p.R + 63) / 64) * 64);
    if (extract)
        hipLaunchKernelGGL((backup_a_lifo_kernel<double, true>), dim3(p.tiles), dim3(threads),
                           bytes, s, p);
    else if (storage_fp32)
        hipLaunchKernelGGL((backup_a_lifo_kernel<float, false>), dim3(p.tiles), dim3(threads),
                           bytes, s, p);
    else
        hipLaunchKernelGGL((backup_a_lifo_kernel<double, false>), dim3(p.tiles), dim3(threads),
                           bytes, s, p);
    return hipGetLastError();
}

}  // namespace pvi

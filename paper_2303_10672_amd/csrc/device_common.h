// Device helpers shared by the kernel files (header-only, no relocatable code).
#pragma once

#include <hip/hip_runtime.h>

#include <cfloat>
#include <cmath>

#include "pvi_internal.h"

namespace pvi {

__device__ __forceinline__ int xcd_remap(int bid, int nb) {
    // Workgroups are dispatched round-robin over the 8 XCDs; give each XCD a
    // contiguous range of tiles so the V blocks a range touches stay in one L2.
    const int q = nb >> 3, r = nb & 7, x = bid & 7, l = bid >> 3;
    return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + l;
}

// Maximum and minimum over a wavefront, the same in every lane: four exchanges inside the
// rows of 16 lanes (DPP, no LDS), then the four rows' values from the scalar side.  Every
// lane of the wavefront must be active.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)(unsigned)lo | (long long)hi << 32);
}
__device__ __forceinline__ double lane_f64(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double((long long)(unsigned)lo | (long long)hi << 32);
}
__device__ __forceinline__ double wave_max(double v) {
    v = fmax(v, dpp_f64<0xb1>(v));   // quad_perm: xor 1
    v = fmax(v, dpp_f64<0x4e>(v));   // quad_perm: xor 2
    v = fmax(v, dpp_f64<0x141>(v));  // row_half_mirror
    v = fmax(v, dpp_f64<0x140>(v));  // row_mirror
    return fmax(fmax(lane_f64(v, 0), lane_f64(v, 16)), fmax(lane_f64(v, 32), lane_f64(v, 48)));
}
__device__ __forceinline__ double wave_min(double v) { return -wave_max(-v); }

// Block-wide reduction of 4 values (max, min, max, min); result valid in thread 0.
__device__ inline void block_reduce4(double& a, double& b, double& c, double& d, double* red) {
    a = wave_max(a);
    b = wave_min(b);
    c = wave_max(c);
    d = wave_min(d);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    if (lane == 0) {
        red[4 * w + 0] = a;
        red[4 * w + 1] = b;
        red[4 * w + 2] = c;
        red[4 * w + 3] = d;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < nw; ++i) {
            a = fmax(a, red[4 * i + 0]);
            b = fmin(b, red[4 * i + 1]);
            c = fmax(c, red[4 * i + 2]);
            d = fmin(d, red[4 * i + 3]);
        }
    }
}

// Stopping rule applied to the reduced (max dv, min dv, max v', min v') of one sweep,
// on a copy of the control block that the caller writes back.
// With FP32 storage (V = c + v) it also moves the centring: c <- gamma c + mu and
// mu <- mu + mid(v').  Called by one thread after the whole sweep is reduced.
__device__ inline void span_update(Ctl& ctl, double a0, double a1, double a2, double a3,
                                   int fp32, int fixed, double gamma) {
    double dmax = a0, dmin = a1;
    if (fp32) {
        const double shift = (gamma - 1.0) * ctl.c + ctl.mu;
        dmax += shift;
        dmin += shift;
        ctl.c = gamma * ctl.c + ctl.mu;
        ctl.mu += 0.5 * (a2 + a3);
    }
    const double span = dmax - dmin;
    // stopping criterion: the span (rule 0) or max |V_new - V| (rule 1)
    // (the periodic rule, 2, is decided by its own kernels after this one)
    const double crit = ctl.rule == 1   ? fmax(fabs(dmax), fabs(dmin))
                        : ctl.rule == 2 ? INFINITY
                                         : span;
    ctl.dmax = dmax;
    ctl.dmin = dmin;
    ctl.span = span;
    ctl.sweeps += 1;
    if (fixed) return;
    if (fp32) {
        const double vabs = fmax(fabs(a2), fabs(a3));
        ctl.vabs = vabs;
        if (span < ctl.best_span * 0.999) {
            ctl.best_span = span;
            ctl.stall = 0;
        } else {
            ctl.stall += 1;
        }
        // the FP32 phase hands over to FP64 at the FP32 floor (span based for
        // either rule) or when the rule itself is met
        if (crit < ctl.thr || span <= ctl.floor32 * vabs || ctl.stall >= 3) {
            ctl.stop = 1;
            ctl.stop_sweep = ctl.sweeps;
        }
    } else if (crit < ctl.thr) {
        ctl.stop = 1;
        ctl.stop_sweep = ctl.sweeps;
    }
}

// Orders a wavefront's LDS stores before its later LDS reads of other lanes' data
// (no instruction: LDS requests of one wavefront are served in issue order).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// max without the extra instruction that quiets signalling NaNs (no arithmetic result is one)
__device__ __forceinline__ double max_f64(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// ------------------------------------------------------------------ SpanBuf
__device__ __forceinline__ unsigned long long span_key(double x) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    return b >> 63 ? ~b : b | (1ull << 63);
}
__device__ __forceinline__ double span_value(unsigned long long k) {
    return __longlong_as_double((long long)(k >> 63 ? k ^ (1ull << 63) : ~k));
}

// What a sweep's wavefront reads at its start: the control block as the sweep before left
// it and the lane's slot of that sweep's keys (requested together, before anything waits).
struct SpanIn {
    Ctl ctl;
    unsigned long long k[4];
};
// Field by field: a struct copy would go through private memory, and wait for it.
__device__ __forceinline__ void ctl_copy(Ctl& to, const Ctl& from) {
    to.mu = from.mu;
    to.c = from.c;
    to.dmax = from.dmax;
    to.dmin = from.dmin;
    to.span = from.span;
    to.best_span = from.best_span;
    to.thr = from.thr;
    to.floor32 = from.floor32;
    to.vabs = from.vabs;
    to.stop = from.stop;
    to.sweeps = from.sweeps;
    to.stop_sweep = from.stop_sweep;
    to.stall = from.stall;
    to.fp32_phase = from.fp32_phase;
    to.rule = from.rule;
    to.pending = from.pending;
}
// Without a SpanBuf the control block of the solve alone is read (and the keys, unused, from
// it): no branch parts the loads from those that follow.
template <bool FP32>
__device__ __forceinline__ void span_fetch(const SpanBuf* b, const Ctl* ctl, int sweep,
                                           SpanIn& in) {
    // by vector loads (the offset 0 is one the compiler cannot see): scalar loads return out
    // of order, so the next wait for a kernel argument would wait for these
    uint32_t zero;
    asm("v_mov_b32 %0, 0" : "=v"(zero));
    const Ctl* c = b ? &b->ctl[sweep & 1] : ctl;
    ctl_copy(in.ctl, *reinterpret_cast<const Ctl*>(reinterpret_cast<const char*>(c) + zero));
    const unsigned long long* k =
        b ? b->key[(sweep + 3) & 3][threadIdx.x & (kSpanSlots - 1)]
          : reinterpret_cast<const unsigned long long*>(ctl);
    in.k[0] = k[0];
    in.k[1] = k[1];
    if (FP32) {
        in.k[2] = k[2];
        in.k[3] = k[3];
    }
}

// Applies the sweep before to in.ctl (every lane with the same result).
template <bool FP32>
__device__ __forceinline__ void span_reduce(SpanIn& in, int fixed, double gamma) {
    if (in.ctl.stop || !in.ctl.pending) return;
    // (a slot nothing was written to decodes to a NaN, which the maxima pass over)
    double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < (FP32 ? 4 : 2); ++i) v[i] = wave_max(span_value(in.k[i]));
    span_update(in.ctl, v[0], -v[1], v[2], -v[3], FP32, fixed, gamma);
}

// The same at a sweep's start, every wavefront for itself; the first workgroup stores it for
// the next sweep and clears that sweep's keys.  Returns whether the rule has fired; this
// sweep then does no work.  Without a SpanBuf the launches between the sweeps have done so.
template <bool FP32>
__device__ __forceinline__ bool span_apply(SpanBuf* b, int sweep, SpanIn& in, int fixed,
                                           double gamma) {
    in.ctl.stop = __builtin_amdgcn_readfirstlane(in.ctl.stop);
    if (!b) return in.ctl.stop;
    in.ctl.pending = __builtin_amdgcn_readfirstlane(in.ctl.pending);
    in.ctl.rule = __builtin_amdgcn_readfirstlane(in.ctl.rule);
    span_reduce<FP32>(in, fixed, gamma);
    in.ctl.pending = !in.ctl.stop;
    if (blockIdx.x == 0 && threadIdx.x < kSpanSlots) {
        if (threadIdx.x == 0) ctl_copy(b->ctl[(sweep + 1) & 1], in.ctl);
        unsigned long long* k = b->key[(sweep + 1) & 3][threadIdx.x];
        k[0] = k[1] = k[2] = k[3] = 0;
    }
    return __builtin_amdgcn_readfirstlane(in.ctl.stop);
}

// One wavefront's (or workgroup's) increments into the keys of its sweep, by one lane.
template <bool FP32>
__device__ __forceinline__ void span_emit(SpanBuf* b, int sweep, int slot, double dmx, double dmn,
                                          double vmx, double vmn) {
    unsigned long long* k = b->key[sweep & 3][slot & (kSpanSlots - 1)];
    __hip_atomic_fetch_max(k, span_key(dmx), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_max(k + 1, span_key(-dmn), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (FP32) {
        __hip_atomic_fetch_max(k + 2, span_key(vmx), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_max(k + 3, span_key(-vmn), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

}  // namespace pvi

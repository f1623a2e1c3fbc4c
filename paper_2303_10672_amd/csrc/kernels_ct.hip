// Scenario C's arrival merges by antidiagonals (kernels_c.hip derives the sums).
//
// A merge of life class j forms, for every remaining count r and stock x of that class,
//   T_j(r, x) = sum_{y<=r} w(r, y) S[r - y][c(x + y)],   c(.) the cap at a_max,
// from the slab S[s][z].  With one lane per x every term is a read of its own.  But with
// t = x + r the term (r, y) is S[s][c(t - s)], s = r - y: it depends on t and s only, so a
// lane that holds the vector D[s] = S[s][c(t - s)] in registers forms every row r of its
// antidiagonal, x = t - r, from R reads instead of R(R + 1)/2.  The first merge,
//   T_2(r, x_1) = sum_{y<=r} w(r, y) U(c(x_2 + y), c(x_1 + r - y)),
// has the same form with t = x_1 + r and D[y] = U(c(x_2 + y), c(t - y)).  Wavefronts take a
// few neighbouring t each, so the rows 0 <= t - r <= a_max that exist are nearly the same
// for its lanes (87% of the multiply-adds count at 21 orders); the weights are the same
// for all lanes.  Each sum has the terms of the plain
// kernels in their order, y = 0, 1, .., r, and nothing else, so values are bit-identical;
// lanes whose x = t - r does not exist compute from clamped reads and store nothing.
//
// The tables of the level below the top, which c_top_kernel and c_order_kernel read, are
// laid out [tau][(y_m, r) pair][x_{m-1}][lower digits padded to tlo, whole lines]
// (row stride trow).  Where the first two merges write them (m = 5), the lower digits come
// in the order x_2, x_3, x_1: a wavefront's store of one row is then one run of up to 64
// values, not one short run per x_3 (2.3 TB/s of partial lines).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <type_traits>

#include "device_common.h"
#include "pvi_internal.h"

namespace pvi {

namespace {

typedef const __attribute__((address_space(4))) double* ConstF64;
typedef const __attribute__((address_space(4))) int32_t* ConstI32;

constexpr int kLo = kTopLo;      // low-digit values per workgroup of c_top_kernel
constexpr int kTopWaves = 12;    // 4 antidiagonals of kLo values per wavefront, 2 R - 1 <= 48
constexpr int kLdsMax = 160 * 1024;

// A copy the compiler takes for new: what is formed from it is formed here, not hoisted
// ahead of loops and row blocks (all masks, offsets and addresses of an unrolled triangle
// at once do not fit the registers).
template <class T>
__device__ __forceinline__ T here_s(T x) {
    asm volatile("" : "+s"(x));
    return x;
}
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
template <class T>
__device__ __forceinline__ T here_v(T x) {
    asm volatile("" : "+v"(x));
    return x;
}

// Weights of one level: the triangle w(r, y), y <= r, packed row by row and spread over the
// 16 lanes of a DPP row, entry e in lane e % 16 of register e / 16 (each of the four rows
// holds a copy).  v_fmac_f64 takes its first factor from one lane of the row
// (row_newbcast) at the full rate, so a weight costs no load per use and no scalar
// register, whose shortage had the compiler spill; 24 orders take 19 registers.
template <int RC>
constexpr int kWRegs = (RC * (RC + 1) / 2 + 15) / 16;

template <int RC>
__device__ __forceinline__ void tri_weights(double (&W)[kWRegs<RC>], const double* src,
                                            int lane, int rhi) {
    // four registers at a time, as far as rows up to rhi (and the pair's other row) use them
#pragma unroll
    for (int b = 0; b < kWRegs<RC>; b += 4)
        if (16 * b < (rhi + 2) * (rhi + 3) / 2) {
#pragma unroll
            for (int i = b; i < b + 4 && i < kWRegs<RC>; ++i) W[i] = src[i * 16 + (lane & 15)];
        }
}

// acc += w D, w the value of lane n of each 16-lane row of W.  The wait states cover a W
// that the instruction before wrote (a DPP read needs two); every lane of the wavefront is
// active here.
#define PVI_DPP " row_newbcast:%c"
#define PVI_FMAC(acc, w, d, n) \
    "v_fmac_f64_dpp %" #acc ", %" #w ", %" #d PVI_DPP #n " row_mask:0xf bank_mask:0xf\n"
template <int n>
__device__ __forceinline__ void fmac1(double& a, double w, double d) {
    asm("s_nop 1\n" PVI_FMAC(0, 1, 2, 3) : "+v"(a) : "v"(w), "v"(d), "n"(n));
}
// two rows, one term each
template <int n0, int n1>
__device__ __forceinline__ void fmac2(double& a, double& b, double wa, double wb, double da,
                                      double db) {
    asm("s_nop 1\n" PVI_FMAC(0, 2, 4, 6) PVI_FMAC(1, 3, 5, 7)
        : "+v"(a), "+v"(b)
        : "v"(wa), "v"(wb), "v"(da), "v"(db), "n"(n0), "n"(n1));
}
// two rows, four terms each, the rows in turn
template <int a0, int a1, int a2, int a3, int b0, int b1, int b2, int b3>
__device__ __forceinline__ void fmac8(double& a, double& b, double wa0, double wa1, double wa2,
                                      double wa3, double wb0, double wb1, double wb2, double wb3,
                                      const double (&da)[4], const double (&db)[4]) {
    asm("s_nop 1\n" PVI_FMAC(0, 2, 10, 18) PVI_FMAC(1, 6, 14, 22) PVI_FMAC(0, 3, 11, 19)
            PVI_FMAC(1, 7, 15, 23) PVI_FMAC(0, 4, 12, 20) PVI_FMAC(1, 8, 16, 24)
                PVI_FMAC(0, 5, 13, 21) PVI_FMAC(1, 9, 17, 25)
        : "+v"(a), "+v"(b)
        : "v"(wa0), "v"(wa1), "v"(wa2), "v"(wa3), "v"(wb0), "v"(wb1), "v"(wb2), "v"(wb3),
          "v"(da[0]), "v"(da[1]), "v"(da[2]), "v"(da[3]), "v"(db[0]), "v"(db[1]), "v"(db[2]),
          "v"(db[3]), "n"(a0), "n"(a1), "n"(a2), "n"(a3), "n"(b0), "n"(b1), "n"(b2), "n"(b3));
}

// Terms y .. r of row r and y .. r + 1 of row r + 1.
template <int RC, bool REV, int r, int y>
__device__ __forceinline__ void tri_pair(double& a, double& b, const double (&D)[RC],
                                         const double (&W)[kWRegs<RC>]) {
    constexpr int ea = r * (r + 1) / 2 + y, eb = (r + 1) * (r + 2) / 2 + y;
    if constexpr (y + 3 <= r) {
        const double da[4] = {D[REV ? r - y : y], D[REV ? r - y - 1 : y + 1],
                              D[REV ? r - y - 2 : y + 2], D[REV ? r - y - 3 : y + 3]};
        const double db[4] = {D[REV ? r + 1 - y : y], D[REV ? r - y : y + 1],
                              D[REV ? r - y - 1 : y + 2], D[REV ? r - y - 2 : y + 3]};
        fmac8<ea % 16, (ea + 1) % 16, (ea + 2) % 16, (ea + 3) % 16, eb % 16, (eb + 1) % 16,
              (eb + 2) % 16, (eb + 3) % 16>(
            a, b, W[ea / 16], W[(ea + 1) / 16], W[(ea + 2) / 16], W[(ea + 3) / 16], W[eb / 16],
            W[(eb + 1) / 16], W[(eb + 2) / 16], W[(eb + 3) / 16], da, db);
        tri_pair<RC, REV, r, y + 4>(a, b, D, W);
    } else if constexpr (y <= r) {
        fmac2<ea % 16, eb % 16>(a, b, W[ea / 16], W[eb / 16], D[REV ? r - y : y],
                                D[REV ? r + 1 - y : y]);
        tri_pair<RC, REV, r, y + 1>(a, b, D, W);
    } else {
        fmac1<eb % 16>(b, W[eb / 16], D[REV ? r + 1 - y : y]);
    }
}

// Terms y .. r of row r.
template <int RC, bool REV, int r, int y>
__device__ __forceinline__ void tri_one(double& a, const double (&D)[RC],
                                        const double (&W)[kWRegs<RC>]) {
    if constexpr (y <= r) {
        constexpr int e = r * (r + 1) / 2 + y;
        fmac1<e % 16>(a, W[e / 16], D[REV ? r - y : y]);
        tri_one<RC, REV, r, y + 1>(a, D, W);
    }
}

// Rows r .. of one lane from its vector D, two at a time.  Pairs outside [rlo, rhi] are
// skipped; a row of a pair outside it is formed and ignored.  REV: term y of row r is
// D[r - y] (else D[y]).  f(row, sum) takes each row as a compile-time constant.
template <int RC, bool REV, int r, class F>
__device__ __forceinline__ void tri_rows(const double (&D)[RC], const double (&W)[kWRegs<RC>],
                                         int rlo, int rhi, F&& f) {
    if constexpr (r < RC) {
        if (r > rhi) return;
        if (r + 1 >= rlo) {
            double a = 0.0, b = 0.0;
            if constexpr (r + 1 < RC) {
                tri_pair<RC, REV, r, 0>(a, b, D, W);
                f(r, a);
                f(r + 1, b);
            } else {
                tri_one<RC, REV, r, 0>(a, D, W);
                f(r, a);
            }
        }
        tri_rows<RC, REV, r + 2>(D, W, rlo, rhi, f);
    }
}

// D[0 .. rhi] by load(i), eight entries at a time (those past rhi are never used by a row
// that exists and keep what they held)
template <int RC, class L>
__device__ __forceinline__ void tri_load(double (&D)[RC], int rhi, L&& load) {
#pragma unroll
    for (int b = 0; b < RC; b += kTriLoad)
        if (b <= rhi) {
#pragma unroll
            for (int i = b; i < b + kTriLoad && i < RC; ++i) D[i] = load(i);
        }
}

// A barrier that orders LDS only: __syncthreads() would also wait until every global store
// before it has arrived, a memory round trip per step of the loops below.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// State offset of the lower digits at place `lo` of a table of level m-2.
__device__ __forceinline__ int state_lo(const CDev& p, int lo) {
    if (!p.swap23) return lo;
    const int R = p.R, hi = lo / R, x1 = lo - hi * R, x2 = hi / R, x3 = hi - x2 * R;
    return (x3 * R + x2) * R + x1;
}

template <typename VT>
__device__ __forceinline__ double lds_at(const unsigned char* base, int byte_off) {
    return (double)*reinterpret_cast<const VT*>(base + byte_off);
}

}  // namespace

// The walk over x_2 of c_merge23_tri_kernel for at most R / 2 rows: the slab then holds
// R / nr values of x_2 side by side, and a pair of phases between barriers serves them all
// (a single x_2 would leave most wavefronts with little to do in each).
template <typename VT, int RC>
__device__ __forceinline__ void c_merge23_short(unsigned char* smem, const double* wtab, VT* T,
                                                uint32_t orow, int s3, int s2, int R, int nr,
                                                int TL, int wave, int lane) {
    constexpr int B = sizeof(VT), RR = RC * RC, kSlab = RR * RC * B, H = RC / 2;
    constexpr int NW = 16 * kWRegs<RC>;
    const int nw = blockDim.x >> 6, nq = (nr + R - 1 + TL - 1) / TL, group = R / nr;
    const int sub = lane / R, ln = min(lane - sub * R, R - 1);
    double D[H], W[kWRegs<H>];
#pragma unroll
    for (int i = 0; i < H; ++i) D[i] = 0.0;
#pragma unroll
    for (int i = 0; i < kWRegs<H>; ++i) W[i] = 0.0;
    __syncthreads();
    for (int x0 = 0; x0 < R; x0 += group) {
        const int ntask = nq * min(group, R - x0);
        tri_weights<H>(W, wtab, lane, nr - 1);
        for (int id = wave; id < ntask; id += nw) {
            const int g = uniform(id / nq), q = (id - g * nq) * TL, x2 = x0 + g, t = here_v(q + sub);
            const int rlo = max(0, q - (R - 1)), rhi = min(nr - 1, q + TL - 1);
            const int plane = ln * (RR * B), last = plane + (R - 1) * B, get = plane + t * B;
            tri_load<H>(D, rhi, [&](int y) {
                return lds_at<VT>(smem, min(max(get - y * B, plane), last) +
                                            min(x2 + y, R - 1) * (RC * B));
            });
            const int put = kSlab + g * nr * (RR * B) + ln * (RC * B) + t * B;
            tri_rows<H, false, 0>(D, W, rlo, rhi, [&](int r, double acc) {
                if (sub < TL && r < nr && (unsigned)(t - r) < (unsigned)R)
                    *reinterpret_cast<VT*>(smem + put + r * (RR - 1) * B) = (VT)acc;
            });
        }
        lds_barrier();
        tri_weights<H>(W, wtab + NW, lane, nr - 1);
        for (int id = wave; id < ntask; id += nw) {
            const int g = uniform(id / nq), q = (id - g * nq) * TL, x2 = x0 + g, t = here_v(q + sub);
            const int rlo = max(0, q - (R - 1)), rhi = min(nr - 1, q + TL - 1);
            const int glo = kSlab + g * nr * (RR * B) + ln * B, ghi = glo + (R - 1) * (RC * B);
            const int get = glo + t * (RC * B);
            tri_load<H>(D, rhi, [&](int s) {
                return lds_at<VT>(smem, min(max(get - s * (RC * B), glo), ghi) +
                                            min(s, nr - 1) * (RR * B));
            });
            unsigned char* out = reinterpret_cast<unsigned char*>(T + x2 * s2);
            const uint32_t step = here_s((orow - (uint32_t)s3) * B);
            const uint32_t at = (uint32_t)(t * s3 + ln) * B;
            tri_rows<H, true, 0>(D, W, rlo, rhi, [&](int r, double acc) {
                if (sub < TL && r < nr && (unsigned)(t - r) < (unsigned)R)
                    *reinterpret_cast<VT*>(out + step * (uint32_t)r + at) = (VT)acc;
            });
        }
        lds_barrier();
    }
}

// Merges of life classes 2 and 3 (m >= 5), T_3 straight from U.  One workgroup per
// (y_m, tau, digits above 3), longest rows (small y_m) first: the cube U(tau, y_m, ..,
// z_3, z_2, z_1) in LDS, then for every x_2 the slab T_2(r', z_3, x_1) (lanes (t, z_3)),
// and from it T_3(r, x_3, x_2, x_1) (lanes (t, x_1)).  LDS strides are RC, known at compile
// time, so the entries of a lane's vectors sit at constant offsets and only the cap costs
// address arithmetic.  Cube and slab take
// 148 KB at RC = 21 in FP64, so one workgroup of up to 14 wavefronts per CU.
// Measured at R = 21, m = 5 (2.5 GB written): 0.68 ms, 3.7 TB/s; the plain kernel, with one
// LDS read per multiply-add, took 1.41 ms.
template <typename VT, int RC>
__global__ __launch_bounds__(1024) void c_merge23_tri_kernel(CDev p, const void* u_, void* out_) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (!p.extract && p.ctl->stop) return;
    constexpr int B = sizeof(VT), RR = RC * RC, R3 = RR * RC, NW = 16 * kWRegs<RC>;
    const int R = p.R, tid = threadIdx.x;
    VT* cube = reinterpret_cast<VT*>(smem);                         // U[z_3][z_2][z_1]
    constexpr int kSlab = R3 * B;                                   // T_2[r'][z_3][x_1]
    double* wtab = reinterpret_cast<double*>(smem + (2 * kSlab + 15) / 16 * 16);  // levels 2, 3
    const int nu = R * R * R;
    const int nhi = (int)(p.nblk / nu);  // values of the digits above 3
    int b = blockIdx.x;
    const int ym = b / (p.P * nhi);
    b -= ym * p.P * nhi;
    const int tau = b / nhi, hi = b - tau * nhi;
    const int nr = min(R - ym, p.alim - ym + 1);
    if (nr <= 0) return;
    {
        const VT* U = reinterpret_cast<const VT*>(u_) + ((int64_t)tau * R + ym) * p.nblk +
                      (int64_t)hi * nu;
        // eight loads in flight per thread
        for (int i0 = tid; i0 < nu; i0 += 8 * blockDim.x) {
            VT v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = U[min(i0 + k * (int)blockDim.x, nu - 1)];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int i = i0 + k * (int)blockDim.x, z32 = i / R, z3 = z32 / R;
                if (i < nu) cube[z3 * RR + (z32 - z3 * R) * RC + i - z32 * R] = v[k];
            }
        }
    }
    for (int i = tid; i < 2 * NW; i += blockDim.x) wtab[i] = p.binp[2 * NW + i];
    const int lane = tid & 63, wave = uniform(tid >> 6);
    const int TL = 64 / R;  // antidiagonals per wavefront
    VT* T = reinterpret_cast<VT*>(out_) + ((int64_t)tau * p.npair + p.pair_base[ym]) * p.orow +
            (int64_t)hi * p.ohi;
    // strides of x_3 and x_2 in the table
    const int s3 = p.swap23 ? R : R * R, s2 = p.swap23 ? R * R : R;
    if (2 * nr <= R) {
        c_merge23_short<VT, RC>(smem, wtab, T, (uint32_t)p.orow, s3, s2, R, nr, TL, wave, lane);
        return;
    }
    const int sub = lane / R, ln = min(lane - sub * R, R - 1);
    const int q = wave * TL, t = q + sub;
    // rows that exist on this wavefront's antidiagonals
    const int rlo = max(0, q - (R - 1)), rhi = min(nr - 1, q + TL - 1);
    const bool work = q < nr + R - 1;
    const uint32_t orow = (uint32_t)p.orow;  // times 8 R below 2^32 (checked by the launcher)
    // byte offsets: entry y of the first merge's vector in a plane of the cube, the same
    // for every x_2; the slab's column of T_2 written (row r, x_1 = t - r: constant steps);
    // entry s of the second merge's vector before its cap; the value stored
    int cap2[RC];
#pragma unroll
    for (int y = 0; y < RC; ++y) cap2[y] = ln * (RR * B) + min(max(t - y, 0), R - 1) * B;
    const int put = kSlab + ln * (RC * B) + t * B;
    const int get0 = kSlab + ln * B + t * (RC * B);
    const int glo = kSlab + ln * B, ghi = glo + (R - 1) * (RC * B);
    const uint32_t at = (uint32_t)(t * s3 + ln) * B;
    // rows of this lane that exist; the masks stay in scalar registers for all x_2
    bool has[RC];
#pragma unroll
    for (int r = 0; r < RC; ++r)
        has[r] = sub < TL && r < nr && (unsigned)(t - r) < (unsigned)R;
    double D[RC], W[kWRegs<RC>];
#pragma unroll
    for (int i = 0; i < RC; ++i) D[i] = 0.0;
#pragma unroll
    for (int i = 0; i < kWRegs<RC>; ++i) W[i] = 0.0;
    __syncthreads();
    for (int x2 = 0; x2 < R; ++x2) {
        if (work) {
            tri_load<RC>(D, rhi, [&](int y) {
                return lds_at<VT>(smem, cap2[y] + min(x2 + y, R - 1) * (RC * B));
            });
            tri_weights<RC>(W, wtab, lane, rhi);
            tri_rows<RC, false, 0>(D, W, rlo, rhi, [&](int r, double acc) {
                if (has[r])
                    *reinterpret_cast<VT*>(smem + put + r * (RR - 1) * B) = (VT)acc;
            });
        }
        lds_barrier();
        if (work) {
            tri_load<RC>(D, rhi, [&](int s) {
                return lds_at<VT>(smem, min(max(get0 - s * (RC * B), glo), ghi) + s * (RR * B));
            });
            tri_weights<RC>(W, wtab + NW, lane, rhi);
            unsigned char* out = reinterpret_cast<unsigned char*>(T + x2 * s2);
            const uint32_t step = here_s((orow - (uint32_t)s3) * B);
            tri_rows<RC, true, 0>(D, W, rlo, rhi, [&](int r, double acc) {
                // row r, x_3 = t - r
                if (has[r])
                    *reinterpret_cast<VT*>(out + step * (uint32_t)r + at) = (VT)acc;
            });
        }
        lds_barrier();
    }
}

// Top merge (life class m-1, m >= 4, order-independent life) with the final sum and the
// max over orders:
//   Q(tau, x, a) = -C_f [a > 0] + sum_{y_m<=a} Bin(y_m; a, p_m) T_{m-1}(tau, y_m, x; a - y_m).
// One workgroup per (tau, kLo values of the digits below m-1).  Row r of slab y_m at
// antidiagonal t belongs to order a = y_m + r of the state x_{m-1} = t - r, so
// u = t + y_m = x_{m-1} + a does not change with y_m: a lane keeps u for the whole loop
// and the running sums B of its orders in registers (B[r] is order y_m + r; it shifts
// down by one per step).  Order a = y_m is complete after step y_m, its terms added in
// the order 0, 1, .., a; its lane then updates the state's best (second best, argmax)
// in LDS, orders ascending.  The slabs T_{m-2}(y_m, z, lo; r') come into LDS straight from
// memory, the next one while this one is used.
// Bound by reading T_{m-2} once (2.5 GB in FP64 at R = 21, m = 5): 0.64 ms, 4.0 TB/s; the
// plain kernel, with one LDS read per multiply-add, took 0.71 ms for the sweeps and the
// extraction ran the unfused chain.
template <typename VT, int RC, bool EXTRACT>
__global__ __launch_bounds__(64 * kTopWaves) void c_top_kernel(CDev p, const void* in_,
                                                               int nslots) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[64];
    if (!EXTRACT && p.ctl->stop) return;
    constexpr int LPR = kLo * (int)sizeof(VT) / 16;  // staging lanes per row of kLo values
    constexpr int RPI = 64 / LPR;                    // rows per staging instruction
    static_assert(RPI == c_top_rows(sizeof(VT)), "layout of the slab");
    const int R = p.R, j = p.m - 1, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
    constexpr int kRowB = kLo * (int)sizeof(VT);  // bytes of a row of the slab
    const int slabb = (R * RC + RPI - 1) / RPI * RPI * kRowB;  // [s][z < RC][kLo], twice
    double* sbest = reinterpret_cast<double*>(smem + 2 * slabb);  // [R][kLo]
    double* ssec = sbest + R * kLo;
    int* sarg = reinterpret_cast<int*>(ssec + R * kLo);
    const int nlo = (int)p.pow_r[j - 1];  // R^(m-2): the digits below m-1
    const int nlob = (nlo + kLo - 1) / kLo;
    const int lid = xcd_remap(blockIdx.x, gridDim.x);
    const int tau = lid / nlob, lo0 = (lid - tau * nlob) * kLo;
    const int l = lane & (kLo - 1), ub = wave * 4, u = ub + lane / kLo;
    for (int i = tid; i < R * kLo; i += blockDim.x) {
        sbest[i] = ssec[i] = -DBL_MAX;
        sarg[i] = 0;
    }
    const int64_t trow0 = (int64_t)tau * p.npair;
    const ConstI32 pb = (ConstI32)p.pair_base;
    auto stage = [&](int ym, int b) {
        const VT* src = reinterpret_cast<const VT*>(in_) + (trow0 + pb[ym]) * p.trow + lo0 +
                        (lane % LPR) * (16 / sizeof(VT));
        const int n = (R - ym) * RC;
        for (int i = wave * RPI; i < n; i += nw * RPI) {
            const int row = min(i + lane / LPR, n - 1), s = row / RC, z = min(row - s * RC, R - 1);
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)(src + (int64_t)s * p.trow +
                                                                (int64_t)z * p.tlo),
                (__attribute__((address_space(3))) void*)(smem + b * slabb + i * kRowB), 16, 0, 0);
        }
    };
    double W[kWRegs<RC>];
    tri_weights<RC>(W, p.binp + (size_t)j * 16 * kWRegs<RC>, lane, RC);
    const ConstF64 bm = (ConstF64)p.binmp;
    double B[RC + 1], D[RC];
#pragma unroll
    for (int r = 0; r < RC; ++r) B[r] = D[r] = 0.0;
    B[RC] = 0.0;
    stage(0, 0);
    // one step: slab ym, the running sums of order ym + r in B[r + off]
    auto step = [&](int ym, auto off_) {
        constexpr int off = decltype(off_)::value;
        const int nr = R - ym;
        // this slab has landed, and every wavefront is done with the other one
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (ym + 1 < R) stage(ym + 1, (ym + 1) & 1);
        const int t = u - ym, tb = ub - ym;  // the wavefront has tb .. tb + 3
        const int rlo = max(0, tb - (R - 1)), rhi = min(nr - 1, tb + 3);
        if (rlo <= rhi) {
            // entry s at z = c(t - s): constant offsets but for the cap, and for the entries
            // that fewer orders than RC may not have
            const int base = (ym & 1) * slabb + l * (int)sizeof(VT);
            const int get0 = base + t * kRowB, ghi = base + (R - 1) * kRowB;
            tri_load<RC>(D, rhi, [&](int s) {
                return lds_at<VT>(smem, min(max(get0 - s * kRowB, base), ghi) +
                                            c_top_entry(s, R, RC) * (RC * kRowB));
            });
            const ConstF64 bmy = here_s(bm + ym * (RC + 1));  // row ym + r, entry ym
            const int nl = here_s(nr);
            tri_rows<RC, true, 0>(D, W, rlo, rhi, [&](int r, double acc) {
                if (r < nl) B[r + off] = fma(bmy[r * RC], (double)(VT)acc, B[r + off]);
            });
        }
        if ((unsigned)t < (unsigned)R) {  // order ym of the state x_{m-1} = t
            const int at = t * kLo + l;
            const double q = (ym > 0 ? -p.cfixed : 0.0) + B[off], best = sbest[at];
            if (q > best) {
                if (EXTRACT) {
                    ssec[at] = best;
                    sarg[at] = ym;
                }
                sbest[at] = q;
            } else if (EXTRACT && q > ssec[at]) {
                ssec[at] = q;
            }
        }
    };
    for (int ym = 0; ym < R; ym += 2) {  // two steps per shift of the running sums
        step(ym, std::integral_constant<int, 0>{});
        if (ym + 1 < R) step(ym + 1, std::integral_constant<int, 1>{});
#pragma unroll
        for (int r = 0; r + 2 <= RC; ++r) B[r] = B[r + 2];
        B[RC - 1] = B[RC] = 0.0;
    }
    __syncthreads();
    double dmx = -DBL_MAX, dmn = DBL_MAX, vmx = -DBL_MAX, vmn = DBL_MAX;
    for (int i = tid; i < R * kLo; i += blockDim.x) {
        const int x = i / kLo, lo = lo0 + i - x * kLo;
        if (lo >= nlo) continue;
        const int64_t s = (int64_t)tau * p.nblk + (int64_t)x * nlo + state_lo(p, lo);
        if (EXTRACT) {
            p.pi[s] = sarg[i];
            p.gap[s] = sbest[i] - ssec[i];
        } else {
            const double mu = sizeof(VT) == 4 ? p.ctl->mu : 0.0;
            const VT o = (VT)(sbest[i] - mu);
            reinterpret_cast<VT*>(p.v_out)[s] = o;
            const double out = (double)o;
            const double dv = out - (double)reinterpret_cast<const VT*>(p.v_in)[s];
            dmx = fmax(dmx, dv);
            dmn = fmin(dmn, dv);
            vmx = fmax(vmx, out);
            vmn = fmin(vmn, out);
        }
    }
    if (EXTRACT) return;
    block_reduce4(dmx, dmn, vmx, vmn, red);
    if (tid == 0) {
        for (int k = lid; k < nslots; k += gridDim.x) {
            double* pp = p.partials + 4 * (size_t)k;
            const bool mine = k == lid;
            pp[0] = mine ? dmx : -DBL_MAX;
            pp[1] = mine ? dmn : DBL_MAX;
            pp[2] = mine ? vmx : -DBL_MAX;
            pp[3] = mine ? vmn : DBL_MAX;
        }
    }
}

// Order-dependent life (m >= 4): the top merge and the final sum of one order a,
//   Q(a) = -C_f [a > 0] + sum_{y_m<=a} Bin(y_m; a, p_m(a)) sum_{y<=r} w(r, y)
//          T_{m-2}(y_m, c(x_{m-1} + y); r - y),   r = a - y_m,
// whose every table value serves one state (but for the cap), so lanes read them straight
// from memory; p.binq and T are order a's.  The running best stays in the gap buffer
// between the orders' launches (extraction: second best in `sec`, argmax in the policy);
// the last order's launch finishes the state.  YS = 1: a wavefront forms all inner sums of
// its 64 states.  YS = 4: the four wavefronts of a workgroup share 64 states and form the
// inner sums of y_m = w, w + 4, .. side by side, the first adding them in order.
// Bound by reading T_{m-2}, (a + 1)(a + 2)/2 rows of R^(m-1) values: 5.5 TB/s at R = 21,
// m = 5 with YS = 1 (74 us a launch on average, 81 us with YS = 4); small instances wait
// for a lane's short runs of loads one after the other (34,391 states: 1.9 ms for five
// sweeps with YS = 1, 1.6 ms with YS = 4).
template <typename VT, int YS, bool EXTRACT>
__global__ __launch_bounds__(256) void c_order_kernel(CDev p, const void* in_, int a) {
    __shared__ double sum[YS > 1 ? 32 : 1][64];  // inner sum of y_m per state
    if (!EXTRACT && p.ctl->stop) return;
    const int R = p.R, tau = blockIdx.y, j = p.m - 1;
    const int nlo = (int)p.pow_r[j - 1], lane = threadIdx.x & 63;
    const int wave = uniform(threadIdx.x >> 6);
    const int slot = YS > 1 ? blockIdx.x : blockIdx.x * 4 + wave;  // 64 states each
    const int D = slot * 64 + lane;
    const bool ok = D < p.nblk;
    const int x = ok ? D / nlo : 0, lo = ok ? D - x * nlo : 0;
    const ConstF64 bm = (ConstF64)(p.binm + a * R);
    double q = 0.0;
    {
        const ConstI32 pb = (ConstI32)p.pair_base;
        const ConstF64 w = (ConstF64)(p.binq + (size_t)j * R * R);
        const int64_t trow0 = (int64_t)tau * p.npair;
        const VT* T = reinterpret_cast<const VT*>(in_) + lo;
        for (int ym = YS > 1 ? wave : 0; ym <= a; ym += YS) {
            const int r = a - ym;
            const VT* row = T + (trow0 + pb[ym] + r) * p.trow;
            const ConstF64 wr = w + r * R;
            double acc = 0.0;
#pragma unroll 4
            for (int y = 0; y <= r; ++y)
                acc = fma(wr[y], (double)row[-(int64_t)y * p.trow + min(x + y, R - 1) * p.tlo],
                          acc);
            if constexpr (YS > 1)
                sum[ym][lane] = (double)(VT)acc;
            else
                q = fma(bm[ym], (double)(VT)acc, q);
        }
    }
    if constexpr (YS > 1) {
        __syncthreads();
        if (wave != 0) return;
        for (int ym = 0; ym <= a; ++ym) q = fma(bm[ym], sum[ym][lane], q);
    }
    double dmx = -DBL_MAX, dmn = DBL_MAX, vmx = -DBL_MAX, vmn = DBL_MAX;
    if (ok) {
        q = (a > 0 ? -p.cfixed : 0.0) + q;
        const int64_t s = (int64_t)tau * p.nblk + x * nlo + state_lo(p, lo);
        double best = a > 0 ? p.gap[s] : -DBL_MAX, second = -DBL_MAX;
        int arg = 0;
        if (EXTRACT && a > 0) {
            second = p.sec[s];
            arg = p.pi[s];
        }
        if (q > best) {
            second = best;
            best = q;
            arg = a;
        } else if (q > second) {
            second = q;
        }
        if (EXTRACT) {
            p.pi[s] = arg;
            p.sec[s] = second;
            p.gap[s] = a == R - 1 ? best - second : best;
        } else if (a < R - 1) {
            p.gap[s] = best;
        } else {
            const double mu = sizeof(VT) == 4 ? p.ctl->mu : 0.0;
            const VT o = (VT)(best - mu);
            reinterpret_cast<VT*>(p.v_out)[s] = o;
            const double out = (double)o;
            const double dv = out - (double)reinterpret_cast<const VT*>(p.v_in)[s];
            dmx = dmn = dv;
            vmx = vmn = out;
        }
    }
    if (EXTRACT || a < R - 1) return;
    dmx = wave_max(dmx);
    dmn = wave_min(dmn);
    vmx = wave_max(vmx);
    vmn = wave_min(vmn);
    const int nslot = (int)((p.nblk + 63) / 64);
    if (lane == 0 && slot < nslot) {
        double* pp = p.partials + 4 * ((size_t)tau * nslot + slot);
        pp[0] = dmx;
        pp[1] = dmn;
        pp[2] = vmx;
        pp[3] = vmn;
    }
}

// The first two merges take this kernel for 17 to 21 orders: below, the plain fused pair is
// faster (periodic solves of m = 5: 2.68 ms against 3.56 at 13 orders, 1.57 against 1.97 at
// 11, while 21.5 against 31.2 the other way at 19), since a workgroup's antidiagonals no
// longer fill its wavefronts.
template <typename VT>
bool c_merge23_tri_fits(const CDev& p) {
    const size_t r3 = (size_t)p.R * p.R * p.R;
    const size_t rc = c_tri_bound(p.R), rc3 = rc * rc * rc;  // LDS strides are the bound's
    const size_t lds = 2 * rc3 * sizeof(VT) + 16 + 2 * c_tri_weights(p.R) * sizeof(double);
    return p.m >= 5 && p.R > 16 && p.R <= 21 && lds <= (size_t)kLdsMax &&
           p.nblk % (int64_t)r3 == 0 && p.R * p.nblk <= 0x1f000000 &&
           p.R * p.P * (p.nblk / (int64_t)r3) <= 0x7fffffff;
}
template bool c_merge23_tri_fits<double>(const CDev&);
template bool c_merge23_tri_fits<float>(const CDev&);

template <typename VT>
hipError_t launch_merge23_tri(const CDev& p, const void* u, void* out, hipStream_t s) {
    if (!c_merge23_tri_fits<VT>(p)) return hipErrorInvalidConfiguration;
    const int64_t r3 = (int64_t)p.R * p.R * p.R;
    const dim3 grid((unsigned)(p.R * p.P * (p.nblk / r3)));
    const size_t rc = c_tri_bound(p.R);
    const size_t lds = 2 * rc * rc * rc * sizeof(VT) + 16 + 2 * c_tri_weights(p.R) * sizeof(double);
    // one wavefront per 64 / R antidiagonals (14 at R = 21, the most up to R = 21)
    const int tasks = (2 * p.R - 1 + 64 / p.R - 1) / (64 / p.R);
    if (tasks > 16) return hipErrorInvalidConfiguration;
    const dim3 block(64 * std::max(4, tasks));
    hipLaunchKernelGGL((c_merge23_tri_kernel<VT, 21>), grid, block, lds, s, p, u, out);
    return hipGetLastError();
}
template hipError_t launch_merge23_tri<double>(const CDev&, const void*, void*, hipStream_t);
template hipError_t launch_merge23_tri<float>(const CDev&, const void*, void*, hipStream_t);

template <typename VT, bool EXTRACT>
hipError_t launch_c_top(const CDev& p, const void* in, hipStream_t s) {
    const int64_t nlo = p.pow_r[p.m - 2], nlob = (nlo + kLo - 1) / kLo;
    const int64_t nslots = c_partial_slots(p.P, nlo), nwg = nlob * p.P;
    const size_t lds = c_top_lds(p.R, sizeof(VT));
    if (p.m < 4 || p.R > 24 || !p.exogenous || lds > kLdsMax - 1024 || nslots > 0x7fffffff ||
        nwg > nslots || p.tlo % kLo != 0 || p.tlo < nlo || nlo * p.R != p.nblk)
        return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)nwg), block(64 * ((2 * p.R - 1 + 3) / 4));
    const int ns = (int)nslots;
    if (p.R <= 8)
        hipLaunchKernelGGL((c_top_kernel<VT, 8, EXTRACT>), grid, block, lds, s, p, in, ns);
    else if (p.R <= 12)
        hipLaunchKernelGGL((c_top_kernel<VT, 12, EXTRACT>), grid, block, lds, s, p, in, ns);
    else if (p.R <= 16)
        hipLaunchKernelGGL((c_top_kernel<VT, 16, EXTRACT>), grid, block, lds, s, p, in, ns);
    else if (p.R <= 21)
        hipLaunchKernelGGL((c_top_kernel<VT, 21, EXTRACT>), grid, block, lds, s, p, in, ns);
    else
        hipLaunchKernelGGL((c_top_kernel<VT, 24, EXTRACT>), grid, block, lds, s, p, in, ns);
    return hipGetLastError();
}
template hipError_t launch_c_top<double, false>(const CDev&, const void*, hipStream_t);
template hipError_t launch_c_top<float, false>(const CDev&, const void*, hipStream_t);
template hipError_t launch_c_top<double, true>(const CDev&, const void*, hipStream_t);

template <typename VT, bool EXTRACT>
hipError_t launch_c_order(const CDev& p, const void* in, int a, hipStream_t s) {
    if (p.m < 4 || p.R > 32 || p.nblk > 0x7fffffff - 256 || !p.sec) return hipErrorInvalidConfiguration;
    // one wavefront per 64 states once that alone is 16 wavefronts per SIMD
    const unsigned n = (unsigned)((p.nblk + 63) / 64);
    if ((int64_t)n * p.P >= 16384)
        hipLaunchKernelGGL((c_order_kernel<VT, 1, EXTRACT>), dim3((n + 3) / 4, p.P), dim3(256), 0,
                           s, p, in, a);
    else
        hipLaunchKernelGGL((c_order_kernel<VT, 4, EXTRACT>), dim3(n, p.P), dim3(256), 0, s, p, in,
                           a);
    return hipGetLastError();
}
template hipError_t launch_c_order<double, false>(const CDev&, const void*, int, hipStream_t);
template hipError_t launch_c_order<float, false>(const CDev&, const void*, int, hipStream_t);
template hipError_t launch_c_order<double, true>(const CDev&, const void*, int, hipStream_t);

}  // namespace pvi

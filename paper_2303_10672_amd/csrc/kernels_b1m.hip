// Scenario B as the paper runs it (two products, lead time 1), on the FP64 matrix
// cores.  The decomposition into W, Y and the final maximum is the one derived in
// kernels_b1.hip; here each of the three sums is a matrix product.
//
// Write x = (y, X_1) with y the older digits (a "path group").  All R stock vectors of
// one group walk the same FIFO path row_0, row_1, .., row_K (K = sum of y), and their
// sums differ only in the weights:
//   out[X_1][col] = sum_k weight(X_1, k) V[row_k][col],
// an (R x K+1) by (K+1 x columns) product whose columns are whatever the path does not
// touch: the 16 joint orders of a tile in all three kernels.  v_mfma_f64_16x16x4_f64 adds
// its four terms k = 0..3 to the accumulator one after the other with one rounding each
// (checked bit by bit against fma chains over random tiles, zeros and denormals
// included), so the terms, their order and their roundings are those of the vector
// kernels and values are bit-identical.  Terms past a group's path have weight 0 and
// value 0.
//
// Lane l of the instruction holds A[l % 16][l / 16], B[l / 16][l % 16] and the results
// D[l / 16 + 4 r][l % 16], r = 0..3.
//
// Tables: W[x_b][g_a][A] and Y[I_b][x_a][A] with the joint order A fastest, padded to a
// multiple of 16 (nap), so that every kernel reads and writes whole 128-byte lines.
// Padding orders repeat the last real one; the final kernel never lets them win.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>

#include "device_common.h"
#include "pvi_internal.h"

namespace pvi {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef unsigned short us4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;         // wavefronts per workgroup
constexpr int kRow = 16;          // joint orders per tile
constexpr int kSlabRow = 17;      // LDS row of the stage kernels' slabs (written transposed)
constexpr int kTabPad = 48;       // zeros past the demand tables: X_1 + k stays inside

__device__ __forceinline__ d4 mfma(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ double lds_f64(uint32_t a) {
    return *(const __attribute__((address_space(3))) double*)(size_t)a;
}

__device__ __forceinline__ uint32_t lds_u16(uint32_t a) {
    return *(const __attribute__((address_space(3))) uint16_t*)(size_t)a;
}
template <typename T>
__device__ __forceinline__ uint32_t lds_address(const T* p) {
    return (uint32_t)(size_t)(const __attribute__((address_space(3))) T*)p;
}

}  // namespace

// W(A, x_b, g) for one g and one tile of 16 joint orders: the slab V(A^a, g, A^b, .) in
// LDS, row = aged index of b; each wavefront takes path groups of b.
// Bound by writing W: 2.1 GB at 16 orders per product and m = 3 in 0.52 ms (4.1 TB/s; the
// vector kernel took 3.5 ms there).
template <typename VT>
__global__ __launch_bounds__(64 * kWaves) void b1m_stage_w_kernel(B1Dev p) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (!p.extract && p.ctl->stop) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lid = xcd_remap(blockIdx.x, gridDim.x);
    const int g = lid / p.ntile, t = lid - g * p.ntile;
    const int tabn = p.HB + 1 + kTabPad;
    double* slab = reinterpret_cast<double*>(smem);  // [nb1][kSlabRow]
    double* sp = slab + (size_t)p.nb1 * kSlabRow;    // [tabn] P(D_b = h)
    double* sf = sp + tabn;                          // [tabn] P(D_b <= h)
    const VT* V = reinterpret_cast<const VT*>(p.v_in);
    for (int i = tid; i < tabn; i += blockDim.x) {
        sp[i] = i <= p.HB ? p.pb[i] : 0.0;
        sf[i] = i <= p.HB ? p.fb[i] : 0.0;
    }
    const int nact = p.Ra * p.Rb;
    for (int i = tid; i < kRow * p.nb1; i += blockDim.x) {
        const int c = i / p.nb1, b = i - c * p.nb1;
        const int A = min(t * kRow + c, nact - 1), aa = A / p.Rb, ab = A - aa * p.Rb;
        slab[b * kSlabRow + c] =
            (double)V[(int64_t)(aa * p.na1 + g) * p.NB + (int64_t)ab * p.nb1 + b];
    }
    __syncthreads();
    const int kk = lane >> 4, col = lane & 15;
    for (int y = wave; y < p.nb1; y += kWaves) {
        const int K = __builtin_amdgcn_readfirstlane(p.bkk[y]);
        const int nk = K > 0 ? K : 1;  // points k < nk carry h_b < I_b
        const us4* path = reinterpret_cast<const us4*>(p.bpath) + (size_t)y * p.nchb * 4 + kk;
        for (int mt = 0; mt * 16 < p.Rb; ++mt) {
            const int x1 = 16 * mt + col;  // A operand row
            d4 acc = {0.0, 0.0, 0.0, 0.0};
            for (int c = 0; 16 * c < nk; ++c) {
                const us4 row = path[c * 4];
                double v[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) v[s] = slab[row[s] * kSlabRow + col];
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    if (16 * c + 4 * s >= nk) break;
                    const int k = 16 * c + 4 * s + kk;
                    double w = sp[x1 + k];
                    if (k == 0)  // everything up to X_1, or h_b < X_1 with no older stock
                        w = K > 0 ? sf[x1] : (x1 > 0 ? sf[x1 - 1] : 0.0);
                    if (k >= nk) w = 0.0;
                    acc = mfma(w, k < nk ? v[s] : 0.0, acc);
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int xr = 16 * mt + kk + 4 * r;
                // no stock of b: an empty sum (its weight 0 times an infinite value is none)
                if (xr < p.Rb)
                    p.w[((int64_t)(y * p.Rb + xr) * p.na1 + g) * p.nap + t * kRow + col] =
                        y + xr > 0 ? acc[r] : 0.0;
            }
        }
    }
}

// Y(A, I_b, x_a) for one I_b and one tile of joint orders: the slab V(A^a, ., A^b, 0) in
// LDS; each wavefront takes path groups of a.  0.16 ms at 16 orders per product and m = 3
// (1.2 ms with one lane per x_a and scattered weights).
template <typename VT>
__global__ __launch_bounds__(64 * kWaves) void b1m_stage_y_kernel(B1Dev p) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (!p.extract && p.ctl->stop) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t = blockIdx.x, Ib = blockIdx.y;
    double* slab = reinterpret_cast<double*>(smem);  // [na1][kSlabRow]
    const VT* V = reinterpret_cast<const VT*>(p.v_in);
    const int nact = p.Ra * p.Rb;
    for (int i = tid; i < kRow * p.na1; i += blockDim.x) {
        const int g = i / kRow, c = i - g * kRow;
        const int A = min(t * kRow + c, nact - 1), aa = A / p.Rb, ab = A - aa * p.Rb;
        slab[g * kSlabRow + c] = (double)V[(int64_t)(aa * p.na1 + g) * p.NB + (int64_t)ab * p.nb1];
    }
    __syncthreads();
    const int kk = lane >> 4, col = lane & 15;
    const double* J = p.j + (size_t)Ib * p.HA * p.HA;
    const double* JC = p.jc + (size_t)Ib * p.HA * p.HA;
    for (int g = wave; g < p.na1; g += kWaves) {
        const int K = __builtin_amdgcn_readfirstlane(p.akk[g]);
        const us4* path = reinterpret_cast<const us4*>(p.apath) + (size_t)g * p.ncha * 4 + kk;
        for (int mt = 0; mt * 16 < p.Ra; ++mt) {
            const int x1 = min(16 * mt + col, p.Ra - 1);  // rows past the real ones repeat it
            const double* Jr = J + (size_t)(K + x1) * p.HA + x1;
            const double j0 = JC[(size_t)(K + x1) * p.HA + x1];
            d4 acc = {0.0, 0.0, 0.0, 0.0};
            for (int c = 0; 16 * c <= K; ++c) {
                const us4 row = path[c * 4];
                double v[4], w[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int k = 16 * c + 4 * s + kk;
                    v[s] = slab[row[s] * kSlabRow + col];
                    w[s] = Jr[min(k, K)];
                    if (k == 0) w[s] = j0;
                    if (k > K) w[s] = v[s] = 0.0;
                }
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    if (16 * c + 4 * s > K) break;
                    acc = mfma(w[s], v[s], acc);
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int xr = 16 * mt + kk + 4 * r;
                if (xr < p.Ra)
                    p.y[((int64_t)Ib * p.NA + g * p.Ra + xr) * p.nap + t * kRow + col] = acc[r];
            }
        }
    }
}

// Q over the joint orders and the maximum for XB stock vectors x_b of one I_b and
// kWaves * GPW path groups of a.  The workgroup walks the tiles of 16 joint orders; the W
// rows of a tile (all g, 16 orders, XB vectors) come into LDS straight from memory,
// double buffered, and each wavefront forms, per path group, the products of its 16 MT
// values of X_1 with the tile, adds Y and the costs and keeps the maximum per (X_1,
// order % 16) in registers; the 16 columns meet once at the end.
// Sweeps write the maximum to best[x_b][x_a]; the extraction keeps the second best and
// the argmax as well and writes policy and gap.
// What bounds it: the Y rows are shared by the XB vectors of a workgroup and the W tile by
// its path groups, so registers (the running maxima, 2 KB per path group and vector) set
// how much of L2's traffic is saved: 17 GB of Y and 8.6 GB of W per sweep at 16 orders
// per product and m = 3 (XB = 2, GPW = 8), beside 1.5e11 flop.  Those take 3.3 ms at the rate
// of a chain of these instructions alone (45 ns each), and two wavefronts per SIMD hide little
// beside them, so everything else is kept off the vector units: the weights of a step are one
// LDS read, only a path's last step selects, padding orders lose by their cost, both vectors'
// rows lie side by side and the maxima are single instructions.  60 such instructions per
// path group and tile instead of 130: 5.04 ms per sweep, 5.75 before.
template <int XB, int MT, int GPW, bool EXTRACT>
__global__ __launch_bounds__(64 * kWaves) void b1m_final_kernel(B1Dev p) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (!EXTRACT && p.ctl->stop) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nblk = (p.na1 + kWaves * GPW - 1) / (kWaves * GPW);
    const int lid = xcd_remap(blockIdx.x, gridDim.x);
    const int xi = lid / nblk, blk = lid - xi * nblk;
    int xb[XB];
#pragma unroll
    for (int i = 0; i < XB; ++i)
        xb[i] = __builtin_amdgcn_readfirstlane(XB == 1 ? p.xb_order[xi] : p.xb_pair[XB * xi + i]);
    const int na1p = (p.na1 + 7) & ~7;  // a staging instruction moves eight rows
    const int tabn = p.HA + 1 + kTabPad;
    double* ws = reinterpret_cast<double*>(smem);             // [2][na1p][XB][kRow]
    double* wp = ws + (size_t)2 * XB * na1p * kRow;           // [tabn] P(D_a = h)
    double* wg = wp + tabn;                                   // [tabn] P(D_a >= h)
    double* wr = wg + tabn;                                   // [tabn] revenue of I_a at I_b
    // [kWaves * GPW][4 ncha][4]: rows of a path's points, four per step; two steps past the
    // last path are read, not used
    uint16_t* sp = reinterpret_cast<uint16_t*>(wr + tabn);
    int Ib = 0;
    for (int v = xb[0]; v > 0; v /= p.Rb) Ib += v % p.Rb;
    Ib = __builtin_amdgcn_readfirstlane(Ib);
    for (int i = tid; i < tabn; i += blockDim.x) {
        wp[i] = p.pa1[i];  // zeros past HA, as are those of ga
        wg[i] = p.ga[i];
        wr[i] = i < p.HA ? p.rev[(size_t)i * p.HB + Ib] : 0.0;
    }
    // path groups of this workgroup: the list is sorted by path length and dealt to
    // workgroups, then wavefronts, forwards and backwards in turn, so that all get about
    // the same work
    auto group_at = [&](int w, int gi) {
        const int j = gi * kWaves + ((gi & 1) ? kWaves - 1 - w : w);
        const int i = j * nblk + ((j & 1) ? nblk - 1 - blk : blk);
        return i < p.na1 ? p.asort[i] : -1;
    };
    for (int i = tid; i < kWaves * GPW * p.ncha * 4; i += blockDim.x) {
        const int slot = i / (p.ncha * 4), g = group_at(slot / GPW, slot % GPW);
        const int chunk = (i >> 2) - slot * p.ncha, lk = i & 3;
        const us4* src = reinterpret_cast<const us4*>(p.apath);
        const us4 row = src[((size_t)max(g, 0) * p.ncha + chunk) * 4 + lk];
#pragma unroll
        for (int s = 0; s < 4; ++s) sp[(i >> 2) * 16 + s * 4 + lk] = row[s];
    }
    int grp[GPW], Kg[GPW];
#pragma unroll
    for (int gi = 0; gi < GPW; ++gi) {
        grp[gi] = __builtin_amdgcn_readfirstlane(group_at(wave, gi));
        Kg[gi] = __builtin_amdgcn_readfirstlane(p.akk[max(grp[gi], 0)]);
    }
    const int kk = lane >> 4, col = lane & 15;
    const int nrow8 = na1p / 8;
    // tile t into buffer b: eight runs of 16 orders per instruction, 16 bytes per lane
    auto stage = [&](int t, int b) {
        for (int i = wave; i < XB * nrow8; i += kWaves) {
            const int run = i * 8 + (lane >> 3), g = min(run / XB, p.na1 - 1);
            int x = xb[0];
            if constexpr (XB > 1) x = run % XB ? xb[1] : xb[0];
            const double* src =
                p.w + ((int64_t)x * p.na1 + g) * p.nap + t * kRow + (lane & 7) * 2;
            double* dst = ws + ((size_t)b * XB * na1p + i * 8) * kRow;
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)src,
                (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
        }
    };
    double best[GPW][XB][MT][4], second[GPW][XB][MT][4];
    int arg[GPW][XB][MT][4];
#pragma unroll
    for (int gi = 0; gi < GPW; ++gi)
#pragma unroll
        for (int i = 0; i < XB; ++i)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    best[gi][i][mt][r] = second[gi][i][mt][r] = -DBL_MAX;
                    arg[gi][i][mt][r] = 0;
                }
    // Y rows of a path group, one order per lane: a uniform base per group and tile, and the
    // lane's row offsets
    const double* ybase = p.y + (int64_t)Ib * p.NA * p.nap;
    uint32_t yoff[MT][4];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            yoff[mt][r] = (uint32_t)(min(16 * mt + kk + 4 * r, p.Ra - 1) * p.nap + col) * 8u;
    auto load_y = [&](int gi, int t, double (&y)[MT][4]) {
        const char* src = reinterpret_cast<const char*>(
            ybase + (int64_t)max(grp[gi], 0) * (p.Ra * p.nap) + t * kRow);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                y[mt][r] = *reinterpret_cast<const double*>(src + yoff[mt][r]);
    };
    double w0[MT];  // weights of the first four points: the first one's is cumulative
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int x1 = 16 * mt + col;
        w0[mt] = kk == 0 ? p.fa[x1] : p.pa1[x1 + kk];
    }
    // LDS addresses of the lane: column of a tile, weights of the first four points, weights
    // of a path's end and revenue at K = 0
    const uint32_t ws0 = lds_address(ws) + col * 8u, wp0 = lds_address(wp) + (col + kk) * 8u;
    const uint32_t wg0 = lds_address(wg) + col * 8u, wr0 = lds_address(wr) + kk * 8u;
    const uint32_t sp0 = lds_address(sp) + (uint32_t)(wave * GPW * p.ncha) * 32u + kk * 2u;
    stage(0, 0);
    for (int t = 0; t < p.ntile; ++t) {
        // the staged tile has landed, and every wavefront is done with the other buffer
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        double y[2][MT][4];
        load_y(0, t, y[0]);
        if (t + 1 < p.ntile) stage(t + 1, (t + 1) & 1);
        const uint32_t wt = ws0 + (uint32_t)((t & 1) * XB * na1p) * (kRow * 8u);
        const int A = t * kRow + col, aa = A / p.Rb, ab = A - aa * p.Rb;
        // padding orders never win: their cost is the lowest value
        const bool real = A < p.Ra * p.Rb;
        const double cost = real ? fma(-p.cvb, (double)ab, -p.cva * aa) : -DBL_MAX;
#pragma unroll
        for (int gi = 0; gi < GPW; ++gi) {
            if (gi + 1 < GPW) load_y(gi + 1, t, y[(gi + 1) & 1]);
            if (grp[gi] < 0) continue;
            // an opaque copy: the comparisons with K would otherwise be hoisted out of the
            // tile loop for every group at once
            int K = Kg[gi];
            asm volatile("" : "+s"(K));
            const int last = K >> 2;  // step of four points that holds the path's end
            // the operands of a step are on their way while the one before is multiplied, and
            // its rows' places in the tile one step earlier
            struct Step {
                double w[MT], v[XB];
            };
            uint32_t pa = sp0 + (uint32_t)(gi * p.ncha) * 32u, wa = wp0;
            auto load = [&](Step& o, uint32_t row, uint32_t w) {
                const uint32_t from = wt + row * (XB * kRow * 8u);
#pragma unroll
                for (int i = 0; i < XB; ++i) o.v[i] = lds_f64(from + i * (kRow * 8u));
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) o.w[mt] = lds_f64(w + 16 * mt * 8u);
            };
            d4 acc[XB][MT];
            auto multiply = [&](const Step& o) {
#pragma unroll
                for (int i = 0; i < XB; ++i)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) acc[i][mt] = mfma(o.w[mt], o.v[i], acc[i][mt]);
            };
            Step a, c;
            load(a, lds_u16(pa), wa);
            uint32_t row = lds_u16(pa + 8);
            double wl[MT];  // weights of the path's last point
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                a.w[mt] = w0[mt];
                wl[mt] = lds_f64(wg0 + (uint32_t)(K + 16 * mt) * 8u);
                if (K == 0) wl[mt] = 1.0;
            }
#pragma unroll
            for (int i = 0; i < XB; ++i)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[i][mt] = d4{0.0, 0.0, 0.0, 0.0};
            int left = K >> 2;  // steps before the one that holds the path's end
            for (; left >= 2; left -= 2) {
                load(c, row, wa + 32);
                row = lds_u16(pa + 16);
                multiply(a);
                load(a, row, wa + 64);
                row = lds_u16(pa + 24);
                multiply(c);
                wa += 64;
                pa += 16;
            }
            if (left) {
                load(c, row, wa + 32);
                multiply(a);
                a = c;
            }
            // the last step: points before the end as ever, the end, and nothing past it
            {
                const int rem = K & 3;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    a.w[mt] = kk < rem ? a.w[mt] : kk == rem ? wl[mt] : 0.0;
#pragma unroll
                for (int i = 0; i < XB; ++i) a.v[i] = kk <= rem ? a.v[i] : 0.0;
                multiply(a);
            }
            const uint32_t wk = wr0 + (uint32_t)K * 8u;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const double base = cost + lds_f64(wk + (16 * mt + 4 * r) * 8u);
#pragma unroll
                    for (int i = 0; i < XB; ++i) {
                        double q = fma(p.gamma, acc[i][mt][r] + y[gi & 1][mt][r], base);
                        if constexpr (EXTRACT) {
                            if (!real) q = -DBL_MAX;  // also where values are infinite
                            if (q > best[gi][i][mt][r]) {
                                second[gi][i][mt][r] = best[gi][i][mt][r];
                                best[gi][i][mt][r] = q;
                                arg[gi][i][mt][r] = A;
                            } else if (q > second[gi][i][mt][r]) {
                                second[gi][i][mt][r] = q;
                            }
                        } else {
                            best[gi][i][mt][r] = max_f64(best[gi][i][mt][r], q);
                        }
                    }
                }
        }
    }
    // the 16 columns of a state meet; ties go to the lowest order
#pragma unroll
    for (int gi = 0; gi < GPW; ++gi) {
        if (grp[gi] < 0) continue;
#pragma unroll
        for (int i = 0; i < XB; ++i)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    double b = best[gi][i][mt][r], sc = second[gi][i][mt][r];
                    int a = arg[gi][i][mt][r];
                    for (int o = 1; o < 16; o <<= 1) {
                        const double ob = __shfl_xor(b, o, 64);
                        if constexpr (EXTRACT) {
                            const double os = __shfl_xor(sc, o, 64);
                            const int oa = __shfl_xor(a, o, 64);
                            const bool other = ob > b || (ob == b && oa < a);
                            sc = fmax(fmax(sc, os), fmin(b, ob));
                            b = fmax(b, ob);
                            a = other ? oa : a;
                        } else {
                            b = fmax(b, ob);
                        }
                    }
                    best[gi][i][mt][r] = b;
                    second[gi][i][mt][r] = sc;
                    arg[gi][i][mt][r] = a;
                }
                // lane column r writes the state X_1 = 16 mt + kk + 4 r
                double b = best[gi][i][mt][0], sc = second[gi][i][mt][0];
                int a = arg[gi][i][mt][0];
#pragma unroll
                for (int r = 1; r < 4; ++r)
                    if (col == r) {
                        b = best[gi][i][mt][r];
                        sc = second[gi][i][mt][r];
                        a = arg[gi][i][mt][r];
                    }
                const int x1 = 16 * mt + kk + 4 * col;
                if (col < 4 && x1 < p.Ra) {
                    const int64_t xa = (int64_t)grp[gi] * p.Ra + x1;
                    if constexpr (EXTRACT) {
                        const int64_t s = xa * p.NB + xb[i];
                        p.pi[s] = a;
                        p.gap[s] = p.Ra * p.Rb > 1 ? b - sc : 0.0;
                    } else {
                        p.best[(int64_t)xb[i] * p.NA + xa] = b;
                    }
                }
            }
    }
}

// best[x_b][x_a] into V'[x_a][x_b] (64 x 64 tiles through LDS, whole lines both ways),
// with the increments' range.  Writing V' from the final kernel would touch one 8-byte
// value per line.
template <typename VT>
__global__ __launch_bounds__(256) void b1m_finish_kernel(B1Dev p) {
    __shared__ double tile[64][65];
    __shared__ double red[64];
    if (p.ctl->stop) return;
    const int nta = (p.NA + 63) / 64;
    const int tb = blockIdx.x / nta, ta = blockIdx.x - tb * nta;
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int i = w; i < 64; i += 4) {
        const int xb = tb * 64 + i, xa = ta * 64 + l;
        if (xb < p.NB && xa < p.NA) tile[i][l] = p.best[(int64_t)xb * p.NA + xa];
    }
    __syncthreads();
    const double mu = sizeof(VT) == 4 ? p.ctl->mu : 0.0;
    double dmx = -DBL_MAX, dmn = DBL_MAX, vmx = -DBL_MAX, vmn = DBL_MAX;
    for (int i = w; i < 64; i += 4) {
        const int xa = ta * 64 + i, xb = tb * 64 + l;
        if (xb < p.NB && xa < p.NA) {
            const int64_t s = (int64_t)xa * p.NB + xb;
            const VT o = (VT)(tile[l][i] - mu);
            reinterpret_cast<VT*>(p.v_out)[s] = o;
            const double out = (double)o;
            const double dv = out - (double)reinterpret_cast<const VT*>(p.v_in)[s];
            dmx = fmax(dmx, dv);
            dmn = fmin(dmn, dv);
            vmx = fmax(vmx, out);
            vmn = fmin(vmn, out);
        }
    }
    block_reduce4(dmx, dmn, vmx, vmn, red);
    if (threadIdx.x == 0) {
        // this workgroup's slot, and neutral values in the slots past the grid
        for (int k = blockIdx.x; k < p.nslots; k += gridDim.x) {
            double* pp = p.partials + 4 * (size_t)k;
            const bool mine = k == (int)blockIdx.x;
            pp[0] = mine ? dmx : -DBL_MAX;
            pp[1] = mine ? dmn : DBL_MAX;
            pp[2] = mine ? vmx : -DBL_MAX;
            pp[3] = mine ? vmn : DBL_MAX;
        }
    }
}

namespace {

size_t final_lds(const B1Dev& p, int xb, int gpw) {
    const size_t na1p = (size_t)((p.na1 + 7) & ~7);
    return sizeof(double) * (2 * xb * na1p * kRow + 3 * (size_t)(p.HA + 1 + kTabPad)) +
           sizeof(us4) * ((size_t)kWaves * gpw * p.ncha * 4 + 2);
}

template <int XB, int MT, int GPW, bool EXTRACT>
hipError_t launch_final(const B1Dev& p, hipStream_t s) {
    const int64_t nx = XB == 1 ? p.NB : p.npair;
    const int64_t n = nx * ((p.na1 + kWaves * GPW - 1) / (kWaves * GPW));
    const size_t lds = final_lds(p, XB, GPW);
    if (n > 0x7fffffff || lds > kB1mLds) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((b1m_final_kernel<XB, MT, GPW, EXTRACT>), dim3((unsigned)n),
                       dim3(64 * kWaves), lds, s, p);
    return hipGetLastError();
}

template <typename VT, bool EXTRACT>
hipError_t launch_t(const B1Dev& p, hipStream_t s) {
    const size_t lw = sizeof(double) * ((size_t)p.nb1 * kSlabRow +
                                        2 * (size_t)(p.HB + 1 + kTabPad));
    const size_t ly = sizeof(double) * (size_t)p.na1 * kSlabRow;
    if (lw > kB1mLds || ly > kB1mLds || p.Ra > 32 || p.Rb > 32) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((b1m_stage_w_kernel<VT>), dim3((unsigned)(p.na1 * p.ntile)),
                       dim3(64 * kWaves), lw, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((b1m_stage_y_kernel<VT>), dim3((unsigned)p.ntile, (unsigned)p.HB),
                       dim3(64 * kWaves), ly, s, p);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if constexpr (EXTRACT) {
        return p.Ra <= 16 ? launch_final<1, 1, 4, true>(p, s) : launch_final<1, 2, 2, true>(p, s);
    } else {
        // pairs of x_b share the Y rows once the launch fills the chip without them (256
        // workgroups of eight wavefronts, twice over) and both W tiles fit twice in LDS
        const bool pairs = p.npair * ((p.na1 + 63) / 64) >= 512 && final_lds(p, 2, 8) <= kB1mLds;
        if (p.Ra <= 16)
            e = pairs ? launch_final<2, 1, 8, false>(p, s) : launch_final<1, 1, 8, false>(p, s);
        else
            e = pairs ? launch_final<2, 2, 4, false>(p, s) : launch_final<1, 2, 4, false>(p, s);
        if (e != hipSuccess) return e;
        const int64_t nf = (int64_t)((p.NA + 63) / 64) * ((p.NB + 63) / 64);
        if (nf > p.nslots) return hipErrorInvalidConfiguration;
        hipLaunchKernelGGL((b1m_finish_kernel<VT>), dim3((unsigned)nf), dim3(256), 0, s, p);
        return hipGetLastError();
    }
}

}  // namespace

hipError_t launch_backup_b1m(const B1Dev& p, int storage_fp32, int extract, hipStream_t s) {
    if (extract) return launch_t<double, true>(p, s);
    if (storage_fp32) return launch_t<float, false>(p, s);
    return launch_t<double, false>(p, s);
}

bool b1m_fits(const B1Dev& p) {
    const size_t stage = sizeof(double) * ((size_t)std::max(p.na1, p.nb1) * kSlabRow +
                                           2 * (size_t)(p.HB + 1 + kTabPad));
    const int64_t rows = (int64_t)std::max(p.na1, p.nb1);
    return p.Ra <= 32 && p.Rb <= 32 && rows <= 65535 && stage <= kB1mLds &&
           final_lds(p, 1, 8) <= kB1mLds;
}

}  // namespace pvi

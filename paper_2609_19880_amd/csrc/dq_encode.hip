// Append path: bf16 K/V tokens -> fixed-size D-Quant records (Fig. 1, Alg. 1).
//
// Two kernels:
//  * key_mean: eight wavefronts per (batch, head, 128-token window).  They
//    rotate the tokens (Hadamard, Sec. 4.2), whose channels are then summed in
//    token order in fp64, and the channel mean is stored as INT8 with one fp16
//    scale (Sec. 4.2, App. B).
//  * encode: one workgroup per (batch, head, 4 to 64 consecutive tokens; at most
//    32 for per-token streams, see streams_per_group).  Each wavefront takes a
//    stream at a time with its n values spread over the lanes and keeps them in
//    registers through Alg. 1 (FitMinMax -> Drift -> Refit -> fp16 -> Drift); no
//    n x M distortion matrix goes to memory.  A drift counts values beyond level
//    thresholds where the rates allow it (fold_drift); elsewhere it tries every
//    level (drift; the distortions of up to 8 or 16 levels stay in registers,
//    those of more are formed again at every step), and the code length is
//    reduced across the wavefront, as Sec. 4.5 describes for the encoder.  The
//    symbols of the workgroup's streams then go through LDS to lane-per-stream
//    backward rANS (divisions by f as exact multiply-high reciprocals), and the
//    records are written as one contiguous span.
//
// What decides the bytes is fp64 in a fixed order without contraction (this file
// is built with -ffp-contract=off), so the records are bit-identical to the
// reference definition of the format.  The threshold search of long streams runs in
// fp32, but only finds the point that fp64 bounds then certify.
#include <float.h>
#include <limits.h>

#include <type_traits>

#include "dq_common.h"

namespace dq {
namespace {

constexpr int kEncStreams = 64;   // streams per workgroup
// Per-token streams (n = 1024) stage 32: their symbols and records then take about
// 27 KB of a workgroup's 36 KB of LDS up to 16 levels (packed_symbols), so that four
// workgroups share a CU, and 48 of 56 KB above (64 streams would leave one
// wavefront per SIMD).
constexpr int kEncStreamsTok = 32;
constexpr int kEncWaves = 4;
constexpr int kEncThreads = kEncWaves * kWave;
constexpr int kD = 128;           // head_dim of the heads in a per-token stream

__device__ __forceinline__ uint32_t lo32(double v) { return (uint32_t)__double_as_longlong(v); }
__device__ __forceinline__ uint32_t hi32(double v) { return (uint32_t)((uint64_t)__double_as_longlong(v) >> 32); }
__device__ __forceinline__ double join(uint32_t lo, uint32_t hi) {
    return __longlong_as_double((long long)((uint64_t)lo | ((uint64_t)hi << 32)));
}

// Exchanges a's upper half-wavefront with b's lower one (swap_halves), or a's
// odd rows of 16 lanes with b's even ones (swap_rows).
__device__ __forceinline__ void swap_halves(double& a, double& b) {
    const auto l = __builtin_amdgcn_permlane32_swap(lo32(a), lo32(b), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi32(a), hi32(b), false, false);
    a = join(l[0], h[0]);
    b = join(l[1], h[1]);
}
__device__ __forceinline__ void swap_rows(double& a, double& b) {
    const auto l = __builtin_amdgcn_permlane16_swap(lo32(a), lo32(b), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi32(a), hi32(b), false, false);
    a = join(l[0], h[0]);
    b = join(l[1], h[1]);
}

// Lanes hold the channels of a head so that every butterfly partner is one
// DPP operation away: within a row of 16 lanes, channel bit 0, 1, 2, 3 is
// flipped by lane ^ 1, ^ 2, ^ 7 (row_half_mirror), ^ 8 (row_ror:8), i.e. lane
// bits 0 to 3 are c0 ^ c2, c1 ^ c2, c2, c3.
__device__ __forceinline__ int row_channel(int lane) { return (lane & 60) | ((lane ^ ((lane & 4) ? 3 : 0)) & 3); }

template <int BIT>
__device__ __forceinline__ double row_partner(double v) {
    constexpr int ctrl = BIT == 0 ? 0xB1 : BIT == 1 ? 0x4E : BIT == 2 ? 0x141 : 0x128;
    return join((uint32_t)__builtin_amdgcn_mov_dpp((int)lo32(v), ctrl, 0xF, 0xF, false),
                (uint32_t)__builtin_amdgcn_mov_dpp((int)hi32(v), ctrl, 0xF, 0xF, false));
}

// +1 or -1 per channel bit 0 to 3 of the lane.
struct RowSigns {
    double s[4];
};
__device__ __forceinline__ RowSigns row_signs(int lane) {
    const int c = row_channel(lane);
    RowSigns r;
#pragma unroll
    for (int b = 0; b < 4; ++b) r.s[b] = join(0u, 0x3FF00000u | ((uint32_t)((c >> b) & 1) << 31));
    return r;
}

// Stage of channel bit BIT across lanes: the lower lane of a pair (a, b) takes
// a + b, the upper a - b, as partner + (+-1) own value in one fused
// multiply-add, whose product is exact: the same rounding.
template <int BIT>
__device__ __forceinline__ void row_stage(double& v, const RowSigns& sg) {
    v = __builtin_fma(v, sg.s[BIT], row_partner<BIT>(v));
}

__device__ __forceinline__ void pair_stage(double& a, double& b) {
    const double s = a + b, d = a - b;
    a = s;
    b = d;
}

// Channel of a 128-value head that register r of lane l holds before the
// rotation (head_channel) and after it (row_channel(l) + 64 r).  The transform
// moves the register index from channel bit 4 to bit 6: stages 1 to 8 run
// across lanes, stage 16 is inside the lane, and before stages 32 and 64 one
// swap of rows or halves brings the pair into one lane.  34 VALU instructions
// and no LDS traffic per head (72 and 24 LDS permutes with lane stages
// throughout).
__device__ __forceinline__ int head_channel(int lane, int r) {
    return (row_channel(lane) & 15) | (r << 4) | ((lane >> 4) << 5);
}

__device__ __forceinline__ void fwht_head(double& a, double& b, const RowSigns& sg) {
    row_stage<0>(a, sg);
    row_stage<0>(b, sg);
    row_stage<1>(a, sg);
    row_stage<1>(b, sg);
    row_stage<2>(a, sg);
    row_stage<2>(b, sg);
    row_stage<3>(a, sg);
    row_stage<3>(b, sg);
    pair_stage(a, b);
    swap_rows(a, b);
    pair_stage(a, b);
    swap_halves(a, b);
    pair_stage(a, b);
}

// Unnormalized FWHT of a stream of 64 VPL values (head_dim 64 or 256); lane l
// holds elements row_channel(l) + 64 k.  Stages run h = 1, 2, ..., 32 VPL as in
// the definition.
template <int VPL>
__device__ __forceinline__ void fwht_wave(double (&v)[VPL], int lane, const RowSigns& sg) {
#pragma unroll
    for (int k = 0; k < VPL; ++k) {
        row_stage<0>(v[k], sg);
        row_stage<1>(v[k], sg);
        row_stage<2>(v[k], sg);
        row_stage<3>(v[k], sg);
        // (a, b) in every lane: the even and odd rows', then the halves' values
        double a = v[k], b = v[k];
        swap_rows(a, b);
        const double r = a + ((lane & 16) ? -b : b);
        a = b = r;
        swap_halves(a, b);
        v[k] = a + ((lane & 32) ? -b : b);
    }
#pragma unroll
    for (int s = 1; s < VPL; s <<= 1) {
#pragma unroll
        for (int k = 0; k < VPL; ++k)
            if (!(k & s)) pair_stage(v[k], v[k + s]);
    }
}

// Fold-in-halves sums of the n = 64 VPL values of P and of Q (v[i] += v[i +
// len/2] until one is left; element i = row_channel(lane) + 64 k).  After the first lane step the lower half of the
// wavefront carries P's sums and the upper half Q's.
template <int VPL>
__device__ __forceinline__ void fold_sums(const double (&P)[VPL], const double (&Q)[VPL], double& sp, double& sq) {
    double p[VPL], q[VPL];
#pragma unroll
    for (int k = 0; k < VPL; ++k) {
        p[k] = P[k];
        q[k] = Q[k];
    }
#pragma unroll
    for (int len = VPL; len > 1; len >>= 1) {
#pragma unroll
        for (int k = 0; k < len / 2; ++k) {
            p[k] = p[k] + p[k + len / 2];
            q[k] = q[k] + q[k + len / 2];
        }
    }
    swap_halves(p[0], q[0]);
    double s = p[0] + q[0], t = s;
    swap_rows(s, t);
    s = s + t;
    s = s + row_partner<3>(s);
    s = s + row_partner<2>(s);
    s = s + row_partner<1>(s);
    s = s + row_partner<0>(s);
    auto at = [&](int l) {
        return join((uint32_t)__builtin_amdgcn_readlane((int)lo32(s), l),
                    (uint32_t)__builtin_amdgcn_readlane((int)hi32(s), l));
    };
    sp = at(0);
    sq = at(32);
}

__device__ __forceinline__ uint64_t ballot(bool c) { return __builtin_amdgcn_ballot_w64(c); }
__device__ __forceinline__ bool uniform_all(bool c) { return ballot(c) == ~0ull; }

struct DriftCtx {
    const double* rate;    // LDS [M]: R_m / 2^16
    const int32_t* cost;   // LDS [M]
    const float* lam;      // LDS [512]
    int M;
    int cheapest;
    int rmin;
};

// max / min of two non-NaN doubles as one v_max_f64 / v_min_f64 (fmax and
// fmin would first quiet possible signalling NaNs, one more instruction per
// operand).  Distortions and penalties are >= +0, so which of two equal zeros
// comes out never matters.
__device__ __forceinline__ double max_nn(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double min_nn(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// DPP copy of a double; lanes that a row mask leaves out are undefined, which
// a reduction read back from lane 63 never sees.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_copy(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint64_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, ROW_MASK, 0xF, false);
    const uint64_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, ROW_MASK, 0xF, false);
    return __longlong_as_double((long long)(lo | (hi << 32)));
}

// Wavefront max / min of non-NaN doubles with no -0 (the distortions).
template <bool MAX>
__device__ __forceinline__ double wave_ext_nn(double v) {
    auto op = [](double a, double b) { return MAX ? max_nn(a, b) : min_nn(a, b); };
    v = op(v, dpp_copy<0xB1, 0xF>(v));
    v = op(v, dpp_copy<0x4E, 0xF>(v));
    v = op(v, dpp_copy<0x141, 0xF>(v));
    v = op(v, dpp_copy<0x140, 0xF>(v));
    v = op(v, dpp_copy<0x142, 0xA>(v));
    v = op(v, dpp_copy<0x143, 0xC>(v));
    return lane63(v);
}

// The two wait states between an arithmetic result and a lane swap that reads it,
// for results of assembly, which the compiler does not count (max_nn, min_nn).
__device__ __forceinline__ void settle(double& a, double& b) { asm("s_nop 1" : "+v"(a), "+v"(b)); }

// Wavefront minimum and maximum of non-NaN doubles as one reduction of
// max(-x) and max(x) (the sign of a zero result is not kept).
__device__ __forceinline__ void wave_minmax_nn(double& mn, double& mx) {
    double a = join(lo32(mn), hi32(mn) ^ 0x80000000u), b = mx;
    settle(a, b);
    swap_halves(a, b);
    double v = max_nn(a, b), t = v;
    settle(v, t);
    swap_rows(v, t);
    v = max_nn(v, t);
    v = max_nn(v, dpp_copy<0xB1, 0xF>(v));
    v = max_nn(v, dpp_copy<0x4E, 0xF>(v));
    v = max_nn(v, dpp_copy<0x141, 0xF>(v));
    v = max_nn(v, dpp_copy<0x140, 0xF>(v));
    mn = join((uint32_t)__builtin_amdgcn_readlane((int)lo32(v), 0),
              (uint32_t)__builtin_amdgcn_readlane((int)hi32(v), 0) ^ 0x80000000u);
    mx = lane63(v);
}

// Assignment at one lambda: each value takes argmin_m D_im + lambda r_m (ties to
// the smallest m); returns the wavefront's total Q16 cost.  MB > 0: the
// distortions D[k][m] of the M <= MB levels were computed once per drift;
// MB = 0: they are recomputed here (t = s m, u = o + t, e = x - u, D = e e).
// rt: the rates R_m / 2^16 of the MB levels in registers (MB > 0).
template <int VPL, int MB>
__device__ __forceinline__ int assign_cost(const double (&x)[VPL], const double (&D)[VPL][MB > 0 ? MB : 1],
                                           const double (&rt)[MB > 0 ? MB : 1], double s, double o,
                                           double lam, const DriftCtx& c, int (&m)[VPL]) {
    double best[VPL];
    if (MB > 0) {
        const double pen0 = lam * rt[0];
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            best[k] = D[k][0] + pen0;
            m[k] = 0;
        }
#pragma unroll
        for (int mm = 1; mm < (MB > 0 ? MB : 1); ++mm) {
            if (mm < c.M) {
                const double pen = lam * rt[mm];
#pragma unroll
                for (int k = 0; k < VPL; ++k) {
                    const double J = D[k][mm] + pen;
                    m[k] = J < best[k] ? mm : m[k];
                    best[k] = min_nn(best[k], J);
                }
            }
        }
    } else {
        {
            const double t = s * 0.0;
            const double u = o + t;
            const double pen = lam * c.rate[0];
#pragma unroll
            for (int k = 0; k < VPL; ++k) {
                const double e = x[k] - u;
                best[k] = e * e + pen;
                m[k] = 0;
            }
        }
        for (int mm = 1; mm < c.M; ++mm) {
            const double t = s * (double)mm;
            const double u = o + t;
            const double pen = lam * c.rate[mm];
            if constexpr (VPL <= 2) {
                // the costs of all values before any comparison: left alone, the
                // scheduler takes value after value (0.8 % at 64 levels)
                double J[VPL];
#pragma unroll
                for (int k = 0; k < VPL; ++k) {
                    const double e = x[k] - u;
                    J[k] = e * e + pen;
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < VPL; ++k) {
                    m[k] = J[k] < best[k] ? mm : m[k];
                    best[k] = min_nn(best[k], J[k]);
                }
            } else {
#pragma unroll
                for (int k = 0; k < VPL; ++k) {
                    const double e = x[k] - u;
                    const double J = e * e + pen;
                    m[k] = J < best[k] ? mm : m[k];
                    best[k] = min_nn(best[k], J);
                }
            }
        }
    }
    int cst = 0;
#pragma unroll
    for (int k = 0; k < VPL; ++k) cst += c.cost[m[k]];
    return wave_sum_i32(cst);
}

// Drift(x, s, o, r, B) of Alg. 1: bisection on log2(lambda) over a
// 40-octave bracket below hi = ceil(log2(8 (max D - min D))), lambda on the
// 2^(U/512) grid, 12 steps, assignment at the final hi; nearest cheapest
// symbol if even that overflows; cheapest symbol if all distortions are equal.
template <int VPL, int MB>
__device__ void drift(const double (&x)[VPL], double s, double o, int64_t budget,
                      const DriftCtx& c, int (&m)[VPL]) {
    double D[VPL][MB > 0 ? MB : 1], rt[MB > 0 ? MB : 1];
    double dmax = -DBL_MAX, dmin = DBL_MAX;
    if (MB > 0) {
#pragma unroll
        for (int mm = 0; mm < (MB > 0 ? MB : 1); ++mm) {
            rt[mm] = mm < c.M ? c.rate[mm] : 0.0;
            const double t = s * (double)mm;
            const double u = o + t;
#pragma unroll
            for (int k = 0; k < VPL; ++k) {
                const double e = x[k] - u;
                D[k][mm] = e * e;
                if (mm < c.M) {
                    dmax = max_nn(dmax, D[k][mm]);
                    dmin = min_nn(dmin, D[k][mm]);
                }
            }
        }
    } else {
        for (int mm = 0; mm < c.M; ++mm) {
            const double t = s * (double)mm;
            const double u = o + t;
#pragma unroll
            for (int k = 0; k < VPL; ++k) {
                const double e = x[k] - u;
                const double Dv = e * e;
                dmax = max_nn(dmax, Dv);
                dmin = min_nn(dmin, Dv);
            }
        }
    }
    dmax = wave_ext_nn<true>(dmax);
    dmin = wave_ext_nn<false>(dmin);
    if (dmax == dmin) {
#pragma unroll
        for (int k = 0; k < VPL; ++k) m[k] = c.cheapest;
        return;
    }
    int ex = 0;
    const double mant = frexp(8.0 * (dmax - dmin), &ex);
    const int hi = (mant == 0.5) ? ex - 1 : ex;
    int u_hi = hi * kLambdaSteps;
    int u_lo = u_hi - kBracketUnits;
    // the code length is an int: comparing it with the budget clamped to
    // INT_MAX decides the same and stays a scalar compare
    const int budget32 = (int)(budget < INT_MAX ? budget : INT_MAX);
    // m holds the assignment at u_hi once a step has moved u_hi: the final
    // assignment at u_hi is then that step's, and within the budget.  With 16
    // values per lane the copy's registers cost more occupancy than the
    // final assignment it saves, which is then recomputed.
    constexpr bool kKeepHi = VPL <= 4;
    bool at_hi = false;
    for (int it = 0; it < kBisectSteps; ++it) {
        const int u_mid = (u_lo + u_hi) >> 1;
        const double lam = ldexp((double)c.lam[u_mid & (kLambdaSteps - 1)], u_mid >> 9);
        int tmp[VPL];
        const int cst = assign_cost<VPL, MB>(x, D, rt, s, o, lam, c, tmp);
        if (cst <= budget32) {
            u_hi = u_mid;
            if (kKeepHi) {
                at_hi = true;
#pragma unroll
                for (int k = 0; k < VPL; ++k) m[k] = tmp[k];
            }
        } else {
            u_lo = u_mid;
        }
    }
    if (at_hi) return;
    const double lam = ldexp((double)c.lam[u_hi & (kLambdaSteps - 1)], u_hi >> 9);
    const int cst = assign_cost<VPL, MB>(x, D, rt, s, o, lam, c, m);
    if (cst > budget32) {
        double best[VPL];
#pragma unroll
        for (int k = 0; k < VPL; ++k) best[k] = DBL_MAX;
        for (int mm = 0; mm < c.M; ++mm) {
            if (c.cost[mm] != c.rmin) continue;
            const double t = s * (double)mm;
            const double u = o + t;
#pragma unroll
            for (int k = 0; k < VPL; ++k) {
                const double e = x[k] - u;
                const double Dv = e * e;
                if (Dv < best[k]) {
                    best[k] = Dv;
                    m[k] = mm;
                }
            }
        }
    }
}

// ------------------------------------------------------------ folded drift
//
// The same assignment without trying every level at every step.  With the
// symmetric tables of Sec. 4.2 a value's level depends only on its distance
// from the middle of the grid, c = o + s (M - 1) / 2: for |x - c| = y, moving
// from one level to the next one outward changes the Lagrangian cost by
//     (D + lambda r)(outer) - (D + lambda r)(inner) = -(z - T_j),
//     z = 2 s y,   T_j = 2 s^2 (j + 1 or j + 1/2) + lambda (r_outer - r_inner),
// so while the T_j increase in j the level is the number of T_j below z, and
// the code length of the stream is n r_centre + sum_j (r_outer - r_inner)
// #{i: z_i > T_j}: one comparison per value and threshold, a population count
// and a scalar multiply-add per threshold, against five VALU instructions per
// value and level before.  A convex rate makes the T_j increase for every
// lambda; at most the outermost level may break it (its frequency is rounded up
// to an integer), and then the level before it drops out where T_last < T_last-1,
// both thresholds taking the mean.
//
// The thresholds decide in exact arithmetic, the format in fp64 with Alg. 1's
// operation order.  The two agree wherever no z lies within delta of its
// threshold, delta bounding both sides' rounding: with K >= |x|, |u_m|, the
// fp64 costs are off by at most 2^-53 (14 K^2 + 30 lambda) and z - T_j by
// 2^-50 (K^2 + 16 lambda); delta = 2^-44 (K^2 + 16 lambda) leaves a factor of
// 16.  fold_drift therefore searches with the thresholds and then certifies
// what Alg. 1's bisection returns, U:
//  * at U no z is within delta of a threshold, and the code length fits;
//  * one grid step below U it does not fit, whatever the values within delta
//    of a threshold do (the count at T_j + delta).
// The other points that the bisection visits are at least one grid step
// (0.68 %) away, and there a value's fp64 choice m against its certain choice g
// at U (or a step below) obeys (lambda - lambda_U) (r_m - r_g) <= 2 E, E the
// error of a cost near the minimum, at most 2^-53 (6 K S + 22 K sqrt(lambda) +
// 30 lambda) with S = s + the distance of the values from the grid.  Rates are
// multiples of 2^-16, so r_m <= r_g (>= below U) once lambda >= 2^-25 K S:
// every point above U fits and every point below does not, and the bisection
// ends at U.  When already the nearest levels fit, the bisection goes down to
// its last grid point: no z may lie between T_j(0) - delta and T_j(lambda_top) +
// delta for lambda_top = 2^-29 K S, below which every assignment is then the
// same and above which the bound holds.
// A stream that does not pass (a value within 2^-44 of a tie, no certain
// bracket) goes through drift() as it is.
constexpr int kFoldMax = (DQ_MAX_LEVELS - 1) / 2;
struct FoldArgs {
    int32_t J;             // thresholds, (M - 1) / 2
    int32_t base;          // n R_centre
    int32_t pool;          // the outermost rate difference is below the one before
    int32_t even;          // M even: the centre is a boundary between two levels
    double off;            // distance of the first threshold from the centre in steps: 1 or 1/2
    int32_t W[kFoldMax];   // R_outer - R_inner (Q16)
    double w[kFoldMax];    // the same as a rate
    float wf[kFoldMax];
};

// T_j(lambda) + d in precision F, JM of them in registers or (JM = 0) formed
// one at a time, the pooled pair together.
template <typename F, int JM, bool POOL>
struct Thresholds {
    const FoldArgs& f;
    F ss;                                      // 2 s^2
    F B[JM > 0 ? JM : 1];
    __device__ __forceinline__ Thresholds(const FoldArgs& f_, F ss_) : f(f_), ss(ss_) {
#pragma unroll
        for (int j = 0; j < JM; ++j) B[j] = ss * ((F)j + (F)f.off);
    }
    __device__ __forceinline__ F raw(int j, F lam) const {
        const F b = JM > 0 ? B[JM > 0 ? j : 0] : ss * ((F)j + (F)f.off);
        if constexpr (sizeof(F) == 4) return __builtin_fmaf(lam, f.wf[j], b);
        else return __builtin_fma(lam, f.w[j], b);
    }
    __device__ __forceinline__ int count() const { return JM > 0 ? JM : f.J; }
    __device__ __forceinline__ F at(int j, F lam) const {
        const F T = raw(j, lam);
        const int J = count();
        if constexpr (POOL) {
            if (j >= J - 2) {
                const F To = raw(2 * J - 3 - j, lam), m = (F)0.5 * (T + To);
                return j == J - 2 ? (T < m ? T : m) : (T > m ? T : m);
            }
        }
        return T;
    }
};

// Code length beyond f.base at lambda.
template <typename F, int VPL, int JM, bool POOL>
__device__ __forceinline__ int fold_cost(const F (&z)[VPL], const Thresholds<F, JM, POOL>& th, F lam) {
    int cost = 0;
    auto add = [&](int j) {
        const F T = th.at(j, lam);
        int c = 0;
#pragma unroll
        for (int k = 0; k < VPL; ++k) c += (int)__popcll(ballot(z[k] > T));
        cost += c * th.f.W[j];
    };
    if constexpr (JM > 0) {
#pragma unroll
        for (int j = 0; j < JM; ++j) add(j);
    } else {
        for (int j = 0; j < th.f.J; ++j) add(j);
    }
    return cost;
}

// ceil(log2(8 d)) of a positive normal double held in scalar registers.
__device__ __forceinline__ int ceil_log2_8(double d) {
    const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)lo32(d)) |
                       ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)hi32(d)) << 32);
    return (int)((u - 1) >> 52) - 1022 + 3;
}

// Drift by thresholds; false if the result is not certain (m is then not
// set).  xmin, xmax: extrema of the stream.
template <int VPL, int JM, bool POOL>
__device__ __forceinline__ bool fold_drift(const double (&x)[VPL], double xmin, double xmax, double s, double o,
                                           int64_t budget, const DriftCtx& c, const FoldArgs& f, int (&m)[VPL]) {
    const int M = c.M;
    const double top = s * (double)(M - 1), uM = o + top;
    const double K = max_nn(fabs(xmin), fabs(xmax)) + fabs(o) + top;
    const double out = max_nn(o - xmin, xmax - uM), S = s + max_nn(out, 0.0);
    // (also false for a scale of 0 and for infinities and NaN)
    if (!uniform_all(s > 0.0 && K <= 65536.0 * s)) return false;
    // max D and min D as Alg. 1 computes them: u_m and x - u_m round
    // monotonically, so the largest distortion is that of an extreme value at
    // an extreme level; the smallest lies between 0 and those of the extreme
    // values at their own ends, and is computed only where that leaves the
    // bracket open
    auto sq = [](double e) { return e * e; };
    const double dmax = max_nn(max_nn(sq(xmax - o), sq(xmin - o)), max_nn(sq(xmax - uM), sq(xmin - uM)));
    double dlow = min_nn(sq(xmin - o), sq(xmax - uM));
    if (!uniform_all(dmax - dlow > 1e-280)) return false;
    int hi = ceil_log2_8(dmax - dlow);
    if (hi != ceil_log2_8(dmax)) {
        for (int mm = 0; mm < M; ++mm) {
            const double t = s * (double)mm;
            const double u = o + t;
#pragma unroll
            for (int k = 0; k < VPL; ++k) dlow = min_nn(dlow, sq(x[k] - u));
        }
        dlow = wave_ext_nn<false>(dlow);
        hi = ceil_log2_8(dmax - dlow);
    }
    const int u0 = hi * kLambdaSteps - kBracketUnits;
    // what the budget leaves beyond the centre level's rate for every value (a
    // scalar, so that the search's branches and bracket stay scalar)
    const int room = __builtin_amdgcn_readfirstlane((int)(budget < INT_MAX / 2 ? budget : INT_MAX / 2)) - f.base;
    const int room1 = room + 1;

    const double s2 = s + s, ss = s2 * s, ctr = o + s * (0.5 * (double)(M - 1));
    const double d0 = K * K * 0x1p-44;
    auto delta = [&](double lam) { return __builtin_fma(lam, 0x1p-40, d0); };
    auto lam_at = [&](int k) {                 // lambda of grid point k of the bracket, as Alg. 1 has it
        const int u = u0 + 5 * k;
        return ldexp((double)c.lam[u & (kLambdaSteps - 1)], u >> 9);
    };
    // all the search has to find is the grid point to certify: in fp32 where
    // the z are many registers (then formed again for the certificate)
    constexpr bool kWide = VPL <= 4;
    using F = std::conditional_t<kWide, double, float>;
    F zs[VPL];
#pragma unroll
    for (int k = 0; k < VPL; ++k) zs[k] = (F)fabs((x[k] - ctr) * s2);
    const Thresholds<F, JM, POOL> ts(f, (F)ss);
    const Thresholds<double, JM, POOL> th(f, ss);
    int cnt[VPL];
#pragma unroll
    for (int k = 0; k < VPL; ++k) cnt[k] = 0;
    double near = ss;                          // smallest distance of a z from its decisions
    double dc = d0;                            // and what makes them certain
    // f(z, value) over the stream, j-th threshold pair outside or inside: the
    // z of many values are formed where they are used
    auto each = [&](auto&& body) {
        if constexpr (JM > 0) {
#pragma unroll
            for (int k = 0; k < VPL; ++k) {
                const double z = kWide ? (double)zs[k] : fabs((x[k] - ctr) * s2);
#pragma unroll
                for (int j = 0; j < JM; ++j) body(k, j, z);
            }
        } else {
            for (int j = 0; j < f.J; ++j) {
#pragma unroll
                for (int k = 0; k < VPL; ++k) body(k, j, kWide ? (double)zs[k] : fabs((x[k] - ctr) * s2));
            }
        }
    };
    if (fold_cost(zs, ts, (F)0) <= room) {
        // the nearest levels fit: the last grid point.  No z between T_j(0) -
        // delta and T_j(lambda_top) + delta
        const double lt = max_nn(0x1p-29 * K * S, 2.0 * lam_at(1)), dt = delta(lt);
        int cost = 0;
        uint64_t between = 0;
        each([&](int k, int j, double z) {
            const bool above = z > th.at(j, 0.0) - d0;
            const uint64_t a = ballot(above);
            between |= a ^ ballot(z > th.at(j, lt) + dt);
            cost += (int)__popcll(a) * f.W[j];
            cnt[k] += above ? 1 : 0;
        });
        if (between || cost > room || !uniform_all(16.0 * lt <= ss)) return false;
    } else {
        // the bracket's upper 20 octaves, Alg. 1's bisection less its first
        // step: lambda goes with it by the factors 2^(+-5), 2^(+-2.5), ...,
        // as high words of doubles (2e-7) or as fp32
        constexpr uint32_t kUp[11] = {
            0x40400000, 0x4016A09E, 0x400306FE, 0x3FF8ACE5, 0x3FF3DEA6, 0x3FF1D487,
            0x3FF0E3EC, 0x3FF0706B, 0x3FF037D4, 0x3FF01BD2, 0x3FF00DE3};
        constexpr uint32_t kDn[11] = {
            0x3FA00000, 0x3FC6A09E, 0x3FDAE8A0, 0x3FE4BFDB, 0x3FE9C492, 0x3FECB721,
            0x3FEE502F, 0x3FEF252B, 0x3FEF91D8, 0x3FEFC8BC, 0x3FEFE452};
        constexpr uint32_t kUpF[11] = {
            0x42000000, 0x40B504F3, 0x401837F0, 0x3FC5672A, 0x3F9EF532, 0x3F8EA43A,
            0x3F871F62, 0x3F838359, 0x3F81BEA1, 0x3F80DE8F, 0x3F806F17};
        constexpr uint32_t kDnF[11] = {
            0x3D000000, 0x3E3504F3, 0x3ED744FD, 0x3F25FED7, 0x3F4E248C, 0x3F65B907,
            0x3F728177, 0x3F79295A, 0x3F7C8EC0, 0x3F7E45E2, 0x3F7F2291};
        int klo = 2048;
        F lam = (F)ldexp(1.0, hi - 10);
#pragma unroll
        for (int it = 0; it < 11; ++it) {
            // all ones if it fits (selects on a scalar condition cost two
            // more scalar instructions each than masking)
            uint32_t fits;
            asm("s_ashr_i32 %0, %1, 31" : "=s"(fits) : "s"(fold_cost(zs, ts, lam) - room1) : "scc");
            klo += (1024 >> it) & ~fits;
            if constexpr (kWide) lam *= join(0u, kUp[it] ^ ((kUp[it] ^ kDn[it]) & fits));
            else lam *= __uint_as_float(kUpF[it] ^ ((kUpF[it] ^ kDnF[it]) & fits));
        }
        // certify klo + 1; a value within the fp32 search's rounding of its
        // threshold may have moved it by a grid point
        double lg, lb, dg;
        int cg, cb;
        auto certify = [&]() {
            lg = lam_at(klo + 1);
            lb = lam_at(klo);
            dg = delta(lg);
            const double db = delta(lb);
            cg = cb = 0;
            each([&](int k, int j, double z) {
                const double T = th.at(j, lg);
                const bool above = z > T;
                cg += (int)__popcll(ballot(above)) * f.W[j];
                cb += (int)__popcll(ballot(z > th.at(j, lb) + db)) * f.W[j];
                near = min_nn(near, fabs(z - T));
                cnt[k] += above ? 1 : 0;
            });
        };
        if (klo == 4095) return false;
        certify();
        if constexpr (!kWide) {
#pragma unroll 1
            for (int tries = 0; (cb <= room || cg > room) && tries < 2; ++tries) {
                klo += cb <= room ? -1 : 1;
                if (klo == 4095) return false;
                near = ss;
#pragma unroll
                for (int k = 0; k < VPL; ++k) cnt[k] = 0;
                certify();
            }
        }
        if (cb <= room || cg > room) return false;
        if (!uniform_all(lb >= 0x1p-25 * K * S)) return false;
        if constexpr (POOL) {
            // the outermost thresholds are not about to trade places, and a
            // pooled pair stays above the one before it
            const int j = f.J - 1;
            const double wa = f.w[j - 1], wb = f.w[j];
            const double gap_g = ss + lg * (wb - wa), gap_b = ss + lb * (wb - wa);
            bool ok = fabs(gap_g) > 8.0 * dg && fabs(gap_b) > 8.0 * dg;
            if (j >= 2) ok = ok && 1.5 * ss + lg * (0.5 * (wa + wb) - f.w[j - 2]) > 8.0 * dg;
            if (!uniform_all(ok)) return false;
        }
        dc = dg;
    }
    const int below = (M - 1) / 2, above = M / 2;
#pragma unroll
    for (int k = 0; k < VPL; ++k) {
        m[k] = x[k] < ctr ? below - cnt[k] : above + cnt[k];
        if (f.even) near = min_nn(near, fabs((x[k] - ctr) * s2));
    }
    return uniform_all(near > dc);
}

__device__ __forceinline__ uint16_t f64_to_half_bits(double v) {
    return __half_as_ushort(__float2half_rn((float)v));
}

// Input channel of register k of lane l of a head (or of a 64- or 256-value
// stream): the channels fwht_head starts from, or with rotate = 0 (the input
// is already in the rotated basis) the ones it ends with.
template <int VPL>
__device__ __forceinline__ int in_channel(int lane, int k, int rotate) {
    return VPL == 2 && rotate ? head_channel(lane, k) : row_channel(lane) + kWave * k;
}

// (the address space stated: the compiler loses it in some instantiations)
#define GLOBAL_PTR(T, p) reinterpret_cast<__attribute__((address_space(1))) T*>(reinterpret_cast<uintptr_t>(p))

template <int VPL>
__device__ __forceinline__ void load_raw(const uint16_t* src, uint16_t (&r)[VPL], int lane, int rotate) {
#pragma unroll
    for (int k = 0; k < VPL; ++k) r[k] = GLOBAL_PTR(const uint16_t, src)[in_channel<VPL>(lane, k, rotate)];
}

template <int VPL>
__device__ __forceinline__ void rotated(const uint16_t (&r)[VPL], double (&v)[VPL], int lane, const RowSigns& sg, int rotate) {
#pragma unroll
    for (int k = 0; k < VPL; ++k) v[k] = (double)bf16_to_f32(r[k]);
    if (rotate) {
        if constexpr (VPL == 2) fwht_head(v[0], v[1], sg);
        else fwht_wave<VPL>(v, lane, sg);
    }
}

// Key means: a workgroup of eight wavefronts per (window, KV head, sequence).
// Each wavefront requests its 16 tokens up front and rotates them two at a
// time; every 16 rotated tokens go through LDS (two buffers, one barrier each)
// to thread j < n, which adds channel j's values in token order.  One wavefront
// per window, rotating and adding 128 tokens in turn, was bound by that chain.
constexpr int kMeanWaves = 8;
constexpr int kMeanBatch = 2 * kMeanWaves;         // tokens per buffer
constexpr int kMeanRounds = DQ_MEAN_WINDOW / kMeanBatch;

template <int VPL>
__global__ __launch_bounds__(kMeanWaves* kWave) void key_mean_kernel(const uint16_t* __restrict__ kv,
                                                         int64_t sb, int64_t st, int64_t sh, int H,
                                                         int t0, int t_cap, Pages pg,
                                                         int8_t* __restrict__ mean_q,
                                                         uint16_t* __restrict__ mean_scale,
                                                         uint32_t* status, int rotate) {
    constexpr int n = kWave * VPL;
    __shared__ double buf[2][kMeanBatch][n];
    __shared__ double s_max[kMeanWaves];
    const int w = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const uint16_t* base = kv + (int64_t)b * sb + (int64_t)h * sh + (int64_t)w * DQ_MEAN_WINDOW * st;
    uint16_t raw[kMeanRounds][2][VPL];
#pragma unroll
    for (int r = 0; r < kMeanRounds; ++r)
#pragma unroll
        for (int u = 0; u < 2; ++u)
            load_raw<VPL>(base + (int64_t)(r * kMeanBatch + 2 * wave + u) * st, raw[r][u], lane, rotate);
    const RowSigns sg = row_signs(lane);
    const int ch = row_channel(lane);
    double acc = 0.0;
#pragma unroll
    for (int r = 0; r < kMeanRounds; ++r) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            double v[VPL];
            rotated<VPL>(raw[r][u], v, lane, sg, rotate);
#pragma unroll
            for (int k = 0; k < VPL; ++k) buf[r & 1][2 * wave + u][ch + kWave * k] = v[k];
        }
        __syncthreads();
        if (tid < n) {
#pragma unroll
            for (int t = 0; t < kMeanBatch; ++t) acc = acc + buf[r & 1][t][tid];
        }
    }
    const double mu = acc / (double)DQ_MEAN_WINDOW;
    const bool mine = tid < n;
    const double wmax = wave_max(mine ? fmax(0.0, fabs(mu)) : 0.0);
    if (lane == 0) s_max[wave] = wmax;
    const int nonfinite = __syncthreads_or(mine && !isfinite(mu));
    double amax = 0.0;
#pragma unroll
    for (int i = 0; i < VPL; ++i) amax = fmax(amax, s_max[i]);
    const uint16_t sbits = f64_to_half_bits(amax / 127.0);
    const double sc = (double)__half2float(__ushort_as_half(sbits));
    bool bad_page = false;
    const int64_t widx = window_index(pg, H, t_cap, b, h, t0 / DQ_MEAN_WINDOW + w, bad_page);
    if (bad_page) {             // nothing is written through a block-table entry outside the pool
        if (tid == 0 && status) atomicOr(status, DQ_STATUS_PAGE);
        return;
    }
    if (mine) {
        double qv = 0.0;
        if (sc > 0.0) qv = fmin(127.0, fmax(-127.0, rint(mu / sc)));
        mean_q[widx * n + tid] = (int8_t)qv;
    }
    if (tid == 0) {
        mean_scale[widx] = sbits;
        if ((nonfinite || !isfinite(sc)) && status) atomicOr(status, DQ_STATUS_RANGE);
    }
}

struct EncArgs {
    TabArgs ta;
    const uint16_t* kv;
    int64_t sb, st, sh;
    int H, t0, n_new, t_cap;
    int ns;                      // streams per workgroup, a power of two
    Pages pg;                    // records and key means: contiguous or paged
    int rec_stride;              // per-token records: bytes per record slot (multiple of 16)
    uint8_t* records;
    const int8_t* mean_q;        // NULL for values
    const uint16_t* mean_scale;
    uint32_t* status;
    int rotate;                  // 0: the input is already in the rotated basis
    FoldArgs f;
};

// LDS of a workgroup: fixed arrays, then per stream the symbols (one padding
// dword per row: the coder's lanes read the same position of 64 rows, which
// then fall in different banks) and the record bytes as the coder emits them,
// from the row's end backwards (an odd number of dwords per row).
struct EncLayout {
    int rate, cost, lam, ent, mean, budget, s16, o16, flag, state, emitted, sym, rec, total;
    int sym_row, rec_row;
};

// Symbols of per-token streams of up to 16 levels are packed, elements i and i +
// 64 of every 128 in one byte: four workgroups of 32 1024-value streams then
// share a CU.
__host__ __device__ inline bool packed_symbols(bool tok, int M) { return tok && M <= 16; }

__host__ __device__ inline EncLayout enc_layout(int n, int C, int ns, bool tok, int M) {
    EncLayout L;
    int off = 0;
    auto take = [&](int bytes) {
        const int at = off;
        off = (off + bytes + 15) & ~15;
        return at;
    };
    L.rate = take(8 * DQ_MAX_LEVELS);
    L.cost = take(4 * DQ_MAX_LEVELS);
    L.lam = take(4 * kLambdaSteps);
    L.ent = take(16 * DQ_MAX_LEVELS);
    L.mean = take(tok ? 4 * n : 0);
    L.budget = take(8 * ns);
    L.s16 = take(2 * ns);
    L.o16 = take(2 * ns);
    L.flag = take(4 * ns);
    L.state = take(4 * ns);
    L.emitted = take(4 * ns);
    L.sym_row = (packed_symbols(tok, M) ? n / 2 : n) + 4;
    L.rec_row = 4 * (((C + 3) / 4) | 1);
    L.sym = take(ns * L.sym_row);
    L.rec = take(ns * L.rec_row + 8);
    L.total = off;
    return L;
}

// Nearest level on the grid (o, s): argmin_m (x - (o + s m))^2, the same
// arithmetic as the distortions of a drift, ties to the smallest m.
template <int VPL>
__device__ __forceinline__ void nearest(const double (&x)[VPL], double s, double o, int M, int (&m)[VPL]) {
    double best[VPL];
#pragma unroll
    for (int k = 0; k < VPL; ++k) {
        best[k] = DBL_MAX;
        m[k] = 0;
    }
    for (int mm = 0; mm < M; ++mm) {
        const double t = s * (double)mm;
        const double u = o + t;
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const double e = x[k] - u;
            const double D = e * e;
            if (D < best[k] || mm == 0) {
                best[k] = D;
                m[k] = mm;
            }
        }
    }
}

// Wavefronts per SIMD that the registers are held to.  The folded search: six for
// streams of up to 128 values with two thresholds (4 x 8192 tokens, K and V, 787
// us, 808 with five and 837 with eight), five with more (four thresholds spill with
// six: 328 and 314 us for 2 x 4096 tokens), four for longer streams (per token
// their LDS fits four workgroups).  Where every step tries every level: as many as
// the distortions leave room for in registers (three with those of 16 levels or of
// 256-value streams), else six or five, which a few registers more would cost:
// unbounded, 2 x 16384 tokens of 8 heads, head_dim 256, 2 levels take 1454 us, not
// 1146, 1 x 8192, 64 levels 6.13 ms, not 5.98.
__host__ __device__ constexpr int enc_waves(int vpl, int mb, bool tok, int jm) {
    if (jm >= 0) return tok || vpl > 2 ? 4 : jm == 2 ? 6 : 5;
    if (mb == 0) return vpl <= 2 ? 6 : vpl == 4 && !tok ? 5 : 3;
    return mb == 16 || tok || vpl == 4 ? 3 : 1;
}

// What bounds it: instruction issue (eleven steps of the search per drift, then the
// coder's 128 serial steps per lane): vector instructions are 79 % of the time at 4
// cycles each, scalar ones 71 % at one a cycle.  Memory, register spills included
// (about 1 GB of writes beyond the 0.15 GB of records at 16 x 32768 tokens), moves
// 0.5 TB/s.
// Keys and values together, 4 x 8192 tokens of 8 heads, 36-byte records (6 levels): 2398 us when every step of the
// search assigned every level anew in 64 bits, 792 with the folded drift;
// 48- and 32-byte records, 2 x 4096: 981 and 320; per token, 4 x 8192: 2936 and
// 777; 4 x 128, with key means and grids that fill the CUs: 475 and 63.
// JM: thresholds of the folded drift in registers (fold_drift), 0: any number,
// -1: the rates do not allow it, every step tries every level (drift with MB).
// POOL: the outermost two may have to share their mean.
// FIXED: the fixed-width comparator of App. B -- the same preprocessing and
// refit with nearest-level rounding in place of both drifts, and b-bit
// symbols (M = 2^b, b = 8 (C - 4) / n rounded down) packed after the 4-byte
// header, least significant bit first, instead of the rANS payload.
template <int VPL, int MB, bool TOK, int JM, bool POOL, bool FIXED = false>
__global__ __launch_bounds__(kEncThreads, enc_waves(VPL, MB, TOK, JM)) void encode_kernel(EncArgs a) {
    constexpr int n = kWave * VPL;
    constexpr int HV = TOK ? 2 : VPL;             // registers per head
    constexpr int NH = VPL / HV;                  // heads per stream
    extern __shared__ __align__(16) uint8_t smem[];
    const TabArgs& ta = a.ta;
    const int C = ta.C, ns = a.ns;
    const EncLayout L = enc_layout(n, C, ns, TOK, ta.M);
    double* s_rate = reinterpret_cast<double*>(smem + L.rate);
    int32_t* s_cost = reinterpret_cast<int32_t*>(smem + L.cost);
    float* s_lam = reinterpret_cast<float*>(smem + L.lam);
    uint4* s_ent = reinterpret_cast<uint4*>(smem + L.ent);    // coder entry per symbol
    float* s_mean = reinterpret_cast<float*>(smem + L.mean);
    int64_t* s_budget = reinterpret_cast<int64_t*>(smem + L.budget);
    uint16_t* s_s16 = reinterpret_cast<uint16_t*>(smem + L.s16);
    uint16_t* s_o16 = reinterpret_cast<uint16_t*>(smem + L.o16);
    int32_t* s_flag = reinterpret_cast<int32_t*>(smem + L.flag);
    uint32_t* s_state = reinterpret_cast<uint32_t*>(smem + L.state);
    int32_t* s_emitted = reinterpret_cast<int32_t*>(smem + L.emitted);
    uint8_t* s_sym = smem + L.sym;
    uint8_t* s_rec = smem + L.rec;

    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const RowSigns sg = row_signs(lane);
    const int ch = row_channel(lane);             // element of the stream: ch + 64 k in register k
    const int b = blockIdx.z, h = blockIdx.y;
    const int first = a.t0 + blockIdx.x * ns;
    const int active = min(ns, a.t0 + a.n_new - first);

    // the wavefront's streams arrive one ahead: stream i + 4 is requested
    // before stream i is worked on
    const uint16_t* src = a.kv + (int64_t)b * a.sb + (TOK ? 0 : (int64_t)h * a.sh);
    uint16_t raw[NH][HV];
    auto load_stream = [&](int i) {
        const uint16_t* row = src + (int64_t)(first - a.t0 + i) * a.st;
#pragma unroll
        for (int g = 0; g < NH; ++g) load_raw<HV>(row + (int64_t)g * a.sh, raw[g], lane, a.rotate);
    };
    if (!TOK && wave < active) load_stream(wave);

    for (int i = tid; i < (FIXED ? 0 : ta.M); i += kEncThreads) {
        s_cost[i] = ta.t.cost[i];
        s_rate[i] = (double)ta.t.cost[i] * (1.0 / 65536.0);
        // floor(x / f) = mulhi(x, rcp) >> (sh - 1) for x < 2^31, where
        // sh = ceil(log2 f) and rcp = ceil(2^(31 + sh) / f); for f = 1 the
        // product with 2^32 - 1 gives x - 1 (x > 0), and the addend makes up
        // for the missing multiple
        const uint32_t f = (uint32_t)ta.t.freq[i], P = 1u << ta.p;
        const uint32_t sh = f > 1 ? 32u - (uint32_t)__builtin_clz(f - 1u) : 1u;
        s_ent[i] = uint4{((kRansL >> ta.p) << 8) * f, P - f,
                         f > 1 ? (uint32_t)(((1ull << (31 + sh)) + f - 1) / f) : 0xFFFFFFFFu,
                         (sh - 1) | (((uint32_t)ta.t.cum[i] + (f > 1 ? 0u : P - 1u)) << 8)};
    }
    for (int i = tid; i < (FIXED ? 0 : kLambdaSteps); i += kEncThreads) s_lam[i] = ta.t.lam[i];
    for (int i = tid; i < ns; i += kEncThreads) {
        s_budget[i] = ta.budget;
        s_flag[i] = 0;
    }
    // the dequantized key means of the workgroup's window (with means t0 is a
    // multiple of the window, so no workgroup straddles two): scale times int8
    // is exact in fp32
    // (a bad block-table entry reads page 0; the record write then skips it)
    double mean[TOK ? 1 : VPL];                   // (0 for values: x - 0 is x)
    if constexpr (!TOK) {
#pragma unroll
        for (int k = 0; k < VPL; ++k) mean[k] = 0.0;
    }
    if (a.mean_q) {
        bool bad = false;
        if constexpr (TOK) {
            for (int j = tid; j < n; j += kEncThreads) {
                const int64_t wi = window_index(a.pg, a.H, a.t_cap, b, j / kD, first / DQ_MEAN_WINDOW, bad);
                s_mean[j] = half_bits_to_f32(a.mean_scale[wi]) * (float)a.mean_q[wi * kD + j % kD];
            }
        } else {
            const int64_t wi = window_index(a.pg, a.H, a.t_cap, b, h, first / DQ_MEAN_WINDOW, bad);
            const float sc = half_bits_to_f32(a.mean_scale[wi]);
#pragma unroll
            for (int k = 0; k < VPL; ++k) mean[k] = (double)(sc * (float)a.mean_q[wi * n + ch + kWave * k]);
        }
    }
    __syncthreads();
    DriftCtx dc{s_rate, s_cost, s_lam, ta.M, ta.cheapest, ta.rmin};
    const bool packed = packed_symbols(TOK, ta.M);

    bool range_bad = false;
    for (int pass = 0;; ++pass) {
        // Drift, wavefront per stream.
        for (int i = wave; i < active; i += kEncWaves) {
            if (pass > 0 && !s_flag[i]) continue;
            if (TOK || pass > 0) load_stream(i);
            double x[VPL];
#pragma unroll
            for (int g = 0; g < NH; ++g) {
                double v[HV];
                rotated<HV>(raw[g], v, lane, sg, a.rotate);
#pragma unroll
                for (int k = 0; k < HV; ++k) x[HV * g + k] = v[k];
            }
            if (!TOK && pass == 0 && i + kEncWaves < active) load_stream(i + kEncWaves);
            if constexpr (TOK) {
                if (a.mean_q) {
#pragma unroll
                    for (int k = 0; k < VPL; ++k) x[k] = x[k] - (double)s_mean[ch + kWave * k];
                }
            } else {
#pragma unroll
                for (int k = 0; k < VPL; ++k) x[k] = x[k] - mean[k];
            }
            double mn = x[0], mx = x[0];
            bool fin = isfinite(x[0]);
#pragma unroll
            for (int k = 1; k < VPL; ++k) {
                mn = min_nn(mn, x[k]);
                mx = max_nn(mx, x[k]);
                fin = fin && isfinite(x[k]);
            }
            fin = uniform_all(fin);
            wave_minmax_nn(mn, mx);
            if (!uniform_all(fin && mn != 0.0 && mx != 0.0)) {
                // NaN, and which zero it is, as plain comparisons over lanes in
                // channel order have it (rare: kept a branch)
                asm volatile("" : "+v"(x[0]));
                mn = mx = x[0];
#pragma unroll
                for (int k = 0; k < VPL; ++k) {
                    mn = fmin(mn, x[k]);
                    mx = fmax(mx, x[k]);
                }
                // (row_channel: the second and fourth quad of a row reversed)
                auto quads = [](uint32_t v) {
                    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x1B, 0xF, 0xA, false);
                };
                auto ordered = [&](double v) { return join(quads(lo32(v)), quads(hi32(v))); };
                mn = wave_min(ordered(mn));
                mx = wave_max(ordered(mx));
            }
            // the two drifts of Alg. 1: on the min-max grid, then on the
            // refitted grid in fp16 (a retry repeats only the second)
            double s = 0.0, o = 0.0;
            if (pass > 0) {
                s = (double)half_bits_to_f32(s_s16[i]);
                o = (double)half_bits_to_f32(s_o16[i]);
            } else {
                s = (mx - mn) / (double)(ta.M - 1);
                o = mn;
            }
            int m[VPL];
#pragma unroll 1
            for (int d = pass > 0 ? 1 : 0;; ++d) {
                if constexpr (FIXED) {
                    nearest<VPL>(x, s, o, ta.M, m);
                } else {
                    int64_t budget = s_budget[i];
                    asm volatile("" : "+v"(budget));       // (a select of the two addresses would be a flat load)
                    if (!d) budget = ta.budget;
                    bool done = false;
                    if constexpr (JM >= 0) done = fin && fold_drift<VPL, JM, POOL>(x, mn, mx, s, o, budget, dc, a.f, m);
                    if (!done) drift<VPL, MB>(x, s, o, budget, dc, m);
                }
                if (d) break;
                // least-squares refit
                int sm = 0, smm = 0;
                double mx_[VPL];
#pragma unroll
                for (int k = 0; k < VPL; ++k) {
                    sm += m[k];
                    smm += m[k] * m[k];
                    mx_[k] = (double)m[k] * x[k];
                }
                sm = wave_sum_i32(sm);
                smm = wave_sum_i32(smm);
                double Sx, Smx;
                fold_sums<VPL>(x, mx_, Sx, Smx);
                // (integers below 2^53: exact)
                const double smf = (double)sm, den = (double)n * (double)smm - smf * smf;
                if (uniform_all(den != 0.0)) {
                    const double s1 = ((double)n * Smx - smf * Sx) / den;
                    const double o1 = (Sx - s1 * smf) / (double)n;
                    if (isfinite(s1) && s1 > 0.0) {
                        s = s1;
                        o = o1;
                    }
                }
                const uint16_t sb16 = f64_to_half_bits(s), ob16 = f64_to_half_bits(o);
                const float sf = half_bits_to_f32(sb16), of = half_bits_to_f32(ob16);
                if (!fin || !isfinite(sf) || !isfinite(of)) range_bad = true;
                if (lane == 0) {
                    s_s16[i] = sb16;
                    s_o16[i] = ob16;
                }
                s = (double)sf;
                o = (double)of;
            }
            uint8_t* sym = s_sym + i * L.sym_row + ch;
            if (packed) {
#pragma unroll
                for (int k = 0; k + 1 < VPL; k += 2) sym[kWave * (k / 2)] = (uint8_t)(m[k] | m[k + 1] << 4);
            } else {
#pragma unroll
                for (int k = 0; k < VPL; ++k) sym[kWave * k] = (uint8_t)m[k];
            }
        }
        __syncthreads();

        if (FIXED) {
            // b-bit symbols after the header, lane per stream
            if (tid < active) {
                const int i = tid;
                uint8_t* rec = s_rec + i * L.rec_row;
                const uint8_t* sym = s_sym + i * L.sym_row;
                const int bb = 31 - __builtin_clz(ta.M);
                for (int k = 0; k < C - 4; ++k) {
                    uint32_t v = 0;
                    for (int t = 0; t < 8; ++t) {
                        const int g = 8 * k + t, j = g / bb;
                        if (j < n) v |= (uint32_t)((sym[j] >> (g - j * bb)) & 1) << t;
                    }
                    rec[4 + k] = (uint8_t)v;
                }
                const uint16_t sb = s_s16[i], ob = s_o16[i];
                rec[0] = (uint8_t)(sb & 0xFF);
                rec[1] = (uint8_t)(sb >> 8);
                rec[2] = (uint8_t)(ob & 0xFF);
                rec[3] = (uint8_t)(ob >> 8);
            }
            __syncthreads();
            break;
        }
        // Backward rANS, lane per stream (Eq. rans, encoded in reverse).  The
        // symbols of four steps and their entries are read ahead of the chain,
        // a step's byte is stored whether or not it counts, and the record is
        // put together when it is written out.  The wavefront runs at a raised
        // issue priority: the workgroup waits for its serial chain.
        if (tid < active && (pass == 0 || s_flag[tid])) {
            const int i = tid;
            uint8_t* const row = s_rec + i * L.rec_row;
            uint8_t* at = row + C - 1;                // next byte, downwards
            uint8_t* const low = row + kPayloadOffset - 1;
            const uint32_t* sym4 = reinterpret_cast<const uint32_t*>(s_sym + i * L.sym_row);
            const int cap = C - kPayloadOffset;
            // x < 256 L and x_max = (L >> p) 256 f: one byte brings x below
            // x_max when p <= 8, two when p <= 12
            const bool two = ta.p > 8;
            uint32_t xs = kRansL;
            bool over = false;
            __builtin_amdgcn_s_setprio(3);
            auto emit = [&](uint32_t xmax) {
                const bool e = xs >= xmax;
                *at = (uint8_t)xs;
                at -= e ? 1 : 0;
                xs = e ? xs >> 8 : xs;
            };
            for (int j = n / 4 - 1; j >= 0; --j) {
                // (packed: elements 64 .. 127 of every 128 in the high halves)
                const uint32_t w = packed ? sym4[(j >> 5) * 16 + (j & 15)] >> ((j >> 4 & 1) * 4) : sym4[j];
                const uint32_t mask = packed ? 0xFu : 0xFFu;
                uint4 ent[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) ent[u] = s_ent[(w >> (8 * u)) & mask];
#pragma unroll
                for (int u = 3; u >= 0; --u) {
                    emit(ent[u].x);
                    if (two) emit(ent[u].x);
                    // Enc(x, m) = floor(x / f) 2^p + (x mod f) + c = x + q (2^p - f) + c;
                    // after renormalization x < 2^29 and q < 2^(29 - p)
                    const uint32_t q = __umulhi(xs, ent[u].z) >> (ent[u].w & 31u);
                    xs = __umul24(q, ent[u].y) + (xs + (ent[u].w >> 8));
                }
                // four steps store at most eight bytes: a stream past its
                // record stays in its row
                over = over || at < low;
                at = at < low ? low : at;
            }
            __builtin_amdgcn_s_setprio(0);
            const int emitted = over ? cap + 1 : (int)(row + C - 1 - at);
            if (emitted > cap) {
                // Defensive: with L = 2^21 the coded length is at most
                // sum r + n (2^-17 + log2(1 + 2^p / L)) bits, under 8 bits
                // past the budget for n <= 1024, so a drifted stream always
                // fits.  Should one not, retry 8 bits lower; when the budget
                // runs out the record is all zeros (decoding flags it corrupt).
                s_flag[i] = 1;
                s_budget[i] -= (int64_t)8 * 65536;
                if (s_budget[i] < (int64_t)n * ta.rmin) {
                    s_flag[i] = 0;
                    s_s16[i] = s_o16[i] = 0;
                    s_state[i] = 0;
                    s_emitted[i] = 0;
                    if (a.status) atomicOr(a.status, DQ_STATUS_OVERFLOW);
                }
            } else {
                s_flag[i] = 0;
                s_state[i] = xs;
                s_emitted[i] = emitted;
            }
        }
        const int again = __syncthreads_or(tid < active ? s_flag[tid] : 0);
        if (!again) break;
    }
    if (range_bad && lane == 0 && a.status) atomicOr(a.status, DQ_STATUS_RANGE);

    // Dword w of stream i's record: the header, the state, the payload (the
    // last `emitted` bytes of the row, moved up to offset 8), zeros.
    auto rec_dword = [&](int i, int w) -> uint32_t {
        const uint32_t* row = reinterpret_cast<const uint32_t*>(s_rec + i * L.rec_row);
        if (FIXED) return row[w];
        if (w == 0) return (uint32_t)s_s16[i] | ((uint32_t)s_o16[i] << 16);
        if (w == 1) return s_state[i];
        const int left = s_emitted[i] - 4 * (w - 2);           // payload bytes from here on
        if (left <= 0) return 0u;
        const int at = C - left;
        const uint32_t v = __builtin_amdgcn_alignbyte(row[at / 4 + 1], row[at / 4], (uint32_t)at & 3u);
        return left >= 4 ? v : v & ((1u << (8 * left)) - 1u);
    };

    bool bad_page = false;
    if (TOK) {
        // 64-token tiles, 8-byte chunk major: chunk c of the token in row r at
        // ((r / 64) S / 8 + c) 512 + (r % 64) 8, the row of token t through
        // the block table when there is one.  A thread serves one stream and
        // every (threads / ns)-th chunk, neighbouring threads neighbouring rows.
        const int i = tid & (ns - 1);
        if (i < active) {
            const int64_t row = token_row(a.pg, a.t_cap, b, first + i, bad_page);
            if (!bad_page) {
                uint8_t* tile = a.records + (row & ~(int64_t)63) * a.rec_stride + (row & 63) * 8;
                for (int c = tid / ns; c < a.rec_stride / 8; c += kEncThreads / ns) {
                    const uint2 v = uint2{rec_dword(i, 2 * c), rec_dword(i, 2 * c + 1)};
                    *reinterpret_cast<uint2*>(tile + (int64_t)c * 512) = v;
                }
            }
        }
    } else {
        // sixteen lanes per record
        const bool dwords = (C & 3) == 0 && (reinterpret_cast<uintptr_t>(a.records) & 3) == 0;
        for (int i = tid / 16; i < active; i += kEncThreads / 16) {
            bool bad = false;
            const int64_t row = record_row(a.pg, a.H, a.t_cap, b, h, first + i, bad);
            if (bad) {
                bad_page = true;
                continue;
            }
            uint8_t* dst = a.records + row * C;
            if (dwords) {
                for (int w = tid & 15; w < C / 4; w += 16) reinterpret_cast<uint32_t*>(dst)[w] = rec_dword(i, w);
            } else {
                for (int k = tid & 15; k < C; k += 16) dst[k] = (uint8_t)(rec_dword(i, k / 4) >> (8 * (k & 3)));
            }
        }
    }
    if (__any(bad_page) && lane == 0 && a.status) atomicOr(a.status, DQ_STATUS_PAGE);
}

// Streams per workgroup: as many as the coder has lanes for (64, or 32 for
// per-token streams: kEncStreamsTok), fewer
// while the grid would leave a CU with fewer than four workgroups: a small append
// is bound by the streams that a wavefront takes in turn.  K and V, us, stopping
// at one / two / four workgroups per CU: 16 x 128 tokens 164 / 121 / 108, 1 x
// 4096 191 / 191 / 161, per-token 4 x 2048 572 / 476 / 458; below 1 x 128 tokens
// the same.
int streams_per_group(int most, int64_t tokens, int64_t rows) {
    int ns = most;
    while (ns > kEncWaves && (tokens + ns - 1) / ns * rows < 4 * (int64_t)cu_count()) ns /= 2;
    return ns;
}

// Rates the folded drift can take: symmetric, non-decreasing away from the
// centre and convex, the outermost level excepted.
bool fold_args(const dq_tables* tab, int n, FoldArgs& f) {
    const int M = tab->cfg.levels, J = (M - 1) / 2;
    const int32_t* R = tab->cost;
    if (J < 1) return false;
    for (int m = 0; m < M; ++m)
        if (R[m] != R[M - 1 - m]) return false;
    f.J = J;
    f.base = n * R[M / 2];
    f.pool = 0;
    f.even = M % 2 == 0;
    f.off = f.even ? 1.0 : 0.5;
    for (int j = 0; j < kFoldMax; ++j) {
        f.W[j] = j < J ? R[M / 2 + j + 1] - R[M / 2 + j] : 0;
        f.w[j] = f.W[j] / 65536.0;
        f.wf[j] = (float)f.w[j];
    }
    for (int j = 0; j < J; ++j) {
        if (f.W[j] < 0) return false;
        if (j > 0 && f.W[j] < f.W[j - 1]) {
            if (j < J - 1) return false;
            f.pool = 1;
        }
    }
    return true;
}

template <int VPL, int MB, bool TOK, int JM, bool POOL = false>
int launch_encode_as(const EncArgs& a, dim3 grid, hipStream_t stream) {
    const int smem = enc_layout(kWave * VPL, a.ta.C, a.ns, TOK, a.ta.M).total;
    if (int rc = hip_check("hipFuncSetAttribute",
                           hipFuncSetAttribute(reinterpret_cast<const void*>(&encode_kernel<VPL, MB, TOK, JM, POOL>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, smem)))
        return rc;
    encode_kernel<VPL, MB, TOK, JM, POOL><<<grid, kEncThreads, smem, stream>>>(a);
    return hip_check("encode launch", hipGetLastError());
}

// Thresholds in registers where the level counts of the default operating
// points meet them (128 values: 5 to 10 levels; 512 and 1024 values: 5 to 8),
// else formed one at a time; the distortions of drift() in registers for up to
// 8 levels (16 with two values per lane) where every step needs them.
template <int VPL, bool TOK>
int launch_encode_vpl(const EncArgs& a, bool fold, dim3 grid, hipStream_t stream) {
    if (fold) {
        if constexpr ((VPL == 2 && !TOK) || VPL >= 8) {
            if (a.f.J == 2 && !a.f.pool) return launch_encode_as<VPL, 0, TOK, 2>(a, grid, stream);
            if (a.f.J == 3) {
                if constexpr (TOK)
                    if (a.f.pool) return launch_encode_as<VPL, 0, TOK, 3, true>(a, grid, stream);
                if (!a.f.pool) return launch_encode_as<VPL, 0, TOK, 3>(a, grid, stream);
            }
            if constexpr (!TOK)
                if (a.f.J == 4 && !a.f.pool) return launch_encode_as<VPL, 0, TOK, 4>(a, grid, stream);
        }
        return a.f.pool ? launch_encode_as<VPL, 0, TOK, 0, true>(a, grid, stream)
                        : launch_encode_as<VPL, 0, TOK, 0>(a, grid, stream);
    }
    if constexpr (VPL <= 4)
        if (a.ta.M <= 8) return launch_encode_as<VPL, 8, TOK, -1>(a, grid, stream);
    if constexpr (VPL <= 2)
        if (a.ta.M <= 16) return launch_encode_as<VPL, 16, TOK, -1>(a, grid, stream);
    return launch_encode_as<VPL, 0, TOK, -1>(a, grid, stream);
}

template <int VPL>
int launch_key_mean(const EncArgs& a, int B, int8_t* mean_q, uint16_t* mean_scale, hipStream_t stream) {
    key_mean_kernel<VPL><<<dim3(a.n_new / DQ_MEAN_WINDOW, a.H, B), kMeanWaves * kWave, 0, stream>>>(
        a.kv, a.sb, a.st, a.sh, a.H, a.t0, a.t_cap, a.pg, mean_q, mean_scale, a.status, a.rotate);
    return hip_check("key_mean launch", hipGetLastError());
}

int launch_key_mean(int vpl, const EncArgs& a, int B, int8_t* mean_q, uint16_t* mean_scale, hipStream_t stream) {
    switch (vpl) {
        case 1: return launch_key_mean<1>(a, B, mean_q, mean_scale, stream);
        case 2: return launch_key_mean<2>(a, B, mean_q, mean_scale, stream);
        case 4: return launch_key_mean<4>(a, B, mean_q, mean_scale, stream);
        default: return DQ_ERR_INVALID_ARG;
    }
}

}  // namespace

int launch_encode(const dq_tables* tab, const Pages& pg, const uint16_t* kv, int64_t sb, int64_t st, int64_t sh,
                  int32_t B, int32_t H, int32_t t0, int32_t n_new, int32_t t_cap,
                  uint8_t* records, int8_t* mean_q, uint16_t* mean_scale, uint32_t* status,
                  hipStream_t stream, int token_stride) {
    const bool tok = token_stride > 0;
    const int n = tab->cfg.head_dim;
    const int vpl = n / kWave;
    EncArgs a;
    a.ta = tab_args(tab);
    a.kv = kv;
    a.sb = sb;
    a.st = st;
    a.sh = sh;
    a.H = H;
    a.t0 = t0;
    a.n_new = n_new;
    a.t_cap = t_cap;
    a.pg = pg;
    a.rec_stride = token_stride;
    a.records = records;
    a.mean_q = mean_q;
    a.mean_scale = mean_scale;
    a.status = status;
    a.rotate = tab->cfg.prerotated ? 0 : 1;
    if (mean_q)
        if (int rc = launch_key_mean(tok ? kD / kWave : vpl, a, B, mean_q, mean_scale, stream)) return rc;
    a.ns = streams_per_group(tok ? kEncStreamsTok : kEncStreams, n_new, (int64_t)(tok ? 1 : H) * B);
    const bool fold = fold_args(tab, n, a.f);
    const dim3 grid((n_new + a.ns - 1) / a.ns, tok ? 1 : H, B);
    switch ((tok ? 100 : 0) + vpl) {
        case 1: return launch_encode_vpl<1, false>(a, fold, grid, stream);
        case 2: return launch_encode_vpl<2, false>(a, fold, grid, stream);
        case 4: return launch_encode_vpl<4, false>(a, fold, grid, stream);
        case 102: return launch_encode_vpl<2, true>(a, fold, grid, stream);
        case 104: return launch_encode_vpl<4, true>(a, fold, grid, stream);
        case 108: return launch_encode_vpl<8, true>(a, fold, grid, stream);
        case 116: return launch_encode_vpl<16, true>(a, fold, grid, stream);
        default: return DQ_ERR_INVALID_ARG;
    }
}

int launch_encode_fixed(int32_t n, int32_t record_bytes, const Pages& pg, const uint16_t* kv, int64_t sb,
                        int64_t st, int64_t sh, int32_t B, int32_t H, int32_t t0, int32_t n_new, int32_t t_cap,
                        uint8_t* records, int8_t* mean_q, uint16_t* mean_scale, uint32_t* status,
                        hipStream_t stream) {
    const int vpl = n / kWave;
    const int bits = 8 * (record_bytes - 4) / n;
    if (vpl < 1 || vpl > 4 || bits < 1 || bits > 8) return DQ_ERR_INVALID_ARG;
    EncArgs a{};
    a.ta.n = n;
    a.ta.M = 1 << bits;
    a.ta.C = record_bytes;
    a.kv = kv;
    a.sb = sb;
    a.st = st;
    a.sh = sh;
    a.H = H;
    a.t0 = t0;
    a.n_new = n_new;
    a.t_cap = t_cap;
    a.pg = pg;
    a.rec_stride = 0;
    a.records = records;
    a.mean_q = mean_q;
    a.mean_scale = mean_scale;
    a.status = status;
    a.rotate = 1;
    if (mean_q)
        if (int rc = launch_key_mean(vpl, a, B, mean_q, mean_scale, stream)) return rc;
    a.ns = streams_per_group(kEncStreams, n_new, (int64_t)H * B);
    const dim3 grid((n_new + a.ns - 1) / a.ns, H, B);
    const int smem = enc_layout(n, record_bytes, a.ns, false, a.ta.M).total;
    switch (vpl) {
        case 1: encode_kernel<1, 0, false, -1, false, true><<<grid, kEncThreads, smem, stream>>>(a); break;
        case 2: encode_kernel<2, 0, false, -1, false, true><<<grid, kEncThreads, smem, stream>>>(a); break;
        default: encode_kernel<4, 0, false, -1, false, true><<<grid, kEncThreads, smem, stream>>>(a); break;
    }
    return hip_check("encode_fixed launch", hipGetLastError());
}

}  // namespace dq

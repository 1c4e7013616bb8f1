// k_stats, k_select: the paper's analytic breakpoint selectors (Section 3.3,
// Section 5.1).  k_mse_tile, k_mse_final: error of Eq.3 at a given (m, p).
#pragma once

#include "pwlq_tables.h"
#include "pwlq_refine.h"

namespace pwlq {

// What the kernels of this file need to know of a tensor.  A call of up
// to kStatArgTensors tensors carries these fields in its kernels' arguments and uploads
// no table (two launches of about 4.5 us each per call on 54 tensors); a longer table
// is read from the workspace.
constexpr int kStatArgTensors = 56;
struct StatArgs {
    long long w[kStatArgTensors], gcount[kStatArgTensors], out_group[kStatArgTensors];
    int tile_prefix[kStatArgTensors + 1], group_prefix[kStatArgTensors + 1];
    int nt;                                     // 0: not used, the table is in the workspace
};
struct StatRec {
    const float *w;
    long long gcount, out_group;
    int tpg, tile_base, group_base;
};
__device__ inline StatRec stat_rec(const Tables &tb, const StatArgs &sa, int i)
{
    StatRec s;
    if (sa.nt > 0) {
        s.w = reinterpret_cast<const float *>(sa.w[i]);
        s.gcount = sa.gcount[i];
        s.out_group = sa.out_group[i];
        s.tpg = (int)((s.gcount + kTileMax - 1) / kTileMax);
        s.tile_base = sa.tile_prefix[i];
        s.group_base = sa.group_prefix[i];
    } else {
        const TensorRec &r = tb.recs[i];
        s.w = r.w;
        s.gcount = r.gcount;
        s.out_group = r.out_group;
        s.tpg = r.tpg;
        s.tile_base = r.tile_base;
        s.group_base = r.group_base;
    }
    return s;
}
struct StatTile {
    const float *src;
    long long og;                // the group's index in the caller's arrays
    int len, t;
    bool whole;                  // the only tile of its group
};
// Tile of a wavefront; of a tensor whose groups are cut into several tiles the full
// ones first (see slot_to_tile).
__device__ inline StatTile stat_tile(const Tables &tb, const StatArgs &sa, int slot)
{
    const int i = sa.nt > 0 ? find_tensor(sa.tile_prefix, sa.nt, slot) : find_tensor(tb.tile_prefix, tb.nt, slot);
    const StatRec r = stat_rec(tb, sa, i);
    int g = slot - r.tile_base, tig = 0;
    if (r.tpg > 1) {
        const int end = sa.nt > 0 ? sa.tile_prefix[i + 1] : tb.tile_prefix[i + 1];
        const int nfull = (end - r.tile_base) / r.tpg * (r.tpg - 1);
        const int ls = g;
        g = ls < nfull ? ls / (r.tpg - 1) : ls - nfull;
        tig = ls < nfull ? ls - g * (r.tpg - 1) : r.tpg - 1;
    }
    const long long first = (long long)tig * kTileMax;
    StatTile st;
    st.src = reinterpret_cast<const float *>(uni((long long)reinterpret_cast<uintptr_t>(
        r.w + (long long)g * r.gcount + first)));
    const long long left = r.gcount - first;
    st.len = uni((int)(left < kTileMax ? left : kTileMax));
    st.og = uni(r.out_group + g);
    st.t = uni(r.tile_base + g * r.tpg + tig);
    st.whole = r.tpg == 1;
    return st;
}
// Tensor of group g, where groups first_g to last_g (the same in every lane, 64 at most) ask
// together: as a rule one tensor's, else one of the 64 from first_g's on.  (A walk from there took up to 63 dependent loads where tensors are single
// groups.)
__device__ inline int find_group(const int *__restrict__ prefix, int nt, int first_g, int last_g, int g)
{
    int lo = find_tensor(prefix, nt, first_g);
    if (prefix[lo + 1] > last_g) return lo;
    int hi = nt - lo > 64 ? lo + 64 : nt;              // prefix[lo] <= g < prefix[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (prefix[mid] <= g) lo = mid;
        else hi = mid;
    }
    return lo;
}
__device__ inline StatRec stat_group(const Tables &tb, const StatArgs &sa, int first_g, int last_g, int g)
{
    const int i = sa.nt > 0 ? find_group(sa.group_prefix, sa.nt, first_g, last_g, g)
                            : find_group(tb.group_prefix, tb.nt, first_g, last_g, g);
    return stat_rec(tb, sa, i);
}

// ------------------------------------------------------------------- stats
// Per tile: max|w| (NaN if any element is NaN), sum of w^2 and sum of |w| in
// binary64.  One wavefront per tile (most tiles are a few hundred elements: a
// workgroup per tile spends its time on the reductions and the barrier), every
// element read once, four loads in flight per lane with a partial sum each,
// added in a fixed order.
constexpr int kStatUnroll = 4;

__global__ __launch_bounds__(kWG) void k_stats(Tables tb, StatArgs sa, int n_tiles, float *__restrict__ tile_max,
                                               double *__restrict__ tile_s2,
                                               double *__restrict__ tile_s1)
{
    const int slot = uni((int)(blockIdx.x * kWaves + (threadIdx.x >> 6)));
    if (slot >= n_tiles) return;
    const StatTile ti = stat_tile(tb, sa, slot);
    const int lane = threadIdx.x & 63;
    float mx = 0.0f;
    int bad = 0;
    double s2[kStatUnroll], s1[kStatUnroll];
#pragma unroll
    for (int u = 0; u < kStatUnroll; ++u) s2[u] = s1[u] = 0.0;
    int i = lane;
    for (; i + 64 * (kStatUnroll - 1) < ti.len; i += 64 * kStatUnroll) {
        float a[kStatUnroll];
#pragma unroll
        for (int u = 0; u < kStatUnroll; ++u) a[u] = fabsf(ti.src[i + 64 * u]);
#pragma unroll
        for (int u = 0; u < kStatUnroll; ++u) {
            bad |= (a[u] != a[u]);
            mx = fmaxf(mx, a[u]);
            const double d = (double)a[u];
            s2[u] += d * d;
            s1[u] += d;
        }
    }
    for (; i < ti.len; i += 64) {
        const float a = fabsf(ti.src[i]);
        bad |= (a != a);
        mx = fmaxf(mx, a);
        const double d = (double)a;
        s2[0] += d * d;
        s1[0] += d;
    }
    const double t2 = wave_sum((s2[0] + s2[1]) + (s2[2] + s2[3]));
    const double t1 = wave_sum((s1[0] + s1[1]) + (s1[2] + s1[3]));
    mx = wave_max(mx);
    bad = wave_or(bad);
    if (lane == 0) {
        tile_max[ti.t] = bad ? __builtin_nanf("") : mx;
        tile_s2[ti.t] = t2;
        tile_s1[ti.t] = t1;
    }
}

// ------------------------------------------------------------------ select
// Minimiser of the expected error of Eq.6 over (0, m/2) for a zero-mean law truncated to
// [-m, m]: root of its derivative (Eq.8; Eq.11 is that root written out).  In units of
// the law's scale, x = p / scale and t = m / scale, with the law's mass above x and above
// t, both over the mass inside [-t, t]:
//   g = x - 2 t (above(x) - above(t)) + t (2 x - t) f(x)
// The derivative is increasing there (Lemma 1: the second derivative, Eq.9, is positive),
// so Newton steps are kept inside a shrinking bracket and replaced by its midpoint when
// they leave it; the end t/2 is looked at when a step would pass it.  A Newton step of
// 1e-9 x is the last: the error after it is of the order of its square, below the
// rounding of a binary64.
//
// One thread per group leaves most SIMDs with one wavefront, which runs at the latency of
// its instructions and of fetching them: the loop body is the only copy of the law (its
// first trip evaluates it at t).  27 560 groups, Gaussian: 44 us with three erfc per step
// and steps that ended on the bracket answered by bisection (50 trips in one group of
// 64 weights in a hundred), 5.4 us like this.
__device__ inline double solve_breakpoint(double m, double scale, bool laplace, double start)
{
    const double t = m / scale;
    double lo = 0.0, hi = 0.5 * t, above_t = 0.0, inv_z = 1.0;
    double x = t;                                      // first trip: the mass outside [-t, t]
    double next = start / scale;
    if (!(next > lo && next < hi)) next = 0.5 * (lo + hi);
    bool first = true, at_end = false, end_seen = false;
    for (int it = 0; it < 100; ++it) {
        const double ex = exp(laplace ? -x : -0.5 * x * x);
        const double above = 0.5 * (laplace ? ex : erfc(x * 0.70710678118654752440));
        if (first) {
            above_t = above;
            inv_z = 1.0 / (1.0 - 2.0 * above);
            x = next;
            first = false;
            continue;
        }
        const double f = ex * (laplace ? 0.5 : 0.39894228040143267794) * inv_z;
        const double df = laplace ? -f : -x * f;
        const double lever = t * (2.0 * x - t);
        const double g = x - 2.0 * t * (above - above_t) * inv_z + lever * f;
        if (at_end) {                                  // x is t/2
            if (g <= 0.0) break;
            end_seen = true;
            x = 0.5 * (lo + hi);
            at_end = false;
            continue;
        }
        const double dg = 1.0 + 4.0 * t * f + lever * df;
        if (g > 0.0) hi = x;
        else lo = x;
        const double step = -g / dg;
        next = x + step;
        if (fabs(step) <= 1.0e-9 * x) {                // before the bracket is asked: the last steps may end on it
            x = fmin(fmax(next, lo), hi);
            break;
        }
        if (next >= hi && hi == 0.5 * t && !end_seen) {
            x = hi;
            at_end = true;
            continue;
        }
        x = (next > lo && next < hi) ? next : 0.5 * (lo + hi);
        if (hi - lo <= 2.0e-16 * t) break;
    }
    return x * scale;
}

// Add the tiles' statistics, estimate the scale about zero (sigma^2 = mean w^2,
// beta = mean |w|) and select p.
// selector 0: Section 5.1's logarithmic fit, p = sigma ln(0.8614 m/sigma + 0.6079);
// selector 1: Eq.11 for the truncated Gaussian; 2: for the truncated Laplacian.
// One thread per group, tiles in order; groups of kWideTiles tiles or more (a tensor as one
// group) have one wavefront each, lanes over the tiles, the lanes' sums added in a fixed
// order.  The groups of several tiles come first, the longest of them in front, so a launch
// takes a range: kWide those in front, the other form the rest.  (One launch for all with one
// live lane in the solver took 171 us for two such groups among 82 680 of 64 weights, the two
// launches 45.)
constexpr int kSelectWG = 64;     // one wavefront per workgroup: a few ten thousand groups reach every CU
// One thread / one wavefront, k_select's whole call in us: 1, 64, 1024 and 4096 groups of 16
// tiles 15.1/13.9, 20.8/19.5, 102/104, 362/370; of 8 14.3/13.7, 14.7/15.0, 47/51, 185/196; of
// 32 16.9/14.0, 25.9/22.2, 189/188.
constexpr int kWideTiles = 16;
// Up to this many groups beside the wide ones join their launch, a wavefront each: 1024 of
// them cost about 4 us more in it, a launch of their own 5 to 6.
constexpr int kWideRest = 1024;

// Sum over the tiles of a wavefront's group, of which lane j holds tile j, j + 64, ...: few
// tiles in tile order, as one thread adds them.
__device__ inline double wide_sum(double v, int tiles)
{
    if (tiles >= kWideTiles) return wave_sum(v);
    double s = 0.0;
    for (int j = 0; j < tiles; ++j)
        s += __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), j),
                              __builtin_amdgcn_readlane(__double2loint(v), j));
    return s;
}

template <bool kWide>
__global__ __launch_bounds__(kSelectWG) void k_select(Tables tb, StatArgs sa, int begin, int end, int selector,
                                                const float *__restrict__ tile_max,
                                                const double *__restrict__ tile_s2,
                                                const double *__restrict__ tile_s1,
                                                float *__restrict__ p_out,
                                                float *__restrict__ m_out)
{
    const int first = begin + (kWide ? blockIdx.x : blockIdx.x * kSelectWG);
    const int g = kWide ? first : (first + (int)threadIdx.x < end ? first + (int)threadIdx.x : end - 1);
    const StatRec r = stat_group(tb, sa, first, kWide ? first : first + kSelectWG - 1 < end ? first + kSelectWG - 1 : end - 1, g);
    const int gl = g - r.group_base;
    const long long tile0 = r.tile_base + (long long)gl * r.tpg;
    float mf = 0.0f;
    int bad = 0;
    double s2 = 0.0, s1 = 0.0;
    for (int j = kWide ? threadIdx.x : 0; j < r.tpg; j += kWide ? kSelectWG : 1) {
        const float v = tile_max[tile0 + j];
        bad |= (v != v);
        mf = fmaxf(mf, v);
        s2 += tile_s2[tile0 + j];
        s1 += tile_s1[tile0 + j];
    }
    if (kWide) {
        mf = wave_max(mf);
        bad = wave_or(bad);
        s2 = wide_sum(s2, r.tpg);
        s1 = wide_sum(s1, r.tpg);
    }
    if (kWide) {
        if (threadIdx.x > 0) return;
    } else if (first + (int)threadIdx.x >= end) {
        return;
    }
    if (bad) mf = __builtin_nanf("");
    const long long og = r.out_group + gl;
    m_out[og] = mf;
    if (!(mf < __builtin_inff())) { p_out[og] = __builtin_nanf(""); return; }
    if (mf == 0.0f) { p_out[og] = 0.0f; return; }
    const double m = (double)mf;
    const double count = (double)r.gcount;
    const double sigma = sqrt(s2 / count), beta = s1 / count;
    const double fit = sigma * log(0.8614 * (m / sigma) + 0.6079);
    double p;
    if (selector == 0) p = fit;
    else if (selector == 1) p = solve_breakpoint(m, sigma, false, fit);
    else p = solve_breakpoint(m, beta, true, 0.25 * m);
    if (p > m) p = m;
    if (p < 0.0) p = 0.0;
    p_out[og] = (float)p;
}

// --------------------------------------------------------------------- mse
// Squared error of Eq.3 over one tile with the group's (m, p): canonical
// binary32 code, binary64 error, fixed summation order.  One wavefront per
// tile, as in k_stats.
__global__ __launch_bounds__(kWG) void k_mse_tile(Tables tb, StatArgs sa, int n_tiles, int bits,
                                                  const float *__restrict__ p_in,
                                                  const float *__restrict__ m_in,
                                                  double *__restrict__ tile_sse,
                                                  double *__restrict__ mse)
{
    const int slot = uni((int)(blockIdx.x * kWaves + (threadIdx.x >> 6)));
    if (slot >= n_tiles) return;
    const StatTile ti = stat_tile(tb, sa, slot);
    const Pieces q = make_pieces(m_in[ti.og], p_in[ti.og], bits);
    const int lane = threadIdx.x & 63;
    double acc[kStatUnroll];
#pragma unroll
    for (int u = 0; u < kStatUnroll; ++u) acc[u] = 0.0;
    int i = lane;
    for (; i + 64 * (kStatUnroll - 1) < ti.len; i += 64 * kStatUnroll) {
        float a[kStatUnroll];
#pragma unroll
        for (int u = 0; u < kStatUnroll; ++u) a[u] = fabsf(ti.src[i + 64 * u]);
#pragma unroll
        for (int u = 0; u < kStatUnroll; ++u) acc[u] = exact_add(q, a[u], acc[u]);
    }
    for (; i < ti.len; i += 64) acc[0] = exact_add(q, fabsf(ti.src[i]), acc[0]);
    const double s = wave_sum((acc[0] + acc[1]) + (acc[2] + acc[3]));
    if (lane == 0) {
        if (ti.whole) mse[ti.og] = s / (double)ti.len;      // the group's only tile
        else tile_sse[ti.t] = s;
    }
}

// Groups of several tiles, which come first: tiles added as in k_select.  (Those of one tile
// are done.)
template <bool kWide>
__global__ __launch_bounds__(kSelectWG) void k_mse_final(Tables tb, StatArgs sa, int end,
                                                   const double *__restrict__ tile_sse,
                                                   double *__restrict__ mse)
{
    const int first = kWide ? blockIdx.x : blockIdx.x * kSelectWG;
    const int g = kWide ? first : (first + (int)threadIdx.x < end ? first + (int)threadIdx.x : end - 1);
    const StatRec r = stat_group(tb, sa, first, kWide ? first : first + kSelectWG - 1 < end ? first + kSelectWG - 1 : end - 1, g);
    const int gl = g - r.group_base;
    const long long tile0 = r.tile_base + (long long)gl * r.tpg;
    double s = 0.0;
    for (int j = kWide ? threadIdx.x : 0; j < r.tpg; j += kWide ? kSelectWG : 1) s += tile_sse[tile0 + j];
    if (kWide) {
        s = wide_sum(s, r.tpg);
        if (threadIdx.x > 0) return;
    } else if (first + (int)threadIdx.x >= end) {
        return;
    }
    mse[r.out_group + gl] = s / (double)r.gcount;
}

} // namespace pwlq

// k_fast: candidate evaluation by bucketed prefix sums instead of one pass over
// the elements per candidate.  Same output as k_prep + k_search (the binary32
// filter value of every candidate of a tile, in candidate units), so the exact
// re-evaluation and the argmin that follow are shared.
//
// With u = |w|/m * n, candidate k quantizes the centre elements (u <= k) to the
// grid j*k/L and the tail elements to k + j*(n-k)/L, j = 0..L.  An element of a
// piece with step s and offset z rounds to level j when it lies above j of the
// half-way points b_i = z + (2i+1) s/2, so
//   (u - z - j s)^2 = (u - z)^2 - 2 s sum_{i<L} max(u - b_i, 0).
// Summed over both pieces, with H(b) = sum_u max(b - u, 0), everything that
// depends on the region of an element cancels:
//   SSE(k) = sum_u (n - u)^2 - 2 (k/L) sum_i H((2i+1) k/(2L))
//                            - 2 ((n-k)/L) sum_i H(k + (2i+1) (n-k)/(2L)).
// A candidate costs 2L look-ups of H, whatever the tile's length.
//
// Whole numbers.  Every half-way point is a multiple of 1/(2L), so magnitudes are
// held as integers in units of 1/(2L q), q the largest that keeps n below 2^30:
// half-way points are exact, every sum below is exact, and binary64 enters once
// per candidate, where the three terms meet.  An element is one binary64 product
// rounded to a whole number: it moves by at most 0.52 * 2^-30 n (q is 63 or more,
// so n is at least 0.97 * 2^30 units).  Weights far below the absmax keep that
// many bits too, so a candidate's value is closer to the exact error than prefix
// sums of binary32 magnitudes (two roundings of up to 2^-24 u each) come: rms error
// 0.024 against 0.032 squared candidate units for 1024 Gaussian weights, b = 4,
// n = 1000 (units of 2^-24 n: 0.061), 3.0e-5 against 5.3e-5 for 2048 of a heavy
// tail, b = 8, n = 500 (5.1e-4).
//
// A tile that is a group of its own looks up a grid of candidates and those that it does not exclude
// (fast_pruned), in launches where that is less work (fast_prunes); other tiles all of them.
//
// A look-up needs no full sort: elements are grouped into buckets that are
// monotone in the magnitude (one counting pass in LDS), and a bucket's 64-bit word
// holds the sum (43 bits) and count (14 bits) of the elements before it and its
// own count in whole fours (7 bits).  H(b) is b * count - sum of the bucket of b, plus
// max(b - u, 0) over the bucket's own elements: elements past its end are above b and
// add nothing, so the first three are read without looking at the count, the others
// four at a time.
// Elements that are exactly zero (pruned weights) are counted, never walked.
//
// Bound by vector issue and LDS together, and by what a workgroup waits for alone between its eight barriers: with 38 400
// tiles of 4096, 1000 candidates, b = 4, us: 1498 with binary64
// prefixes of counts, sums and squares and walks of nine elements, 745 with all candidates looked up and an
// element's load and add waited for one by one, 544 with one bound on the candidates, 508 with chords and without the choices for
// elements that do not exist, 386 in workgroups of 256 threads and 26 KB (see k_fast).
#pragma once

#include <type_traits>

#include "pwlq_prep.h"
#include "pwlq_refine.h"
#include "pwlq_tables.h"

namespace pwlq {

// Most buckets per octave, 2^8.  2^9 halves the walks and costs the fourth workgroup of 512 threads per
// CU its LDS (38 400 tiles of 4096, search + quantize, with 24-bit units: 1228 us with 2^9, 1145 with 2^8).
// Workgroups of 256 threads have 2^7: six of them, not four, then fit a CU (k_fast alone, us: 485 with 2^8, 386).
constexpr int kFastOctBits = 8;
constexpr int kFastOct = 7;                        // octaves, or twice as many of half as many buckets each
constexpr int kFastWords = kFastOct << kFastOctBits;   // most buckets per tile
constexpr int kFastBits = 30;
// Largest magnitude: with the offset `low` it is at most 2^30 - 64, the largest
// binary32 below 2^30, so that no bucket number passes the last octave's.
constexpr unsigned kFastTop = (1u << kFastBits) - 64u - (1u << (kFastBits - kFastOct));
static_assert(kFastTop / (65535u * 254u) >= 63u, "every grid fits, with 63 units or more to half its finest step");
constexpr int kFastCrowd = 64;                     // fullest bucket the look-ups may walk: this or 1/16 of the tile, twice
constexpr int kFastCrowdMax = 511;                 // as much in workgroups of 256 threads (fast_crowd), and never more than this
constexpr int kFastCrowdLog = 6, kFastCrowdBits = 9;
static_assert(kFastCrowd <= 1 << kFastCrowdLog && kFastCrowdMax < 1 << kFastCrowdBits, "as powers of two");
constexpr int kFastWalk = 3;                       // elements read unasked (4: 0.5-2 % slower, 6: 3-7 %)
constexpr int kFastWalkOn = 4;                     // ... and then per step
constexpr int kFastShort = 256;                    // longest tile of a launch of 128 or 64 threads
constexpr int kFastLong = 5120;                    // longest tile of a launch of 512 threads: four workgroups' LDS per CU
constexpr int kFastShortest = 9;                   // shortest tile that many short ones have looked up (see fast_min_len)
constexpr int kFastWaveTiles = 8192, kFastWaveCand = 2000;   // a wavefront for a short tile: fewest tiles, most candidates (fast_threads)
constexpr int kFastManyTiles = 2048;               // more tiles of 1025 to kFastLong elements get 256 threads instead of 512
constexpr int kFastGridMax = 1 << 21;              // workgroups of a launch
constexpr int kFastLaunchTiles = 1024;             // fewer tiles join the launch of the next longer ones,
constexpr int kFastOwnTiles = 2048, kFastOwnShort = 6144;   // ... or than these where it has fewer longer ones (own_launch)

// Error of a tile's filter value beyond the rounding of its elements: A is a sum of
// squares added in at most 33 steps (20 per thread, 6 over the wavefront and 4 over a workgroup of
// 256; 10, 6 and 8; 8, 6 and 16) and scaled in three roundings, the rest is exact up to seven roundings
// of a value of at most A, and A is at most n^2 K: below 48 * 2^-53 n^2 K = 5.4e-15
// n^2 K.  kFastRelErr * n^2 * K is added to the slack of the filter (keep_threshold).

// log2 of a tile's buckets per octave, about two buckets per element, 32 at least, and in workgroups of 256 threads 128 at
// most: the parts of H inside one bucket then fit 32 bits.  With 2^m buckets in an octave
// (2^(m-1) where there are 14 octaves) the widest, in the last octave, has 2^(30-m) units, so that its elements
// are at most 2^(30-m) - 1 below a half-way point in it.
__host__ __device__ constexpr int fast_octave_bits(int len, int threads)
{
    const int most = threads == 256 ? kFastOctBits - 1 : kFastOctBits;
    int bits = 5;
    while (bits < most && (8 << bits) <= len) ++bits;
    return bits;
}
// Most elements of a bucket: a tile with more in one is evaluated element by element.  Twice as many in workgroups of 256 threads,
// of long tiles since their buckets are twice as wide, of others since walks are the cheaper by far (4229x573 of
// cubes of normal numbers, b = 4, n = 2962, us, 64 / 128: 549/51).
__host__ __device__ constexpr int fast_crowd(int len, int threads)
{
    int most = (len >> 4) > kFastCrowd ? len >> 4 : kFastCrowd;
    if (threads == 256) most *= 2;
    return most < kFastCrowdMax ? most : kFastCrowdMax;
}
constexpr bool fast_parts_fit(int longest, int threads)
{
    for (int len = 1; len <= longest; ++len)
        if (fast_crowd(len, threads) * ((1ull << (kFastBits - fast_octave_bits(len, threads))) - 1) >> 32) return false;
    return true;
}
static_assert(fast_parts_fit(kFastLong, 256) && fast_parts_fit(kTileMax, 1024), "the parts inside any bucket fit 32 bits");

// inclusive prefix sum of 64-bit words over the wavefront
template <int kCtrl, int kRows>
__device__ inline unsigned long long dpp_u64(unsigned long long v)
{
    const unsigned lo = (unsigned)dpp_i32<kCtrl, kRows>(0, (int)(unsigned)v);
    const unsigned hi = (unsigned)dpp_i32<kCtrl, kRows>(0, (int)(unsigned)(v >> 32));
    return ((unsigned long long)hi << 32) | lo;
}
__device__ inline unsigned long long wave_scan_incl_u64(unsigned long long v)
{
    v += dpp_u64<0x111, 0xf>(v);
    v += dpp_u64<0x112, 0xf>(v);
    v += dpp_u64<0x114, 0xf>(v);
    v += dpp_u64<0x118, 0xf>(v);
    v += dpp_u64<0x142, 0xa>(v);
    v += dpp_u64<0x143, 0xc>(v);
    return v;
}

constexpr int kFastSumBits = kFastBits + 13, kFastCountBits = 14;   // then 7 bits: the bucket's own count / 4
static_assert(kFastSumBits + kFastCountBits == 57 && kFastCrowdMax / kFastWalkOn < 128 && kFastWalkOn == kFastWalk + 1,
              "a bucket of c elements is walked in kFastWalk and c / kFastWalkOn steps of kFastWalkOn");

typedef __attribute__((address_space(3))) const unsigned long long FastWordLds;
typedef __attribute__((address_space(3))) const unsigned FastElemLds;

struct FastLds {
    unsigned words;                // LDS address of the word of bucket 0, less 8 times its number
    FastElemLds *elems;            // grouped by bucket; index 0 is the first of the zero elements
    int shift;                     // bits of the binary32 pattern below a bucket number
};

// Bucket number of value v (magnitude plus `low`): the top bits of its binary32
// pattern, i.e. 2^m buckets per octave (values above 2^24 are rounded to binary32 on
// the way, which keeps their order).  Below `low` the added offset makes them
// equally wide.
__device__ inline unsigned fast_bucket(unsigned v, int shift) { return __float_as_uint((float)v) >> shift; }

struct FastSums {
    unsigned long long c;          // sums of the elements below
    unsigned n, m, d;              // counts; counts times 2i+1; parts inside buckets
};

struct FastWord {
    unsigned before, steps;        // elements before the bucket; steps of a walk past the first elements
    unsigned long long c;
};
__device__ inline FastWord fast_word(const FastLds &L, unsigned b)
{
    const unsigned long long w = *(FastWordLds *)(uintptr_t)((fast_bucket(b, L.shift) << 3) + L.words);
    const unsigned hi = (unsigned)(w >> 32);
    FastWord f;
    f.before = (hi >> (kFastSumBits - 32)) & ((1u << kFastCountBits) - 1u);
    f.steps = hi >> (kFastSumBits - 32 + kFastCountBits);
    f.c = w & ((1ull << kFastSumBits) - 1ull);
    return f;
}

// max(b - u, 0) over kCount elements.
template <int kCount>
__device__ inline unsigned fast_walk(FastElemLds *e, unsigned b)
{
    unsigned x[kCount], d = 0;
#pragma unroll
    for (int i = 0; i < kCount; ++i) x[i] = e[i];
#pragma unroll
    for (int i = 0; i < kCount; ++i) d += __builtin_elementwise_sub_sat(b, x[i]);
    return d;
}

// H at one half-way point of each piece: the two chains of reads run side by side.
__device__ inline void fast_query2(const FastLds &L, unsigned b0, unsigned b1, unsigned odd, FastSums &s0,
                                   FastSums &s1)
{
    const FastWord w0 = fast_word(L, b0), w1 = fast_word(L, b1);
    FastElemLds *e0 = L.elems + w0.before, *e1 = L.elems + w1.before;
    s0.d += fast_walk<kFastWalk>(e0, b0);
    s1.d += fast_walk<kFastWalk>(e1, b1);
    for (unsigned i = 0; i < w0.steps; ++i) s0.d += fast_walk<kFastWalkOn>(e0 + kFastWalk + kFastWalkOn * i, b0);
    for (unsigned i = 0; i < w1.steps; ++i) s1.d += fast_walk<kFastWalkOn>(e1 + kFastWalk + kFastWalkOn * i, b1);
    s0.c += w0.c;
    s1.c += w1.c;
    s0.n += w0.before;
    s1.n += w1.before;
    s0.m += __umul24(odd, w0.before);
    s1.m += __umul24(odd, w1.before);
}

// What a candidate's value needs beside the tables: A = sum (n - u)^2, inv = 2 / (L 2Lq), the
// offset `low` of the stored values, and the look-ups whose parts inside buckets fit 32
// bits together (those of its own elements are below the bucket's width, those past it zero).
struct FastCurve {
    double A, inv;
    unsigned low;
    int n, Li, q, run;
};

// Sum over groups of 2^g lanes, in every lane of the group.
__device__ inline double group_sum(double v, int g)
{
    if (g > 0) v += dpp_f64<0xb1, 0xf>(0.0, v);         // lane ^ 1
    if (g > 1) v += dpp_f64<0x4e, 0xf>(0.0, v);         // lane ^ 2
    if (g > 2) v += dpp_f64<0x141, 0xf>(0.0, v);        // the other four of eight
    if (g > 3) v += dpp_f64<0x140, 0xf>(0.0, v);        // the other eight of sixteen
    if (g > 4) v += __shfl_xor(v, 16, 64);
    if (g > 5) v += __shfl_xor(v, 32, 64);
    return v;
}

// What the bound between two candidates needs: (2 / L) (sum H in the tail - sum H in the centre), and the latter
// part, in squared candidate units per candidate.
struct FastSlope {
    float d, centre;
};

// Filter value of candidate k: by one lane, or (kGroups) by a group of 2^g lanes whose
// lane `sub` takes the half-way points sub, sub + 2^g, ... of both pieces; the loops are the
// same in every lane.  All lanes of the wavefront come here together.
template <bool kGroups, bool kSlope>
__device__ inline float fast_value(const FastLds &Q, const FastCurve &c, int k, int sub, int g, FastSlope &slope)
{
    if (!kGroups) sub = g = 0;
    const unsigned kk = (unsigned)(k * c.q), ww = (unsigned)((c.n - k) * c.q);   // half steps of the two pieces
    const unsigned zt = 2u * (unsigned)c.Li * kk + c.low;
    const unsigned odd0 = 2u * (unsigned)sub + 1u, dc = (2u * kk) << g, dt = (2u * ww) << g;
    FastSums fc = {0, 0, 0, 0}, ft = {0, 0, 0, 0};
    unsigned bc = odd0 * kk + c.low, bt = odd0 * ww + zt;
    const int whole = c.Li >> g;
    for (int i = 0; i < whole;) {
        const int stop = i + c.run < whole ? i + c.run : whole;
        fc.d = ft.d = 0;
        for (; i < stop; ++i) {
            fast_query2(Q, bc, bt, (unsigned)(2 * i << g) + odd0, fc, ft);
            bc += dc;
            bt += dt;
        }
        fc.c -= fc.d;
        ft.c -= ft.d;
    }
    // L + 1 is a power of two: one half-way point is left to every lane but the last
    if (kGroups && sub < (c.Li & ((1 << g) - 1))) {
        fc.d = ft.d = 0;
        fast_query2(Q, bc, bt, (unsigned)(2 * whole << g) + odd0, fc, ft);
        fc.c -= fc.d;
        ft.c -= ft.d;
    }
    // whole numbers below 2^52, so exact in binary64, and so are the group's sums
    double hc = (double)kk * (double)fc.m + (double)c.low * (double)fc.n - (double)(long long)fc.c;
    double ht = (double)ww * (double)ft.m + (double)zt * (double)ft.n - (double)(long long)ft.c;
    if (kGroups) { hc = group_sum(hc, g); ht = group_sum(ht, g); }
    if (kSlope) {
        slope.d = (float)(c.inv * (ht - hc));
        slope.centre = (float)(c.inv * hc);
    }
    const double sse = c.A - c.inv * ((double)k * hc + (double)(c.n - k) * ht);
    return (float)(sse > 0.0 ? sse : 0.0);
}

// put(lead, k, value, slope) for the candidates k_of(0 .. count-1), `lead` in one lane of each
// one's group.  Where there are threads for it a candidate gets several lanes, four half-way points
// of a piece each at least: what comes after the look-ups costs as much as three of them.
template <int kT, bool kSlope = false, typename KOf, typename Put>
__device__ inline void fast_each(const FastLds &Q, const FastCurve &c, int count, KOf k_of, Put put)
{
    int g = 0;
    while ((8 << g) <= c.Li + 1 && (count << (g + 1)) <= kT) ++g;
    const int lane = threadIdx.x & 63, sub = lane & ((1 << g) - 1);
    for (int at = uni((int)threadIdx.x & ~63); at < count << g; at += kT) {
        const int item = (at + lane) >> g;
        const bool live = item < count;
        const int k = k_of(live ? item : count - 1);
        FastSlope slope = {0.0f, 0.0f};
        const float v = g > 0 ? fast_value<true, kSlope>(Q, c, k, sub, g, slope) : fast_value<false, kSlope>(Q, c, k, 0, 0, slope);
        put(live && sub == 0, k, v, slope);
    }
}

// Filter value of every candidate of the tile.
template <int kT>
__device__ inline void fast_candidates(const FastLds &Q, const FastCurve &c, float *__restrict__ row)
{
    fast_each<kT>(Q, c, c.n, [](int i) { return i + 1; },
                  [&](bool lead, int k, float v, const FastSlope &) { if (lead) row[k - 1] = v; });
}

// ---------------------------------------------------------------- fewer candidates
// A tile that is a group of its own needs the candidates within the slack of the minimum
// only, and most candidates can be shown to be past it, from a grid of candidates that are evaluated.
//
// H is convex, and so are its sums over the half-way points of a piece, h(k) in the centre and t(k) in the tail, whose
// half-way points move evenly with k.  Between neighbours k0, k1 of the grid both lie below their chords, and as
// SSE(k) = A - (2/L) (k h(k) + (n-k) t(k)),
//   SSE(k) >= chord of SSE - (k - k0) (k1 - k) (D1 - D0) / (k1 - k0),  D = (2/L) (t - h):
// a parabola per interval, 3 % below SSE in the middle of steps of 8 of 1000 for long-tailed weights at b = 4.  Candidate 0
// is the ends' partner of n: its half-way points are those of n, all in the tail.
//
// Eq.3 takes an element to the nearest of the 2L+1 levels of both pieces (p is a level of both), and a level moves by at
// most c_j candidate units when the breakpoint moves by one: c_j = j/L in the centre,
// 1 - j/L in the tail.  With f = sqrt(SSE), the length of the vector of errors,
//   f(k) >= f(k') - |k - k'| C(k),  C(k)^2 = sum over the elements of c_j^2, j the level under k,
// and c_j <= min(1, u/k + 1/(2L)), so that C(k)^2 <= min(N, U2/k^2 + U1/(Lk) + N/(4L^2)) with
// the sums U1, U2 of u and u^2.  That excludes more where the steps are long for the curve: 2-5 % of the candidates at 8 bits.
//
// The candidates that neither bound excludes are evaluated, and what k_exact is given is the list of candidates within
// the threshold of the minimum, the same as from a row of all values.  Of 1000 candidates this
// evaluates (grid and others) 60 at b = 2 and 3, 100 to 140 at b = 4, 150 to 200 at b = 5, 220 to 300 at b = 6, 430 to 770 at b = 8;
// by the second bound alone, from a grid of 128, 180 to 280 at b = 4.
constexpr int kPruneMin = 300;                     // fewest candidates
constexpr int kPruneGrid = 128;                    // most points of the grid
constexpr int kPruneList = 2048;                   // most candidates between them, else all are evaluated
constexpr int kPruneKeep = 64;                     // most of those within the threshold, else all are evaluated

// log2 of the grid's step.  The gap below the chord goes with the square of the step and, against the error, of L: up to
// four bits half of the points leave fewer candidates in all, which larger workgroups evaluate as fast as few.
__host__ __device__ constexpr int prune_grid(int L, int threads) { return threads <= 256 && L <= 7 ? kPruneGrid / 2 : kPruneGrid; }
__host__ __device__ constexpr int prune_log(int n, int L, int threads)
{
    int log = 2;
    while (n >> log > prune_grid(L, threads)) ++log;
    return log;
}
// number of the last point, which is candidate n.  Of a full grid its neighbour may be up to two steps away: a point more than 64
// or 128 would halve the lanes that each gets (7048x65, b = 3, n = 517, us, 65 points 30.4, 64 28.5).
__host__ __device__ constexpr int prune_points(int n, int L, int threads)
{
    const int log = prune_log(n, L, threads), points = (n + (1 << log) - 1) >> log, grid = prune_grid(L, threads);
    return points < grid ? points : grid;
}
static_assert(prune_points(512, 7, 128) == 64 && prune_points(519, 3, 256) == 64 && prune_points(520, 3, 64) == 33 &&
                  prune_points(528, 7, 128) == 33 && prune_points(1031, 15, 512) == 128 && prune_points(300, 1, 64) == 38,
              "no more points than the grid has");
// LDS beyond the tables: the grid's values and slopes, then the list
__host__ __device__ constexpr int prune_bytes(int n, int L, int threads)
{
    return n < kPruneMin ? 0 : 8 * (prune_points(n, L, threads) + 1) + 2 * (n < kPruneList ? n : kPruneList);
}

struct FastPruneLds {
    unsigned least;                                // binary32 pattern of the least value
    int listed, kept;
    float keep_v[kPruneKeep];
    int keep_k[kPruneKeep];
};

// A row that holds a list instead of values: its first word is the count with the sign bit.
constexpr int kRowIsList = (int)0x80000000;

// U1, U2, count: bounds from above.  False, in every thread: the row has to be evaluated in full.
template <int kT>
__device__ inline bool fast_pruned(const FastLds &Q, const FastCurve &c, float U1, float U2, float count,
                                   FastPruneLds &S, float *value, unsigned short *list, int *__restrict__ row)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int log = prune_log(c.n, c.Li, kT), points = prune_points(c.n, c.Li, kT);
    float *slope = value + points + 1;
    const auto point = [&](int i) { return i < points ? i << log : c.n; };
    const auto least = [&](bool lead, float v) {
        const unsigned w = ~wave_max_u32(lead ? ~__float_as_uint(v) : ~0x7f800000u);      // v >= 0
        if (lane == 0) atomicMin(&S.least, w);
        return __uint_as_float(w);
    };
    // keep_threshold of a value, from above
    const float nf = (float)c.n, eps = nf * 4.7684e-7f;
    const float flat_slack = count * (2.0001f * eps * eps + 2.0001f * (float)kFastRelErr * nf * nf);
    const auto threshold = [&](float v) {
        return v * 1.00007f + 4.0001f * eps * __builtin_amdgcn_sqrtf(count * v) + flat_slack;
    };
    fast_each<kT, true>(Q, c, points, [&](int i) { return point(i + 1); }, [&](bool lead, int k, float v, const FastSlope &s) {
        if (lead) {
            const int i = k < c.n ? k >> log : points;
            value[i] = v;
            slope[i] = s.d;
            if (k == c.n) { value[0] = v; slope[0] = s.centre; }
        }
        least(lead, v);
    });
    __syncthreads();
    // A bound above these excludes a candidate.  A parabola's ends are within 1e-14 n^2 count and a rounding to binary32 of their
    // values, and so is the value that it bounds; 6e-7 n sqrt(count) covers the roundings of the
    // roots, of at most n sqrt(count), and of the values below them.
    const float near = threshold(__uint_as_float(S.least));
    const float top = near * 1.00002f + 4.0f * (float)kFastRelErr * nf * nf * count;
    const float top_root = __builtin_amdgcn_sqrtf(near) * 1.00002f + 6e-7f * nf * __builtin_amdgcn_sqrtf(count);
    const float invL = __builtin_amdgcn_rcpf((float)c.Li), flat = 0.25f * count * invL * invL;
    const int cap = c.n < kPruneList ? c.n : kPruneList;
    for (int at = uni(tid & ~63); at < points; at += kT) {
        // the candidates between grid points i and i + 1: x = lo .. hi past the first
        const int i = at + lane;
        int lo = 1, hi = 0, from = 0;
        if (i < points) {
            from = point(i);
            const int s = point(i + 1) - from;
            const float sf = (float)s, rs = __builtin_amdgcn_rcpf(sf) * 1.000001f;
            const float v0 = value[i], v1 = value[i + 1], d0 = slope[i], d1 = slope[i + 1];
            // the parabola less the threshold is g x^2 + b x + v: g from above, positive
            const float up = d1 - d0 + 2e-7f * (__builtin_fabsf(d0) + __builtin_fabsf(d1));
            const float g = (up > 0.0f ? up * 1.0001f : 0.0f) * rs + 1e-6f * (v0 + v1 + top) * rs * rs;
            const float b = (v1 - v0) * rs - g * sf, v = v0 - top;
            const float disc = b * b - 4.0f * g * v + 4e-6f * (b * b + 4.0f * g * __builtin_fabsf(v));
            hi = s - 1;
            if (disc < 0.0f) hi = 0;
            else {
                const float root = __builtin_amdgcn_sqrtf(disc);
                const float q = -0.5f * (b + (b < 0.0f ? -root : root));
                // the roots q / g and v / q, in either order; 0.01 for the roundings of a quotient of at most s
                const float x0 = q / g, x1 = v / q;
                const float first = fminf(x0, x1) - 0.01f, last = fmaxf(x0, x1) + 0.01f;
                if (first > 1.0f) lo = first < sf ? (int)__builtin_ceilf(first) : s;
                if (last < sf) hi = last > 0.0f ? (int)last : 0;
                hi = hi < s ? hi : s - 1;
            }
            const float r = __builtin_amdgcn_rcpf((float)(from + 1));
            const float y = __builtin_fmaf(__builtin_fmaf(U2, r, U1 * invL), r, flat);
            const float per = __builtin_amdgcn_rcpf(1.0001f * __builtin_amdgcn_sqrtf(y < count ? y : count));
            if (i > 0) {
                const float d = (__builtin_amdgcn_sqrtf(v0) - top_root) * per - 0.01f;
                const int l = d < sf ? (int)__builtin_ceilf(d) : s;
                if (d > 1.0f && l > lo) lo = l;
            }
            const float d = (__builtin_amdgcn_sqrtf(v1) - top_root) * per - 0.01f;
            const int h = d < sf ? s - (int)__builtin_ceilf(d) : 0;
            if (d > 1.0f && h < hi) hi = h;
        }
        const int own = hi >= lo ? hi - lo + 1 : 0;
        const int incl = wave_scan_incl(own);
        int base = 0;
        if (lane == 63 && incl > 0) base = atomicAdd(&S.listed, incl);
        int pos = __builtin_amdgcn_readlane(base, 63) + incl - own;
        for (int j = 0; j < own; ++j, ++pos)
            if (pos < cap) list[pos] = (unsigned short)(from + lo + j);
    }
    __syncthreads();
    const int listed = uni(S.listed);
    if (listed > cap) return false;
    fast_each<kT>(Q, c, listed, [&](int i) { return (int)list[i]; }, [&](bool lead, int k, float v, const FastSlope &) {
        // within the threshold of the least value that the wavefront knows of
        const float own = least(lead, v);
        if (lead && v <= threshold(fminf(own, __uint_as_float(S.least)))) {
            const int at = atomicAdd(&S.kept, 1);
            if (at < kPruneKeep) { S.keep_v[at] = v; S.keep_k[at] = k; }
        }
    });
    __syncthreads();
    const int kept = uni(S.kept);
    if (kept > kPruneKeep) return false;
    if (tid >= 64) return true;                    // one wavefront writes the list (at most 192 entries)
    const float thr = threshold_f32(keep_threshold((double)__uint_as_float(S.least), (double)count, c.n, true));
    int out = 0;
    const auto keep = [&](bool want, int k) {
        const unsigned long long bal = __ballot(want);
        if (want) row[1 + out + __builtin_popcountll(bal & ((1ull << lane) - 1ull))] = k;
        out += __builtin_popcountll(bal);
    };
    static_assert(kPruneGrid + 1 + kPruneKeep < kPruneMin && kPruneKeep <= 64, "the list fits a row, the kept one wavefront");
    for (int at = 0; at < points; at += 64) {
        const int i = at + lane + 1;
        keep(i <= points && value[i <= points ? i : 1] <= thr, point(i));
    }
    keep(lane < kept && S.keep_v[lane < kept ? lane : 0] <= thr, S.keep_k[lane < kept ? lane : 0]);
    if (lane == 0) row[0] = kRowIsList | out;
    return true;
}

// A tile whose values crowd into a few buckets (many equal magnitudes: a bucket
// holding more than fast_crowd) would make every look-up walk a long bucket; it is evaluated element by element
// instead, from binary32 magnitudes in candidate units, with the chunked sums of the
// plain search kernel (all lanes read the same LDS word, which is a broadcast).
//
// Four elements to a read: element by element a wavefront waits out the LDS for every ten vector instructions (tiles crowded all
// of them, us, one by one / four to a read: 512x1155 of log-uniform weights, b = 4, n = 600, in 512 threads, 109/72;
// 1141x2738 of cubes of normal numbers, b = 7, n = 463, 389/291; 2361x5110 of these, b = 4, n = 2464, in 256 threads, 6580/5150).
//
// kPairs: two candidates of a thread at a time, half of the reads and two chains of additions, for workgroups of few threads
// (up to 5120 elements in 256 threads: 4100x5000 of log-uniform weights, b = 4, n = 600, us: 1638 one by one, 1573 so).
// A wavefront takes a pair where any of its lanes has two candidates left, so that no wavefront walks the
// tile for a part of its pairs and once more for the rest.
//
// fast_plain_row: candidates k0 and k0 + apart, those up to n.
template <int kC>
__device__ inline void fast_plain_row(const unsigned *__restrict__ elems, int len, int n, float Lf, int k0, int apart,
                                      float *__restrict__ row)
{
    float kf[kC], rc[kC], rt[kC], ct[kC], stepc[kC], stept[kC], outer[kC], acc[kC];
#pragma unroll
    for (int x = 0; x < kC; ++x) {
        const int k = k0 + x * apart < n ? k0 + x * apart : n;
        kf[x] = (float)k;
        rc[x] = Lf / kf[x];
        rt[x] = (k < n) ? Lf / (float)(n - k) : 0.0f;
        ct[x] = -kf[x] * rt[x];
        stepc[x] = kf[x] / Lf;
        stept[x] = (float)(n - k) / Lf;
        // else the compiler divides once per element, after the choice of the piece: 21 vector instructions
        // instead of 10 (4096x512 of log-uniform weights, b = 4, n = 2000, us: 2106, 817 now)
        asm("" : "+v"(stepc[x]), "+v"(stept[x]));
        outer[x] = 0.0f;
    }
    const auto add = [&](unsigned e) {
        const float u = __uint_as_float(e);
#pragma unroll
        for (int x = 0; x < kC; ++x) {
            const bool tail = u > kf[x];
            const float t = tail ? __builtin_fmaf(u, rt[x], ct[x]) : u * rc[x];
            const float err = (t - __builtin_rintf(t)) * (tail ? stept[x] : stepc[x]);
            acc[x] = __builtin_fmaf(err, err, acc[x]);
        }
    };
    static_assert(kChunk % 4 == 0, "chunks of whole 16-byte words");
    for (int cb = 0; cb < len; cb += kChunk) {
        const int ce = (cb + kChunk < len) ? cb + kChunk : len;
#pragma unroll
        for (int x = 0; x < kC; ++x) acc[x] = 0.0f;
        int i = cb;
        for (; i + 4 <= ce; i += 4) {
            const uint4 e = *reinterpret_cast<const uint4 *>(elems + i);
            add(e.x);
            add(e.y);
            add(e.z);
            add(e.w);
        }
        for (; i < ce; ++i) add(elems[i]);
#pragma unroll
        for (int x = 0; x < kC; ++x) outer[x] += acc[x];
    }
#pragma unroll
    for (int x = 0; x < kC; ++x)
        if (k0 + x * apart <= n) row[k0 + x * apart - 1] = outer[x];
}

template <int kT, bool kPairs>
__device__ inline void fast_plain(const unsigned *__restrict__ elems, int len, int n, int Li,
                                  float *__restrict__ row)
{
    const int tid = threadIdx.x;
    int at = 0;                                    // candidates at + 1 .. at + kT, one per thread
    const int wave = uni(tid & ~63);
    if constexpr (kPairs)
        for (; at + kT + wave < n; at += 2 * kT) fast_plain_row<2>(elems, len, n, (float)Li, at + tid + 1, kT, row);
    for (; at + wave < n; at += kT) fast_plain_row<1>(elems, len, n, (float)Li, at + tid + 1, kT, row);
}

// What depends on n and bits alone: magnitudes are held in units of 1/unit of a candidate,
// m as `top`; m at or below `keep_all` makes n / m overflow binary32.
struct FastUnits {
    double per_unit, per_unit2, inv;       // 1 / (2 L q), 1 / (2 L q)^2, 2 / (L 2L q)
    unsigned top;                          // 2 L q n: 0.97 * 2^30 or more
    int q;
    float keep_all;
};
inline FastUnits fast_units(int n, int bits)
{
    const int L = (1 << (bits - 1)) - 1;
    FastUnits f;
    f.q = (int)kFastTop / (n * 2 * L);
    const double unit = (double)(2 * L * f.q);
    f.per_unit = 1.0 / unit;
    f.per_unit2 = 1.0 / (unit * unit);
    f.inv = 1.0 / ((double)L * (double)L * (double)f.q);
    f.top = (unsigned)(n * 2 * L * f.q);
    f.keep_all = (float)((double)n / (3.4028235677973366e38));      // 2^128 - 2^103
    return f;
}

// The elements of a thread in batches, e0 .. e0 + count - 1: batch(first, count), both compile-time.  What a wavefront does with
// a batch depends on whether the tile ends in it: batches are as many as the tiles of a launch's range end in
// usefully, and no longer than the LDS adds that a thread can hold in flight within 64 registers.  In workgroups of
// 1024 threads, where a tile may end in any, four where the wavefront has `all` of its elements and else two (always four / always two / so,
// against no batches: 60 calls of groups of many tiles, whole but for the last, 0.986 / 1.001 / 0.986 of the time, 60 of tiles of 5121 to 8192
// 0.979 / 0.975 / 0.970, 40 with shorter tiles in the launch 0.973 / 0.961 / 0.964; 59x7021 and 1533x1051, b = 4, n = 97, us, 46.7/45.1).
template <int kPer, typename F>
__device__ inline void fast_batches([[maybe_unused]] bool all, F batch)
{
    static_assert(kPer == 2 || kPer == 4 || kPer == 8 || kPer == 10 || kPer == 20, "no batches for this many");
    const auto call = [&](auto e0, auto count) { batch(e0, count); };
#define PWLQ_BATCH(E, C) call(std::integral_constant<int, E>(), std::integral_constant<int, C>())
    if constexpr (kPer == 2) PWLQ_BATCH(0, 2);
    if constexpr (kPer == 4) PWLQ_BATCH(0, 4);
    if constexpr (kPer == 20) { PWLQ_BATCH(0, 4); PWLQ_BATCH(4, 4); PWLQ_BATCH(8, 4); PWLQ_BATCH(12, 4); PWLQ_BATCH(16, 4); }
    if constexpr (kPer == 8) {
        if (all) { PWLQ_BATCH(0, 4); PWLQ_BATCH(4, 4); }
        else { PWLQ_BATCH(0, 2); PWLQ_BATCH(2, 2); PWLQ_BATCH(4, 2); PWLQ_BATCH(6, 2); }
    }
    if constexpr (kPer == 10) { PWLQ_BATCH(0, 5); PWLQ_BATCH(5, 5); }
#undef PWLQ_BATCH
}

// Long tiles in 256 threads (kPer 20) where a launch has many: what every wavefront of a tile does once (reductions, prefixes,
// candidates' ends) is done by four instead of eight, all of them have candidates to look up, and six workgroups fit a CU's
// LDS where 512 threads are four at most (transformer_fast 925 -> 801 us, 5608 tiles of 1152 to 4608 82 -> 69).
template <int kT, int kPer>
__global__ __launch_bounds__(kT, kPer == 20 ? 6 : 8) void k_fast(Tables tb, int tile_begin, int n, int bits, FastUnits F,
                                             const float *__restrict__ tile_max,
                                             float *__restrict__ gm,
                                             float *__restrict__ sse32)
{
    // dynamic LDS: the buckets' words (first the counts and sums of the buckets
    // themselves, then of everything before them), then the grouped elements
    extern __shared__ __attribute__((aligned(16))) unsigned long long fast_lds[];
    constexpr int kW = kT / 64;
    constexpr int kScan = ((kFastOct << fast_octave_bits(kT * kPer, kT)) + kT - 1) / kT;   // words a thread holds at most
    __shared__ unsigned redm[kW];
    __shared__ float redsum[kW];
    __shared__ int wfull[kW];                                // a bucket fuller than 16, than kFastCrowd, crowded
    __shared__ unsigned long long wsum[kW];
    __shared__ double redA[kW];
    __shared__ FastPruneLds pruned;

    int t;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = uni(tid >> 6);
    TensorRec r;
    TileInfo ti = tile_of(tb, tile_begin + blockIdx.x, r, t);
    if (!r.fast) return;
    const int len = ti.len;
    const int Li = (1 << (bits - 1)) - 1;

    // Whether the wavefront has elements in a batch, and whether all of its lanes have all of them: no
    // lane of a whole batch looks at the length (half of the instructions of a thread's 8 elements did).
    const int wave_end = len - wave * 64;                  // elements from the wavefront's first on
    const auto none = [&](int e0) { return e0 * kT >= wave_end; };
    const auto all = [&](int e0, int count) { return (e0 + count - 1) * kT + 64 <= wave_end; };

    // No load depends on the length: past the end it reads the tile's last element.
    float a[kPer];
    {
        const GlobalFloat *src = (const GlobalFloat *)ti.src;
        const unsigned last = (unsigned)len - 1u;
        fast_batches<kPer>(all(0, kPer), [&](auto first, auto count) {
            constexpr int e0 = decltype(first)::value, e1 = e0 + decltype(count)::value;
            if (none(e0)) {
#pragma unroll
                for (int e = e0; e < e1; ++e) a[e] = 0.0f;
            } else if (all(e0, e1 - e0)) {
#pragma unroll
                for (int e = e0; e < e1; ++e) a[e] = (src + e * kT)[(unsigned)tid];
            } else {
#pragma unroll
                for (int e = e0; e < e1; ++e) a[e] = src[tid + e * kT < last ? tid + e * kT : last];
            }
        });
    }
    if (tid == 0) {
        pruned.least = 0x7f800000u;
        pruned.listed = pruned.kept = 0;
    }
    int obits = fast_octave_bits(len, kT);
    const int T = kFastOct << obits;
    for (int i = tid; i < T / 2; i += kT) reinterpret_cast<ulonglong2 *>(fast_lds)[i] = make_ulonglong2(0ull, 0ull);

    // group absmax: from the registers (single-tile group) or the tile maxima; the
    // tile's mean magnitude places the buckets.  Binary32 patterns of magnitudes are in the
    // magnitudes' order, NaN above infinity.
    unsigned mb = 0, lowest = ~0u;
    float sum = 0.0f;
    fast_batches<kPer>(all(0, kPer), [&](auto first, auto count) {
        constexpr int e0 = decltype(first)::value, e1 = e0 + decltype(count)::value;
        if (none(e0)) return;
        if (!all(e0, e1 - e0)) {
            asm volatile("");                                  // a branch: not a choice for every element of every batch
#pragma unroll
            for (int e = e0; e < e1; ++e) {
                const bool within = tid + e * kT < len;
                const unsigned ab = __float_as_uint(fabsf(a[e]));
                lowest = within && ab < lowest ? ab : lowest;
                a[e] = within ? a[e] : 0.0f;
            }
        }
        const bool whole = all(e0, e1 - e0);
#pragma unroll
        for (int e = e0; e < e1; ++e) {
            a[e] = fabsf(a[e]);
            if (whole) lowest = __float_as_uint(a[e]) < lowest ? __float_as_uint(a[e]) : lowest;
            const unsigned ab = __float_as_uint(a[e]);
            mb = ab > mb ? ab : mb;
            sum += a[e];
        }
    });
    if (r.tpg > 1) {
        const int tile0 = r.tile_base + ti.group_local * r.tpg;
        for (int j = tid; j < r.tpg; j += kT) {
            const unsigned v = __float_as_uint(fabsf(tile_max[tile0 + j]));
            mb = v > mb ? v : mb;
        }
    }
    mb = wave_max_u32(mb);
    sum = (float)wave_sum((double)sum);
    if (lane == 0) { redm[wave] = mb; redsum[wave] = sum; }
    __syncthreads();
    mb = redm[0];
    sum = redsum[0];
#pragma unroll 8
    for (int i = 1; i < kW; ++i) { mb = redm[i] > mb ? redm[i] : mb; sum += redsum[i]; }
    mb = (unsigned)uni((int)mb);
    sum = uni(sum);
    const float m = mb > 0x7f800000u ? __builtin_nanf("") : __uint_as_float(mb);
    if (ti.tile_in_group == 0 && tid == 0) gm[ti.group] = m;

    const bool usable = (m > 0.0f) && (m < __builtin_inff());
    const double scale = uni(usable ? (double)F.top / (double)m : 0.0);
    // A group so small that n / m overflows binary32: the weights' own steps are too coarse
    // there for the filter's slack.  Every element counts as m then, which gives all
    // candidates the value 0 and keeps them.
    const bool keep_all = usable && m <= F.keep_all;
    if (!usable || keep_all) {
#pragma unroll
        for (int e = 0; e < kPer; ++e) a[e] = (usable && a[e] > 0.0f) ? m : 0.0f;
    }

    // Values run from `low` to top + low, whose exponents are 30 - octaves and 29.  Seven
    // octaves, and 14 of half as many buckets where the mean lies in the lowest: near zero
    // these are 64 times as fine, elsewhere half as fine.
    const bool deep = uni((double)sum * (double)F.top <
                          (double)len * (double)(1u << (kFastBits - 1 - kFastOct)) * (double)m ? 1 : 0) != 0;
    obits -= deep ? 1 : 0;
    const unsigned low = 1u << (kFastBits - (deep ? 2 * kFastOct : kFastOct));
    FastLds Q;
    Q.shift = 23 - obits;
    const unsigned bucket0 = fast_bucket(low, Q.shift);
    Q.words = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)fast_lds - (bucket0 << 3);

    // values, counts and sums per bucket; the count an add returns is the element's
    // rank inside its bucket
    unsigned v[kPer];
    unsigned rank[kPer];
    double A = 0.0;
    // 2^52 + a scale, rounded once, holds the whole number in its low word: at most top, since
    // a <= m and scale is within 2^-53 of top / m
    const double one52 = 4503599627370496.0, full52 = one52 + (double)F.top;
    // A batch's adds are in flight before the first result is looked at: one at a time, under a
    // branch, a thread waits out the LDS for each of its elements (more at once: past 64
    // registers).  So zero elements and threads past the end add nothing to a word of their own; where a
    // wavefront has neither in a batch, it does without the choice.
    static_assert(64 <= kFastOct << 5, "a word for every lane");
    const float past = usable ? m : 0.0f;                      // counts as m: nothing in A
    // whether the wavefront has magnitudes that may round to zero
    const bool zeros_here = __ballot((double)__uint_as_float(lowest) * scale < 1.0) != 0ull;
    typedef __attribute__((address_space(3))) unsigned long long WordLds;
    fast_batches<kPer>(all(0, kPer), [&](auto first, auto count) {
        constexpr int e0 = decltype(first)::value, kCount = decltype(count)::value;
        if (none(e0)) return;
        const bool whole = all(e0, kCount);
        if (!whole) {
            asm volatile("");                                  // a branch: not a choice for every element of every batch
#pragma unroll
            for (int e = e0; e < e0 + kCount; ++e) a[e] = tid + e * kT < len ? a[e] : past;
        }
#pragma unroll
        for (int e = e0; e < e0 + kCount; ++e) {
            const double w = __builtin_fma((double)a[e], scale, one52);
            const double d = full52 - w;                       // exact
            A = __builtin_fma(d, d, A);
            v[e] = (unsigned)__double2loint(w) + low;
        }
        unsigned long long was[kCount];
        if (whole && !zeros_here) {
#pragma unroll
            for (int x = 0; x < kCount; ++x)
                was[x] = __hip_atomic_fetch_add((WordLds *)(uintptr_t)((fast_bucket(v[e0 + x], Q.shift) << 3) + Q.words),
                                                (1ull << kFastSumBits) | v[e0 + x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        } else {
#pragma unroll
            for (int x = 0; x < kCount; ++x) {
                const int e = e0 + x;
                const bool counts = tid + e * kT < len && v[e] > low;
                v[e] = counts ? v[e] : low;
                const unsigned at = counts ? fast_bucket(v[e], Q.shift) - bucket0 : (unsigned)lane;
                was[x] = atomicAdd(&fast_lds[at], counts ? (1ull << kFastSumBits) | v[e] : 0ull);
            }
        }
#pragma unroll
        for (int x = 0; x < kCount; ++x) {
            rank[e0 + x] = (unsigned)(was[x] >> kFastSumBits);
            asm volatile("" : "+v"(rank[e0 + x]));             // here, not where it is used: half the registers
        }
        __builtin_amdgcn_sched_barrier(0);
    });
    A = wave_sum(A);
    __syncthreads();

    const int crowd = fast_crowd(len, kT);
    // exclusive prefix of counts and sums, both fields in one word
    const int per = (T + kT - 1) / kT;             // divides T
    const int lo = tid * per;
    const bool holds = lo < T;
    int zeros = len;                               // less the elements counted in the buckets
    {
        unsigned long long w[kScan], tot = 0;
        unsigned fullest = 0;
#pragma unroll
        for (int x = 0; x < kScan; ++x) {
            w[x] = (holds && x < per) ? fast_lds[lo + x] : 0ull;
            tot += w[x];
            const unsigned c = (unsigned)(w[x] >> kFastSumBits);
            fullest = c > fullest ? c : fullest;
        }
        const unsigned long long incl = wave_scan_incl_u64(tot);
        const int over = (__ballot(fullest > 16u) != 0ull ? 1 : 0) |
                         (__ballot(fullest > (unsigned)kFastCrowd) != 0ull ? 2 : 0) |
                         (__ballot(fullest > (unsigned)crowd) != 0ull ? 4 : 0);
        if (lane == 63) { wsum[wave] = incl; wfull[wave] = over; redA[wave] = A; }
        __syncthreads();
        // (sums that are the same in every lane, in scalar registers)
        unsigned long long before = 0;
#pragma unroll
        for (int i = 0; i < kW; ++i) {
            const unsigned long long s = (unsigned long long)uni((long long)wsum[i]);
            zeros -= (int)(s >> kFastSumBits);
            before += i < wave ? s : 0ull;
        }
        // the zero elements come before everything
        before += ((unsigned long long)zeros << kFastSumBits) + (unsigned long long)zeros * low;
        unsigned long long run = incl - tot + before;
        if (holds) {
#pragma unroll
            for (int x = 0; x < kScan; ++x) {
                if (x < per) {
                    // (a count that does not fit is a crowded tile's)
                    const unsigned long long own = w[x] >> kFastSumBits;
                    fast_lds[lo + x] = run | ((own / kFastWalkOn) << (kFastSumBits + kFastCountBits));
                    run += w[x];
                }
            }
        }
    }
    A = 0.0;
    int full = 0;
#pragma unroll 8
    for (int i = 0; i < kW; ++i) { A += redA[i]; full |= wfull[i]; }
    A = uni(A * F.per_unit2);
    full = uni(full);
    __syncthreads();
    unsigned *elems = reinterpret_cast<unsigned *>(fast_lds + T);
    Q.elems = (FastElemLds *)elems - zeros;
    fast_batches<kPer>(all(0, kPer), [&](auto first, auto count) {
        constexpr int e0 = decltype(first)::value, kCount = decltype(count)::value;
        if (none(e0)) return;
        unsigned at[kCount];
#pragma unroll
        for (int x = 0; x < kCount; ++x) at[x] = fast_word(Q, v[e0 + x]).before - zeros + rank[e0 + x];
        const bool choose = zeros_here || !all(e0, kCount);    // the same in every lane
#pragma unroll
        for (int x = 0; x < kCount; ++x)
            if (!choose || v[e0 + x] > low) elems[at[x]] = v[e0 + x];
        __builtin_amdgcn_sched_barrier(0);
    });
    // what a walk reads past the last element adds nothing
    if (tid < kFastWalk) elems[len - zeros + tid] = ~0u;
    // look-ups whose parts inside buckets fit 32 bits together: one or two at least (see
    // fast_octave_bits), eight or more as a rule
    int run = (int)(0xffffffffu >> (kFastBits - 1 - obits)) >> (full & 2 ? kFastCrowdBits : full & 1 ? kFastCrowdLog : 4);
    run = run > 0 ? run : 1;                       // (a bucket's own parts fit: fast_parts_fit)
    __syncthreads();
    float *row = sse32 + (long long)t * n;
    if (full & 4) {
        for (int i = tid; i < len - zeros; i += kT)
            elems[i] = __float_as_uint((float)((double)(elems[i] - low) * F.per_unit));
        __syncthreads();
        fast_plain<kT, kPer == 20>(elems, len - zeros, n, Li, row);
        return;
    }
    const FastCurve c = {A, F.inv, low, n, Li, F.q, run};
    if (r.fast == 2 && usable && !keep_all) {
        // the sum is within 2e-6 of the tile's (at most 27 binary32 additions, 2^-24 each)
        const double U1 = (double)sum * (scale * F.per_unit) * 1.000002;
        const double U2 = A - (double)n * (double)n * (double)len + 2.0 * (double)n * U1;
        float *grid = reinterpret_cast<float *>(elems + len + kFastWalk);
        unsigned short *list = reinterpret_cast<unsigned short *>(grid + 2 * (prune_points(n, Li, kT) + 1));
        if (fast_pruned<kT>(Q, c, (float)U1 * 1.0001f, (float)U2 * 1.0001f, (float)len, pruned, grid, list,
                            reinterpret_cast<int *>(row)))
            return;
    }
    fast_candidates<kT>(Q, c, row);
}

} // namespace pwlq

// Host side of libpwlq: argument checks, the per-call tensor table, workspace
// layout and kernel launches.  See include/pwlq.h for the contract.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <atomic>
#include <mutex>
#include <numeric>
#include <vector>

#include "../../include/pwlq.h"
#include "../../include/pwlq_bench.h"
#include "pwlq_kernels.h"

// Scratch of pwlq_search_static: one copy per GPU, resident until the process
// ends.  In host code this name is only a handle for hipGetSymbolAddress; the
// device address it yields is what kernels and copies are given.
static __device__ __align__(256) unsigned char scratch[PWLQ_STATIC_SCRATCH_BYTES];

namespace {

using namespace pwlq;

thread_local char g_error[512] = "";
thread_local long long g_last_tiles = 0, g_last_groups = 0, g_last_units = 0;
thread_local const char *g_last_search_kernel = "k_search";
// What the thread's last search or inner product launched, for pwlq_last_kernels.
struct Launched {
    enum { kNone, kSmall, kSearch, kLinearRows, kLinearSplit, kLinearWide, kLinear } what = kNone;
    int fast_threads[4] = {};      // workgroup sizes of the k_fast launches, in order
    int n_fast = 0;
    int slices = 0;                // of k_search_sliced; 1: k_search; 0: neither
    int bits = 0, planes = 0, row_tile = 0, row_mt = 0;
};
thread_local Launched g_launched;
thread_local char g_launched_text[160] = "";

int fail(int status, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_error, sizeof(g_error), fmt, ap);
    va_end(ap);
    return status;
}

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

constexpr long long kBeside = 1;                   // tiles of k_fast that count for the units' size, per tile that is not

// Everything a call needs to know about its tensors, built on the host.
struct Plan {
    std::vector<TensorRec> recs;
    std::vector<int> tile_prefix, group_prefix, unit_prefix, mgroup_prefix, emit_prefix;
    int nt = 0;
    long long n_tiles = 0, n_groups = 0, n_units = 0, n_mgroups = 0, n_chunks = 0;
    long long n_all_units = 0;     // n_units if k_fast took no tiles
    int n = 0, nblk = 0;
    // workspace offsets in bytes
    size_t off_recs = 0, off_prefix = 0, off_tile_max = 0, off_gm = 0, off_offsets = 0,
           off_sorted = 0, off_sse32 = 0, off_mask = 0, off_part = 0, off_gsum = 0,
           off_stat_max = 0, off_stat_s2 = 0, off_stat_s1 = 0, off_fine = 0, total = 0;
    bool fine = false;     // tiles ordered by candidate, with per-candidate switch positions
};

// per-tile scratch beyond the tensor table
enum Aux { kAuxNone = 0, kAuxStats = 1, kAuxMse = 2 };

int check_common(int bits, int mode)
{
    if (bits < 2 || bits > 8) return fail(PWLQ_EINVAL, "bits=%d outside [2,8]", bits);
    if (mode != PWLQ_PER_CHANNEL && mode != PWLQ_PER_TENSOR)
        return fail(PWLQ_EINVAL, "mode=%d is neither PWLQ_PER_CHANNEL nor PWLQ_PER_TENSOR", mode);
    return PWLQ_OK;
}

// Whether n candidates are enough for a grid of them, and not so many that most tiles would have more within the
// threshold than are kept, and be evaluated in full after all.  The threshold is 6e-5 + 2.4e-5 L above the least
// value, since the rounding in its slack is in proportion to n / m as the error is, and the values are a parabola in
// k / n around the least one: about n sqrt(6e-5 + 2.4e-5 L) candidates, in proportion.  At 112 of that measure no
// weights but uniform ones lose (64x5000, all / pruned: b = 4, n = 7000 137/108, n = 12000 166/173; b = 6, n = 3000
// 87/63, n = 6000 155/161; b = 8, n = 2000 179/159, n = 5000 408/424); from n = 8000 on at two and three bits some do
// (200x700, b = 3, n = 10000 78/84).
bool grid_pays(int n, int L)
{
    return n >= kPruneMin && n <= 8000 && (long long)n * n * (60 + 24 * L) <= 112LL * 112 * 1000000;
}

// Threads that k_fast gives a tile, by the longest of a launch's tiles.  A short tile is
// served fastest by few threads where there are many tiles (see k_fast), but a thread then
// walks many candidates one after the other: where the tiles are too few to hide that
// (b = 4, n = 4000, us, 128 or 256 / 512 threads: 512x121 72/37, 512x300 46/39; n = 1000,
// 1024x121 24.7/22.6, 2048x121 31.8/36.1; n = 300, 1024x121 14.9/17.2) they get 512.
//
// Longer tiles likewise: 256 threads where a launch has many and their look-ups are few, 512 where not (us, 512 / 256:
// 38 400 tiles of 4096, n = 1000, b = 4, k_fast alone 508/386; but 2500x4608, 512 threads with fewer candidates left out than
// now: n = 290, without the grid of candidates, b = 5, 68/75, b = 6 85/101; b = 7, n = 700 146/196).
//
// One wavefront to a short tile where a launch has many and its look-ups are few (at b = 3 and 4 a grid leaves 60 to 140 of 1000
// candidates; at b = 2 all below 704 are looked up, two each): both wavefronts of 128 threads repeat the reductions and prefixes, and
// one waits for the other.  8192 and 25 000 tiles of 9 to 256, time with 64 threads / 128: b = 2, n = 300 to 703 0.89 to 1.03, 704 to 1200,
// which 128 threads look up without a grid, 0.45 to 0.73, 1500 and 2000 0.84 to 0.98; b = 3, n = 300 to 1000 0.63 to 0.90, to
// 2000 0.84 to 1.00; b = 4, n = 300 to 1000 0.76 to 0.93, to 1500 0.80 to 1.00, 2000 0.87 to 1.02, 3000 0.90 to 1.08; b = 2, n = 5000
// up to 1.34.  Not at five bits (1.01 to 1.13), nor for few tiles (2100, b = 4, n = 1000 up to 1.05).
int fast_threads(int longest, long long tiles, int n, int L)
{
    if (longest > kFastLong) return 1024;
    if (longest > kSmallTile)
        return tiles > kFastManyTiles && L <= 15 && (n >= kPruneMin || n * L <= 2500) ? 256 : 512;
    const bool short_tiles = longest <= kFastShort;
    if (short_tiles && tiles >= kFastWaveTiles && L <= 7 && n <= kFastWaveCand && grid_pays(n, L)) return 64;
    if (tiles <= (short_tiles ? 1024 : 512) && (long long)n * L >= 3500) return 512;
    return short_tiles ? 128 : 256;
}

// Whether the tiles of a launch that are groups of their own look up a grid of candidates first and
// then only those that it does not exclude (see fast_pruned): where a thread would have 11 or
// more pairs of look-ups for all candidates, or 20 where the workgroups are fewer than the CUs, and each
// waits out the three steps alone (us, all / pruned: 512 threads, 4096x4608, b = 4, n = 1000
// 119/108, n = 400 88/93; 256 threads, 4096x1024, n = 700 55/46, n = 300 41/41; 128 threads,
// 20000x128, n = 1000 191/101, n = 4000 740/155, n = 256 89/86; 1024 threads, 700x8192, n = 1000
// 60/61, n = 4000 188/168; 64x600, n = 1000 15.5/16.1, n = 4000 31/20).
//
// At 7 and 8 bits the grid leaves about 60 and 76 of 100 candidates.  Fewer workgroups than CUs take as long
// as a thread's candidates, so these have to get fewer (250x2000, b = 7: n = 1000 47/51, n = 1300 61/52; 64x5000, b = 8: n = 1500
// 143/149, n = 1700 169/155); more of them gain from n = 600 and 1500 on, or always (1024x1155, b = 7: n = 500 51/54,
// n = 700 66/59; 2500x4608 n = 500 182/158; 300x7000, b = 8, n = 1500 213/196; 64x5000, n = 1000 93/102).
bool fast_prunes(int threads, int tiles, int n, int L)
{
    if (!grid_pays(n, L)) return false;
    if ((long long)n * L < (tiles < 256 ? 20 : 11) * threads) return false;
    if (L < 63) return true;
    const auto rounds = [&](int count) { return (count + threads - 1) / threads; };
    if (tiles < 256) return rounds(n * (L == 63 ? 60 : 76) / 100) < rounds(n);
    return L == 63 ? n >= 600 || tiles >= 2048 : n >= 1500;
}

// Tiles by length, longest first: those of a class need workgroups and LDS of one size.
int size_class(int len) { return len > kFastLong ? 0 : len > kSmallTile ? 1 : len > kFastShort ? 2 : 3; }

// Whether the `shorter` tiles of at most `next` elements behind the `longer` ones of at most `longest` of a launch get a
// launch of their own: where both sides have enough of them, or the shorter ones alone.  Workgroups of 512 and 1024 threads
// are much too large for them (us, together / apart: 500x8000 and 5000x9, b = 4, n = 1000 159/76, 77x5816 and 3776x377,
// n = 1128 130/70; 1281 tiles of 838 behind 39 of 5652 38/41).  Of 256 threads, which tiles of more than kFastShort elements
// would have in either case, only those that get fewer, and only where they are many (12x607 and 4308x59, b = 2, n = 1223 47/58,
// 70x4518 and 5564x77, b = 3, n = 1628 72/64, 41x3171 and 8351x19, n = 369 64/44).
bool own_launch(int longest, long long longer, int next, long long shorter, int n, int L)
{
    if (shorter < kFastLaunchTiles) return false;
    if (longer >= kFastLaunchTiles) return true;
    if (fast_threads(longest, longer + shorter, n, L) >= 512) return shorter >= kFastOwnTiles;
    return next <= kFastShort && (shorter >= kFastWaveTiles || (shorter >= kFastOwnShort &&
                                                                fast_prunes(fast_threads(next, shorter, n, L), (int)shorter, n, L)));
}

// Whether tiles from `low` elements on are handed to the prefix-sum evaluator, shorter ones than its look-ups of all
// candidates pay for: where 2048 tiles and more look up a grid of them first (see grid_pays) a
// tile costs the same whatever its length, and less than its pass, down to the 3x3 kernels of a depthwise layer
// (kFastShortest): at up to four bits at every length (us, passes / look-ups: 7136x9, b = 4, n = 1000 44/34, n = 3000
// 108/41, b = 3, n = 300 32/32; the searches of MobileNetV2's shapes, b = 4, n = 1000 164/118, for which the shortest
// tiles need no launches of their own; 16384 tiles of 18 to 119, n = 1000, 0.60 to 0.33 of the time), at five bits at
// every length from 1000 candidates on and else from 64 (n = 300, 16384x48 1.00, x64 0.93 of the time), at six from
// 150 and 1000 (16384x150 0.81, x64 1.07; n = 300 1.25).
//
// Where launches of the short tiles alone look up all candidates after all (b = 2 below 1408 candidates, or 704 in one
// wavefront; b = 3 below 470) these are few enough for any length but nine, whose pass is two vectors: tiles of nine alone
// lose from some number on (b = 3, n = 400, 4000 tiles 0.96, 7136 1.06 of the time; b = 2, n = 700, 20000 tiles 0.96, 60000
// 1.06; with the grid b = 5, n = 1000, 12000 tiles 1.00, 20000 1.05, 60000 1.21, but n = 1100, one more block of candidates
// in the pass, 0.79).
//
// Not where they would share workgroups of 512 or 1024 threads with a few longer tiles (see own_launch).
bool many_short(const std::vector<TensorRec> &recs, int low, int always, int n, int L)
{
    long long counts[4] = {}, tiles = 0, nine = 0;             // by size_class
    for (const TensorRec &r : recs) {
        if (r.tile_len < low) continue;
        counts[size_class(r.tile_len)] += r.ntiles;
        if (r.tile_len < always && r.tile_len <= kSmallTile) tiles += r.ntiles;
        if (r.tile_len == kFastShortest) nine += r.ntiles;
    }
    if (tiles < 2048) return false;
    const long long small = counts[2] + counts[3];
    const int next = counts[2] > 0 ? kSmallTile : kFastShort;
    const bool cut = counts[0] > 0 && counts[1] > 0 && own_launch(kTileMax, counts[0], kFastLong, counts[1] + small, n, L);
    const long long longer = counts[1] + (cut ? 0 : counts[0]);
    const int longest = longer > counts[1] ? kTileMax : kFastLong;
    if (longer > 0 && !own_launch(longest, longer, next, small, n, L) && fast_threads(longest, longer + small, n, L) > 256) return false;
    if (4 * nine <= 3 * small) return true;
    if (L == 15) return n > 1024 || small <= 12288;
    return small * L <= 16384 || fast_prunes(fast_threads(kFastShort, small, n, L), (int)small, n, L);
}

// Shortest tile handed to the prefix-sum evaluator by the fast search: its cost per
// candidate grows with the number of half-way points (2L look-ups) and hardly depends on
// the tile length, the plain evaluation costs one pass over the tile.  16384 tiles, 1000
// candidates, b = 4, us, look-ups of all candidates / pass: 160 elements 168 / 249, 96 elements 162 / 178,
// 64 elements 157 / 144; but a line at 6 * 2L cost MobileNetV2 shapes 216 -> 238, one more
// launch beside the passes over the shorter tiles, which stay.  At b = 8 and many
// candidates the line is a little longer (2048 and 1024 tiles of 2048, n = 1000: 297/286,
// 169/160; n = 300: 149/194, 78/120).
//
// Below 2048 tiles the look-ups of a tile, L pairs for every candidate of a thread one after
// the other at about 0.3 us, take as long for one tile as for all, and the passes are spread over
// the chip: tiles not far above that length are handed over only where the look-ups'
// time is less than the passes' at 1.6e13 evaluations a second on a full chip and 6 us for
// their launch (16x121, n = 20000, us, look-ups / pass 99/54; 64x2048, b = 8, n = 2000 116/46; 512x121,
// n = 1000 15.5/20.3).
int fast_min_len(const std::vector<TensorRec> &recs, int bits, int n)
{
    const int L = (1 << (bits - 1)) - 1;
    const int shortest = (bits == 8 && n >= 800 ? 9 : 8) * (2 * L) + 8, always = 16 * (2 * L + 1) + 64;
    long long tiles = 0, elements = 0;
    if (grid_pays(n, L) && (L <= 15 || (L == 31 && n >= 1000))) {
        const int low = L == 31 ? 150 : L == 15 && n < 1000 ? 64 : kFastShortest;
        if (many_short(recs, low, always, n, L)) return low;
    }
    int longest = 0;
    for (const TensorRec &r : recs) {
        if (r.tile_len < shortest || r.tile_len >= always) continue;
        tiles += r.ntiles;
        elements += (long long)r.ntiles * r.tile_len;
        longest = std::max(longest, r.tile_len);
    }
    if (tiles >= 2048) return shortest;
    const int threads = fast_threads(longest, tiles, n, L);
    const long long look_ups_ns = (long long)((n + threads - 1) / threads) * L * 300;
    const long long wavefronts = tiles * ((n + kBlk - 1) / kBlk);
    const long long per_ns = 16000 * std::min(wavefronts + 1024, 8192LL) / 8192;
    const long long passes_ns = 6000 + elements * n / per_ns;
    return look_ups_ns <= passes_ns ? shortest : always;
}

struct FastLaunch {
    int begin, end, threads, longest;
    bool prunes;
};

// The launches of k_fast.  A launch's workgroups and LDS are sized for its longest tile; shorter
// tiles get launches of their own where both sides have enough of them.  Tensors are ordered
// longest tile first, so the fast tiles are 0 .. fast_tiles-1.
int plan_fast_launches(Plan &pl, int fast_tiles, int n, int L, FastLaunch (&out)[4])
{
    int launches = 0, begin = 0, seen = 0, longest = 0;
    size_t first = 0;
    for (size_t i = 0; i < pl.recs.size() && pl.recs[i].fast; ++i) {
        longest = std::max(longest, pl.recs[i].tile_len);
        seen += pl.recs[i].ntiles;
        const bool last = seen == fast_tiles;
        if (!last && (size_class(pl.recs[i + 1].tile_len) == size_class(longest) ||
                      !own_launch(longest, seen - begin, pl.recs[i + 1].tile_len, fast_tiles - seen, n, L)))
            continue;
        const int threads = fast_threads(longest, seen - begin, n, L);
        const bool prunes = fast_prunes(threads, seen - begin, n, L);
        out[launches++] = {begin, seen, threads, longest, prunes};
        for (; first <= i; ++first) pl.recs[first].fast = prunes && pl.recs[first].tpg == 1 ? 2 : 1;
        begin = seen;
        longest = 0;
    }
    return launches;
}

// n_cand == 0 builds a plan without search scratch (quantizer, selectors, error).
// fast_bits > 0: the bit width of a fast search.
int build_plan(Plan &pl, const pwlq_tensor_desc *desc, int n_tensors, int n_cand, int mode,
               bool need_pointers, const int64_t *code_byte_offset = nullptr,
               const int64_t *flag_byte_offset = nullptr, Aux aux = kAuxNone,
               int fast_bits = 0)
{
    if (!desc) return fail(PWLQ_ENULL, "tensor descriptor table is NULL");
    if (n_tensors < 1) return fail(PWLQ_EINVAL, "n_tensors=%d must be >= 1", n_tensors);
    pl.nt = n_tensors;
    pl.n = n_cand;
    pl.nblk = (n_cand + kBlk - 1) / kBlk;

    struct Item { int idx; int tile_len; };
    std::vector<Item> order(n_tensors);
    std::vector<TensorRec> tmp(n_tensors);
    for (int i = 0; i < n_tensors; ++i) {
        const pwlq_tensor_desc &d = desc[i];
        if (need_pointers && !d.w) return fail(PWLQ_ENULL, "desc[%d].w is NULL", i);
        if (d.C < 1 || d.K < 1) return fail(PWLQ_EINVAL, "desc[%d]: C=%lld K=%lld must be >= 1", i,
                                            (long long)d.C, (long long)d.K);
        if (d.group_offset < 0 || d.elem_offset < 0)
            return fail(PWLQ_EINVAL, "desc[%d]: negative offset", i);
        if (d.C > (1LL << 40) / d.K) return fail(PWLQ_EINVAL, "desc[%d]: tensor too large", i);
        TensorRec r;
        memset(&r, 0, sizeof(r));
        r.w = d.w;
        const long long groups = (mode == PWLQ_PER_CHANNEL) ? d.C : 1;
        r.gcount = (mode == PWLQ_PER_CHANNEL) ? d.K : d.C * d.K;
        r.out_elem = d.elem_offset;
        r.out_group = d.group_offset;
        r.out_code_byte = code_byte_offset ? code_byte_offset[i] : 0;
        r.out_flag_byte = flag_byte_offset ? flag_byte_offset[i] : 0;
        if (r.out_code_byte < 0 || r.out_flag_byte < 0)
            return fail(PWLQ_EINVAL, "desc[%d]: negative byte offset", i);
        const long long tpg = (r.gcount + kTileMax - 1) / kTileMax;
        r.tile_len = (tpg == 1) ? (int)r.gcount : kTileMax;
        r.last_len = (int)(r.gcount - (tpg - 1) * (long long)r.tile_len);
        if (groups * tpg > 0x3fffffffLL) return fail(PWLQ_EINVAL, "desc[%d]: too many tiles", i);
        r.tpg = (int)tpg;
        r.ngroups = (int)groups;
        r.ntiles = (int)(groups * tpg);
        r.stride = (r.tile_len + kVec - 1) / kVec * kVec + kVec;   // one spare vector: loads may run one ahead
        tmp[i] = r;
        order[i] = {i, r.tile_len};
    }
    if (fast_bits > 0) {
        const int min_len = fast_min_len(tmp, fast_bits, n_cand);
        for (TensorRec &r : tmp) r.fast = r.tile_len >= min_len ? 1 : 0;
    }
    // a search workgroup walks tpu tiles one after the other; keep enough
    // workgroups to fill the chip when the call is small.  Tiles that k_fast evaluates are in no unit, but
    // as many of them as others count here: fewer and larger units and workgroups beside them are faster (us, sized for the others
    // alone / so: 470x6256 and 8056x104, b = 7, n = 985, 180/171; 553x5959 and 3924x338, b = 6, n = 77, 103/97; 1735x632 and 7957x118,
    // b = 4, n = 209, 81/78), but not where few are left (all counted: up to 1.03 times the time, on the average the same).
    const auto size_units = [&](bool all) {
        long long total_tiles = 0, tiny_tiles = 0, fast_tiles = 0, fast_tiny = 0, units = 0;
        const auto tiny = [](const TensorRec &r) { return r.tile_len <= kTinyTile && r.tpg == 1; };
        for (const TensorRec &r : tmp) {
            const bool in = all || !r.fast;
            (in ? total_tiles : fast_tiles) += r.ntiles;
            if (tiny(r)) (in ? tiny_tiles : fast_tiny) += r.ntiles;
        }
        total_tiles += std::min(fast_tiles, kBeside * total_tiles);
        tiny_tiles += std::min(fast_tiny, kBeside * tiny_tiles);
        const int cap = (int)std::max(1LL, total_tiles / kMinUnits);
        // tiles of at most kTinyTile elements cost a unit little each (no offsets, loads one
        // tile ahead): up to kTinyUnit per unit while they still make about a thousand units
        const int tiny_cap = (int)std::min((long long)kTinyUnit, std::max((long long)cap, tiny_tiles / 1024));
        for (TensorRec &r : tmp)
            if (all || !r.fast) {
                r.tpu = std::min(std::max(1, kUnitElems / r.tile_len), tiny(r) ? tiny_cap : cap);
                units += (r.ntiles + r.tpu - 1) / r.tpu;
            }
        return units;
    };
    pl.n_all_units = size_units(true);
    if (fast_bits > 0) size_units(false);
    // longest tiles first: the search kernel's workgroups are dispatched in
    // index order, so the big items start early and the small ones fill gaps
    // (selectors and error: of these, the groups of most tiles in front)
    std::stable_sort(order.begin(), order.end(), [&](const Item &a, const Item &b) {
        if (a.tile_len != b.tile_len || aux == kAuxNone) return a.tile_len > b.tile_len;
        return tmp[a.idx].tpg > tmp[b.idx].tpg;
    });
    pl.recs.resize(n_tensors);
    pl.tile_prefix.assign(n_tensors + 1, 0);
    pl.group_prefix.assign(n_tensors + 1, 0);
    pl.unit_prefix.assign(n_tensors + 1, 0);
    pl.mgroup_prefix.assign(n_tensors + 1, 0);
    pl.emit_prefix.assign(n_tensors + 1, 0);
    long long tiles = 0, groups = 0, units = 0, mgroups = 0, parts = 0, sorted = 0, chunks = 0;
    for (int s = 0; s < n_tensors; ++s) {
        TensorRec r = tmp[order[s].idx];
        r.tile_base = (int)tiles;
        r.group_base = (int)groups;
        r.unit_base = (int)units;
        r.mgroup_base = (int)mgroups;
        r.sorted_base = sorted;
        r.part_base = (r.tpg > 1) ? (int)parts : -1;
        pl.tile_prefix[s] = (int)tiles;
        pl.group_prefix[s] = (int)groups;
        pl.unit_prefix[s] = (int)units;
        pl.mgroup_prefix[s] = (int)mgroups;
        pl.emit_prefix[s] = (int)chunks;
        r.emit_base = (int)chunks;
        chunks += ((long long)r.ngroups * r.gcount + kEmitChunk - 1) / kEmitChunk;
        tiles += r.ntiles;
        groups += r.ngroups;
        if (!r.fast) units += (r.ntiles + r.tpu - 1) / r.tpu;
        if (r.tpg > 1) { mgroups += r.ngroups; parts += r.ntiles; }
        if (!r.fast) sorted += (long long)r.ntiles * r.stride;
        if (tiles > 0x3fffffffLL || units > 0x3fffffffLL || chunks > 0x3fffffffLL)
            return fail(PWLQ_EINVAL, "call has too many tiles");
        pl.recs[s] = r;
    }
    pl.tile_prefix[n_tensors] = (int)tiles;
    pl.group_prefix[n_tensors] = (int)groups;
    pl.unit_prefix[n_tensors] = (int)units;
    pl.mgroup_prefix[n_tensors] = (int)mgroups;
    pl.emit_prefix[n_tensors] = (int)chunks;
    pl.n_chunks = chunks;
    pl.n_tiles = tiles;
    pl.n_groups = groups;
    pl.n_units = units;
    pl.n_mgroups = mgroups;

    size_t off = 0;
    auto take = [&](size_t bytes) { size_t at = off; off = align_up(off + bytes, 256); return at; };
    pl.off_recs = take(sizeof(TensorRec) * (size_t)n_tensors);
    pl.off_prefix = take(sizeof(int) * 5 * (size_t)(n_tensors + 1));
    if (n_cand > 0) {
        pl.off_tile_max = take(sizeof(float) * (size_t)tiles);
        pl.off_gm = take(sizeof(float) * (size_t)groups);
        pl.off_offsets = take(sizeof(int) * (size_t)tiles * (size_t)(pl.nblk + 1));
        pl.off_sorted = take(sizeof(float) * (size_t)sorted);
        pl.off_sse32 = take(sizeof(float) * (size_t)tiles * (size_t)n_cand);
        pl.fine = n_cand <= kFineMax;
        if (pl.fine) pl.off_fine = take(sizeof(unsigned short) * (size_t)tiles * (size_t)(n_cand + 1));
        pl.off_mask = take(sizeof(int) * (size_t)mgroups * (size_t)(n_cand + 1));
        pl.off_part = take(sizeof(double) * (size_t)parts * (size_t)n_cand);
        pl.off_gsum = take(sizeof(double) * (size_t)mgroups * (size_t)n_cand);
    }
    if (aux == kAuxStats) {
        pl.off_stat_max = take(sizeof(float) * (size_t)tiles);
        pl.off_stat_s2 = take(sizeof(double) * (size_t)tiles);
        pl.off_stat_s1 = take(sizeof(double) * (size_t)tiles);
    } else if (aux == kAuxMse) {
        pl.off_stat_s2 = take(sizeof(double) * (size_t)tiles);
    }
    pl.total = off;
    return PWLQ_OK;
}

int check_workspace(const Plan &pl, const void *workspace, size_t bytes)
{
    if (!workspace) return fail(PWLQ_EWORKSPACE, "workspace is NULL (%zu bytes needed)", pl.total);
    if (((uintptr_t)workspace & 255) != 0)
        return fail(PWLQ_EWORKSPACE, "workspace is not 256-byte aligned");
    if (bytes < pl.total)
        return fail(PWLQ_EWORKSPACE, "workspace holds %zu bytes, %zu needed", bytes, pl.total);
    return PWLQ_OK;
}

// Writes the tensor table into the head of the workspace and returns the
// device-side view.  Tables of up to kUploadMaxBytes travel in the arguments of
// k_upload launches (asynchronous, nothing on the host has to outlive the call,
// recordable into a graph); longer ones are copied from a host image that lives
// only for this call, so the call waits for the copy, and cannot be recorded.
constexpr size_t kUploadMaxBytes = 16 * sizeof(UploadChunk);

int upload_tables(const Plan &pl, char *ws, hipStream_t stream, Tables &tb)
{
    memset(&tb, 0, sizeof(tb));
    tb.nt = pl.nt;
    tb.n_units = (int)pl.n_units;
    if (pl.nt == 1) {            // the record travels in the kernel arguments
        tb.one = pl.recs[0];
        return PWLQ_OK;
    }
    // host image of [off_recs, off_prefix + prefix bytes): records, padding, the five prefix arrays
    static_assert(sizeof(TensorRec) % 4 == 0, "the table is copied in 32-bit words");
    const size_t prefix_bytes = sizeof(int) * 5 * (size_t)(pl.nt + 1);
    const size_t bytes = pl.off_prefix - pl.off_recs + prefix_bytes;
    std::vector<unsigned int> image(bytes / 4, 0u);
    memcpy(image.data(), pl.recs.data(), sizeof(TensorRec) * (size_t)pl.nt);
    int *prefix = reinterpret_cast<int *>(image.data() + (pl.off_prefix - pl.off_recs) / 4);
    const std::vector<int> *parts[5] = {&pl.tile_prefix, &pl.group_prefix, &pl.unit_prefix,
                                        &pl.mgroup_prefix, &pl.emit_prefix};
    for (int i = 0; i < 5; ++i)
        memcpy(prefix + (size_t)i * (pl.nt + 1), parts[i]->data(), sizeof(int) * (size_t)(pl.nt + 1));
    if (bytes <= kUploadMaxBytes) {
        UploadChunk chunk;
        for (size_t w0 = 0; w0 < image.size(); w0 += kUploadWords) {
            const size_t nw = std::min((size_t)kUploadWords, image.size() - w0);
            memcpy(chunk.words, image.data() + w0, nw * 4);
            k_upload<<<1, kWG, 0, stream>>>(chunk, reinterpret_cast<unsigned int *>(ws + pl.off_recs) + w0,
                                            (int)nw);
        }
        if (hipGetLastError() != hipSuccess) return fail(PWLQ_EHIP, "table upload launch failed");
    } else {
        // this copy reads host memory that is gone when the call returns: a graph that
        // recorded it would read freed memory at every replay
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(stream, &cap) == hipSuccess && cap != hipStreamCaptureStatusNone)
            return fail(PWLQ_EINVAL, "a call with this many tensors copies its table from host memory "
                                     "and cannot be recorded into a graph");
        hipError_t e = hipMemcpyAsync(ws + pl.off_recs, image.data(), bytes, hipMemcpyHostToDevice, stream);
        if (e == hipSuccess) e = hipStreamSynchronize(stream);    // `image` is gone when this function returns
        if (e != hipSuccess) return fail(PWLQ_EHIP, "table upload: %s", hipGetErrorString(e));
    }
    tb.recs = reinterpret_cast<const TensorRec *>(ws + pl.off_recs);
    const int *p = reinterpret_cast<const int *>(ws + pl.off_prefix);
    tb.tile_prefix = p;
    tb.group_prefix = p + (pl.nt + 1);
    tb.unit_prefix = p + 2 * (pl.nt + 1);
    tb.mgroup_prefix = p + 3 * (pl.nt + 1);
    tb.emit_prefix = p + 4 * (pl.nt + 1);
    return PWLQ_OK;
}

// The quantize kernels' view of a small tensor table, for the kernel arguments.
bool fill_emit_args(const Plan &pl, EmitArgs &ea)
{
    memset(&ea, 0, sizeof(ea));
    if (pl.nt < 2 || pl.nt > kEmitArgTensors) return false;
    for (int i = 0; i < pl.nt; ++i) {
        const TensorRec &r = pl.recs[i];
        ea.w[i] = (long long)reinterpret_cast<uintptr_t>(r.w);
        ea.gcount[i] = r.gcount;
        ea.out_elem[i] = r.out_elem;
        ea.out_group[i] = r.out_group;
        ea.out_code_byte[i] = r.out_code_byte;
        ea.out_flag_byte[i] = r.out_flag_byte;
        ea.ngroups[i] = r.ngroups;
        ea.emit_prefix[i] = pl.emit_prefix[i];
    }
    ea.emit_prefix[pl.nt] = pl.emit_prefix[pl.nt];
    ea.nt = pl.nt;
    return true;
}

// The same for the selectors and the error.
bool fill_stat_args(const Plan &pl, StatArgs &sa)
{
    memset(&sa, 0, sizeof(sa));
    if (pl.nt > kStatArgTensors) return false;
    for (int i = 0; i < pl.nt; ++i) {
        const TensorRec &r = pl.recs[i];
        sa.w[i] = (long long)reinterpret_cast<uintptr_t>(r.w);
        sa.gcount[i] = r.gcount;
        sa.out_group[i] = r.out_group;
        sa.tile_prefix[i] = pl.tile_prefix[i];
        sa.group_prefix[i] = pl.group_prefix[i];
    }
    sa.tile_prefix[pl.nt] = pl.tile_prefix[pl.nt];
    sa.group_prefix[pl.nt] = pl.group_prefix[pl.nt];
    sa.nt = pl.nt;
    return true;
}

// How many groups of a plan for the selectors get a wavefront each: those whose tiles are too
// many for one thread, which come first, and a few others with them.
int wide_groups(const Plan &pl)
{
    const int groups = (int)pl.n_groups;
    int wide = 0;
    for (const TensorRec &r : pl.recs) {
        if (r.tpg < kWideTiles) break;
        wide += r.ngroups;
    }
    return wide > 0 && groups - wide <= kWideRest ? groups : wide;
}

// Whether a launch holds so many workgroups of so many threads: from 2^32 threads on the
// runtime starts what is left after the wrap and reports nothing.
bool launch_fits(long long workgroups, int threads)
{
    return workgroups * threads <= 0xffffffffLL;
}

int launch_status(const char *what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(PWLQ_EHIP, "%s: %s", what, hipGetErrorString(e));
    return PWLQ_OK;
}

// Optional event timing of the dominant kernels (benchmarks only).
// A ring of the last kProfRing recorded launches per role, so that a benchmark
// can time a run of calls without waiting inside it.
constexpr int kProfRoles = 4, kProfRing = 64;
unsigned g_profile = 0;         // bit r: events are recorded around the kernel of role r
hipEvent_t g_ev[kProfRoles][kProfRing][2];
bool g_ev_made = false;
long long g_ev_count[kProfRoles] = {0, 0, 0, 0};     // launches recorded so far

// idx = 2*role for the event before the kernel, 2*role+1 for the one after it
void profile_mark(int idx, hipStream_t stream)
{
    if (!((g_profile >> (idx >> 1)) & 1u) || !g_ev_made) return;
    const int role = idx >> 1;
    (void)hipEventRecord(g_ev[role][g_ev_count[role] % kProfRing][idx & 1], stream);
    if (idx & 1) ++g_ev_count[role];
}

// Largest number of groups a search call may have and still run as one fused launch
// (PWLQ_SMALL_CALL_TILES overrides the default once; pwlq_set_small_call_tiles at any time).
std::atomic<int> &small_call_tiles()
{
    static std::atomic<int> v([] {
        const char *e = getenv("PWLQ_SMALL_CALL_TILES");
        return e ? atoi(e) : kSmallCallTiles;
    }());
    return v;
}

int run_search(const pwlq_tensor_desc *desc, int n_tensors, int bits, int n_cand, int mode,
               float *p_star, float *m_out, int32_t *k_star, double *mse, void *workspace,
               size_t workspace_bytes, void *stream_v, bool fast = false)
{
    int rc = check_common(bits, mode);
    if (rc) return rc;
    if (n_cand < 1 || n_cand > 65535) return fail(PWLQ_EINVAL, "n_cand=%d outside [1,65535]", n_cand);
    if (!p_star || !m_out || !k_star || !mse) return fail(PWLQ_ENULL, "an output pointer is NULL");
    Plan pl;
    rc = build_plan(pl, desc, n_tensors, n_cand, mode, true, nullptr, nullptr, kAuxNone,
                    fast ? bits : 0);
    if (rc) return rc;
    rc = check_workspace(pl, workspace, workspace_bytes);
    if (rc) return rc;
    // every limit is checked before the first launch: a failing call enqueues nothing
    const int ny = (pl.nblk + kSearchWaves - 1) / kSearchWaves;
    int bpw_log2 = 0, upw = 1;             // candidate blocks per unit in a workgroup, as a power of two; units per workgroup
    const auto search_wgs = [&](long long units) {
        const long long sized = std::min(pl.n_all_units, (1 + kBeside) * units);
        bpw_log2 = 0;
        while ((1 << bpw_log2) < std::min(pl.nblk, kSearchWaves)) ++bpw_log2;
        // ... but a small call keeps one unit per workgroup rather than a handful of workgroups
        while (bpw_log2 < 4 && sized / (kSearchWaves >> bpw_log2) < 2048) ++bpw_log2;
        upw = kSearchWaves >> bpw_log2;
        const long long unit_groups = (units + upw - 1) / upw;
        return (unit_groups + 7) / 8 * 8 * ny;
    };
    // (a fast search is refused where the exhaustive one of the same tensors would be)
    const long long all_wgs = search_wgs(pl.n_all_units), wgs = search_wgs(pl.n_units);
    // Too few wavefronts to keep the SIMDs busy: the tiles' elements are cut into slices.  With
    // 16 candidate blocks or more k_search's workgroups are full without slices, and those
    // past 2048 wavefronts gain only on long tiles (n = 4000, 4032 wavefronts, us, one / two
    // slices: tiles of 300 27.0/29.2, 550 34.8/37.5, 2048 81.9/86.0; n = 1000, 2080: 400
    // 21.7/23.0, 1150 39.4/39.2, 2048 59.9/55.6; n = 10000, 2512: 300 40.7/45.0, 2048 93.3/96.7,
    // 4608 221/220); beyond kFineMax candidates tiles of less than 512 lose too (471: 256
    // 33.5/35.1, 550 42.9/39.9).
    int slices = 1;
    {
        int longest_plain = 0;
        bool one_tile = true;
        for (const TensorRec &r : pl.recs)
            if (!r.fast) { longest_plain = std::max(longest_plain, r.tile_len); one_tile &= r.tpu == 1; }
        const long long wavefronts = pl.n_units * pl.nblk;
        const bool pays = (pl.nblk < kSearchWaves || wavefronts <= 2048 || longest_plain >= (pl.fine ? 2048 : 4096)) &&
                          (pl.fine || longest_plain >= 4 * kSliceMin);
        while (one_tile && pays && slices < 8 && 2 * slices * wavefronts <= kSlicedWaves &&
               longest_plain >= 2 * slices * kSliceMin)
            slices *= 2;
    }
    const long long group_sum_wgs = pl.n_mgroups * (long long)((n_cand + kSumCand - 1) / kSumCand);
    if (!launch_fits(group_sum_wgs, kWG) || !launch_fits(pl.n_mgroups ? pl.n_tiles : 0, kWG))
        return fail(PWLQ_EINVAL, "too many groups longer than one tile");
    const int NT = (int)pl.n_tiles;
    int longest = 0, fast_tiles = 0;
    // tiles of at most kSmallTile elements (a suffix of the tile order) get one wavefront each
    int nt_large = 0, longest_small = 0;
    for (const TensorRec &r : pl.recs) {
        if (r.fast) fast_tiles += r.ntiles;
        else longest = std::max(longest, r.tile_len);
        if (r.tile_len > kSmallTile) nt_large += r.ntiles;
        else if (!r.fast) longest_small = std::max(longest_small, r.tile_len);
    }
    if (NT - nt_large < 1024) nt_large = NT;     // too few short tiles to pay for launches of their own
    const int nt_small = NT - nt_large;
    // Single-tile groups only: the short tiles above 512 elements (next in the tile order) join
    // the two-wavefront launch of k_exact, so that the one-wavefront launch holds 8 elements per
    // thread instead of 16 and fits six wavefronts per SIMD like the other.
    int nt_mid = 0;
    if (pl.n_mgroups == 0 && nt_large > 0 && nt_small > 0)
        for (const TensorRec &r : pl.recs)
            if (r.tile_len <= kSmallTile && r.tile_len > 512) nt_mid += r.ntiles;
    if ((fast_tiles < NT && slices == 1 && !launch_fits(std::max(wgs, all_wgs), kSearchWaves * 64)) || !launch_fits(nt_small, 64) ||
        (longest > kSmallTile && !launch_fits(nt_large, pl.fine && longest > 256 * 16 ? 512 : kWG)) ||
        !launch_fits(nt_large + nt_mid, 128))
        return fail(PWLQ_EINVAL, "search grid too large");

    FastLaunch fast_launches[4];
    const int n_fast_launches = plan_fast_launches(pl, fast_tiles, n_cand, (1 << (bits - 1)) - 1, fast_launches);
    hipStream_t stream = (hipStream_t)stream_v;
    char *ws = (char *)workspace;
    Tables tb;
    rc = upload_tables(pl, ws, stream, tb);
    if (rc) return rc;
    float *tile_max = (float *)(ws + pl.off_tile_max);
    float *gm = (float *)(ws + pl.off_gm);
    int *offsets = (int *)(ws + pl.off_offsets);
    float *sorted = (float *)(ws + pl.off_sorted);
    float *sse32 = (float *)(ws + pl.off_sse32);
    unsigned short *fine = pl.fine ? (unsigned short *)(ws + pl.off_fine) : nullptr;
    int *klist = (int *)(ws + pl.off_mask);
    double *part64 = (double *)(ws + pl.off_part);
    double *gsum = (double *)(ws + pl.off_gsum);

    // A call too small to fill the chip: everything for a group in one workgroup, one launch.
    {
        int longest_any = 0;
        long long evals = 0;
        for (const TensorRec &r : pl.recs) {
            longest_any = std::max(longest_any, r.tile_len);
            evals += (long long)r.ntiles * r.tile_len * n_cand;
        }
        // (also for a fast search: at this size the fused exhaustive launch is the faster way
        // to the same result)
        if (pl.n_mgroups == 0 && NT <= small_call_tiles().load() && evals <= kSmallCallEvals &&
            longest_any <= kSmallLen && n_cand <= kSmallCand) {
            profile_mark(fast ? 4 : 0, stream);
            k_small<<<NT, kSmallWG, 0, stream>>>(tb, n_cand, pl.nblk, bits, p_star, m_out, k_star, mse);
            profile_mark(fast ? 5 : 1, stream);
            g_last_tiles = pl.n_tiles;
            g_last_groups = pl.n_groups;
            g_last_units = pl.n_tiles;
            g_last_search_kernel = "k_small";
            g_launched = Launched();
            g_launched.what = Launched::kSmall;
            return launch_status("search launch");
        }
    }
    g_last_search_kernel = fast ? "k_fast" : "k_search";
    Launched launched;
    launched.what = Launched::kSearch;
    if (pl.n_mgroups > 0) k_tile_absmax<<<NT, kWG, 0, stream>>>(tb, tile_max);
    if (fast_tiles > 0) {
        static_assert(sizeof(unsigned long long) * kFastWords + sizeof(unsigned) * (kTileMax + kFastWalk) +
                          8 * (kPruneGrid + 2) + 2 * kPruneList <= 63 * 1024,
                      "k_fast must fit the LDS a launch gets without asking for more");
        auto lds_bytes = [&](const FastLaunch &fl) {
            return sizeof(unsigned long long) * ((size_t)kFastOct << fast_octave_bits(fl.longest, fl.threads)) +
                   sizeof(unsigned) * (size_t)(fl.longest + kFastWalk) + (size_t)(fl.prunes ? prune_bytes(n_cand, (1 << (bits - 1)) - 1, fl.threads) : 0);
        };
        const FastUnits units = fast_units(n_cand, bits);
        profile_mark(4, stream);
        for (int i = 0; i < n_fast_launches; ++i) {
            const FastLaunch &fl = fast_launches[i];
            const size_t lds = lds_bytes(fl);
            launched.fast_threads[launched.n_fast++] = fl.threads;
            // a launch has less than 2^32 threads
            for (int at = fl.begin; at < fl.end; at += kFastGridMax) {
                const unsigned wgs = (unsigned)std::min(fl.end - at, kFastGridMax);
                switch (fl.threads) {
                    case 1024:
                        k_fast<1024, kTileMax / 1024><<<wgs, 1024, lds, stream>>>(tb, at, n_cand, bits, units, tile_max, gm, sse32);
                        break;
                    case 512:
                        k_fast<512, kFastLong / 512><<<wgs, 512, lds, stream>>>(tb, at, n_cand, bits, units, tile_max, gm, sse32);
                        break;
                    case 64:
                        k_fast<64, kFastShort / 64><<<wgs, 64, lds, stream>>>(tb, at, n_cand, bits, units, tile_max, gm, sse32);
                        break;
                    case 128:
                        k_fast<128, kFastShort / 128><<<wgs, 128, lds, stream>>>(tb, at, n_cand, bits, units, tile_max, gm, sse32);
                        break;
                    default:
                        if (fl.longest > kSmallTile)
                            k_fast<256, kFastLong / 256><<<wgs, 256, lds, stream>>>(tb, at, n_cand, bits, units, tile_max, gm, sse32);
                        else
                            k_fast<256, kSmallTile / 256><<<wgs, 256, lds, stream>>>(tb, at, n_cand, bits, units, tile_max, gm, sse32);
                }
            }
        }
        profile_mark(5, stream);
    }
    if (fast_tiles < NT) {
        auto stage_bytes = [](int len) { return sizeof(float) * (size_t)((len + kVec - 1) / kVec * kVec); };
        const int nb2 = (pl.nblk + 1) / 2;
        // tiles that are not k_fast's, which come first
        const int large0 = std::min(fast_tiles, nt_large), small0 = std::max(fast_tiles, nt_large);
        const int n_large = nt_large - large0, n_small = NT - small0;
        const bool large = n_large > 0, small = n_small > 0;
        // long tiles are ordered by candidate (one bin per candidate and the switch
        // positions written out: worth it only where buckets can be long), short
        // ones by block of 64 candidates
        if (pl.fine) {
            if (large) {    // 512 threads x 16 elements: 256 x 32 measured 7-27 % slower, 1024 x 8 slower still
                if (longest <= 256 * 16)    // tiles of at most 4096 elements: smaller workgroups, twice as many in flight
                    k_prep<false, true, 256, 16><<<n_large, 256, sizeof(int) * n_cand + stage_bytes(longest), stream>>>(
                        tb, large0, n_cand, pl.nblk, tile_max, gm, offsets, fine, sorted);
                else
                    k_prep<false, true, 512, 16><<<n_large, 512, sizeof(int) * n_cand + stage_bytes(longest), stream>>>(
                        tb, large0, n_cand, pl.nblk, tile_max, gm, offsets, fine, sorted);
            }
            if (small)
                k_prep<true, false, 64, kSmallPer><<<n_small, 64, sizeof(int) * nb2 * 64 + stage_bytes(longest_small), stream>>>(
                    tb, small0, n_cand, pl.nblk, tile_max, gm, offsets, fine, sorted);
        } else if (pl.nblk <= 32) {
            if (large)
                k_prep<true, false, kWG, kPerThread><<<n_large, kWG, sizeof(int) * nb2 * kWG + stage_bytes(longest), stream>>>(
                    tb, large0, n_cand, pl.nblk, tile_max, gm, offsets, fine, sorted);
            if (small)
                k_prep<true, false, 64, kSmallPer><<<n_small, 64, sizeof(int) * nb2 * 64 + stage_bytes(longest_small), stream>>>(
                    tb, small0, n_cand, pl.nblk, tile_max, gm, offsets, fine, sorted);
        } else {
            if (large)
                k_prep<false, false, kWG, kPerThread><<<n_large, kWG, sizeof(int) * pl.nblk + stage_bytes(longest), stream>>>(
                    tb, large0, n_cand, pl.nblk, tile_max, gm, offsets, fine, sorted);
            if (small)
                k_prep<false, false, 64, kSmallPer><<<n_small, 64, sizeof(int) * pl.nblk + stage_bytes(longest_small), stream>>>(
                    tb, small0, n_cand, pl.nblk, tile_max, gm, offsets, fine, sorted);
        }
        profile_mark(0, stream);
        launched.slices = slices;
        if (slices > 1) {
            const int search_ny = (pl.nblk * slices + kSearchWaves - 1) / kSearchWaves;
            const int bw = (pl.nblk + search_ny - 1) / search_ny;
            k_search_sliced<<<(unsigned)(pl.n_units * search_ny), (unsigned)(bw * slices) * 64, 0, stream>>>(
                tb, n_cand, pl.nblk, bits, search_ny, bw, slices, offsets, sorted, fine, pl.fine ? nt_large : 0, sse32);
        } else
            k_search<<<(unsigned)wgs, kSearchWaves * 64, 0, stream>>>(tb, n_cand, pl.nblk, bits, ny, upw, bpw_log2,
                                                        offsets, sorted, fine, pl.fine ? nt_large : 0, sse32);
        profile_mark(1, stream);
    }
    if (pl.n_mgroups > 0) {
        k_group_sum<<<(unsigned)group_sum_wgs, kWG, 0, stream>>>(tb, n_cand, sse32, gsum);
        k_flag<<<(int)pl.n_mgroups, kWG, 0, stream>>>(tb, n_cand, gm, gsum, klist);
    }
    if (nt_large > 0) {
        // single-tile groups only: workgroups of two wavefronts, twice as many in flight (the
        // stage is bound by latency); with groups spread over tiles, where a tile's threads
        // share the evaluation of the group's whole list, four wavefronts measured faster
        if (pl.n_mgroups == 0)
            k_exact<128><<<nt_large + nt_mid, 128, 0, stream>>>(tb, 0, n_cand, bits, gm, sse32, klist, part64,
                                                                p_star, m_out, k_star, mse);
        else
            k_exact<kWG><<<nt_large, kWG, 0, stream>>>(tb, 0, n_cand, bits, gm, sse32, klist, part64, p_star,
                                                       m_out, k_star, mse);
    }
    if (nt_small > 0) {
        if (nt_mid > 0) {
            if (nt_small > nt_mid)
                k_exact<64, 8><<<nt_small - nt_mid, 64, 0, stream>>>(tb, nt_large + nt_mid, n_cand, bits, gm, sse32,
                                                                      klist, part64, p_star, m_out, k_star, mse);
        } else {
            k_exact<64><<<nt_small, 64, 0, stream>>>(tb, nt_large, n_cand, bits, gm, sse32, klist, part64,
                                                     p_star, m_out, k_star, mse);
        }
    }
    if (pl.n_mgroups > 0)
        k_final<<<(int)pl.n_mgroups, kWG, 0, stream>>>(tb, n_cand, gm, klist, part64, p_star, m_out,
                                                       k_star, mse);
    g_last_tiles = pl.n_tiles;
    g_last_groups = pl.n_groups;
    g_last_units = pl.n_units;
    g_launched = launched;
    return launch_status("search launch");
}

int run_quantize(const pwlq_tensor_desc *desc, int n_tensors, int bits, int mode,
                 const float *p_star, const float *m, uint8_t *codes, uint8_t *flags, float *w_hat,
                 void *workspace, size_t workspace_bytes, void *stream_v)
{
    int rc = check_common(bits, mode);
    if (rc) return rc;
    if (!p_star || !m || !codes || !flags || !w_hat)
        return fail(PWLQ_ENULL, "an input or output pointer is NULL");
    Plan pl;
    rc = build_plan(pl, desc, n_tensors, 0, mode, true);
    if (rc) return rc;
    if (pl.nt > 1) {
        rc = check_workspace(pl, workspace, workspace_bytes);
        if (rc) return rc;
    }
    if (!launch_fits(pl.n_chunks, kWG)) return fail(PWLQ_EINVAL, "call has too many elements");
    hipStream_t stream = (hipStream_t)stream_v;
    Tables tb;
    static_assert(sizeof(Tables) + sizeof(EmitArgs) + 64 <= 4096, "a launch passes at most 4 KB");
    EmitArgs ea;
    if (pl.nt > 1 && fill_emit_args(pl, ea)) {          // the table travels with the launch
        memset(&tb, 0, sizeof(tb));
        tb.nt = pl.nt;
    } else {
        rc = upload_tables(pl, (char *)workspace, stream, tb);
        if (rc) return rc;
    }
    profile_mark(2, stream);
    if (pl.nt == 1) k_emit<<<(int)pl.n_chunks, kWG, 0, stream>>>(tb, EmitOne{0}, bits, p_star, m, codes, flags, w_hat);
    else k_emit<<<(int)pl.n_chunks, kWG, 0, stream>>>(tb, ea, bits, p_star, m, codes, flags, w_hat);
    profile_mark(3, stream);
    return launch_status("quantize launch");
}

int run_quantize_packed(const pwlq_tensor_desc *desc, int n_tensors, int bits, int mode,
                        const float *p_star, const float *m, uint8_t *packed_codes,
                        const int64_t *code_byte_offset, uint8_t *packed_flags,
                        const int64_t *flag_byte_offset, float *w_hat, void *workspace,
                        size_t workspace_bytes, void *stream_v)
{
    int rc = check_common(bits, mode);
    if (rc) return rc;
    if (!p_star || !m || !packed_codes || !packed_flags)
        return fail(PWLQ_ENULL, "an input or output pointer is NULL");
    if (n_tensors > 1 && (!code_byte_offset || !flag_byte_offset))
        return fail(PWLQ_ENULL, "byte offset tables are NULL");
    Plan pl;
    rc = build_plan(pl, desc, n_tensors, 0, mode, true, code_byte_offset, flag_byte_offset);
    if (rc) return rc;
    if (pl.nt > 1) {
        rc = check_workspace(pl, workspace, workspace_bytes);
        if (rc) return rc;
    }
    if (!launch_fits(pl.n_chunks, kEmitChunk / (w_hat ? 8 : 16)))
        return fail(PWLQ_EINVAL, "call has too many elements");
    hipStream_t stream = (hipStream_t)stream_v;
    Tables tb;
    EmitArgs ea;
    if (pl.nt > 1 && fill_emit_args(pl, ea)) {
        memset(&tb, 0, sizeof(tb));
        tb.nt = pl.nt;
    } else {
        rc = upload_tables(pl, (char *)workspace, stream, tb);
        if (rc) return rc;
    }
#define PWLQ_PACKED(B, PER, ARGS)                                                                  \
    k_emit_packed<B, PER><<<(int)pl.n_chunks, kEmitChunk / PER, 0, stream>>>(                      \
        tb, ARGS, p_star, m, packed_codes, packed_flags, w_hat)
#define PWLQ_PACKED_CASE(B)                                                                        \
    case B:                                                                                        \
        if (w_hat) {                                                                               \
            if (pl.nt == 1) PWLQ_PACKED(B, 8, EmitOne{0});                                         \
            else PWLQ_PACKED(B, 8, ea);                                                            \
        } else {                                                                                   \
            if (pl.nt == 1) PWLQ_PACKED(B, 16, EmitOne{0});                                        \
            else PWLQ_PACKED(B, 16, ea);                                                           \
        }                                                                                          \
        break;
    switch (bits) {
        PWLQ_PACKED_CASE(2)
        PWLQ_PACKED_CASE(3)
        PWLQ_PACKED_CASE(4)
        PWLQ_PACKED_CASE(5)
        PWLQ_PACKED_CASE(6)
        PWLQ_PACKED_CASE(7)
        PWLQ_PACKED_CASE(8)
    }
#undef PWLQ_PACKED_CASE
#undef PWLQ_PACKED
    return launch_status("packed quantize launch");
}

int run_select(const pwlq_tensor_desc *desc, int n_tensors, int mode, int selector, float *p_out,
               float *m_out, void *workspace, size_t workspace_bytes, void *stream_v)
{
    int rc = check_common(2, mode);
    if (rc) return rc;
    if (selector < PWLQ_SELECT_GAUSS_FIT || selector > PWLQ_SELECT_LAPLACE_SOLVE)
        return fail(PWLQ_EINVAL, "selector=%d is not a pwlq_selector", selector);
    if (!p_out || !m_out) return fail(PWLQ_ENULL, "an output pointer is NULL");
    Plan pl;
    rc = build_plan(pl, desc, n_tensors, 0, mode, true, nullptr, nullptr, kAuxStats);
    if (rc) return rc;
    rc = check_workspace(pl, workspace, workspace_bytes);
    if (rc) return rc;
    if (!launch_fits((pl.n_tiles + kWaves - 1) / kWaves, kWG) || !launch_fits(pl.n_mgroups, kSelectWG))
        return fail(PWLQ_EINVAL, "call has too many tiles");
    hipStream_t stream = (hipStream_t)stream_v;
    char *ws = (char *)workspace;
    Tables tb;
    StatArgs sa;
    static_assert(sizeof(Tables) + sizeof(StatArgs) + 128 <= 4096, "a launch passes at most 4 KB");
    if (fill_stat_args(pl, sa)) {
        memset(&tb, 0, sizeof(tb));
        tb.nt = pl.nt;
    } else {
        rc = upload_tables(pl, ws, stream, tb);
        if (rc) return rc;
    }
    float *tile_max = (float *)(ws + pl.off_stat_max);
    double *tile_s2 = (double *)(ws + pl.off_stat_s2);
    double *tile_s1 = (double *)(ws + pl.off_stat_s1);
    const unsigned tile_wgs = (unsigned)((pl.n_tiles + kWaves - 1) / kWaves);
    const int groups = (int)pl.n_groups, wide = wide_groups(pl);
    k_stats<<<tile_wgs, kWG, 0, stream>>>(tb, sa, (int)pl.n_tiles, tile_max, tile_s2, tile_s1);
    if (wide > 0)
        k_select<true><<<(unsigned)wide, kSelectWG, 0, stream>>>(tb, sa, 0, wide, selector, tile_max, tile_s2, tile_s1,
                                                                 p_out, m_out);
    if (wide < groups)
        k_select<false><<<(unsigned)((groups - wide + kSelectWG - 1) / kSelectWG), kSelectWG, 0, stream>>>(
            tb, sa, wide, groups, selector, tile_max, tile_s2, tile_s1, p_out, m_out);
    return launch_status("select launch");
}

int run_mse(const pwlq_tensor_desc *desc, int n_tensors, int bits, int mode, const float *p,
            const float *m, double *mse, void *workspace, size_t workspace_bytes, void *stream_v)
{
    int rc = check_common(bits, mode);
    if (rc) return rc;
    if (!p || !m || !mse) return fail(PWLQ_ENULL, "an input or output pointer is NULL");
    Plan pl;
    rc = build_plan(pl, desc, n_tensors, 0, mode, true, nullptr, nullptr, kAuxMse);
    if (rc) return rc;
    rc = check_workspace(pl, workspace, workspace_bytes);
    if (rc) return rc;
    if (!launch_fits((pl.n_tiles + kWaves - 1) / kWaves, kWG) || !launch_fits(pl.n_mgroups, kSelectWG))
        return fail(PWLQ_EINVAL, "call has too many tiles");
    hipStream_t stream = (hipStream_t)stream_v;
    char *ws = (char *)workspace;
    Tables tb;
    StatArgs sa;
    if (fill_stat_args(pl, sa)) {
        memset(&tb, 0, sizeof(tb));
        tb.nt = pl.nt;
    } else {
        rc = upload_tables(pl, ws, stream, tb);
        if (rc) return rc;
    }
    double *tile_sse = (double *)(ws + pl.off_stat_s2);
    const unsigned tile_wgs = (unsigned)((pl.n_tiles + kWaves - 1) / kWaves);
    // groups of several tiles, which come first, a wavefront each where the first is a wide one:
    // there is nothing to solve, so the others lose nothing by it
    const int groups = (int)pl.n_mgroups;
    k_mse_tile<<<tile_wgs, kWG, 0, stream>>>(tb, sa, (int)pl.n_tiles, bits, p, m, tile_sse, mse);
    if (groups > 0 && pl.recs[0].tpg >= kWideTiles)
        k_mse_final<true><<<(unsigned)groups, kSelectWG, 0, stream>>>(tb, sa, groups, tile_sse, mse);
    else if (groups > 0)
        k_mse_final<false><<<(unsigned)((groups + kSelectWG - 1) / kSelectWG), kSelectWG, 0, stream>>>(
            tb, sa, groups, tile_sse, mse);
    return launch_status("mse launch");
}

// Whether an inner product goes to k_linear_rows, against k_linear_split where that is
// possible and k_linear where not.  Its workgroups of eight wavefronts, two to a CU, decode
// the weights once per row tile: one tile, or up to 512 workgroups in one pass over the chip,
// beat both at every K, bit width and form (b = 4, us, rows / split / k_linear: K = 4096,
// 250x4096 26.1/31.6/48.8, 441x1000 19.1/28.6/46.1, 8x11008 12/-/59, 63x50000 102/-/186;
// K = 1024, 250x4096 10.3/13.4/18.9; sums apart, K = 4096, 250x4096 33.1/-/52.2).  Against
// that:
//  - b = 8 decodes a lane's weights in more registers and, on reductions beyond 2048, loses
//    to k_linear_split past one workgroup per CU (K = 4096: 256 workgroups 21.7/30.8, 512
//    36.5/31.0; K = 2048: 0.86-1.12 of it at 470 to 512).
//  - One tile of 32 to 63 rows, sums apart, short reductions, many channels: the call is its
//    output, which k_linear writes in longer runs (63x200000, K = 64 / 256: 122/102, 138/120,
//    faster by rows from K = 1024; 63x50000 36/33 and 40/39, at odd widths 38/42).
// Past 512 workgroups there is a second pass:
//  - k_linear_split is the better one (K = 4096, 441x4096 48.9/33.8, 1024x1000 38.3/30.5), but
//    for two row tiles up to K = 2048 (K = 1024, 126x11008 15.2/15.7; 2048: 0.87-0.97 of it),
//    or of up to 38 rows, whose upper halves read one row (K = 4096, N = 11008: 64 rows
//    32.8/36.8, 76 34.3/36.9, 88 38.3/37.0; b = 2, 112 rows 34.7/39.0, 126 42.3/39.1), at
//    b = 8 for those up to K = 1024; and at K = 512, its shortest, up to 768 workgroups
//    (0.90-1.05 of it; b = 8 1.10).
//  - With the sums apart k_linear, but for two row tiles, a third of its 192 rows (K = 1024,
//    126x11008 22.1/25.4, K = 4096 57.3/57.5; K = 64: 1.07 of it), and at up to 5 bits on
//    reductions from 1024 (189 to 378 rows, 640 to 768 workgroups: 0.85-1.04 of it; 896:
//    441x4096 29.0/23.9).
//  - Else, against k_linear, up to 900 workgroups, 740 on long reductions from 3 bits on (K =
//    4112, 378x4096, 378x4800, us, b = 2 50.8/55.7, 55.8/57.5, b = 3 57.4/60.4, 65.4/62.8; K =
//    4096, 378x4096 0.96 of it at b = 4, 0.99 at 7; b = 8 1.08-1.3 past 512).
bool linear_by_rows(int planes, int bits, long long K, int row_cap, long long row_tiles, long long row_cols,
                    int rows_per_tile, bool can_split)
{
    const long long wgs = row_tiles * row_cols;
    const bool wide = bits == 8 && K > 2048;
    if (row_tiles == 1) {
        if (planes == 3) return !(row_cap == 63 && K <= 256 && wgs > 2048);
        return !(can_split && wide && wgs > 512);
    }
    if (wgs <= 512) return !(can_split && wide && wgs > 256);
    const bool two = row_tiles == 2 && wgs <= 700, short_tiles = rows_per_tile <= (bits == 2 ? 56 : 38);
    if (can_split && bits < 8) return (two && (K <= 2048 || short_tiles)) || (K <= 512 && wgs <= 770);
    if (can_split) return two && K <= 1024 && short_tiles;
    if (planes == 3)
        return (two && K >= 256 && (!wide || (short_tiles && K <= 4096))) || (bits <= 5 && K >= 1024 && wgs <= 770);
    return wgs <= (K <= 2048 || bits == 2 ? 900 : bits == 8 ? 512 : 740);
}

// Workgroups of k_linear_rows: `tile` channels by up to cap = tile mt - 1 rows (and one of ones).
struct RowShape {
    int tile, mt, cap, rows;               // rows of a workgroup, the same in all but the last
    long long tiles, cols;                 // workgroups along the rows and along the channels
};
RowShape row_shape(long long M, long long N, int tile, int mt)
{
    RowShape rs;
    rs.tile = tile;
    rs.mt = mt;
    rs.cap = tile * mt - 1;
    rs.tiles = (M + rs.cap - 1) / rs.cap;
    rs.cols = (N + tile - 1) / tile;
    rs.rows = (int)((M + rs.tiles - 1) / rs.tiles);
    return rs;
}

// Smaller workgroups than 63 rows by 32 channels, where those leave CUs idle: a workgroup takes as
// long for its share of the reduction and its decoding whatever runs beside it, so the
// smallest share that one workgroup per CU covers the call with is the fastest, though more of
// them decode the same weights.  us by 32 x 63 / 16 x 31 / 32 x 31 / 16 x 63 (channels x rows):
// 63x2048x1000, b = 4 9.3/5.2/6.5/7.6 (189 workgroups of the second shape); 63x4096x1500 14.3/
// 11.2/9.6/11.7 (141 of the third); 250x2048x1000, b = 6, three sums, 12.2/12.2/12.7/10.1 (252 of
// the fourth).  Past one per CU they lose in the folded form (100x1024x4000 7.3/9.0/7.3/8.0; 63x4096x4096, 256 of the
// fourth, 14.9/16.1/15.5/15.5), but for short reductions, to two per CU of the third (126x256x3000
// 6.0/6.4/5.2/6.5); with the sums apart some calls past it would gain (700x512x1000, b = 6, 14.9/11.3 by the third).
// The fourth has twice the columns of workgroups, and each column reads all activations: only where
// these fit an XCD's 4 MiB of L2, or at 8 bits in the folded form, where it gains more than the
// reads cost (32 x 63 / 16 x 63: 2000x1024x100, b = 4, 7.2/6.4; 3000x4096x80 17.3/23.1; b = 8, 3000x8192x80 35.3/30.5).
// Few channels, where 32 x 63 are a handful of workgroups, gain most (16 x 31: 63x2304x64, b = 4, 9.9/5.4; 1900x4096x64 14.2/8.6).
RowShape smaller_row_shape(const RowShape &rs, long long M, long long K, long long N, int bits, int planes)
{
    if (rs.cap < 63) return rs;
    const auto wgs = [](const RowShape &r) { return r.tiles * r.cols; };
    const RowShape a = row_shape(M, N, 16, 2), b = row_shape(M, N, 32, 1), c = row_shape(M, N, 16, 4);
    if (wgs(a) <= 256) return a;
    if (wgs(b) <= (K <= 512 ? 512 : 256)) return b;
    return wgs(c) < 256 && (M * K <= 4 << 20 || (bits == 8 && planes == 2)) ? c : rs;
}

// Whether a call of y alone goes to k_linear_wide: its estimated time (us) against 0.97 of that of k_linear with k_linear_wsum,
// from 898 calls of 65 to 4096 rows and 90 to 1600 tiles of 256 x 128, most of them near the line (each within 7 % on
// the average).  Both pay per pass over the chip, of 256 workgroups (k_linear: half a pass; `xcd_wgs` of its workgroups are on the
// fullest XCD), for its start, its end and the reduction; and for y, k_linear_wide more where rows of y are no whole
// vectors, and then no less than a pass of full tiles does.  k_linear_wsum goes with N and N K.  Taken so, the calls' mean is
// 0.900 of the time by k_linear and k_linear_split (0.898 if the faster one were known each time), 7 of them lose more than
// 5 % and the worst 10: 1024x2064x8000 60.6/40.8, 4096x4096x5500 212/166, 100x4096x30000 91/58, 1721x7968x6440 242/211, but
// 4096x272x11008 64/70, 1072x16x3782 10.8/12.8, 1183x592x2977 16.5/19.1, 4096x64x3001 18.7/23.9.
// Below 100 tiles most of its CUs are idle (2048x4096x1600, 104 tiles, 49/54; 768x4096x2048, 48, 33/52), and
// k_linear_split, which has at most 384 workgroups, is beaten from 129 tiles on (128x4096x17000 60.1/55.5; 2600x4096x1000, 88
// tiles, 50/54).  A quarter of a tile's rows, or less, is left to k_linear, and so are the
// shortest reductions past one pass, which are their output (2048x64x11008 26.7/27.9).
bool linear_wide(long long M, long long K, long long N, const LinWideTiles &tiles, long long xcd_wgs, bool can_split)
{
    const long long count = (long long)tiles.rows * tiles.chans;
    if (M <= kLinWideBM / 4 || count < (can_split ? 129 : 100) || (count > 256 && K < 128)) return false;
    const auto passes = [](long long wgs, int per) { return (double)((wgs + per - 1) / per); };
    const double k = (double)K / 1000.0, full = (double)M / (double)(kLinWideBM * (long long)tiles.rows), part = (double)count / 256.0;
    const double wide = 1.5 + passes((count + 7) / 8, 32) * (5.4 + 13.1 * k) + full * (N % 4 ? 7.1 * std::max(part, 1.0) : 2.5 * part);
    const double tall = 7.1 + 2.8 * passes(xcd_wgs, 64) + 9.1 * passes(xcd_wgs, 32) * k + 2.2 * (double)xcd_wgs / 64.0 +
                        2.2e-4 * (double)N + 8.7e-5 * (double)N * k;
    return wide < 0.97 * tall;
}

int run_linear(const int8_t *xq, int64_t M, int64_t K, float s_x, float z_x,
               const uint8_t *packed_codes, const uint8_t *packed_flags, int64_t N, int bits,
               const float *p, const float *m, float *y, int32_t *acc, void *workspace,
               size_t workspace_bytes, void *stream_v)
{
    int rc = check_common(bits, PWLQ_PER_CHANNEL);
    if (rc) return rc;
    if (!xq || !packed_codes || !packed_flags || !p || !m || !y)
        return fail(PWLQ_ENULL, "an input or output pointer is NULL");
    if (M < 1 || N < 1 || K < 1) return fail(PWLQ_EINVAL, "M=%lld N=%lld K=%lld must be >= 1",
                                             (long long)M, (long long)N, (long long)K);
    if (K % 16 != 0) return fail(PWLQ_EINVAL, "K=%lld is not a multiple of 16", (long long)K);
    if (M > (1LL << 31) / 4 || N > (1LL << 31) / 4 || K > (1LL << 22))
        return fail(PWLQ_EINVAL, "matrix too large");
    if ((((uintptr_t)xq) | ((uintptr_t)packed_codes)) & 15)
        return fail(PWLQ_EINVAL, "xq and packed_codes must be 16-byte aligned");
    if (((uintptr_t)packed_flags) & 1) return fail(PWLQ_EINVAL, "packed_flags must be 2-byte aligned");
    const size_t need = align_up(sizeof(float) * (size_t)N, 256);
    if (!workspace) return fail(PWLQ_EWORKSPACE, "workspace is NULL (%zu bytes needed)", need);
    if (((uintptr_t)workspace & 255) != 0) return fail(PWLQ_EWORKSPACE, "workspace is not 256-byte aligned");
    if (workspace_bytes < need)
        return fail(PWLQ_EWORKSPACE, "workspace holds %zu bytes, %zu needed", workspace_bytes, need);
    // the three sums apart only when the caller asks for them; else the folded form
    const int planes = acc ? 3 : 2;
    const long long tiles_m = (M + lin_bm(planes) - 1) / lin_bm(planes), tiles_n = (N + kLinBN - 1) / kLinBN;
    const long long tn_per_xcd = (tiles_n + 7) / 8;
    const long long wgs = 8 * tn_per_xcd * tiles_m;
    float *wconst = (float *)workspace;
    const unsigned wsum_wgs = (unsigned)((N + kLinWG / 64 - 1) / (kLinWG / 64));
    RowShape rs = row_shape(M, N, M <= 31 ? 16 : 32, M <= 15 ? 1 : 2);
    // Where the rows leave it, k_linear_split up to one and a half of its workgroups per CU (each XCD counted as full as its
    // fullest: few channel tiles fill few XCDs); above that k_linear has as many
    // wavefronts without the second half's LDS traffic (K = 4096, b = 4, workgroups: us, k_linear
    // against k_linear_split: 256: 50.8/33.3, 320: 51.3/47.7, 352: 56.4/52.5, 384: 51.6/49.2,
    // 512: 52.5/54.3, 704: 77.2/79.0, 1024: 83/99).
    const long long split_m = (M + kSplitBM - 1) / kSplitBM, split_wgs = 8 * tn_per_xcd * split_m;
    const bool can_split = planes == 2 && K % (2 * kLinBK) == 0 && K >= kSplitMinK && split_wgs <= kSplitMaxWgs;
    const bool by_rows = linear_by_rows(planes, bits, K, rs.cap, rs.tiles, rs.cols, rs.rows, can_split);
    LinWideTiles wide;
    wide.rows = (int)((M + kLinWideBM - 1) / kLinWideBM);
    wide.chans = (int)((N + kLinWideBN - 1) / kLinWideBN);
    wide.cols = (wide.chans + 7) / 8;
    const long long wide_tiles = (long long)wide.rows * wide.chans;
    const bool by_wide = planes == 2 && !by_rows && wide_tiles <= kLinWideMaxTiles &&
                         linear_wide(M, K, N, wide, tn_per_xcd * tiles_m, can_split);
    const bool by_split = !by_rows && !by_wide && can_split;
    if (by_rows) rs = smaller_row_shape(rs, M, K, N, bits, planes);
    const dim3 row_grid((unsigned)rs.cols, (unsigned)rs.tiles);
    if (by_rows ? !launch_fits(rs.cols, 64 * kRowWaves)
        : by_wide ? !launch_fits(wide_tiles + 7, kLinWideWG)
                : !launch_fits(wgs, kLinWG) || !launch_fits((N + kLinWG / 64 - 1) / (kLinWG / 64), kLinWG))
        return fail(PWLQ_EINVAL, "grid too large");
    hipStream_t stream = (hipStream_t)stream_v;
    g_launched = Launched();
    g_launched.what = by_rows ? Launched::kLinearRows : by_wide ? Launched::kLinearWide : by_split ? Launched::kLinearSplit : Launched::kLinear;
    g_launched.bits = bits;
    g_launched.planes = planes;
    g_launched.row_tile = rs.tile;
    g_launched.row_mt = rs.mt;
#define PWLQ_LINEAR_ROWS(B, P, T, ...)                                                             \
    k_linear_rows<B, P, T, __VA_ARGS__><<<row_grid, 64 * kRowWaves, 0, stream>>>(                  \
        xq, M, K, s_x, z_x, packed_codes, packed_flags, N, p, m, y, acc, rs.rows)
#define PWLQ_LINEAR_CASE(B)                                                                       \
    case B:                                                                                        \
        if (by_rows) {                                                                             \
            profile_mark(6, stream);                                                               \
            if (planes == 3) {                                                                     \
                if (rs.tile == 16 && rs.mt == 1) PWLQ_LINEAR_ROWS(B, 3, 16, 1);                    \
                else if (B == 4 && rs.tile == 16 && rs.mt == 2 && rs.tiles * rs.cols > kRows31WavesWgs) \
                    PWLQ_LINEAR_ROWS(4, 3, 16, 2, kLookUps, kRows31Waves);                         \
                else if (rs.tile == 16 && rs.mt == 2) PWLQ_LINEAR_ROWS(B, 3, 16, 2);               \
                else if (rs.tile == 16) PWLQ_LINEAR_ROWS(B, 3, 16, 4);                             \
                else if (rs.mt == 1) PWLQ_LINEAR_ROWS(B, 3, 32, 1);                                \
                else PWLQ_LINEAR_ROWS(B, 3, 32, 2);                                                \
            } else {                                                                               \
                if (rs.tile == 16 && rs.mt == 1) PWLQ_LINEAR_ROWS(B, 2, 16, 1);                    \
                else if (rs.tile == 16 && rs.mt == 2) PWLQ_LINEAR_ROWS(B, 2, 16, 2);               \
                else if (rs.tile == 16) PWLQ_LINEAR_ROWS(B, 2, 16, 4);                             \
                else if (rs.mt == 1) PWLQ_LINEAR_ROWS(B, 2, 32, 1);                                \
                else if (B == 8 && K > kRows63BorrowsK && rs.tiles * rs.cols > 256)                \
                    PWLQ_LINEAR_ROWS(8, 2, 32, 2, kBorrows);                                       \
                else PWLQ_LINEAR_ROWS(B, 2, 32, 2);                                                \
            }                                                                                      \
            profile_mark(7, stream);                                                               \
            break;                                                                                 \
        }                                                                                          \
        if (by_wide) {                                                                             \
            profile_mark(6, stream);                                                               \
            k_linear_wide<B><<<(unsigned)((wide_tiles + 7) / 8 * 8), kLinWideWG, 0, stream>>>(        \
                xq, M, K, s_x, z_x, packed_codes, packed_flags, N, p, m, y, wide);                 \
            profile_mark(7, stream);                                                               \
            break;                                                                                 \
        }                                                                                          \
        if (planes == 3)                                                                           \
            k_linear_wsum<B, 3><<<wsum_wgs, kLinWG, 0, stream>>>(packed_codes, packed_flags, N, K, \
                                                                 p, m, wconst);                    \
        else                                                                                       \
            k_linear_wsum<B, 2><<<wsum_wgs, kLinWG, 0, stream>>>(packed_codes, packed_flags, N, K, \
                                                                 p, m, wconst);                    \
        profile_mark(6, stream);                                                                   \
        if (by_split && B == 8 && K <= kSplitBorrowsMaxK)                                          \
            k_linear_split<8, kBorrows><<<(unsigned)split_wgs, 2 * kLinWG, 0, stream>>>(           \
                xq, M, K, s_x, z_x, packed_codes, packed_flags, N, p, m, wconst, y,                \
                (int)split_m, (int)tiles_n, (int)tn_per_xcd);                                      \
        else if (by_split)                                                                         \
            k_linear_split<B, kLookUps><<<(unsigned)split_wgs, 2 * kLinWG, 0, stream>>>(           \
                xq, M, K, s_x, z_x, packed_codes, packed_flags, N, p, m, wconst, y,                \
                (int)split_m, (int)tiles_n, (int)tn_per_xcd);                                      \
        else if (planes == 3)                                                                      \
            k_linear<B, 3><<<(unsigned)wgs, kLinWG, 0, stream>>>(                                  \
                xq, M, K, s_x, z_x, packed_codes, packed_flags, N, p, m, wconst, y, acc,           \
                (int)tiles_m, (int)tiles_n, (int)tn_per_xcd);                                      \
        else                                                                                       \
            k_linear<B, 2><<<(unsigned)wgs, kLinWG, 0, stream>>>(                                  \
                xq, M, K, s_x, z_x, packed_codes, packed_flags, N, p, m, wconst, y, nullptr,       \
                (int)tiles_m, (int)tiles_n, (int)tn_per_xcd);                                      \
        profile_mark(7, stream);                                                                   \
        break;
    switch (bits) {
        PWLQ_LINEAR_CASE(2)
        PWLQ_LINEAR_CASE(3)
        PWLQ_LINEAR_CASE(4)
        PWLQ_LINEAR_CASE(5)
        PWLQ_LINEAR_CASE(6)
        PWLQ_LINEAR_CASE(7)
        PWLQ_LINEAR_CASE(8)
    }
#undef PWLQ_LINEAR_CASE
    return launch_status("linear launch");
}

// Device address of `scratch` on the current device, looked up once per device.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};

int static_scratch(void **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(PWLQ_EHIP, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(PWLQ_EHIP, "device index %d not supported", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return fail(PWLQ_EHIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev,
                        hipGetErrorString(e));
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return PWLQ_OK;
}

} // namespace

extern "C" {

int pwlq_search_static(const float *w, int64_t C, int64_t K, int bits, int n_cand, int mode,
                       float *p_star, float *m_out, int32_t *k_star, double *mse, void *stream)
{
    if (!w) return fail(PWLQ_ENULL, "w is NULL");
    int rc = check_common(bits, mode);
    if (rc) return rc;
    if (n_cand < 1 || n_cand > 65535) return fail(PWLQ_EINVAL, "n_cand=%d outside [1,65535]", n_cand);
    pwlq_tensor_desc d = {w, C, K, 0, 0};
    Plan pl;
    rc = build_plan(pl, &d, 1, n_cand, mode, true);
    if (rc) return rc;
    if (pl.total > (size_t)PWLQ_STATIC_SCRATCH_BYTES)
        return fail(PWLQ_EWORKSPACE,
                    "this search needs %zu bytes of scratch, the library's static buffer holds %zu: "
                    "call pwlq_search with a workspace of the caller's",
                    pl.total, (size_t)PWLQ_STATIC_SCRATCH_BYTES);
    void *ptr = nullptr;
    rc = static_scratch(&ptr);
    if (rc) return rc;
    return run_search(&d, 1, bits, n_cand, mode, p_star, m_out, k_star, mse, ptr,
                      (size_t)PWLQ_STATIC_SCRATCH_BYTES, stream);
}

size_t pwlq_linear_workspace_bytes(int64_t N)
{
    if (N < 1) return 0;
    return align_up(sizeof(float) * (size_t)N, 256);
}

int pwlq_linear_i8(const int8_t *xq, int64_t M, int64_t K, float s_x, float z_x,
                   const uint8_t *packed_codes, const uint8_t *packed_flags, int64_t N, int bits,
                   const float *p, const float *m, float *y, int32_t *acc, void *workspace,
                   size_t workspace_bytes, void *stream)
{
    return run_linear(xq, M, K, s_x, z_x, packed_codes, packed_flags, N, bits, p, m, y, acc,
                      workspace, workspace_bytes, stream);
}

size_t pwlq_select_list_workspace_bytes(const pwlq_tensor_desc *desc, int n_tensors, int mode)
{
    if (check_common(2, mode)) return 0;
    Plan pl;
    if (build_plan(pl, desc, n_tensors, 0, mode, false, nullptr, nullptr, kAuxStats)) return 0;
    return pl.total;
}

size_t pwlq_select_workspace_bytes(int64_t C, int64_t K, int mode)
{
    pwlq_tensor_desc d = {nullptr, C, K, 0, 0};
    return pwlq_select_list_workspace_bytes(&d, 1, mode);
}

int pwlq_select_analytic_list(const pwlq_tensor_desc *desc, int n_tensors, int mode, int selector,
                              float *p_out, float *m_out, void *workspace, size_t workspace_bytes,
                              void *stream)
{
    return run_select(desc, n_tensors, mode, selector, p_out, m_out, workspace, workspace_bytes,
                      stream);
}

int pwlq_select_analytic(const float *w, int64_t C, int64_t K, int mode, int selector,
                         float *p_out, float *m_out, void *workspace, size_t workspace_bytes,
                         void *stream)
{
    if (!w) return fail(PWLQ_ENULL, "w is NULL");
    pwlq_tensor_desc d = {w, C, K, 0, 0};
    return run_select(&d, 1, mode, selector, p_out, m_out, workspace, workspace_bytes, stream);
}

size_t pwlq_mse_list_workspace_bytes(const pwlq_tensor_desc *desc, int n_tensors, int mode)
{
    if (check_common(2, mode)) return 0;
    Plan pl;
    if (build_plan(pl, desc, n_tensors, 0, mode, false, nullptr, nullptr, kAuxMse)) return 0;
    return pl.total;
}

size_t pwlq_mse_workspace_bytes(int64_t C, int64_t K, int mode)
{
    pwlq_tensor_desc d = {nullptr, C, K, 0, 0};
    return pwlq_mse_list_workspace_bytes(&d, 1, mode);
}

int pwlq_mse_list(const pwlq_tensor_desc *desc, int n_tensors, int bits, int mode, const float *p,
                  const float *m, double *mse, void *workspace, size_t workspace_bytes,
                  void *stream)
{
    return run_mse(desc, n_tensors, bits, mode, p, m, mse, workspace, workspace_bytes, stream);
}

int pwlq_mse(const float *w, int64_t C, int64_t K, int bits, int mode, const float *p,
             const float *m, double *mse, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!w) return fail(PWLQ_ENULL, "w is NULL");
    pwlq_tensor_desc d = {w, C, K, 0, 0};
    return run_mse(&d, 1, bits, mode, p, m, mse, workspace, workspace_bytes, stream);
}

size_t pwlq_search_list_workspace_bytes(const pwlq_tensor_desc *desc, int n_tensors, int bits,
                                        int n_cand, int mode)
{
    if (check_common(bits, mode) || n_cand < 1 || n_cand > 65535) return 0;
    Plan pl;
    if (build_plan(pl, desc, n_tensors, n_cand, mode, false)) return 0;
    return pl.total;
}

size_t pwlq_search_workspace_bytes(int64_t C, int64_t K, int bits, int n_cand, int mode)
{
    pwlq_tensor_desc d = {nullptr, C, K, 0, 0};
    return pwlq_search_list_workspace_bytes(&d, 1, bits, n_cand, mode);
}

int pwlq_search_list(const pwlq_tensor_desc *desc, int n_tensors, int bits, int n_cand, int mode,
                     float *p_star, float *m_out, int32_t *k_star, double *mse, void *workspace,
                     size_t workspace_bytes, void *stream)
{
    return run_search(desc, n_tensors, bits, n_cand, mode, p_star, m_out, k_star, mse, workspace,
                      workspace_bytes, stream);
}

int pwlq_search(const float *w, int64_t C, int64_t K, int bits, int n_cand, int mode,
                float *p_star, float *m_out, int32_t *k_star, double *mse, void *workspace,
                size_t workspace_bytes, void *stream)
{
    if (!w) return fail(PWLQ_ENULL, "w is NULL");
    pwlq_tensor_desc d = {w, C, K, 0, 0};
    return run_search(&d, 1, bits, n_cand, mode, p_star, m_out, k_star, mse, workspace,
                      workspace_bytes, stream);
}

int pwlq_search_fast_list(const pwlq_tensor_desc *desc, int n_tensors, int bits, int n_cand,
                          int mode, float *p_star, float *m_out, int32_t *k_star, double *mse,
                          void *workspace, size_t workspace_bytes, void *stream)
{
    return run_search(desc, n_tensors, bits, n_cand, mode, p_star, m_out, k_star, mse, workspace,
                      workspace_bytes, stream, true);
}

int pwlq_search_fast(const float *w, int64_t C, int64_t K, int bits, int n_cand, int mode,
                     float *p_star, float *m_out, int32_t *k_star, double *mse, void *workspace,
                     size_t workspace_bytes, void *stream)
{
    if (!w) return fail(PWLQ_ENULL, "w is NULL");
    pwlq_tensor_desc d = {w, C, K, 0, 0};
    return run_search(&d, 1, bits, n_cand, mode, p_star, m_out, k_star, mse, workspace,
                      workspace_bytes, stream, true);
}

size_t pwlq_quantize_list_workspace_bytes(const pwlq_tensor_desc *desc, int n_tensors, int bits,
                                          int mode)
{
    if (check_common(bits, mode)) return 0;
    Plan pl;
    if (build_plan(pl, desc, n_tensors, 0, mode, false)) return 0;
    return pl.total;
}

int pwlq_quantize_list(const pwlq_tensor_desc *desc, int n_tensors, int bits, int mode,
                       const float *p_star, const float *m, uint8_t *codes, uint8_t *flags,
                       float *w_hat, void *workspace, size_t workspace_bytes, void *stream)
{
    return run_quantize(desc, n_tensors, bits, mode, p_star, m, codes, flags, w_hat, workspace,
                        workspace_bytes, stream);
}

int pwlq_quantize(const float *w, int64_t C, int64_t K, int bits, int mode, const float *p_star,
                  const float *m, uint8_t *codes, uint8_t *flags, float *w_hat, void *stream)
{
    if (!w) return fail(PWLQ_ENULL, "w is NULL");
    pwlq_tensor_desc d = {w, C, K, 0, 0};
    return run_quantize(&d, 1, bits, mode, p_star, m, codes, flags, w_hat, nullptr, 0, stream);
}

size_t pwlq_packed_code_bytes(int64_t count, int bits)
{
    if (count < 0 || bits < 2 || bits > 8) return 0;
    return (size_t)((count * bits + 7) / 8);
}

size_t pwlq_packed_flag_bytes(int64_t count) { return count < 0 ? 0 : (size_t)((count + 7) / 8); }

int pwlq_quantize_packed(const float *w, int64_t C, int64_t K, int bits, int mode,
                         const float *p_star, const float *m, uint8_t *packed_codes,
                         uint8_t *packed_flags, float *w_hat, void *stream)
{
    if (!w) return fail(PWLQ_ENULL, "w is NULL");
    pwlq_tensor_desc d = {w, C, K, 0, 0};
    return run_quantize_packed(&d, 1, bits, mode, p_star, m, packed_codes, nullptr, packed_flags,
                               nullptr, w_hat, nullptr, 0, stream);
}

int pwlq_quantize_packed_list(const pwlq_tensor_desc *desc, int n_tensors, int bits, int mode,
                              const float *p_star, const float *m, uint8_t *packed_codes,
                              const int64_t *code_byte_offset, uint8_t *packed_flags,
                              const int64_t *flag_byte_offset, float *w_hat, void *workspace,
                              size_t workspace_bytes, void *stream)
{
    return run_quantize_packed(desc, n_tensors, bits, mode, p_star, m, packed_codes,
                               code_byte_offset, packed_flags, flag_byte_offset, w_hat, workspace,
                               workspace_bytes, stream);
}

const char *pwlq_last_error(void) { return g_error; }

void pwlq_profile_enable(int roles)
{
    // the events are made here, on the first call that enables anything, so that no
    // call that launches kernels pays for them
    if (roles && !g_ev_made) {
        for (auto &role : g_ev)
            for (auto &slot : role)
                for (auto &ev : slot) (void)hipEventCreate(&ev);
        g_ev_made = true;
    }
    g_profile = (unsigned)roles & ((1u << kProfRoles) - 1u);
}

double pwlq_profile_ms(int role, int back)
{
    if (role < 0 || role >= kProfRoles || !g_ev_made) return -1.0;
    if (back < 0 || back >= kProfRing || back >= g_ev_count[role]) return -1.0;
    hipEvent_t *pair = g_ev[role][(g_ev_count[role] - 1 - back) % kProfRing];
    float ms = -1.0f;
    if (hipEventSynchronize(pair[1]) != hipSuccess) return -1.0;
    if (hipEventElapsedTime(&ms, pair[0], pair[1]) != hipSuccess) return -1.0;
    return (double)ms;
}

double pwlq_profile_last_ms(int role) { return pwlq_profile_ms(role, 0); }

void pwlq_last_search_shape(int64_t *n_tiles, int64_t *n_groups, int64_t *n_units)
{
    if (n_tiles) *n_tiles = g_last_tiles;
    if (n_groups) *n_groups = g_last_groups;
    if (n_units) *n_units = g_last_units;
}

int pwlq_set_small_call_tiles(int tiles)
{
    return small_call_tiles().exchange(tiles < 0 ? kSmallCallTiles : tiles);
}

const char *pwlq_last_search_kernel(void) { return g_last_search_kernel; }

const char *pwlq_last_kernels(void)
{
    const Launched &l = g_launched;
    char *const text = g_launched_text;
    const size_t room = sizeof(g_launched_text);
    text[0] = 0;
    size_t at = 0;
    switch (l.what) {
        case Launched::kNone: break;
        case Launched::kSmall: snprintf(text, room, "k_small"); break;
        case Launched::kSearch:
            for (int i = 0; i < l.n_fast; ++i)
                at += (size_t)snprintf(text + at, room - at, "%sk_fast<%d>", at ? " " : "", l.fast_threads[i]);
            if (l.slices > 1) snprintf(text + at, room - at, "%sk_search_sliced(%d)", at ? " " : "", l.slices);
            else if (l.slices == 1) snprintf(text + at, room - at, "%sk_search", at ? " " : "");
            break;
        case Launched::kLinearRows:
            snprintf(text, room, "k_linear_rows<%d, %d, %d, %d>", l.bits, l.planes, l.row_tile, l.row_mt);
            break;
        case Launched::kLinearSplit: snprintf(text, room, "k_linear_split<%d>", l.bits); break;
        case Launched::kLinearWide: snprintf(text, room, "k_linear_wide<%d>", l.bits); break;
        case Launched::kLinear: snprintf(text, room, "k_linear<%d, %d>", l.bits, l.planes); break;
    }
    return text;
}

const char *pwlq_kernel_name(int role)
{
    if (role == 0) return "k_search";
    if (role == 1) return "k_emit";
    if (role == 2) return "k_fast";
    if (role == 3) return "k_linear";
    return nullptr;
}

} // extern "C"

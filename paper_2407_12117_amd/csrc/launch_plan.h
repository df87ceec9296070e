// How a launch is cut into workgroups: the orders of work, and the choice of shape and order by estimated time.
// Host arithmetic on sizes alone (no HIP), included by the kernel sources and by the test that asks which shape a size gets.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <numeric>
#include <utility>

namespace memo {

inline constexpr int kXcds = 8, kChunk = 32;   // XCDs per device; compute units (one workgroup each) per XCD

// Two orders of work.  Every workgroup of a head streams that head's K/V rows (forward, dQ) or Q/dO
// rows (dK/dV), and a tile's sweep is as long as its distance from the end of the causal triangle.
//
// Folded (launches of many whole rounds): a workgroup works a PAIR of tiles of one head, the p-th longest
// and the p-th shortest, so every workgroup of a launch has the same length (ntiles + 1 tile units).
// Chunks of kChunk consecutive pairs go to one XCD (the dispatcher deals consecutive workgroup
// ids round-robin to the 8 XCDs; an XCD has 32 compute units and these kernels run one workgroup
// per unit), consecutive chunks to the 8 XCDs of a round.  The long tile is swept from the end all
// tiles share towards its own end, the short tile the other way round (forward and dQ: keys upwards
// from row 0, then downwards to row 0; dK/dV: queries downwards from row S-1, then upwards to it).
// Workgroup s of a chunk ends its first sweep a fixed number of steps per s before workgroup 0 and
// begins its second one as many steps further from the shared end, so the lengths cancel and the
// workgroups of an XCD read the same rows at about the same time in both sweeps, which is what
// lets that XCD's L2 serve most of those reads (measured: 32 workgroups, one fetch from the fabric,
// up to S = 256K; at S = 1M the forward keeps that, the two backward kernels drift apart over their
// 16384 steps and fetch about half of what they stream).
//
// Longest first (everything else): one tile per workgroup, in order of falling length, heads fastest, each
// unit taking the next tile when it is done.  A launch of 1.2 rounds of pairs costs two rounds, in
// this order 1.2 to 1.3 (S = 40000, H = 4: forward 2202 -> 1516 us); on whole rounds it is 2 % slower
// than folded (S = 128K: 14.84 against 14.59 ms), because the units of an XCD no longer sweep together.
enum BlockOrder { kFolded = 0, kLongestFirst = 1 };

// Every workgroup has 512 threads, and a HIP launch takes fewer than 2^32 of them: a longer grid would run in part, without an error.
inline constexpr int64_t kThreads = 512, kMaxBlocks = ((int64_t)1 << 32) / kThreads - 1;

inline int64_t order_grid(int64_t ntiles, int64_t heads, int order)
{
    if (order == kLongestFirst) return ntiles * heads;
    const int64_t round = kXcds * kChunk;
    return ((ntiles + 1) / 2 * heads + round - 1) / round * round;
}

// What a launch loses longest first when an XCD works many heads at a time.  Heads run fastest and workgroups are dealt
// round-robin, so an XCD meets heads / gcd(heads, 8) different ones, up to one per unit, and its L2 serves the fewer units
// the more heads it holds; folded chunks keep an XCD on one or two.  It costs nothing while the rows (1 KB of Q, K, V and dO
// each) are few enough for the cache behind the L2s, and grows with the doublings of the heads beyond that.  Measured,
// us, longest first against folded pairs.  Backward, one joint launch: S = 8192, 64 heads 3128 : 3052, 128 heads 6722 : 6272,
// 256 heads 14358 : 12799; S = 50000, 5 heads 8649 : 8290; but S = 4096, 32 heads 423 : 430, S = 25000, 8 heads (one per XCD)
// 3358 : 4221.  Forward: S = 400000, 5 heads 179997 : 173781, 4 heads (one) 137131 : 140589.
inline constexpr double kCrowdRows = 180e3;
inline double crowding(int64_t S, int64_t heads)
{
    const double met = (double)std::min<int64_t>(kChunk, heads / std::gcd(heads, (int64_t)kXcds));
    return std::log2(met) * std::max(0.0, 1.0 - kCrowdRows / ((double)S * heads));
}
inline constexpr double kCrowdedJoint = 0.08, kCrowdedAlone = 0.02;       // of the time, per doubling; 256-row launches of one kernel lose less

// Division by a launch constant d >= 1 as one high product: floor(2^32 / d) makes the quotient right or one too small.
struct Division { uint32_t quot, rem; };
struct Divisor {
    uint32_t d, inv;
    constexpr explicit Divisor(int64_t by) : d((uint32_t)by), inv(by == 1 ? 0xffffffffu : (uint32_t)(((uint64_t)1 << 32) / (uint64_t)by)) {}
    constexpr Division operator()(uint32_t x) const
    {
        const uint32_t quot = (uint32_t)(((uint64_t)x * inv) >> 32), rem = x - quot * d;
        return rem >= d ? Division{quot + 1, rem - d} : Division{quot, rem};
    }
};

// The order of one launch that works key tiles (dK/dV) and query tiles (dQ): all key tiles, longest first, and then all query tiles, longest
// first.  Position p stands for one tile of every head.  The key tiles take longer, their starts and ends most of all, the short query tiles
// fill the end, and units that work tiles of one kind share what they stream.  Key tiles shorter than the longest query tile spread among the query
// tiles instead, in launches of one to two rounds of workgroups: 134 sizes of 1 to 32 heads 2.2 % slower on average, us in front : spread,
// S = 825 H = 16 21.2 : 23.3, S = 1017 H = 32 44.7 : 48.5, S = 675 H = 6 13.3 : 14.4, S = 2041 H = 4 26.0 : 27.5, S = 1998 H = 6 33.4 : 34.0; the other way
// round where the key tiles nearly fill the first round, with up to five heads: S = 2962 H = 5 52.4 : 50.5, S = 8185 H = 1 74.0 : 71.7.  With fewer of
// them spread it is 0.5 % slower or more.  Beyond two rounds: S = 5000 H = 5 125 : 131, S = 12000 H = 5 554 : 571, S = 90000 H = 4 22307 : 22762.
struct JointSlot { bool key; uint32_t rank; };      // rank 0: the longest tile of its kind
constexpr JointSlot joint_slot(uint32_t key_tiles, uint32_t pos)
{
    return pos < key_tiles ? JointSlot{true, pos} : JointSlot{false, pos - key_tiles};
}

// Launches of 16- or 32-row workgroups that leave units idle: a tile goes to so many workgroups, each of which forms the scores again
// and its part of the output columns, as long as all of them find a unit.  What shrinks with the parts is the second half of a
// step's contractions, the accumulators to clear and the sums through the LDS at the end; output bits do not change.  us in 1 : 2 : 4
// parts, bf16 forward S = 32 H = 2 4.0 : 3.4 : 3.2, S = 640 H = 2 6.8 : 6.0 : 5.7, S = 2000 H = 1 12.0 : 10.9 : 10.8; bf16 backward with the D_i
// launch S = 32 H = 2 8.1 : 6.9 : 6.3, S = 500 H = 2 11.0 : 9.2 : 8.8.  With more workgroups than units it loses: two parts of S = 1000 H = 4
// backward 14.9 : 16.6, S = 2000 H = 4 forward 12.8 : 14.9.
// The units are idle only if nobody else wants them.  Beside a copy to the host no more is lost than in one part, and the copy takes as long.
// But calls on several streams at once meet that limit together: us for a forward and backward on every one of 1, 2, 3, 4 streams, one part : as
// here, S = 640 H = 2 18.6 : 16.0, 21.0 : 18.8, 23.4 : 22.5, 25.2 : 34.8; S = 1000 H = 2 23.1 : 20.2, 25.7 : 25.4, 28.5 : 36.1, 31.7 : 53.8.
inline int column_parts(int64_t blocks)
{
    const int64_t units = kXcds * kChunk;
    return blocks * 4 <= units ? 4 : blocks * 2 <= units ? 2 : 1;
}

// fp32, head dim 64, launches in one part: whether the rows that all waves of a workgroup need are brought in once (F32Fill::shared) or
// by each wave for itself.  Sharing them puts a barrier in front of the sweep.  us, each wave for itself : shared.
// Forward: a unit with one workgroup has nothing to do before the barrier (S = 2000 H = 2 22.20 : 22.48, S = 4000 H = 1 40.37 : 40.94); from the
// second workgroup of a unit on sharing is ahead (S = 1500 H = 3 19.23 : 19.06, S = 4000 H = 3 64.30 : 63.79), and over long sweeps, where the
// starts are a small part, behind again (S = 5000 H = 2 70.5 : 71.2, H = 4 116.4 : 117.8, S = 10000 H = 1 136.1 : 137.1).
// Backward: ahead by 1 us and more per round of workgroups (S = 300 B = 16 H = 4 45.5 : 41.0, S = 2000 H = 3 64.2 : 61.5, S = 5000 H = 1 138.8 : 137.2),
// but its loop, which holds other registers, is 1 to 2 % slower (S = 6000 H = 2 302.9 : 304.7, S = 8000 H = 1 266.0 : 270.1, S = 12000 H = 2 1104 : 1114,
// S = 30000 H = 1 3338 : 3398).  The lines lie where the two meet; S = 6000 H = 1 (175.3 : 171.3) is on the wrong side of its.
inline bool f32_fwd_shares_rows(int64_t tiles, int64_t heads) { return tiles * heads > kXcds * kChunk && tiles <= 256; }
inline bool f32_bwd_shares_rows(int64_t tiles) { return tiles <= 320; }

// fp32: from so many rows on a launch goes to the fp16 matrix instructions (attn_f32_split.hip).  Its workgroups of 32 rows start and end 3 to 5 us later than
// those of 16 rows on fp32 instructions, which also share out a tile's columns where units are idle, and take half the time per pair: it wins where a launch fills
// the chip.  One line for forward and backward, since a backward has to form its scores as the forward did whose logsumexp it is given; it lies where the two meet
// forward, over 270 sizes of 1 to 40 heads (us, fp32 instructions : fp16; d = 64 S = 3601 H = 1 37.1 : 38.2, 4501 H = 1 48.2 : 46.6, 1306 H = 4 18.2 : 18.4, 1567 H = 4
// 22.1 : 20.8, 811 H = 20 22.3 : 25.4, 1151 H = 20 37.8 : 34.2; d = 128 1945 H = 1 31.0 : 34.0, 2201 H = 1 40.2 : 37.4, 1179 H = 4 24.4 : 24.9, 1262 H = 4 25.6 : 25.4,
// 318 H = 40 23.7 : 20.4), which is later than backward (d = 64 2500 H = 1 71.0 : 47.8, 1100 H = 4 37.6 : 27.1; d = 128 1560 H = 1 59.3 : 51.8, 840 H = 4 36.5 : 34.4).
// d = 128, where each XCD's L2 brings in three heads or more: later (S = 1678 H = 3 32.3 : 33.8, 1333 H = 5 27.9 : 29.0, 1130 H = 6 25.2 : 23.9).
// Nor is the output of head dim 64 as exact in shorter sums (S = 504 H = 4 1.45e-7 : 1.44e-7 of fp32 instructions, 750 1.50e-7 : 1.52e-7).
inline bool f32_splits(int64_t S, int64_t heads, int d)
{
    const double h = (double)heads;
    const bool many = heads / std::gcd(heads, (int64_t)kXcds) >= 3;
    const double line = d == 64 ? std::max(1050.0, 4300.0 / std::pow(h, 0.75)) : std::max(2200.0 / std::pow(h, 0.45), many ? std::min(1750.0, 7000.0 / h) : 0.0);
    return (double)S >= line;
}

// One way to cut a launch into workgroups, and what it costs: `rows` owned rows per workgroup, the time of
// 2^20 (row, key) pairs on one compute unit with the whole chip busy, and the time a workgroup spends before
// and after its sweep.  `waves` of a workgroup, and the sequences it is for: more than `over` rows and up to `upto`.
struct TileChoice { int rows, order; double us_per_mpair, us_per_item; int waves = 8; int64_t over = 0, upto = INT64_MAX; };

// Estimated time of a launch, us.  Folded: rounds of 256 equal pairs of tiles.  Longest first: the n
// tiles an XCD gets have lengths n, n-1, .. 1 (in units of ntiles / n tiles); the first 32 start
// together, the next 32 go to the units that end first, so that two layers add up to equal sums, and
// what remains after whole double layers ends with the longest remaining tile.
inline double tile_choice_us(const TileChoice &c, int64_t S, int64_t heads, double crowded = kCrowdedAlone)
{
    const int64_t ntiles = (S + c.rows - 1) / c.rows;
    const double mpairs = (double)c.rows * c.rows / (1 << 20);            // a tile unit: rows x rows
    if (c.order == kFolded) {
        const int64_t round = kXcds * kChunk, rounds = ((ntiles + 1) / 2 * heads + round - 1) / round;
        return rounds * ((ntiles + 1) * mpairs * c.us_per_mpair + 2 * c.us_per_item);
    }
    const double n = (double)(ntiles * heads) / kXcds, P = kChunk, j = std::floor(n / (2 * P));
    double makespan = 2 * n * j - 2 * P * j * j + j + n - 2 * P * j;
    if (n < 1) makespan = 1;                                              // fewer tiles than XCDs
    // a partly idle chip clocks higher; the four-wave launches, which power bounds most, also where the second of two rounds ends before the first one's longest
    const double busy = n < P ? n / P : n < 2 * P && c.waves == 4 ? n / (2 * P) : 1.0;
    return makespan * (ntiles / (n < 1 ? 1 : n)) * mpairs * c.us_per_mpair * (0.8 + 0.2 * busy) * (1.0 + crowded * crowding(S, heads)) +
           std::ceil(n / P) * c.us_per_item;
}

template <int N>
inline int cheapest_tiles(const TileChoice (&choices)[N], int64_t S, int64_t heads)
{
    int best = -1;
    double best_us = 0.0;
    for (int i = 0; i < N; ++i) {
        if (S <= choices[i].over || S > choices[i].upto) continue;
        const double us = tile_choice_us(choices[i], S, heads);
        if (best < 0 || us < best_us) {
            best = i;
            best_us = us;
        }
    }
    return best;
}

// One way to work key tiles (dK/dV) and then query tiles (dQ) of `rows` rows in one launch, each longest first, and what it costs: as in TileChoice, with
// `longest` of the longest key tile's estimated time (shorter by what the units that end early leave of the power, longer by its start and end),
// what `crowding` costs and the time around everything.
struct JointChoice { int rows, waves; double key_us_per_mpair, query_us_per_mpair, longest, crowded, us; int64_t over = 0, upto = INT64_MAX; };

// Its estimated time: all work there is, spread over the chip, but no shorter than the longest key tile; the last dQ tiles leave a
// tenth of the longest one uneven.
inline double both_us(const JointChoice &c, int64_t S, int64_t heads)
{
    const double per_row = (double)S / (1 << 20);                         // mpairs per owned row of the longest tile
    const double mean = 0.5 * per_row * (double)(S * heads) / (kXcds * kChunk) * (1.0 + c.crowded * crowding(S, heads));
    const double longest = c.longest * c.rows * per_row * c.key_us_per_mpair;
    const double spread = mean * (c.key_us_per_mpair + c.query_us_per_mpair) + 0.1 * c.rows * per_row * c.query_us_per_mpair;
    return std::max(longest, spread) + c.us;
}

// The order a workgroup shape can work.  The downward sweep over the second tile of a pair starts every key group at the last
// key tile and steps over all of them: it is right for 256-row workgroups alone, whose waves share every key tile.
constexpr int tile_order(int rows, int order) { return rows == 256 ? order : kLongestFirst; }

// ---- bf16 forward
// Costs fitted to launches of every variant (N(0,1) inputs, S = 200 .. 200K, 1 to 10 heads): over 40 random
// (B, H, S) the estimate's choice was within 1.1 % of the fastest variant on average, 21 % at worst; over 36 sizes of 2048 to
// 400000 rows and 2 to 256 heads 0.3 % and, at S = 40000 with 5 heads (128 rows for 256), 4.6 %.  The worst are sizes
// of less than a round of workgroups and a few heads (S = 3000, 16 heads: 64 rows for 128, 19 %).
// 256 rows in four waves of 64 (attn_fwd_long_bf16.hip) take less per pair, but start and end a sweep 3 to 4 us later than in eight of 32, so they are for
// the longer sequences.  us, eight waves : four, folded S = 482 H = 227 39.7 : 49.5, 1468 H = 161 124 : 134, 2498 H = 116 265 : 276, 3249 H = 33 106.8 : 108.7,
// 3410 H = 67 231.7 : 227.0, 4397 H = 145 827 : 784; longest first S = 719 H = 177 54.6 : 64.1, 1468 H = 161 126.5 : 134.4, 1977 H = 50 69.2 : 70.7,
// 2554 H = 81 151 : 156, 2655 H = 91 216 : 204, 2734 H = 70 158 : 160, 2881 H = 145 380 : 362, 3596 H = 96 366 : 343, 4369 H = 82 460 : 426.
// From 3329 rows on their costs are fitted to 304 sizes of up to 120000 rows and 1 to 256 heads, timed by 64 and 128 rows and by both orders of 256: the choice
// is 0.4 to 0.9 % slower than the best on average, 21 % at worst (S = 3373 H = 14, 64 rows for 128).  us, 128 rows : 256, longest first, just beyond a round:
// S = 6000 H = 16 155 : 145, 8422 H = 12 218 : 202, 12715 H = 8 317 : 297, 20000 H = 10 980 : 871, 2667 H = 33 92 : 77, 40000 H = 5 1985 : 1702.
inline constexpr TileChoice kFwdChoices[] = {
    {256, kFolded, 115.5, 4.0, 8, 0, 3328}, {256, kFolded, 108.0, 4.0, 4, 3328},
    {256, kLongestFirst, 117.0, 8.0, 8, 0, 2560}, {256, kLongestFirst, 117.0, 8.0, 4, 2560, 3328}, {256, kLongestFirst, 109.0, 8.0, 4, 3328},
    {128, kLongestFirst, 125.0, 8.0}, {64, kLongestFirst, 140.0, 6.0}, {32, kLongestFirst, 185.0, 4.5},
};

inline const TileChoice &fwd_plan(int64_t S, int64_t heads) { return kFwdChoices[cheapest_tiles(kFwdChoices, S, heads)]; }

// ---- bf16 backward
// Costs of launches of one gradient (see tile_choice_us): 256 rows in four waves, and 128, which pay for their larger fill traffic.
inline constexpr TileChoice kDkdvChoices[] = {{256, kFolded, 196.5, 7.1, 4}, {256, kLongestFirst, 200.6, 8.5, 4}, {128, kLongestFirst, 222.0, 8.0}};
inline constexpr TileChoice kDqChoices[] = {{256, kFolded, 141.4, 7.1, 4}, {256, kLongestFirst, 146.0, 8.5, 4}, {128, kLongestFirst, 156.0, 8.0}};

// Joint launches.  256 rows go out in four waves of 64 from 3073 rows on, in eight of 32 below: four take less per pair and start and end a sweep later, as in
// the forward.  us, eight waves : four, S = 961 H = 128 150 : 163, 1442 H = 128 291 : 309, 2115 H = 100 447 : 464, 2538 H = 100 584 : 610, 3868 H = 64 796 : 790,
// 8577 H = 20 1168 : 1116, 14528 H = 8 1226 : 1127, 22690 H = 5 1948 : 1804, 42591 H = 4 5452 : 4810, 85099 H = 4 20465 : 18772.
inline constexpr JointChoice kJointChoices[] = {
    {256, 4, 191.2, 154.8, 0.985, 0.086, 12.8, 3072}, {256, 8, 218.0, 149.0, 0.87, kCrowdedJoint, 10.0, 0, 3072},
    {128, 8, 222.0, 156.0, 0.87, kCrowdedJoint, 10.0}, {64, 8, 232.0, 181.0, 0.87, kCrowdedJoint, 10.0},
};

// A launch of 32-row workgroups: no shorter than its longest key tile, nor than all work spread over the chip with the start and
// the end of every workgroup (4.5 us).  Fitted before these kernels' starts and ends became shorter and their columns went out in parts: the estimate
// is 0.92 to 1.17 times what is measured now from 2000 rows on, 1.05 to 1.45 times from 400, and up to 1.6 times below.  So launches of up to one
// round of 32-row workgroups and many heads still go to 64 rows: us, 64 rows (taken) : 32, S = 78 H = 12 9.8 : 7.5, S = 121 H = 16 9.9 : 7.9, S = 300 H = 10
// 12.6 : 11.0, S = 1187 H = 6 24.3 : 21.3; over 250 sizes of 25 to 25593 rows and 1 to 32 heads the choice of rows is 1.8 % slower than the best one on average.
inline double own_us(int64_t S, int64_t heads)
{
    const double per_row = (double)S / (1 << 20), items = 2.0 * ((S + 31) / 32) * heads;
    const double mean = 0.5 * per_row * (double)(S * heads) / (kXcds * kChunk);
    return std::max(0.87 * 32 * per_row * 232.0, mean * 450.0 + 4.5 * items / (kXcds * kChunk)) + 10.0;
}

// Workgroups of `rows` rows and `waves` waves: dK/dV and dQ in one joint launch, or the one after the other in the orders k_order and q_order.
struct BwdPlan { int rows; bool joint; int k_order, q_order, waves; };

// Fitted to 130 sizes of 961 to 113292 rows and 1 to 128 heads, timed as joint launches of 64, 128 and 256 rows and as two launches in each order: the choice
// is 0.4 % slower than the fastest of them on average and 6.5 % at worst (S = 2905 H = 10, 64 rows for 128); with joint launches in eight waves throughout
// and two launches priced as eight waves it was 4 % (us, then : now, S = 25000 H = 4 1930 : 1739, 40000 H = 5 6038 : 5597, 70000 H = 4 13780 : 12669,
// 90000 H = 4 22735 : 21012).
inline BwdPlan bwd_plan(int64_t S, int64_t heads)
{
    BwdPlan best = {256, false, kFolded, kFolded, 4};
    double best_us = 0;
    for (auto [choices, order] : {std::make_pair(kDkdvChoices, &best.k_order), std::make_pair(kDqChoices, &best.q_order)}) {
        const double folded = tile_choice_us(choices[0], S, heads), longest_first = tile_choice_us(choices[1], S, heads);
        *order = longest_first < folded ? kLongestFirst : kFolded;
        best_us += std::min(folded, longest_first);
    }
    auto offer = [&](int rows, bool joint, int waves, double us) {
        if (us >= best_us) return;
        best = {rows, joint, kLongestFirst, kLongestFirst, waves};
        best_us = us;
    };
    // apart: S = 32768, 2 heads 1508 us against 1565 joint (two long sweeps per unit either way); nowhere else
    offer(128, false, 8, tile_choice_us(kDkdvChoices[2], S, heads, kCrowdedJoint) + tile_choice_us(kDqChoices[2], S, heads, kCrowdedJoint));
    for (const JointChoice &c : kJointChoices)
        if (S > c.over && S <= c.upto) offer(c.rows, true, c.waves, both_us(c, S, heads));
    offer(32, true, 8, own_us(S, heads));
    return best;
}

// ---- projection
// Tile shapes, and what a round of tiles costs: us per 128 of K with one compute unit busy and with all of them (the chip
// clocks lower then), and us per tile around it.  Fitted to launches of 300 to 138937 rows, K = 1024 to 5120; the wave
// grids and ring depths are the fastest of the two or three tried for each tile.
struct LinChoice { int bm, bn; double us_alone, us_full, us_tile; };
inline constexpr LinChoice kLinChoices[] = {
    {256, 256, 2.16, 2.95, 5.0}, {256, 128, 1.28, 1.62, 3.5}, {192, 128, 0.95, 1.28, 2.5},
    {128, 128, 0.70, 0.88, 2.0}, {128, 64, 0.48, 0.59, 1.0},  {64, 64, 0.37, 0.43, 0.7},
};

inline double lin_choice_us(const LinChoice &c, int64_t rows, int K, int N)
{
    const double tiles = std::ceil((double)rows / c.bm) * std::ceil((double)N / c.bn), units = kXcds * kChunk;
    const double busy = std::min(1.0, tiles / units);
    return std::ceil(tiles / units) * (K / 128.0 * (c.us_alone + busy * (c.us_full - c.us_alone)) + c.us_tile);
}

// The rows that the buffer of tile `tile` of the rows [begin, end) covers.  Not live (behind a workgroup's last tile): none, and
// first stays inside the matrix, since the address is formed all the same.
struct RowWindow { int64_t first; int rows; };
constexpr RowWindow row_window(int64_t begin, int64_t end, int64_t tile, int tile_rows, bool live)
{
    if (!live) return {begin, 0};
    const int64_t first = begin + tile * tile_rows, left = end - first;
    return {first, left < tile_rows ? (int)left : tile_rows};
}

inline const LinChoice &lin_plan(int64_t rows, int K, int N)
{
    const LinChoice *best = kLinChoices;
    for (const LinChoice &c : kLinChoices)
        if (lin_choice_us(c, rows, K, N) < lin_choice_us(*best, rows, K, N)) best = &c;
    return *best;
}

// every choice of an order is one that its shape can work
template <int N>
constexpr bool orders_fit(const TileChoice (&choices)[N])
{
    for (int i = 0; i < N; ++i)
        if (tile_order(choices[i].rows, choices[i].order) != choices[i].order) return false;
    return true;
}
static_assert(orders_fit(kFwdChoices) && orders_fit(kDkdvChoices) && orders_fit(kDqChoices), "a pair of tiles needs 256-row workgroups");

}  // namespace memo

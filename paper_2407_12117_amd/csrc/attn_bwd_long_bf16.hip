// bf16 causal attention backward for gfx950 (CDNA4), head dim 128: dK and dV by workgroups of 256 keys, dQ by workgroups of 256 rows, one
// per compute unit, for long sequences (shorter ones, what is computed and the operand conventions: attn_bwd_bf16.hip).
//
// dK, dV.  Four waves, one per SIMD, each with 64 key rows: all 256 accumulation registers hold its dV^T and dK^T, and a Q or dO operand read from
// LDS serves four key blocks of 16.  K and V of the 256 keys stay in LDS (128 KB), Q and dO come in tiles of 32 queries through
// two places (32 KB).  A wave works a tile as 32 items of four MFMAs, in one stream that is ordered by hand, every MFMA first and its
// share of the vector instructions behind it (as in attn_fwd_long_bf16.hip):
//   items  0..7   S = Q K^T - LSE/scale   keys 0..31, then 32..63; Q rows stay in registers from one to the other
//   items  8..15  dP = dO V^T - D         P = exp2(scale log2e S) behind the MFMAs of items 4..15
//   items 16..23  dV^T += dO^T P          dS = P dP behind them
//   items 24..31  dK^T += Q^T dS          the last three behind the next tile's barrier, where they cover its first reads
// The MFMAs are inline asm that names the register file (the compiler moves score tiles in and out of the accumulation registers
// otherwise); the waits between an MFMA and vector instructions that touch its result are written here.  The sums are formed in
// the order of eight waves of 32 keys (attn_bwd_bf16.hip), to the same bits.
// S = 128K, H = 4, same card in turn, eight waves -> this: 27.25 -> 25.05 ms (1291 -> 1405 TFLOP/s; all-zero inputs, which the power limit
// does not reach: 1471 -> 1640).  What is left: without vector instructions 1700 (1805), without the exponentials 1478 (1709), without
// the fills 1440 (1622); dK's items all behind the barrier, so that the exponentials have more MFMAs to hide behind: 1400 (1530).
#include "bf16_tiles.h"

namespace memo {
namespace {

constexpr int kLongWaves = 4, kLongKeys = 64 * kLongWaves, kLongQueries = 32;
constexpr int kHalfStage = kLongQueries * 256, kStage = 2 * kHalfStage;        // Q rows, then dO rows
constexpr int kWaveRows = 64 * 256;                                           // a wave's K rows, its V rows behind them
constexpr int kKvOff = 2 * kStage, kDkdvLds = kKvOff + kLongWaves * 2 * kWaveRows;
static_assert(kDkdvLds == 160 * 1024, "LDS is full");

// N: LDS reads that may still be on their way when the operands are needed; -1: they were needed before
constexpr int kHere = -1;
template <int N>
__device__ __forceinline__ void mfma_from(f32x4 &d, const bf16x8 &x, const bf16x8 &y, const f32x4 &c)      // D = A B + C
{
    if constexpr (N >= 0) asm volatile("s_waitcnt lgkmcnt(%4)\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(x), "v"(y), "v"(c), "n"(N));
    else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(x), "v"(y), "v"(c));
}
template <int N>
__device__ __forceinline__ void mfma_on(f32x4 &d, const bf16x8 &x, const bf16x8 &y)                        // D = A B + D, vector registers
{
    if constexpr (N >= 0) asm volatile("s_waitcnt lgkmcnt(%3)\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(x), "v"(y), "n"(N));
    else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(x), "v"(y));
}
template <int N>
__device__ __forceinline__ void mfma_acc(f32x4 &d, const bf16x8 &x, const u32x4 &y)                        // the same, accumulation registers
{
    if constexpr (N >= 0) asm volatile("s_waitcnt lgkmcnt(%3)\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(x), "v"(y), "n"(N));
    else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(x), "v"(y));
}

// When a step's LDS reads are queued, as the MFMA of the step (0..127, the last three items of the tile before first) they come behind.
// A read comes 10 to 20 MFMAs ahead of its use, and the reads are spread so that the LDS, which four waves need for half of a step's time,
// is not asked for much more than it gives (with all reads of an item in one piece three items ahead: 1395 TFLOP/s for 1405).
struct Reads {
    static constexpr int kMost = 4;
    // two rows each: the streamed ones (Q, dO) before the resident ones (K, V); two halves of a transposed operand
    static constexpr int of(int n) { return n < 4 || (n >= 8 && n < 16 && n % 2 == 0) ? 4 : 2; }
    static constexpr int first(int n) { return n < 29 ? 12 + 4 * n : 4 * (n - 29); }       // the item's own first MFMA
    static constexpr bool before(int n, int part) { return n < 4 && part >= 2; }           // resident: read in the step before
    static constexpr int slot(int n, int part)
    {
        if (n < 4) return part < 2 ? 2 * n + part : 93 + 3 * (2 * n + part - 2);
        if (n < 8) return 12 + 2 * (2 * (n - 4) + part);
        if (n < 16) return 26 + 11 * (6 * ((n - 8) / 2) + (n % 2 ? 4 : 0) + part) / 8;
        return n < 24 ? 58 + 4 * (n - 16) + 2 * part : 88 + 4 * (n - 24) + 2 * part;
    }
    static constexpr int at(int x, int i)              // the i-th read (4 n + part) behind MFMA x, or -1
    {
        for (int code = 0; code < 128; ++code)
            if (code % 4 < of(code / 4) && slot(code / 4, code % 4) == x && i-- == 0) return code;
        return -1;
    }
    static constexpr int later(int n)                  // reads queued behind the item's last one when it is needed
    {
        int last = -1, count = 0;
        for (int part = 0; part < of(n); ++part)
            if (!before(n, part) && 128 * slot(n, part) + 4 * n + part > last) last = 128 * slot(n, part) + 4 * n + part;
        for (int code = 0; code < 128; ++code)
            if (code % 4 < of(code / 4) && slot(code / 4, code % 4) < first(n) && 128 * slot(code / 4, code % 4) + code > last) ++count;
        return count < 15 ? count : 15;
    }
};

__device__ __forceinline__ void settle(f32x4 (&x)[2][4])
{
    asm volatile("s_nop 15" : "+v"(x[0][0]), "+v"(x[0][1]), "+v"(x[0][2]), "+v"(x[0][3]), "+v"(x[1][0]), "+v"(x[1][1]), "+v"(x[1][2]), "+v"(x[1][3]));
}

// lds: [stage][Q|dO], [wave][K|V]; t: key tile p (long) and key tile nkt-1-p (short)
__device__ __forceinline__ void dkdv_long_rows(const AttnArgs &a, LDS_AS unsigned char *lds, const PairId t)
{
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh;
    const __bf16 *q = static_cast<const __bf16 *>(a.q) + base;
    const __bf16 *g = static_cast<const __bf16 *>(a.d_o) + base;
    const int64_t stat = ((int64_t)t.b * a.H + t.h) * a.S;
    const int nit = (int)((a.S + kLongQueries - 1) / kLongQueries);
    const float c = a.scale * kLog2e;
    float neg_inv_scale = -1.f / a.scale, neg_one = -1.f;
    asm volatile("" : "+v"(neg_inv_scale), "+v"(neg_one));
    using Fills = TileOffsets<kLongWaves, kLongQueries>;
    const Fills toff = make_tile_offsets<kLongWaves, SwzB, kLongQueries>(a.ss, wave, lane);
    static_assert(Fills::kInstr == 2, "fill_part deals out four");
    const LdsAddr16 ad = make_lds_addr16(lds, lane);
    // -LSE_i/scale and -D_i of the queries 4*g4 .. 4*g4+3 of a block of 16, from one value a lane (attn_bwd_bf16.hip, "Row statistics")
    const uint32_t stat_off = (uint32_t)(4 * g4 + (lane & 3)) * 4;
    const uint32_t stat_bytes = (uint32_t)min(a.S * 4, (int64_t)0x7fffffff);
    const __amdgpu_buffer_rsrc_t lse_buf = __builtin_amdgcn_make_buffer_rsrc(a.lse + stat, 0, stat_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t dlt_buf = __builtin_amdgcn_make_buffer_rsrc(a.delta + stat, 0, stat_bytes, 0x00020000);

    // The long tile walks the query tiles downwards from the last one to its diagonal, the short tile upwards from its diagonal to the
    // last one (launch_plan.h, folded order).
#pragma clang loop unroll(disable)
    for (int pass = 0; pass < 2; ++pass) {
        const int64_t tile = pass == 0 ? t.first : t.second;
        if (tile < 0) break;
        const int64_t col0 = tile * kLongKeys, j0w = col0 + 64 * wave;
        const int it0 = (int)(col0 / kLongQueries), npos = nit - it0;     // the tile's first query tile (its diagonal), and how many
        const int it_first = pass ? it0 : nit - 1, dir = pass ? 1 : -1;
        // this wave's own first query tile, and what part of the sweep it works: [ua, ub]; one that has no keys works none
        const int own = (int)(j0w / kLongQueries) - it0;
        const bool live = j0w < a.S;
        const int ua = !live ? npos : pass ? own : 0, ub = pass ? npos - 1 : npos - 1 - own;
        if (pass) __syncthreads();    // every wave has left the first tile's ring
        {   // this wave's K and V rows; rows past S are zero, masked and never stored
            const __bf16 *kp = static_cast<const __bf16 *>(a.k) + base, *vp = static_cast<const __bf16 *>(a.v) + base;
            const OwnTileFill own_fill(a.ss, lane);
            LDS_AS unsigned char *rows = lds + kKvOff + wave * 2 * kWaveRows;
#pragma unroll
            for (int blk = 0; blk < 2; ++blk) {
                const int64_t r0 = live ? j0w + 32 * blk : a.S;
                own_fill(rows + blk * 8192, kp, a.ss, min(r0, a.S), a.S);
                own_fill(rows + kWaveRows + blk * 8192, vp, a.ss, min(r0, a.S), a.S);
            }
        }
        // Tile u of the sweep as two buffers, from pointers that move on a tile at a time; behind the last one they are empty.
        const int64_t tile_bytes = (int64_t)dir * kLongQueries * a.ss * 2;
        uint32_t full_bytes = (uint32_t)(kLongQueries - 1) * (uint32_t)a.ss * 2 + 256;
        uint32_t last_bytes = (uint32_t)((int)(a.S - (int64_t)(nit - 1) * kLongQueries) - 1) * (uint32_t)a.ss * 2 + 256;
        asm volatile("" : "+s"(full_bytes), "+s"(last_bytes));      // selected without branches
        const int u_last = pass ? npos - 1 : 0;
        const char *qp = reinterpret_cast<const char *>(q + (int64_t)it_first * kLongQueries * a.ss);
        const char *gp = reinterpret_cast<const char *>(g + (int64_t)it_first * kLongQueries * a.ss);
        __amdgpu_buffer_rsrc_t qb, gb;
        int to = 0;                                // the place of the tile that is filled next
        auto prepare = [&](int u) __attribute__((always_inline)) {
            uint32_t bytes = u < npos ? full_bytes : 0;
            bytes = u == u_last ? last_bytes : bytes;
            qb = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(qp), 0, bytes, 0x00020000);
            gb = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(gp), 0, bytes, 0x00020000);
            qp += tile_bytes;
            gp += tile_bytes;
        };
        auto fill_part = [&](auto nc) __attribute__((always_inline)) {
            constexpr int n = decltype(nc)::value;
            toff.part(lds + to + n / 2 * kHalfStage, n / 2 ? gb : qb, n % 2, wave);
        };
        struct { uint32_t l[2], d[2]; } raw;
        auto load_stats = [&](int u) __attribute__((always_inline)) {         // rows past S: zero
            const int at = min(u, npos - 1) * dir + it_first;
#pragma unroll
            for (int qt = 0; qt < 2; ++qt) {
                raw.l[qt] = __builtin_amdgcn_raw_buffer_load_b32(lse_buf, stat_off + 64 * qt, at * (kLongQueries * 4), 0);
                raw.d[qt] = __builtin_amdgcn_raw_buffer_load_b32(dlt_buf, stat_off + 64 * qt, at * (kLongQueries * 4), 0);
            }
        };
        prepare(0);
        static_for<0, 4>(fill_part);
        to = kStage;
        load_stats(ua);

        f32x4 accV[8][4], accK[8][4];              // dV^T, dK^T: [head-dim block][key block]; lane = key
#pragma unroll
        for (int dt = 0; dt < 8; ++dt)
#pragma unroll
            for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                for (int r = 0; r < 4; ++r) accV[dt][kt][r] = accK[dt][kt][r] = 0.f;
        auto settle_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) {
                asm volatile("s_nop 15" : "+a"(accV[dt][0]), "+a"(accV[dt][1]), "+a"(accV[dt][2]), "+a"(accV[dt][3]),
                                          "+a"(accK[dt][0]), "+a"(accK[dt][1]), "+a"(accK[dt][2]), "+a"(accK[dt][3]));
            }
        };
        uint32_t row[4], tr[8], kv[4];             // LDS addresses in the present tile's place; of this wave's K rows
        int at = (ua & 1) * kStage, way = ua & 1 ? -kStage : kStage;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            row[kk] = ad.row16[kk] + at;
            kv[kk] = ad.row16[kk] + kKvOff + wave * 2 * kWaveRows;
        }
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) tr[dt] = ad.tr16[dt] + at;

        f32x4 s[2][4], dp[2][4], nl[2], nd[2];     // [query block][key block]; register r = query 16*qt + 4*g4 + r
        u32x4 pB[4], dsB[4];
        bf16x8 qa[2][4], ga[4][2], bp[8][2];
        TrSlot trs[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) dsB[i] = u32x4{0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < 8; ++i) trs[i].lo = trs[i].hi = s16x4{0, 0, 0, 0};

        // Step u begins: tile u is complete, and nobody reads the other place any more, which tile u + 1 takes from here on.
        auto begin = [&](int u) __attribute__((always_inline)) {
            wait_fills();
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            prepare(u + 1);
        };
        auto idle = [&](int u) __attribute__((always_inline)) {        // a step in which this wave has no queries
            begin(u);
            static_for<0, 4>(fill_part);
            to ^= kStage;
        };
        auto spread_stats = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int qt = 0; qt < 2; ++qt) {
                asm volatile("v_mfma_f32_4x4x1_16b_f32 %0, %1, %2, 0" : "=v"(nl[qt]) : "v"(raw.l[qt]), "v"(neg_inv_scale));
                asm volatile("v_mfma_f32_4x4x1_16b_f32 %0, %1, %2, 0" : "=v"(nd[qt]) : "v"(raw.d[qt]), "v"(neg_one));
            }
        };
        auto read = [&](auto codec) __attribute__((always_inline)) {
            constexpr int n = decltype(codec)::value / 4, P = decltype(codec)::value % 4;
            if constexpr (n < 16) {
                constexpr int kk = n < 8 ? n % 4 : (n - 8) / 2, kt = n < 8 ? n / 4 * 2 : n % 2 * 2, streamed = Reads::of(n) - 2;
                if constexpr (P < streamed) {
                    if constexpr (n < 8) lds_issue_b128<P * 4096>(qa[P][kk], row[kk]);
                    else lds_issue_b128<kHalfStage + P * 4096>(ga[kk][P], row[kk]);
                    if constexpr (n >= 8 && P == 1) row[kk] += way;
                } else {
                    lds_issue_b128<(n < 8 ? 0 : kWaveRows) + (kt + P - streamed) * 4096>(bp[n % 8][P - streamed], kv[kk]);
                }
            } else {
                constexpr int off = n < 24 ? kHalfStage : 0;
                if constexpr (P == 0) lds_issue_tr_half<off>(trs[n % 8].lo, tr[n % 8]);
                else lds_issue_tr_half<off + 4096>(trs[n % 8].hi, tr[n % 8]);
                if constexpr (n >= 24 && P == 1) tr[n % 8] += way;
            }
        };
        auto reads_at = [&](auto xc) __attribute__((always_inline)) {
            static_for<0, Reads::kMost>([&](auto ic) {
                constexpr int code = Reads::at(decltype(xc)::value, decltype(ic)::value);
                if constexpr (code >= 0) read(IntC<code>{});
            });
        };
        // the element-wise chains: el = 8 kt + 4 qt + r
        float x[2], ds[4];
        auto exp_position = [&](auto ic) __attribute__((always_inline)) {      // P: product of el i, exponential of i - 1, rounding of i - 2
            constexpr int i = decltype(ic)::value;
            if constexpr (i >= 2 && i % 2 == 1) {
                constexpr int el = i - 2, kt = el / 8, qt = el / 4 % 2, r = el % 4;
                const f32x2 two = {s[qt][kt][r - 1], s[qt][kt][r]};
                pB[kt][el % 8 / 2] = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2));
                asm volatile("" : "+v"(pB[kt][el % 8 / 2]));
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (i >= 1 && i < 33) {
                constexpr int el = i - 1;
                s[el / 4 % 2][el / 8][el % 4] = __builtin_amdgcn_exp2f(x[el % 2]);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (i < 32) x[i % 2] = s[i / 4 % 2][i / 8][i % 4] * c;
            __builtin_amdgcn_sched_barrier(0);
        };
        auto ds_position = [&](auto ic) __attribute__((always_inline)) {       // dS: product of el i, rounding of i - 1
            constexpr int i = decltype(ic)::value;
            if constexpr (i >= 2 && i % 2 == 0) {
                constexpr int el = i - 1;
                const f32x2 two = {ds[(el - 1) % 4], ds[el % 4]};
                dsB[el / 8][el % 8 / 2] = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2));
                asm volatile("" : "+v"(dsB[el / 8][el % 8 / 2]));
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (i < 32) ds[i % 4] = s[i / 4 % 2][i / 8][i % 4] * dp[i / 4 % 2][i / 8][i % 4];
            __builtin_amdgcn_sched_barrier(0);
        };
        // item n: its four MFMAs, with reads (READS) and vector instructions between them
        constexpr int kExpFrom = 16, kExpSpan = 46, kDsFrom = 64, kDsSpan = 30;      // in MFMAs of items 0..; other spans: 0 to -1 %
        auto item = [&](auto nc, auto reads_c, auto waited_c) __attribute__((always_inline)) {
            constexpr int n = decltype(nc)::value;
            constexpr bool READS = decltype(reads_c)::value, WAITED = decltype(waited_c)::value;
            constexpr int later = WAITED ? kHere : Reads::later(n);
            static_for<0, 4>([&](auto jc) {
                constexpr int j = decltype(jc)::value, m = 4 * n + j, W = j == 0 ? later : kHere;
                if constexpr (n < 8) {
                    constexpr int kk = n % 4, kh = j / 2, kt = n / 4 * 2 + kh, qt = j % 2;
                    if constexpr (kk == 0) mfma_from<W>(s[qt][kt], qa[qt][kk], bp[n % 8][kh], nl[qt]);
                    else mfma_on<W>(s[qt][kt], qa[qt][kk], bp[n % 8][kh]);
                } else if constexpr (n < 16) {
                    constexpr int kk = (n - 8) / 2, kh = j / 2, kt = n % 2 * 2 + kh, qt = j % 2;
                    if constexpr (kk == 0) mfma_from<W>(dp[qt][kt], ga[kk][qt], bp[n % 8][kh], nd[qt]);
                    else mfma_on<W>(dp[qt][kt], ga[kk][qt], bp[n % 8][kh]);
                } else if constexpr (n < 24) {
                    mfma_acc<W>(accV[n % 8][j], tr_operand(trs[n % 8]), pB[j]);
                } else {
                    mfma_acc<W>(accK[n % 8][j], tr_operand(trs[n % 8]), dsB[j]);
                }
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (READS) reads_at(IntC<Reads::first(n) + j>{});
                constexpr auto upto = [](int k, int span, int all) constexpr { return k <= 0 ? 0 : k >= span ? all : (k * all + span - 1) / span; };
                static_for<upto(m - kExpFrom, kExpSpan, 34), upto(m + 1 - kExpFrom, kExpSpan, 34)>(exp_position);
                static_for<upto(m - kDsFrom, kDsSpan, 33), upto(m + 1 - kDsFrom, kDsSpan, 33)>(ds_position);
                if constexpr (n < 4 && j == 3) fill_part(IntC<n>{});
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        // what a tile at the diagonal or at the end of the sequence leaves out, key blocks [2 H, 2 H + 2)
        auto mask = [&](auto hc, int64_t i0) __attribute__((always_inline)) {
            constexpr int H = decltype(hc)::value;
            int ln = lane;
            asm volatile("" : "+v"(ln));
#pragma unroll
            for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                for (int kt = 2 * H; kt < 2 * H + 2; ++kt) {
                    // query offset 16qt + 4g4 + r of the tile is visible to key j iff it is >= j - i0, and there iff below S - i0
                    const int thr = (int)(j0w + 16 * kt + (ln & 15) - i0) - (16 * qt + 4 * (ln >> 4));
                    const int end = (int)min(a.S - i0, (int64_t)kLongQueries) - (16 * qt + 4 * (ln >> 4));
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (r < thr || r >= end) s[qt][kt][r] = -INFINITY;
                }
        };
        using Yes = IntC<1>;
        using No = IntC<0>;

        int u = 0;
#pragma clang loop unroll(disable)
        for (; u < ua; ++u) idle(u);
        if (live) {
            begin(u);
            spread_stats();
            asm volatile("s_nop 15" : "+v"(nl[0]), "+v"(nl[1]), "+v"(nd[0]), "+v"(nd[1]));
            static_for<0, 4>([&](auto n) {
                read(IntC<4 * decltype(n)::value + 2>{});
                read(IntC<4 * decltype(n)::value + 3>{});
            });
            static_for<0, 12>(reads_at);
#pragma clang loop unroll(disable)
            for (;;) {
                const int64_t i0 = ((int64_t)u * dir + it_first) * kLongQueries;
                const bool ragged = i0 + kLongQueries > a.S, edge = i0 < j0w + 63 || ragged;
                load_stats(u + 1);
                static_for<0, 4>([&](auto n) { item(n, Yes{}, No{}); });
                to ^= kStage;
                if (edge) {
                    settle(s);
                    mask(IntC<0>{}, i0);
                }
                static_for<4, 8>([&](auto n) { item(n, Yes{}, No{}); });
                if (edge) {
                    settle(s);
                    mask(IntC<1>{}, i0);
                }
                static_for<8, 16>([&](auto n) { item(n, Yes{}, No{}); });
                if (ragged) {
                    settle(dp);
                    const int end = (int)(a.S - i0);
#pragma unroll
                    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                if (16 * qt + 4 * g4 + r >= end) dp[qt][kt][r] = 0.f;
                }
                static_for<16, 29>([&](auto n) { item(n, Yes{}, No{}); });
                asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(trs[5].lo), "+v"(trs[5].hi), "+v"(trs[6].lo), "+v"(trs[6].hi), "+v"(trs[7].lo), "+v"(trs[7].hi) :: "memory");
                way = -way;
                if (u == ub) break;
                ++u;
                begin(u);
                spread_stats();
                static_for<29, 32>([&](auto n) { item(n, Yes{}, Yes{}); });
            }
            static_for<29, 32>([&](auto n) { item(n, No{}, Yes{}); });
            settle_acc();
            ++u;
        }
#pragma clang loop unroll(disable)
        for (; u < npos; ++u) idle(u);
        wait_fills();

        __bf16 *dv = static_cast<__bf16 *>(a.dv) + base + (j0w + l16) * a.ss + 4 * g4;
        __bf16 *dk = static_cast<__bf16 *>(a.dk) + base + (j0w + l16) * a.ss + 4 * g4;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
            if (j0w + 16 * kt + l16 < a.S) {
#pragma unroll
                for (int dt = 0; dt < 8; ++dt) {
                    store4(dv + 16 * kt * a.ss + 16 * dt, accV[dt][kt], 1.f);
                    store4(dk + 16 * kt * a.ss + 16 * dt, accK[dt][kt], a.scale);
                }
            }
    }   // pass
}

// ============================================================================ dQ
// Four waves, one per SIMD, each with 64 query rows: accumulation registers hold its dQ^T, Q and dO (all 256 of them), and an operand of K,
// V or K^T read from LDS serves four query blocks of 16.  K and V come in tiles of 64 keys through rings of three, with the barrier of a
// step between its two blocks of 32 keys (as in attn_fwd_long_bf16.hip).  A block is worked as 24 items of four MFMAs, one operand each:
//   items  0..7   S^T = K Q^T           keys 0..15, then 16..31
//   items  8..15  dP^T = V dO^T - D     P = exp2(scale log2e S - LSE) behind the MFMAs of items 4..15
//   items 16..23  dQ^T += K^T dS^T      of the block before; dS = P dP of this one behind them
// Same bits as eight waves of 32 rows (attn_bwd_bf16.hip).  S = 128K, H = 4, same card in turn: 18.69 -> 17.5 to 18.05 ms (1411 -> 1462 to
// 1508 TFLOP/s; all-zero inputs 1710 -> 1812).
constexpr int kDqKeys = 64, kDqTile = kDqKeys * 256, kDqRing = 3 * kDqTile;

template <int N>
__device__ __forceinline__ void mfma_zero_a(f32x4 &d, const bf16x8 &x, const bf16x8 &y)                     // D = A B, B in accumulation registers
{
    if constexpr (N >= 0) asm volatile("s_waitcnt lgkmcnt(%3)\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(x), "a"(y), "n"(N));
    else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(x), "a"(y));
}
template <int N>
__device__ __forceinline__ void mfma_from_a(f32x4 &d, const bf16x8 &x, const bf16x8 &y, const f32x4 &c)     // D = A B + C
{
    if constexpr (N >= 0) asm volatile("s_waitcnt lgkmcnt(%4)\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(x), "a"(y), "v"(c), "n"(N));
    else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(x), "a"(y), "v"(c));
}
template <int N>
__device__ __forceinline__ void mfma_on_a(f32x4 &d, const bf16x8 &x, const bf16x8 &y)                       // D = A B + D
{
    if constexpr (N >= 0) asm volatile("s_waitcnt lgkmcnt(%3)\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(x), "a"(y), "n"(N));
    else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(x), "a"(y));
}

// lds: K tile t at t % 3, V tile t behind them likewise
__device__ __forceinline__ void dq_long_rows(const AttnArgs &a, LDS_AS unsigned char *lds, const PairId t)
{
    constexpr int kRows = 64 * kLongWaves;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh;
    const __bf16 *q = static_cast<const __bf16 *>(a.q) + base;
    const __bf16 *k = static_cast<const __bf16 *>(a.k) + base;
    const __bf16 *v = static_cast<const __bf16 *>(a.v) + base;
    const __bf16 *g = static_cast<const __bf16 *>(a.d_o) + base;
    const int64_t stat = ((int64_t)t.b * a.H + t.h) * a.S;
    const float c = a.scale * kLog2e;
    using Fills = TileOffsets<kLongWaves, kDqKeys>;
    const Fills toff = make_tile_offsets<kLongWaves, SwzB, kDqKeys>(a.ss, wave, lane);
    static_assert(Fills::kInstr == 4, "fill_part deals out eight");
    const LdsAddr16 ad = make_lds_addr16(lds, lane);

    // the heavy tile of the pair sweeps the keys upwards from row 0, the light one downwards to row 0
#pragma clang loop unroll(disable)
    for (int pass = 0; pass < 2; ++pass) {
        const int64_t tile = pass == 0 ? (t.second >= 0 ? t.second : t.first) : (t.second >= 0 ? t.first : -1);
        if (tile < 0) break;
        const int64_t row0 = tile * kRows, i0w = row0 + 64 * wave;
        const int64_t last_row = min(row0 + kRows, a.S) - 1;
        const int ntiles = (int)(last_row / kDqKeys) + 1;
        // Tiles by their place in the sweep: this wave works [ua, ub], of which um holds its diagonal; one that has no rows works none.
        const int diagonal = (int)(i0w / kDqKeys);
        const bool live = i0w < a.S;
        const int ua = !live ? ntiles : pass ? ntiles - 1 - diagonal : 0, ub = pass ? ntiles - 1 : diagonal, um = pass ? ua : ub;
        if (pass) __syncthreads();    // every wave has left the first tile's last LDS buffers

        // Tile u of the sweep as two buffers, from pointers that move on a tile at a time; behind the last one they are empty.
        const int64_t tile_bytes = (pass ? -1 : 1) * (int64_t)kDqKeys * a.ss * 2;
        const int64_t first_key = pass ? (int64_t)(ntiles - 1) * kDqKeys : 0;
        uint32_t full_bytes = (uint32_t)(kDqKeys - 1) * (uint32_t)a.ss * 2 + 256;
        uint32_t last_bytes = (uint32_t)(min(a.S - (int64_t)(ntiles - 1) * kDqKeys, (int64_t)kDqKeys) - 1) * (uint32_t)a.ss * 2 + 256;
        asm volatile("" : "+s"(full_bytes), "+s"(last_bytes));      // selected without branches
        const int u_last = pass ? 0 : ntiles - 1;
        const char *kp = reinterpret_cast<const char *>(k + first_key * a.ss), *vp = reinterpret_cast<const char *>(v + first_key * a.ss);
        __amdgpu_buffer_rsrc_t kb, vb;
        int to = -kDqTile;                         // the place of the tile that is filled
        auto prepare = [&](int u) __attribute__((always_inline)) {
            uint32_t bytes = u < ntiles ? full_bytes : 0;
            bytes = u == u_last ? last_bytes : bytes;
            kb = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(kp), 0, bytes, 0x00020000);
            vb = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(vp), 0, bytes, 0x00020000);
            kp += tile_bytes;
            vp += tile_bytes;
            to = to == 2 * kDqTile ? 0 : to + kDqTile;
        };
        auto fill_part = [&](auto nc) __attribute__((always_inline)) {
            constexpr int n = decltype(nc)::value;
            toff.part(lds + to + n / Fills::kInstr * kDqRing, n / Fills::kInstr ? vb : kb, n % Fills::kInstr, wave);
        };
        prepare(0);
        static_for<0, 8>(fill_part);
        prepare(1);
        static_for<0, 8>(fill_part);

        // Q^T and dO^T as B operands: lane = query 16*qt + l16, 8 head-dim values per 32-wide k step
        bf16x8 qB[4][4], gB[4][4];
        float lse2[4];
        f32x4 neg_d[4];               // -D_i in all four registers: dP^T starts from it
#pragma unroll
        for (int qt = 0; qt < 4; ++qt) {
            const int64_t i = i0w + 16 * qt + l16, iq = i < a.S ? i : a.S - 1;      // rows past S are computed and never stored
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                qB[qt][kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(q + iq * a.ss + 32 * kk + 8 * g4));
                gB[qt][kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(g + iq * a.ss + 32 * kk + 8 * g4));
            }
            lse2[qt] = a.lse[stat + iq] * kLog2e;
            const float nd = -a.delta[stat + iq];
            neg_d[qt] = f32x4{nd, nd, nd, nd};
        }
        f32x4 accQ[8][4];             // dQ^T: [head-dim block of 16][query block]; lane = query, rows = head dim
#pragma unroll
        for (int dt = 0; dt < 8; ++dt)
#pragma unroll
            for (int qt = 0; qt < 4; ++qt)
#pragma unroll
                for (int r = 0; r < 4; ++r) accQ[dt][qt][r] = 0.f;
        uint32_t row[4], tr[8];       // LDS addresses in the K tile of the step; the V tile's are kDqRing further
        int at = ua % 3 * kDqTile, way = 0;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) row[kk] = ad.row16[kk] + at;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) tr[dt] = ad.tr16[dt] + at;

        f32x4 s[2][4], dp[2][4];      // [key block of 16][query block]
        u32x4 dsB[2][4];              // [parity of the key block of 32][query block]
        bf16x8 ka[4];
        TrSlot kt[4];
#pragma unroll
        for (int qt = 0; qt < 4; ++qt) dsB[0][qt] = dsB[1][qt] = u32x4{0, 0, 0, 0};

        // In the middle of step u: tile u + 1 is complete, and nobody reads tile u - 1 any more, whose place tile u + 2 takes from here on.
        auto meet = [&](int u) __attribute__((always_inline)) {
            wait_fills();
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            prepare(u + 2);
        };
        auto idle = [&](int u) __attribute__((always_inline)) {        // a step in which this wave has no keys
            meet(u);
            static_for<0, 8>(fill_part);
        };
        // block X of a step (OUT: with dQ of the block before it; LAST: no block follows); the reads of an item are queued three items ahead,
        // from 24 on the next block's
        constexpr int kAhead = 3;
        auto block = [&](auto xc, auto outc, auto lastc, bool masked) __attribute__((always_inline)) {
            constexpr int X = decltype(xc)::value, Y = X ^ 1;
            constexpr bool OUT = decltype(outc)::value, LAST = decltype(lastc)::value;
            constexpr auto reads_of = [](int n) constexpr { return n >= 24 ? (LAST ? 0 : 1) : n >= 16 ? 2 : 1; };
            auto read = [&](auto nc, auto pc) __attribute__((always_inline)) {
                constexpr int n = decltype(nc)::value, P = decltype(pc)::value;
                if constexpr (P >= reads_of(n)) {
                } else if constexpr (n >= 16 && n < 24) {
                    constexpr int off = (X == 0 ? 8192 : 0) + P * 4096;           // block 0 adds up block 1 of the tile before
                    lds_issue_tr_half<off>(P ? kt[n % 4].hi : kt[n % 4].lo, tr[n % 8]);
                    if constexpr (X == 0 && P == 1) tr[n % 8] += way;
                } else {
                    constexpr int XX = n < 24 ? X : Y, m = n % 24, isv = m / 8, kb16 = m % 8 / 4, kk = m % 4;
                    lds_issue_b128<isv * kDqRing + XX * 8192 + kb16 * 4096>(ka[n % 4], row[kk]);
                    if constexpr (X == 1 && n < 24 && isv && kb16) row[kk] += way;
                }
            };
            // the element-wise chains: el = 16 (key block) + 4 qt + r
            float x[2], ds[4];
            auto exp_position = [&](auto ic) __attribute__((always_inline)) {      // P: fma of el i, exponential of i - 1
                constexpr int i = decltype(ic)::value;
                if constexpr (i >= 1) {
                    constexpr int el = i - 1;
                    s[el / 16][el / 4 % 4][el % 4] = __builtin_amdgcn_exp2f(x[el % 2]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (i < 32) x[i % 2] = fmaf(s[i / 16][i / 4 % 4][i % 4], c, -lse2[i / 4 % 4]);
                __builtin_amdgcn_sched_barrier(0);
            };
            auto ds_position = [&](auto ic) __attribute__((always_inline)) {       // dS: product of el i, rounding of i - 1
                constexpr int i = decltype(ic)::value;
                if constexpr (i >= 2 && i % 2 == 0) {
                    constexpr int el = i - 1;
                    const f32x2 two = {ds[(el - 1) % 4], ds[el % 4]};
                    dsB[X][el / 4 % 4][el / 16 * 2 + el % 4 / 2] = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2));
                    asm volatile("" : "+v"(dsB[X][el / 4 % 4][el / 16 * 2 + el % 4 / 2]));
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (i < 32) ds[i % 4] = s[i / 16][i / 4 % 4][i % 4] * dp[i / 16][i / 4 % 4][i % 4];
                __builtin_amdgcn_sched_barrier(0);
            };
            constexpr int kExpFrom = 16, kExpSpan = 46, kDsFrom = 64, kDsSpan = 30;      // in MFMAs of the block
            auto item = [&](auto nc) __attribute__((always_inline)) {
                constexpr int n = decltype(nc)::value;
                constexpr auto behind = [](int i) constexpr { return !OUT && i >= 16 ? i + 8 : i; };       // without dQ the next block follows
                constexpr int later = reads_of(behind(n + 1)) + reads_of(behind(n + 2)), ahead = behind(n + kAhead);
                static_for<0, 4>([&](auto jc) {
                    constexpr int j = decltype(jc)::value, m = 4 * n + j, W = j == 0 ? later : kHere, kk = n % 4, kb16 = n % 8 / 4;
                    if constexpr (n < 8) {
                        if constexpr (kk == 0) mfma_zero_a<W>(s[kb16][j], ka[n % 4], qB[j][kk]);
                        else mfma_on_a<W>(s[kb16][j], ka[n % 4], qB[j][kk]);
                    } else if constexpr (n < 16) {
                        if constexpr (kk == 0) mfma_from_a<W>(dp[kb16][j], ka[n % 4], gB[j][kk], neg_d[j]);
                        else mfma_on_a<W>(dp[kb16][j], ka[n % 4], gB[j][kk]);
                    } else {
                        mfma_acc<W>(accQ[n % 8][j], tr_operand(kt[n % 4]), dsB[Y][j]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (j % 2 == 0) read(IntC<ahead>{}, IntC<j / 2>{});
                    constexpr auto upto = [](int i, int span, int all) constexpr { return i <= 0 ? 0 : i >= span ? all : (i * all + span - 1) / span; };
                    static_for<upto(m - kExpFrom, kExpSpan, 33), upto(m + 1 - kExpFrom, kExpSpan, 33)>(exp_position);
                    if constexpr (OUT) static_for<upto(m - kDsFrom, kDsSpan, 33), upto(m + 1 - kDsFrom, kDsSpan, 33)>(ds_position);
                    if constexpr (X == 1 && n < 8 && j == 3) fill_part(nc);
                    __builtin_amdgcn_sched_barrier(0);
                });
            };
            auto mask = [&](auto hc) __attribute__((always_inline)) {              // keys beyond the query, in the diagonal tile
                constexpr int H = decltype(hc)::value;
                asm volatile("s_nop 15" : "+v"(s[H][0]), "+v"(s[H][1]), "+v"(s[H][2]), "+v"(s[H][3]));
                int thr = l16 - 4 * g4;
                asm volatile("" : "+v"(thr));
#pragma unroll
                for (int qt = 0; qt < 4; ++qt)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (r > thr + 16 * qt - (32 * X + 16 * H)) s[H][qt][r] = -INFINITY;
            };
            if constexpr (!OUT) static_for<0, kAhead>([&](auto n) { read(n, IntC<0>{}); });
            static_for<0, 4>(item);
            if (masked) mask(IntC<0>{});
            static_for<4, 8>(item);
            if (masked) mask(IntC<1>{});
            static_for<8, 16>(item);
            if constexpr (OUT) {
                static_for<16, 24>(item);
            } else {
                settle(dp);
                static_for<0, 33>(ds_position);
            }
        };
        using Yes = IntC<1>;
        using No = IntC<0>;
        wait_fills();
        __syncthreads();
        int u = 0;
#pragma clang loop unroll(disable)
        for (; u < ua; ++u) idle(u);
        if (live) {
            block(IntC<0>{}, No{}, No{}, u == um);
            // the second half of step u; after the loop once more: with one copy and an exit in mid-loop the compiler spills Q
            auto second = [&](auto lastc) __attribute__((always_inline)) {
                way = at == 2 * kDqTile ? -2 * kDqTile : kDqTile;
                at += way;
                meet(u);
                block(IntC<1>{}, Yes{}, lastc, u == um);
            };
#pragma clang loop unroll(disable)
            while (u < ub) {
                second(No{});
                ++u;
                block(IntC<0>{}, Yes{}, No{}, u == um);
            }
            second(Yes{});
            static_for<0, 8>([&](auto n) {        // dQ of the last block
                constexpr int dt = decltype(n)::value;
                lds_issue_tr_pair<8192>(kt[dt % 4], tr[dt]);
                static_for<0, 4>([&](auto jc) { mfma_acc<decltype(jc)::value ? kHere : 0>(accQ[dt][decltype(jc)::value], tr_operand(kt[dt % 4]), dsB[1][decltype(jc)::value]); });
            });
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) asm volatile("s_nop 15" : "+a"(accQ[dt][0]), "+a"(accQ[dt][1]), "+a"(accQ[dt][2]), "+a"(accQ[dt][3]));
            ++u;
        }
#pragma clang loop unroll(disable)
        for (; u < ntiles; ++u) idle(u);
        wait_fills();

        __bf16 *dq = static_cast<__bf16 *>(a.dq) + base + (i0w + l16) * a.ss + 4 * g4;
#pragma unroll
        for (int qt = 0; qt < 4; ++qt)
            if (i0w + 16 * qt + l16 < a.S) {
#pragma unroll
                for (int dt = 0; dt < 8; ++dt) store4(dq + 16 * qt * a.ss + 16 * dt, accQ[dt][qt], a.scale);
            }
    }   // pass
}

// ============================================================================ launches
#define LONG_KERNEL __global__ __launch_bounds__(64 * kLongWaves) __attribute__((amdgpu_waves_per_eu(1, 1))) void

__device__ __forceinline__ int64_t long_tiles(const AttnArgs &a) { return (a.S + kLongKeys - 1) / kLongKeys; }

LONG_KERNEL attn_bwd_dkdv_bf16_long_kernel(AttnArgs a, int order)
{
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kDkdvLds];
    const PairId t = decode_block(a, blockIdx.x, long_tiles(a), order, false);
    if (t.first >= 0) dkdv_long_rows(a, (LDS_AS unsigned char *)smem, t);
}

LONG_KERNEL attn_bwd_dq_bf16_long_kernel(AttnArgs a, int order)
{
    __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * kDqRing];
    const PairId t = decode_block(a, blockIdx.x, long_tiles(a), order, true);
    if (t.first >= 0) dq_long_rows(a, (LDS_AS unsigned char *)smem, t);
}

// both gradients in one launch, single tiles, longest first: all key tiles and then all query tiles.  Against the same launch in eight waves
// (attn_bwd_bf16.hip), us: S = 14528 H = 8 1226 -> 1127, 25000 H = 4 1899 -> 1739, 40000 H = 5 6141 -> 5597, 90000 H = 4 22911 -> 21012; where four waves lose is
// beside kJointChoices (launch_plan.h).
LONG_KERNEL attn_bwd_both_bf16_long_kernel(AttnArgs a, uint32_t dkdv_blocks)
{
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kDkdvLds];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;
    if (blockIdx.x < dkdv_blocks) dkdv_long_rows(a, lds, decode_block(a, blockIdx.x, long_tiles(a), kLongestFirst, false));
    else dq_long_rows(a, lds, decode_block(a, blockIdx.x - dkdv_blocks, long_tiles(a), kLongestFirst, true));
}

}  // namespace

hipError_t launch_attn_bwd_both_bf16_long(const AttnArgs &a, int64_t dkdv_blocks, int64_t blocks, hipStream_t st)
{
    return launch_blocks<64 * kLongWaves>(attn_bwd_both_bf16_long_kernel, blocks, st, a, (uint32_t)dkdv_blocks);
}

hipError_t launch_attn_bwd_dkdv_bf16_long(const AttnArgs &a, int order, int64_t blocks, hipStream_t st)
{
    return launch_blocks<64 * kLongWaves>(attn_bwd_dkdv_bf16_long_kernel, blocks, st, a, order);
}

hipError_t launch_attn_bwd_dq_bf16_long(const AttnArgs &a, int order, int64_t blocks, hipStream_t st)
{
    return launch_blocks<64 * kLongWaves>(attn_bwd_dq_bf16_long_kernel, blocks, st, a, order);
}

}  // namespace memo

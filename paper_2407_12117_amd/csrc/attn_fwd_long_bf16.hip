// bf16 causal attention forward for gfx950 (CDNA4), head dim 128, workgroups of 256 rows: long sequences
// (shorter ones, what is computed and the operand conventions: attn_bf16.hip).
//
// Four waves, one per SIMD, each with 64 query rows (two blocks of 32) and 460 registers.  Long sweeps are bound by power, so what counts
// is the energy of a product and how little of a wave's time its matrix core rests:
//  * An operand of K or V^T read from LDS serves two row blocks, half the LDS reads per product of eight waves of 32 rows.
//  * Scores, exponentials and output of three consecutive blocks of 32 keys run in one stream, dealt out behind the MFMAs by hand:
//    slot b issues the MFMAs of S(b + 1) and of O += V^T P(b - 1), two and two, and behind each about one element's share of
//    P(b) = exp2(..).  The MFMA comes first in each piece and its vector instructions behind it (the other way round: 1272 for
//    1312 TFLOP/s); sums and their test end two MFMAs before the slot does.
//  * K and V come through rings of three tiles; the barrier of a step lies between its two slots, a full step after the fills it waits
//    for were asked for, and the first operands of the next step are read before this one ends.
// The output accumulators and Q live in the accumulation registers, which the compiler does by itself only with moves of the score tiles in
// and out of them: the MFMAs are inline asm that names the register file.  The compiler does not see what is in it, so the waits
// between an MFMA and the vector instructions that touch its result are written here (settle_*).
// S = 128K, H = 4, same card in turn, eight waves of 32 rows (two per SIMD, compiler's order) -> this: 14.56 -> 13.40 ms
// (1208 -> 1312 TFLOP/s; all-zero inputs, no power limit: 51.5 -> 45 cycles per MFMA of 32).
#include "bf16_tiles.h"

namespace memo {
namespace {

constexpr int kLongWaves = 4, kLongRows = 64 * kLongWaves, kLongKeys = 64;

// D = A B + D with the scores in vector registers and the output in accumulation registers.  N: LDS reads that may still be on
// their way when A is needed; -1: it was needed before.
constexpr int kHere = -1;
template <int N>
__device__ __forceinline__ void mfma_scores(f32x16 &d, const bf16x8 &k, const bf16x8 &q)
{
    if constexpr (N >= 0) asm volatile("s_waitcnt lgkmcnt(%3)\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(k), "a"(q), "n"(N));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(k), "a"(q));
}
template <int N>
__device__ __forceinline__ void mfma_scores_first(f32x16 &d, const bf16x8 &k, const bf16x8 &q)      // D = A B
{
    if constexpr (N >= 0) asm volatile("s_waitcnt lgkmcnt(%3)\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(k), "a"(q), "n"(N));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(k), "a"(q));
}
template <int N>
__device__ __forceinline__ void mfma_output(f32x16 &d, const bf16x8 &v, const u32x4 &p)
{
    if constexpr (N >= 0) asm volatile("s_waitcnt lgkmcnt(%3)\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(v), "v"(p), "n"(N));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(v), "v"(p));
}

// An MFMA of 8 passes is written 12 wait states after its issue; vector instructions that touch the result come behind these.
__device__ __forceinline__ void settle_output(f32x16 (&acc)[2][4])
{
    asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[0][0]), "+a"(acc[0][1]), "+a"(acc[0][2]), "+a"(acc[0][3]),
                                          "+a"(acc[1][0]), "+a"(acc[1][1]), "+a"(acc[1][2]), "+a"(acc[1][3]));
}
template <bool ALONE>              // whether no other MFMAs were issued behind the last one of the scores
__device__ __forceinline__ void settle_scores(f32x16 (&s)[2])
{
    if constexpr (ALONE) asm volatile("s_nop 15\n\ts_nop 15" : "+v"(s[0]), "+v"(s[1]));
    else asm volatile("s_nop 3" : "+v"(s[0]), "+v"(s[1]));           // two MFMAs of 8 states each lie between
}

__global__ __launch_bounds__(64 * kLongWaves) __attribute__((amdgpu_waves_per_eu(1, 1))) void attn_fwd_bf16_long_kernel(AttnArgs a, int order)
{
    constexpr int kTile = kLongKeys * 256, kRing = 3 * kTile;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * kRing];     // K tile t at t % 3, V tile t behind them likewise
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;

    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: lives in a scalar register
    const int64_t nqt = (a.S + kLongRows - 1) / kLongRows;
    const PairId t = decode_block(a, blockIdx.x, nqt, order, true);
    if (t.first < 0) return;
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh;
    const __bf16 *q = static_cast<const __bf16 *>(a.q) + base;
    const __bf16 *k = static_cast<const __bf16 *>(a.k) + base;
    const __bf16 *v = static_cast<const __bf16 *>(a.v) + base;
    const float c = a.scale * kLog2e;
    const LdsAddr ad = make_lds_addr(lds, make_lane_addr(lane));
    using Fills = TileOffsets<kLongWaves, kLongKeys>;
    const Fills toff = make_tile_offsets<kLongWaves, SwzA, kLongKeys>(a.ss, wave, lane);
    static_assert(Fills::kInstr == 4, "fill_part deals out eight");

    // the heavy tile of the pair sweeps the keys upwards from row 0, the light one downwards to row 0
    // (online softmax takes the key tiles in any order)
#pragma clang loop unroll(disable)
    for (int pass = 0; pass < 2; ++pass) {
        const int64_t tile = pass == 0 ? (t.second >= 0 ? t.second : t.first) : (t.second >= 0 ? t.first : -1);
        if (tile < 0) break;
        const int64_t row0 = tile * kLongRows, i0w = row0 + 64 * wave;
        const int64_t last_row = min(row0 + kLongRows, a.S) - 1;
        const int ntiles = (int)(last_row / kLongKeys) + 1;
        // Tiles by their place in the sweep: this wave works [ua, ub], of which um holds its diagonal; one that has no rows works none.
        const int diagonal = (int)(i0w / kLongKeys);
        const bool live = i0w < a.S;
        const int ua = !live ? ntiles + 1 : pass ? ntiles - 1 - diagonal : 0, ub = pass ? ntiles - 1 : diagonal, um = pass ? ua : ub;
        if (pass) __syncthreads();    // every wave has left the first tile's last LDS buffers

        // Tile u of the sweep as a buffer (TileOffsets::fill), from a pointer that moves on a tile at a time; behind the last one it is empty.
        const int64_t tile_bytes = (pass ? -1 : 1) * (int64_t)kLongKeys * a.ss * 2;
        const int64_t first_key = pass ? (int64_t)(ntiles - 1) * kLongKeys : 0;
        uint32_t full_bytes = (uint32_t)(kLongKeys - 1) * (uint32_t)a.ss * 2 + 256;
        uint32_t last_bytes = (uint32_t)(min(a.S - (int64_t)(ntiles - 1) * kLongKeys, (int64_t)kLongKeys) - 1) * (uint32_t)a.ss * 2 + 256;
        asm volatile("" : "+s"(full_bytes), "+s"(last_bytes));      // selected without branches
        const int u_last = pass ? 0 : ntiles - 1;
        auto buffer = [&](const char *p, int u) __attribute__((always_inline)) {
            uint32_t bytes = u < ntiles ? full_bytes : 0;
            bytes = u == u_last ? last_bytes : bytes;
            return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p), 0, bytes, 0x00020000);
        };
        const char *kp = reinterpret_cast<const char *>(k + first_key * a.ss), *vp = reinterpret_cast<const char *>(v + first_key * a.ss);
        int kto = 0, vto = kRing;                  // where the next K and V tiles go
        auto advance = [&](const char *&p, int &to, int end) __attribute__((always_inline)) {
            p += tile_bytes;
            to += kTile;
            if (to == end) to -= kRing;
        };
        auto fill_tile = [&](const char *&p, int &to, int end, int u) __attribute__((always_inline)) {
            const __amdgpu_buffer_rsrc_t r = buffer(p, u);
#pragma unroll
            for (int n = 0; n < Fills::kInstr; ++n) toff.part(lds + to, r, n, wave);
            advance(p, to, end);
        };
        fill_tile(kp, kto, kRing, 0);
        fill_tile(vp, vto, 2 * kRing, 0);
        fill_tile(kp, kto, kRing, 1);

        // Q^T as B operand: lane = query row, 8 head-dim values per 16-wide chunk
        bf16x8 qB[2][8];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int64_t i = i0w + 32 * b + l32, iq = i < a.S ? i : a.S - 1;     // rows past S are computed and never stored
#pragma unroll
            for (int kc = 0; kc < 8; ++kc)
                qB[b][kc] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(q + iq * a.ss + 16 * kc + 8 * half));
        }
        f32x16 acc[2][4], s[2][2];        // [row block][column block]; [parity of the key block][row block]
        u32x4 p[2][2][2];                 // [parity of the key block][row block][16-key chunk]
        bf16x8 kr[4];                     // operands on their way
        TrSlot vr[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) kr[i] = qB[0][0], vr[i].lo = vr[i].hi = s16x4{0, 0, 0, 0};
#pragma unroll
        for (int b = 0; b < 2; ++b) {
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[b][cb][e] = 0.f;
#pragma unroll
            for (int x = 0; x < 2; ++x) {
#pragma unroll
                for (int e = 0; e < 16; ++e) s[x][b][e] = 0.f;
                p[x][b][0] = p[x][b][1] = u32x4{0, 0, 0, 0};
            }
        }
        float m[2] = {-INFINITY, -INFINITY}, mc[2] = {-INFINITY, -INFINITY}, lsum[2] = {0.f, 0.f};   // as in attn_fwd_bf16_kernel
        // Row sums of a tile: two chains over both of its key blocks, added to lsum once a tile, as in attn_fwd_bf16_kernel (once a block: rms error
        // of the logsumexp 7.1e-7 for 6.3e-7 at 64K keys, 1.08e-6 for 8.5e-7 at 256K, and no faster); and what they were behind the first block.
        float ps[2][2] = {{0.f, 0.f}, {0.f, 0.f}}, ps_first[2][2] = {{0.f, 0.f}, {0.f, 0.f}};

        uint32_t ka[8], va[4][2];                  // LDS addresses in the K tile of this step and in the V tile of the step before
        int kat = 0, vat = 0, kd = 0, vd = 0;      // places of these tiles, ways to the next ones
        auto ways = [&]() __attribute__((always_inline)) {
            kd = kat == 2 * kTile ? -2 * kTile : kTile;
            vd = vat == 2 * kTile ? -2 * kTile : kTile;
        };
        auto addresses = [&](int u) __attribute__((always_inline)) {
            kat = u % 3 * kTile;
            vat = (u + 2) % 3 * kTile;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                ka[i] = ad.row[i] + kat;
                va[i / 2][i % 2] = ad.tr[i / 2][i % 2] + kRing + vat;
            }
            ways();
        };
        // In the middle of step u: K tile u + 1 and V tile u are complete, and nobody reads K tile u - 1 or V tile u - 2 any more,
        // whose places K tile u + 2 and V tile u + 1 take from here on.
        auto meet = [&]() __attribute__((always_inline)) {
            wait_fills();
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };
        __amdgpu_buffer_rsrc_t kb, vb;
        auto fill_part = [&](auto nc) __attribute__((always_inline)) {
            constexpr int n = decltype(nc)::value;
            if constexpr (n < Fills::kInstr) toff.part(lds + vto, vb, n, wave);
            else toff.part(lds + kto, kb, n - Fills::kInstr, wave);
        };
        auto idle = [&](int u) __attribute__((always_inline)) {        // a step in which this wave has no keys
            meet();
            fill_tile(vp, vto, 2 * kRing, u + 1);
            fill_tile(kp, kto, kRing, u + 2);
        };

        // Step u, two slots of one key block each: slot x forms the scores of block 2u + x (SCORES), the exponentials of the block before
        // it (EXPx) and adds block 2u + x - 2 to the output (OUT: both slots).  Its LDS operands are K items 0..15
        // (slot n / 8, chunk n % 8) and V items 0..15 (slot n / 8, 16 keys n % 8 / 4, 32 columns n % 4), read in the order K0 V0 K1 V1 ..,
        // two items ahead; items from 16 on are the next step's.
        auto step = [&](int u, auto scores_c, auto exp0_c, auto exp1_c, auto out_c, auto first_c) __attribute__((always_inline)) {
            constexpr bool SCORES = decltype(scores_c)::value, EXP0 = decltype(exp0_c)::value, EXP1 = decltype(exp1_c)::value,
                           OUT = decltype(out_c)::value, FIRST = decltype(first_c)::value;
            constexpr int kAhead = 2;
            constexpr auto has_k = [](int) constexpr { return SCORES; };
            constexpr auto has_v = [](int n) constexpr { return n < 16 ? OUT : SCORES; };
            auto issue_k = [&](auto n) __attribute__((always_inline)) {
                constexpr int i = decltype(n)::value;
                if constexpr (has_k(i)) lds_issue_b128<i % 16 / 8 * 8192>(kr[i % 4], ka[i % 8]);
                if constexpr (SCORES && i >= 8 && i < 16) ka[i % 8] += kd;
            };
            auto issue_v = [&](auto n, auto hi) __attribute__((always_inline)) {
                constexpr int i = decltype(n)::value, h = decltype(hi)::value;
                if constexpr (has_v(i)) lds_issue_tr_half<i % 16 / 4 * 4096>(h ? vr[i % 4].hi : vr[i % 4].lo, va[i % 4][h]);
                if constexpr (SCORES && i >= 12 && i < 16) va[i % 4][h] += vd;
            };
            if constexpr (FIRST) static_for<0, kAhead>([&](auto n) { issue_k(n); });
            static_for<0, 2>([&](auto slotc) {
                constexpr int X = decltype(slotc)::value, Y = X ^ 1;      // parity of the scores and of the output; of the exponentials
                constexpr bool EXP = X ? EXP1 : EXP0;
                f32x16 (&se)[2] = s[Y];
                if constexpr (EXP) {
                    if (u - Y == um) {                // the diagonal tile: mask keys j > i
                        int thr = l32 - 4 * half;
                        asm volatile("" : "+v"(thr));
#pragma unroll
                        for (int b = 0; b < 2; ++b)
#pragma unroll
                            for (int e = 0; e < 16; ++e)
                                if (8 * (e >> 2) + (e & 3) > thr + 32 * (b - Y)) se[b][e] = -INFINITY;
                    }
                }
                if constexpr (X == 1) {
                    meet();
                    vb = buffer(vp, u + 1);
                    kb = buffer(kp, u + 2);
                }
                // P = exp2(c S - c m) against the running maximum as it stands, its row sums, rounded to bf16 (attn_fwd_bf16_kernel), as a
                // chain over positions 0..33: fma of element i, exponential of i - 1, sum and rounding of i - 2.  In this order: an
                // exponential right before an MFMA costs 3 cycles of 45.
                float sum[2], x[3], y[4];
                if constexpr (EXP) {
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int i = 0; i < 2; ++i) (Y ? ps_first : ps)[b][i] = Y ? ps[b][i] : 0.f;
                }
                auto position = [&](auto ic) __attribute__((always_inline)) {
                    constexpr int i = decltype(ic)::value;
                    if constexpr (i >= 2) {
                        constexpr int el = i - 2, b = el / 16, e = el % 16;
                        ps[b][e & 1] += y[el & 3];
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (e & 1) {
                            const f32x2 two = {y[(el - 1) & 3], y[el & 3]};
                            p[Y][b][e >> 3][(e & 7) >> 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2));
                            asm volatile("" : "+v"(p[Y][b][e >> 3][(e & 7) >> 1]));
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                    if constexpr (i >= 1 && i < 33) y[(i - 1) & 3] = __builtin_amdgcn_exp2f(x[(i - 1) % 3]);
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (i < 32) x[i % 3] = fmaf(se[i / 16][i % 16], c, -mc[i / 16]);
                    __builtin_amdgcn_sched_barrier(0);
                };
                // what comes behind MFMA j of the slot's 32: all positions behind the first kSpan, the sums and their test behind the last two
                constexpr int kSpan = 30;
                bool high = false;
                auto behind = [&](auto jc) __attribute__((always_inline)) {
                    constexpr int j = decltype(jc)::value;
                    constexpr auto upto = [](int n) constexpr { return n >= kSpan ? 34 : (n * 34 + kSpan - 1) / kSpan; };
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (EXP) {
                        static_for<upto(j), upto(j + 1)>(position);
                        if constexpr (j == kSpan) {
                            sum[0] = ps[0][0] + ps[0][1];
                            sum[1] = ps[1][0] + ps[1][1];
                        }
                        // not (sum <= bound) rather than sum > bound: a NaN sum takes the careful path too
                        if constexpr (j == kSpan + 1) high = __builtin_amdgcn_ballot_w64(!(sum[0] + sum[1] <= kRescaleAbove)) != 0;
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
                static_for<0, 8>([&](auto nc) {
                    constexpr int n = decltype(nc)::value, g = X * 8 + n;
                    // reads queued behind K item g and behind V item g where these are needed
                    constexpr int behind_k = [&]() constexpr {
                        int w = 0;
                        for (int j = g; j < g + kAhead; ++j) w += (has_v(j) ? 2 : 0) + (j > g && has_k(j) ? 1 : 0);
                        return w;
                    }();
                    constexpr int behind_v = [&]() constexpr {
                        int w = has_v(g + kAhead) ? 1 : 0;
                        for (int j = g + 1; j <= g + kAhead; ++j) w += (has_k(j) ? 1 : 0) + (j < g + kAhead && has_v(j) ? 2 : 0);
                        return w;
                    }();
                    if constexpr (SCORES) {
                        if constexpr (n == 0) mfma_scores_first<behind_k>(s[X][0], kr[g % 4], qB[0][n]);
                        else mfma_scores<behind_k>(s[X][0], kr[g % 4], qB[0][n]);
                    }
                    issue_k(IntC<g + kAhead>{});
                    behind(IntC<4 * n>{});
                    if constexpr (SCORES) {
                        if constexpr (n == 0) mfma_scores_first<kHere>(s[X][1], kr[g % 4], qB[1][n]);
                        else mfma_scores<kHere>(s[X][1], kr[g % 4], qB[1][n]);
                    }
                    issue_v(IntC<g + kAhead>{}, IntC<0>{});
                    behind(IntC<4 * n + 1>{});
                    if constexpr (OUT) mfma_output<behind_v>(acc[0][n % 4], tr_operand(vr[g % 4]), p[X][0][n / 4]);
                    issue_v(IntC<g + kAhead>{}, IntC<1>{});
                    behind(IntC<4 * n + 2>{});
                    if constexpr (OUT) mfma_output<kHere>(acc[1][n % 4], tr_operand(vr[g % 4]), p[X][1][n / 4]);
                    if constexpr (X == 1) fill_part(nc);
                    behind(IntC<4 * n + 3>{});
                });
                if constexpr (SCORES) settle_scores<!OUT>(s[X]);
                if constexpr (EXP) {
                    if (high) {                       // some row sum shows a score far above the maximum: bring it up to date, once more
                        settle_output(acc);
#pragma unroll
                        for (int b = 0; b < 2; ++b) {
                            float mb = fmaxf(fmaxf(se[b][0], se[b][1]), se[b][2]);
#pragma unroll
                            for (int e = 3; e < 15; e += 2) mb = fmaxf(fmaxf(mb, se[b][e]), se[b][e + 1]);
                            mb = fmaxf(mb, se[b][15]);
                            if constexpr (FIRST) {    // the maximum of a sweep's first tile, not of its first block alone: P of the largest score is 1, without rounding
#pragma unroll
                                for (int e = 0; e < 16; ++e) {
                                    if (u == um && 8 * (e >> 2) + (e & 3) > l32 - 4 * half + 32 * (b - 1)) s[X][b][e] = -INFINITY;
                                    mb = fmaxf(mb, s[X][b][e]);
                                }
                            }
                            const float m_new = finite_max(m[b], max_across_halves(mb));
                            const float corr = __builtin_amdgcn_exp2f((m[b] - m_new) * c);
                            m[b] = m_new;
                            mc[b] = scaled_max(m_new, c);
                            lsum[b] *= corr;
#pragma unroll
                            for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                                for (int e = 0; e < 16; ++e) acc[b][cb][e] *= corr;
#pragma unroll
                            for (int i = 0; i < 2; ++i) ps[b][i] = Y ? ps_first[b][i] * corr : 0.f;
#pragma unroll
                            for (int e = 0; e < 16; e += 2) {
                                const f32x2 two = {__builtin_amdgcn_exp2f(fmaf(se[b][e], c, -mc[b])), __builtin_amdgcn_exp2f(fmaf(se[b][e + 1], c, -mc[b]))};
                                ps[b][0] += two[0];
                                ps[b][1] += two[1];
                                p[Y][b][e >> 3][(e & 7) >> 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2));
                            }
                            sum[b] = ps[b][0] + ps[b][1];
                        }
                        settle_output(acc);
                    }
                    if constexpr (Y == 1) {
#pragma unroll
                        for (int b = 0; b < 2; ++b) lsum[b] += sum[b];
                    }
                    asm volatile("s_nop 1" : "+v"(p[Y][0][0]), "+v"(p[Y][0][1]), "+v"(p[Y][1][0]), "+v"(p[Y][1][1]));
                }
            });
            if constexpr (SCORES) {
                kat += kd;
                vat += vd;
                ways();
            }
            advance(vp, vto, 2 * kRing);
            advance(kp, kto, kRing);
        };
        using Yes = IntC<1>;
        using No = IntC<0>;
        wait_fills();
        __syncthreads();
        // ntiles + 1 steps for every wave, which meet once in each
        int u = 0;
#pragma clang loop unroll(disable)
        for (; u < min(ua, ntiles + 1); ++u) idle(u);
        if (live) {
            addresses(u);
            step(u, Yes{}, No{}, Yes{}, No{}, Yes{});
#pragma clang loop unroll(disable)
            for (++u; u <= ub; ++u) step(u, Yes{}, Yes{}, Yes{}, Yes{}, No{});
            // The reads queued ahead, of which the last step uses V's alone: K's keep their registers up to here (named in the text for the test).
            asm volatile("s_waitcnt lgkmcnt(0) ; %0 %1" : "+v"(kr[0]), "+v"(kr[1]), "+v"(vr[0].lo), "+v"(vr[0].hi), "+v"(vr[1].lo), "+v"(vr[1].hi) :: "memory");
            step(u, No{}, Yes{}, No{}, Yes{}, No{});
            settle_output(acc);           // here: the compiler may move the accumulators before the waves meet again
            ++u;
        }
#pragma clang loop unroll(disable)
        for (; u <= ntiles; ++u) idle(u);
        wait_fills();

#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int64_t i = i0w + 32 * b + l32;
            const float ltot = add_across_halves(lsum[b]);
            if (i < a.S) {
                store_acc_T(static_cast<__bf16 *>(a.o_out) + base + i * a.ss, acc[b], 1.f / ltot, half);
                if (half == 0) a.lse[((int64_t)t.b * a.H + t.h) * a.S + i] = (mc[b] + __builtin_amdgcn_logf(ltot)) * kLn2;
            }
        }
    }   // pass
}

}  // namespace

hipError_t launch_attn_fwd_bf16_long(const AttnArgs &a, int order, int64_t blocks, hipStream_t st)
{
    return launch_blocks<64 * kLongWaves>(attn_fwd_bf16_long_kernel, blocks, st, a, order);
}

}  // namespace memo

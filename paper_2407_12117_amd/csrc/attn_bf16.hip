// bf16 causal attention forward for gfx950 (CDNA4), head dim 128 (the backward is attn_bwd_bf16.hip).
//
// What is computed (Section 2.1.3 of the paper): O = softmax(scale Q K^T) V under the causal
// mask, tile by tile with per-row running maximum and sum ("compact states"), plus the
// per-row logsumexp that the backward re-forms the probabilities from.
//
// Contractions run on the matrix cores with v_mfma_f32_32x32x16_bf16 (fp32 accumulate);
// softmax runs in fp32 on the VALU with exp2 (scale*log2 e folded into one fma).
// Probabilities are rounded to bf16 before the second contraction.
//
// Operand conventions of the 32x32x16 MFMA, D = A(32xK16) * B(K16x32), lane = 32*half + l32:
//   A : lane holds row  l32, k = 8*half .. 8*half+7      (8 bf16)
//   B : lane holds col  l32, k = 8*half .. 8*half+7      (8 bf16)
//   D : lane holds col  l32, rows 8*g + 4*half + r for register v = 4*g + r (16 fp32)
// Every product is arranged so that the per-row softmax quantities sit in ONE lane: the
// score tile is produced with the key index along D's rows and the query index along D's
// columns.
// The fp32 D registers of the score tile, rounded to bf16, are then directly a B operand
// of the next contraction, whose contraction slot e (0..7) of 16-row chunk q is tile row
//   16*q + 8*(e/4) + 4*half + e%4.
// The matching A operand is a TRANSPOSED read of a row-major LDS tile, done by the LDS
// transpose load ds_read_b64_tr_b16 (two per operand: rows 4*half+0..3 and 8+4*half+0..3).
// All operand reads are issued by hand several MFMAs ahead (see lds_pipeline_* below).
//
// LDS tiles are 64 or 32 rows x 128 bf16, row-major, 256 bytes per row, no padding; the sixteen
// 16-byte chunks of row r are stored at chunk position  c ^ swz(r),
//   swz(r) = ((r & 3) << 2) | ((r >> 2) & 3),
// which makes both access patterns bank-conflict free: 16 lanes reading the same chunk of
// 16 consecutive rows (row-major operand), and 32 lanes reading 4 rows x 64 contiguous
// bytes (transposed operand).
#include "bf16_tiles.h"

namespace memo {
namespace {

// ============================================================================ forward
// Workgroups, by owned rows:
//   256 rows, long sequences: attn_fwd_long_bf16.hip, four waves of 64 rows.  The more rows share a K/V tile, the less fill traffic
//        (L2 -> LDS) each MFMA pays for, and the fewer LDS reads per MFMA with more rows in a wave: the best rate on a full chip.
//   256 rows, shorter ones (launch_plan.h): attn_fwd_bf16_kernel<8>, eight waves of 32 rows, keys not split.  Its sweep starts and ends 3 to 4 us earlier.
//   128: attn_fwd_bf16_kernel<4>, eight waves as four query groups (32 rows each) x two key groups; key group g
//        takes the key tiles g, g + 2, ... of 64 rows through its own double-buffered LDS ring, filled
//        asynchronously (one barrier per step), and the groups of a row are combined at the end.
//   64: keys in eight, all rows in every wave: attn_fwd_bf16_own_kernel.
//   32: keys in eight: attn_fwd_bf16_short_kernel.
// TFLOP/s at S = 128K, H = 4: 1312, 1208, 1130, 1050, 700.
// A short sequence has too few 256-row tiles for 256 compute units, and a sweep is as long as its
// last row: what bounds it is the longest workgroup, which 32 rows make 64 times shorter.  The launcher
// takes the cheapest by estimate (launch_plan.h).  256-row pairs alone -> now, us: S = 640 H = 2 31.0 -> 5.7,
// B = 2 S = 2000 H = 3 67.8 -> 14.8, S = 8192 H = 4 250 -> 77, S = 16461 H = 4 482 -> 264, S = 40000 H = 4 2202 -> 1483.
// The fills address a tile as a buffer (TileOffsets::fill): no per-lane pointers to step and no second path for the
// ragged last tile, 1 to 3 % of every shape.
constexpr int kFwdWaves = 8;                 // waves per workgroup

// a K operand and the Q operands of one or two row blocks
template <int NQ> struct KqSlot { bf16x8 k, q[NQ]; };

template <int N>
__device__ __forceinline__ void lds_wait(KqSlot<1> &x)
{
    static_assert(N >= 0 && N <= 15, "lgkmcnt range");
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(x.k), "+v"(x.q[0]) : "n"(N));
}

template <int N>
__device__ __forceinline__ void lds_wait(KqSlot<2> &x)
{
    static_assert(N >= 0 && N <= 15, "lgkmcnt range");
    asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(x.k), "+v"(x.q[0]), "+v"(x.q[1]) : "n"(N));
}

template <int QG>
__global__ __launch_bounds__(64 * kFwdWaves) void attn_fwd_bf16_kernel(AttnArgs a, int fold)
{
    constexpr int KS = kFwdWaves / QG, kBq = 32 * QG, kBk = 64, JB = kBk / 32;
    constexpr int kTile = kBk * 256;            // bytes of one K or V tile
    constexpr int kStage = 2 * kTile, kGroup = 2 * kStage, kRing = KS * kGroup;
    constexpr int kMerge = KS > 1 ? 8 * 32 * 8 : 0;             // (maximum, sum) of every row of every wave
    static_assert(KS == 1 || kRing == 8 * 16384, "the merge lays eight accumulator sets over the ring");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kRing + kMerge];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;   // [key group][buf][K|V] tiles

    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: lives in a scalar register
    const LaneAddr la = make_lane_addr(lane);
    const int wq = wave % QG, grp = wave / QG;  // query group, key group
    const int64_t nqt = (a.S + kBq - 1) / kBq;
    const int order = tile_order(kBq, fold);
    const PairId t = decode_block(a, blockIdx.x, nqt, order, true);
    if (t.first < 0) return;
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh;
    const __bf16 *q = static_cast<const __bf16 *>(a.q) + base;
    const __bf16 *k = static_cast<const __bf16 *>(a.k) + base;
    const __bf16 *v = static_cast<const __bf16 *>(a.v) + base;
    const float c = a.scale * kLog2e;
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const LdsAddr ad = make_lds_addr(lds + grp * kGroup, la);
    const uint32_t (&row_addr)[8] = ad.row;
    const uint32_t (&tr_addr)[4][2] = ad.tr;

    // the heavy tile of the pair sweeps the keys upwards from row 0, the light one downwards to row 0
    // (online softmax takes the key tiles in any order)
    for (int pass = 0; pass < (QG == 8 ? 2 : 1); ++pass) {
    const int64_t tile = pass == 0 ? (t.second >= 0 ? t.second : t.first) : (t.second >= 0 ? t.first : -1);
    if (tile < 0) break;
    const int64_t row0 = tile * kBq, i0w = row0 + 32 * wq, i = i0w + l32;
    const int64_t last_row = min(row0 + kBq, a.S) - 1;
    const int ntiles = (int)(last_row / kBk) + 1, nsteps = (ntiles + KS - 1) / KS;
    // step n of a key group works tile KS * n + grp (KS = 1: also from the other end)
    const int jfirst = pass ? ntiles - 1 : grp, jstep = pass ? -KS : KS;
    if (pass) __syncthreads();    // every wave has left the first tile's last LDS buffer
    const TileOffsets<QG, kBk> toff = make_tile_offsets<QG, SwzA, kBk>(a.ss, wq, lane);
    auto fill_k = [&](int off, int jt) {
        toff.fill(lds + grp * kGroup + off, k, a.ss, (int64_t)jt * kBk, a.S, wq);
    };
    auto fill_v = [&](int off, int jt) {
        toff.fill(lds + grp * kGroup + off + kTile, v, a.ss, (int64_t)jt * kBk, a.S, wq);
    };
    // Key groups that need the same Q rows bring them in once, as whole rows, in the place of the buffers that the second tiles take: to each
    // wave's registers straight from memory, 32 bytes of a row at a time, they cost a unit 5000 cycles.
    constexpr bool kStaged = KS > 1;
    constexpr int kBlocks = kStage / (32 * 256);      // 32-row blocks in one such buffer
    static_assert(!kStaged || KS * kBlocks >= QG, "room for the Q rows");
    auto staged = [&](int block) { return lds + block / kBlocks * kGroup + kStage + block % kBlocks * 32 * 256; };
    if constexpr (kStaged) {
        const TileOffsets<8, 32> qoff = make_tile_offsets<8, SwzA, 32>(a.ss, wave, lane);
#pragma unroll
        for (int blk = 0; blk < QG; ++blk) qoff.fill(staged(blk), q, a.ss, row0 + 32 * blk, a.S, wave);
    }
    if (jfirst < ntiles) {
        fill_k(0, jfirst);
        fill_v(0, jfirst);
    }

    // Q^T as B operand: lane = query row i, 8 head-dim values per 16-wide chunk
    bf16x8 qB[8];
    if constexpr (!kStaged) {
        const int64_t iq = i < a.S ? i : a.S - 1;     // rows past S are computed and never stored
#pragma unroll
        for (int kc = 0; kc < 8; ++kc)
            qB[kc] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(q + iq * a.ss + 16 * kc + 8 * half));
    }

    f32x16 accO[4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int e = 0; e < 16; ++e) accO[cb][e] = 0.f;
    float m = -INFINITY, mc = -INFINITY, lsum = 0.f;   // running max of raw dots (and times c), running sum
    const int wave_first_tile_masked = min((int)((i0w + 31) / kBk) + 1, ntiles);   // tiles >= this are fully masked
    const int wave_first_diag = (int)(i0w / kBk);                     // tiles >= this need the mask

    if constexpr (kStaged) {
        wait_fills();
        __syncthreads();          // the Q rows are complete; the first step's barrier is what their place waits for
        static_for<0, 8>([&](auto n) {
            lds_issue_b128<0>(qB[decltype(n)::value], (uint32_t)(uintptr_t)staged(wq) + (uint32_t)(la.row_op[0] ^ (decltype(n)::value << 5)));
        });
        static_for<0, 8>([&](auto n) { lds_wait<0>(qB[decltype(n)::value]); });
    }

    // One key/value tile.  BUF is a compile-time buffer index, so every LDS address below is
    // a per-lane register plus an immediate offset.
    auto tile_step = [&](auto bufc, int jt) {
        constexpr int BUF = decltype(bufc)::value;
        constexpr int kOff = BUF * kStage, vOff = kOff + kTile;
        constexpr int nOff = (BUF ^ 1) * kStage;
        const int jn = jt + jstep;
        wait_fills();
        __syncthreads();          // tile jt is complete; nobody still reads the other buffer
        if (jn >= 0 && jn < ntiles) {
            fill_k(nOff, jn);
            fill_v(nOff, jn);
        }
        if (jt >= wave_first_tile_masked) return;         // every key of this tile is masked for this wave

        // S^T tile: rows = 64 keys (JB = 2 blocks of 32), cols = this wave's 32 queries.
        // item n = (jb = n%JB, kc = n/JB): one row operand of K, read 2 MFMAs ahead; two key blocks
        // alternate, so that no MFMA accumulates onto the result of the one issued right before it
        f32x16 s[JB];
        {
            bf16x8 ring[3];
            auto issue = [&](auto n, bf16x8 &slot) {
                constexpr int jb = decltype(n)::value % JB, kc = decltype(n)::value / JB;
                lds_issue_b128<jb * 8192 + kOff>(slot, row_addr[kc]);
            };
            lds_pipeline_prologue<8 * JB, 2, 1>(ring, issue);
            lds_pipeline_body<8 * JB, 2, 1>(ring, issue, [&](auto n, bf16x8 &slot) {
                constexpr int jb = decltype(n)::value % JB, kc = decltype(n)::value / JB;
                s[jb] = mfma32(slot, qB[kc], kc == 0 ? zero : s[jb]);
            });
        }
        // the first V^T operands are requested now: their latency hides behind the softmax
        TrSlot vring[3];
        auto v_issue = [&](auto n, TrSlot &slot) {
            constexpr int kj = decltype(n)::value / 4, cb = decltype(n)::value % 4;
            lds_issue_tr<kj * 4096 + vOff>(slot, tr_addr[cb][0], tr_addr[cb][1]);
        };
        lds_pipeline_prologue<8 * JB, 2, 2>(vring, v_issue);
        if (jt >= wave_first_diag) {                  // diagonal tile: mask keys j > i
            const int thr = (int)(i - (int64_t)jt * kBk) - 4 * half;    // key offset e' is visible iff e' <= thr
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (32 * jb + 8 * (e >> 2) + (e & 3) > thr) s[jb][e] = -INFINITY;
        }
        // P^T = exp2(c S^T - c m) against the running maximum m AS IT STANDS, rounded to bf16 for the second
        // contraction, and its row sums.  Softmax does not need the true maximum, only one that keeps the
        // exponentials in range: O and the logsumexp come out of (accO, lsum, m) the same whatever m is, and
        // fp32 and bf16 keep their relative precision at any exponent.  So the maximum of the tile is not
        // formed at all (16 three-input maxima, an exchange between the half-waves, and the exponentials
        // waiting for both) unless some row sum shows a score far above m, which also covers the first
        // tile, where m = -inf gives +inf or NaN here.
        bf16x8 pB[2 * JB];
        float psum0, psum1;
        auto exponentials = [&]() __attribute__((always_inline)) {
            psum0 = psum1 = 0.f;
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
#pragma unroll
                for (int e = 0; e < 16; e += 2) {
                    const f32x2 two = {__builtin_amdgcn_exp2f(fmaf(s[jb][e], c, -mc)), __builtin_amdgcn_exp2f(fmaf(s[jb][e + 1], c, -mc))};
                    psum0 += two[0];
                    psum1 += two[1];
                    const bf16x2 r = __builtin_convertvector(two, bf16x2);
                    pB[2 * jb + (e >> 3)][e & 7] = r[0];
                    pB[2 * jb + (e >> 3)][(e & 7) + 1] = r[1];
                }
        };
        exponentials();
        // not (sum <= bound) rather than sum > bound: a NaN sum takes the careful path too
        if (__builtin_amdgcn_ballot_w64(!(psum0 + psum1 <= kRescaleAbove)) != 0) {
            // three-input maxima, one chain per key block
            float mb[JB];
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) {
                mb[jb] = fmaxf(fmaxf(s[jb][0], s[jb][1]), s[jb][2]);
#pragma unroll
                for (int e = 3; e < 15; e += 2) mb[jb] = fmaxf(fmaxf(mb[jb], s[jb][e]), s[jb][e + 1]);
                mb[jb] = fmaxf(mb[jb], s[jb][15]);
            }
            const float mt = max_across_halves(fmaxf(mb[0], mb[1]));
            const float m_new = finite_max(m, mt);
            const float corr = __builtin_amdgcn_exp2f((m - m_new) * c);
            m = m_new;
            mc = scaled_max(m_new, c);
            lsum *= corr;
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                for (int e = 0; e < 16; ++e) accO[cb][e] *= corr;
            exponentials();
        }
        lsum += psum0 + psum1;

        // O^T += V^T P^T : A = V^T (transposed LDS read), B = P^T straight from the score registers.
        // item n = (kj = n/4, cb = n%4)
        lds_pipeline_body<8 * JB, 2, 2>(vring, v_issue, [&](auto n, TrSlot &slot) {
            constexpr int kj = decltype(n)::value / 4, cb = decltype(n)::value % 4;
            accO[cb] = mfma32(tr_operand(slot), pB[kj], accO[cb]);
        });
    };

    for (int n = 0; n < nsteps; n += 2) {
        tile_step(IntC<0>{}, jfirst + jstep * n);
        if (n + 1 < nsteps) tile_step(IntC<1>{}, jfirst + jstep * (n + 1));
    }

    const float ltot = add_across_halves(lsum);
    __bf16 *o = static_cast<__bf16 *>(a.o_out) + base + i * a.ss;
    float *lse = a.lse + ((int64_t)t.b * a.H + t.h) * a.S + i;
    if constexpr (KS == 1) {
        if (i < a.S) {
            store_acc_T(o, accO, 1.f / ltot, half);
            if (half == 0) *lse = (mc + __builtin_amdgcn_logf(ltot)) * kLn2;
        }
    } else {
        // The key groups of a row meet in LDS: every wave leaves its accumulators, (c m) and row sums; each
        // then combines 16/KS of the sixteen 4-value pieces of its rows over the groups.  A group that had
        // no tile has m = -inf and weighs exactly zero.
        LDS_AS f32x4 *pieces = (LDS_AS f32x4 *)lds;
        LDS_AS f32x2 *stats = (LDS_AS f32x2 *)(lds + kRing);
        __syncthreads();          // every wave has left the last LDS buffer
#pragma unroll
        for (int e = 0; e < 16; ++e)
            pieces[(wave * 16 + e) * 64 + lane] = f32x4{accO[e >> 2][4 * (e & 3)], accO[e >> 2][4 * (e & 3) + 1],
                                                        accO[e >> 2][4 * (e & 3) + 2], accO[e >> 2][4 * (e & 3) + 3]};
        if (half == 0) stats[wave * 32 + l32] = f32x2{mc, ltot};
        __syncthreads();
        float top = -INFINITY, total = 0.f, weight[KS];
        f32x2 st[KS];
#pragma unroll
        for (int g = 0; g < KS; ++g) {
            st[g] = stats[(g * QG + wq) * 32 + l32];
            top = fmaxf(top, st[g][0]);
        }
#pragma unroll
        for (int g = 0; g < KS; ++g) {
            weight[g] = __builtin_amdgcn_exp2f(st[g][0] - top);
            total += weight[g] * st[g][1];
        }
        if (i < a.S) {
            const float inv = 1.f / total;
#pragma unroll
            for (int n = 0; n < 16 / KS; ++n) {
                const int e = grp * (16 / KS) + n;
                f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int g = 0; g < KS; ++g) {
                    const f32x4 x = pieces[((g * QG + wq) * 16 + e) * 64 + lane];
#pragma unroll
                    for (int r = 0; r < 4; ++r) sum[r] += weight[g] * x[r];
                }
                store4(o + 8 * e + 4 * half, sum, inv);
            }
            if (grp == 0 && half == 0) *lse = (top + __builtin_amdgcn_logf(total)) * kLn2;
        }
    }
    }   // pass
}

// The end of the kernels whose eight waves share out the keys of 32 rows: every wave has left its accumulators as sixteen
// pieces and, per row, its (c m, row sum); each combines two pieces over the waves.  A wave without a tile has m = -inf
// and weighs exactly zero.
template <int CS = 1>
__device__ __forceinline__ void merge_waves(const AttnArgs &a, const LDS_AS f32x4 *pieces, const LDS_AS f32x2 *stats, int64_t base, int64_t stat,
                                            int64_t i, int wave, int l32, int half, int lane, int part = 0)
{
    constexpr int kOwn = CS == 1 ? 2 : 1, kPieces = 16 / CS;
    if (kOwn * wave >= kPieces) return;               // fewer pieces than waves
    f32x2 st[kFwdWaves];
    f32x4 x[kOwn][kFwdWaves];
#pragma unroll
    for (int g = 0; g < kFwdWaves; ++g) st[g] = stats[g * 32 + l32];
#pragma unroll
    for (int n = 0; n < kOwn; ++n)
#pragma unroll
        for (int g = 0; g < kFwdWaves; ++g) x[n][g] = pieces[(g * 16 + kOwn * wave + n) * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);                // all reads are on their way before the first is waited for
    float top = -INFINITY, total = 0.f, weight[kFwdWaves];
#pragma unroll
    for (int g = 0; g < kFwdWaves; ++g) top = fmaxf(top, st[g][0]);
#pragma unroll
    for (int g = 0; g < kFwdWaves; ++g) {
        weight[g] = __builtin_amdgcn_exp2f(st[g][0] - top);
        total += weight[g] * st[g][1];
    }
    if (i >= a.S) return;
    const float inv = 1.f / total;
    __bf16 *o = static_cast<__bf16 *>(a.o_out) + base + i * a.ss + 128 / CS * part;
#pragma unroll
    for (int n = 0; n < kOwn; ++n) {
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int g = 0; g < kFwdWaves; ++g)
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[r] += weight[g] * x[n][g][r];
        store4(o + 8 * (kOwn * wave + n) + 4 * half, sum, inv);
    }
    if (wave == 0 && half == 0 && part == 0) a.lse[stat + i] = (top + __builtin_amdgcn_logf(total)) * kLn2;
}

// 32 rows, the keys in eight: every wave works all rows against key tiles of 32 of its own, without a barrier in the sweep; one
// buffer, whose K half is refilled while V is worked and the other way round.  For sequences so short that a launch is
// little more than its start and its end (S = 640: 13000 of 17000 cycles before), and both are bound by what passes
// through the compute unit's 64 B per cycle from the L2, its 128 B per cycle into the LDS, and single waves' chains of
// instructions.  So the loads go out first and once (kernel arguments in one go; Q to the LDS, not to every wave's registers in
// pieces of 32 bytes), the set-up of addresses and accumulators comes behind them, and at the end a wave leaves its
// accumulators in its own buffer without waiting for the others.  us, columns in one part: S = 32 H = 2 6.0 -> 4.0, S = 640 H = 2 8.1 -> 6.8,
// B = 2 S = 2000 H = 3 18.1 -> 14.8, S = 3000 H = 4 20.6 -> 17.9.
// CS: the columns of O of a tile go to so many workgroups where units would be idle (column_parts, launch_plan.h): S = 32 H = 2 3.2, S = 640 H = 2 5.7.
template <int CS>
__global__ __launch_bounds__(64 * kFwdWaves, 2) void attn_fwd_bf16_short_kernel(AttnArgs a, Divisor heads, Divisor H)
{
    constexpr int NB = 4 / CS;    // blocks of 32 columns of O that the workgroup forms
    constexpr int T = 32, kTile = T * 256, kQ = kFwdWaves * 2 * kTile, kStats = kQ + kTile;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kStats + kFwdWaves * T * 8];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;   // [wave][K|V] tiles, then the Q rows, then (maximum, sum)
    load_args_at_once(a);

    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const auto [rank, hbp] = heads(blockIdx.x);       // CS parts of a head beside each other
    const int part = (int)(hbp % CS);
    const TileId t = head_of(hbp / CS, (int)((a.S + T - 1) / T) - 1 - (int)rank, H);
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh, row0 = (int64_t)t.tile * T;
    const __bf16 *k = static_cast<const __bf16 *>(a.k) + base;
    const __bf16 *v = static_cast<const __bf16 *>(a.v) + base;
    const int ntiles = t.tile + 1;                    // the last one is the diagonal
    const int ring = wave * 2 * kTile;
    const TileOffsets<1, T> toff = make_tile_offsets<1, SwzA, T>(a.ss, 0, lane);
    constexpr int kFills = TileOffsets<1, T>::kInstr;
    auto fill_k = [&](int jt, int to) { toff.fill(lds + to, k, a.ss, (int64_t)jt * T, a.S, 0); };
    auto fill_v = [&](int jt, int to) { toff.fill(lds + to + kTile, v, a.ss, (int64_t)jt * T, a.S, 0); };
    const TileOffsets<8, T> qoff = make_tile_offsets<8, SwzA, T>(a.ss, wave, lane);
    qoff.fill(lds + kQ, static_cast<const __bf16 *>(a.q) + base, a.ss, row0, a.S, wave);
    if (wave < ntiles) {
        fill_k(wave, ring);
        fill_v(wave, ring);
    } else {
        wait_fills();
        __builtin_amdgcn_s_barrier();                 // as below
    }
    __builtin_amdgcn_sched_barrier(0);
    const LaneAddr la = make_lane_addr(lane);
    // pieces of a row operand lie at address ^ (kc << 5), of a transposed one at address ^ (cb << 6)
    const uint32_t row = (uint32_t)(uintptr_t)lds + (uint32_t)la.row_op[0], own = (uint32_t)(uintptr_t)lds + (uint32_t)ring;
    uint32_t ka[8], va[NB][2];
#pragma unroll
    for (int kc = 0; kc < 8; ++kc) ka[kc] = (row + ring) ^ (kc << 5);
#pragma unroll
    for (int cb = 0; cb < NB; ++cb)
#pragma unroll
        for (int sec = 0; sec < 2; ++sec) va[cb][sec] = (own + (uint32_t)la.tr_op[0][sec]) ^ (uint32_t)((part * NB + cb) << 6);
    const float c = a.scale * kLog2e;
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 accO[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) accO[cb] = zero;
    float m = -INFINITY, mc = -INFINITY, lsum = 0.f;
    bf16x8 qB[8];                 // Q^T as B operand: lane = query row l32, 8 head-dim values per 16-wide chunk

#pragma clang loop unroll(disable)
    for (int jt = wave; jt < ntiles; jt += kFwdWaves) {
        const int jn = jt + kFwdWaves;
        const bool first = jt == wave;
        int to = ring;            // opaque: the addresses of the fills are formed where they are used, not in a long preamble of the loop
        asm volatile("" : "+s"(to));
        if (first) {              // in the loop, so that what the compiler moves in front of it is done while the loads are on their way
            wait_fills_but<2 * kFills>();
            __builtin_amdgcn_s_barrier();             // the Q rows are complete
            static_for<0, 8>([&](auto n) { lds_issue_b128<0>(qB[decltype(n)::value], (row + kQ) ^ (decltype(n)::value << 5)); });
            static_for<0, 8>([&](auto n) { lds_wait<0>(qB[decltype(n)::value]); });
        }
        wait_fills_but<kFills>();                     // K has landed; V, queued behind it, may still be on its way
        f32x16 s;                                     // S^T tile: rows = 32 keys, cols = the 32 queries
        {
            bf16x8 slots[3];
            auto issue = [&](auto n, bf16x8 &slot) { lds_issue_b128<0>(slot, ka[decltype(n)::value]); };
            lds_pipeline_prologue<8, 2, 1>(slots, issue);
            lds_pipeline_body<8, 2, 1>(slots, issue, [&](auto n, bf16x8 &slot) {
                constexpr int kc = decltype(n)::value;
                s = mfma32(slot, qB[kc], kc == 0 ? zero : s);
            });
        }
        if (jn < ntiles) {                            // K is used up: the next K tile comes while V is worked
            fill_k(jn, to);
            wait_fills_but<kFills>();
        } else {
            wait_fills();
        }
        TrSlot vring[3];
        auto v_issue = [&](auto n, TrSlot &slot) {
            constexpr int kj = decltype(n)::value / NB, cb = decltype(n)::value % NB;
            lds_issue_tr<kj * 4096 + kTile>(slot, va[cb][0], va[cb][1]);
        };
        lds_pipeline_prologue<2 * NB, 2, 2>(vring, v_issue);
        if (jt == ntiles - 1) {                       // diagonal tile: mask keys j > i
            int thr = l32 - 4 * half;
            asm volatile("" : "+v"(thr));
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (8 * (e >> 2) + (e & 3) > thr) s[e] = -INFINITY;
        }
        // against the running maximum as it stands (see attn_fwd_bf16_kernel); the first tile has none yet
        bf16x8 pB[2];
        float psum0 = INFINITY, psum1 = 0.f;
        auto exponentials = [&]() __attribute__((always_inline)) {
            psum0 = psum1 = 0.f;
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
                const f32x2 two = {__builtin_amdgcn_exp2f(fmaf(s[e], c, -mc)), __builtin_amdgcn_exp2f(fmaf(s[e + 1], c, -mc))};
                psum0 += two[0];
                psum1 += two[1];
                const bf16x2 r = __builtin_convertvector(two, bf16x2);
                pB[e >> 3][e & 7] = r[0];
                pB[e >> 3][(e & 7) + 1] = r[1];
            }
        };
        if (!first) exponentials();
        if (__builtin_amdgcn_ballot_w64(!(psum0 + psum1 <= kRescaleAbove)) != 0) {
            float mt = fmaxf(fmaxf(s[0], s[1]), s[2]);
#pragma unroll
            for (int e = 3; e < 15; e += 2) mt = fmaxf(fmaxf(mt, s[e]), s[e + 1]);
            const float m_new = finite_max(m, max_across_halves(fmaxf(mt, s[15])));
            if (!first) {
                const float corr = __builtin_amdgcn_exp2f((m - m_new) * c);
                lsum *= corr;
#pragma unroll
                for (int cb = 0; cb < NB; ++cb)
#pragma unroll
                    for (int e = 0; e < 16; ++e) accO[cb][e] *= corr;
            }
            m = m_new;
            mc = scaled_max(m_new, c);
            exponentials();
        }
        lsum += psum0 + psum1;
        // O^T += V^T P^T
        lds_pipeline_body<2 * NB, 2, 2>(vring, v_issue, [&](auto n, TrSlot &slot) {
            constexpr int kj = decltype(n)::value / NB, cb = decltype(n)::value % NB;
            accO[cb] = mfma32(tr_operand(slot), pB[kj], accO[cb]);
        });
        if (jn < ntiles) fill_v(jn, to);
    }

    // the waves' parts meet in LDS, as in attn_fwd_bf16_kernel; a wave's sixteen pieces take the place of its own buffer
    LDS_AS f32x4 *pieces = (LDS_AS f32x4 *)lds;
    LDS_AS f32x2 *stats = (LDS_AS f32x2 *)(lds + kStats);
    const float ltot = add_across_halves(lsum);
#pragma unroll
    for (int e = 0; e < 4 * NB; ++e)
        pieces[(wave * 16 + e) * 64 + lane] = f32x4{accO[e >> 2][4 * (e & 3)], accO[e >> 2][4 * (e & 3) + 1],
                                                    accO[e >> 2][4 * (e & 3) + 2], accO[e >> 2][4 * (e & 3) + 3]};
    if (half == 0) stats[wave * T + l32] = f32x2{mc, ltot};
    __syncthreads();
    merge_waves<CS>(a, pieces, stats, base, ((int64_t)t.b * a.H + t.h) * a.S, row0 + l32, wave, l32, half, lane, part);
}

// 64 rows, the keys in eight: every wave works all 64 rows (two blocks of 32) against key tiles of 32 of its own, so
// there is no barrier in the sweep and a K or V operand read feeds two MFMAs.  Q stays in LDS: the accumulators of 64
// rows leave no registers for it.  Bound, like all shapes below 256 rows, by what it streams per MFMA: as many bytes as
// two waves per 32-key tile behind a barrier did, which ran at 885 TFLOP/s on a full chip (S = 8192, H = 4: 87 -> 79 us).
// Its start and end are those of the 32-row kernel.
__global__ __launch_bounds__(64 * kFwdWaves, 2) void attn_fwd_bf16_own_kernel(AttnArgs a, Divisor heads, Divisor H)
{
    constexpr int kBq = 64, T = 32, kTile = T * 256, kQ = kFwdWaves * 2 * kTile, kStats = kQ + kBq * 256;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kStats + kFwdWaves * kBq * 8];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;   // [wave][K|V] tiles, then the Q rows, then (maximum, sum)
    load_args_at_once(a);

    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const TileId t = decode_tile(blockIdx.x, (int)((a.S + kBq - 1) / kBq), heads, H);
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh;
    const __bf16 *k = static_cast<const __bf16 *>(a.k) + base;
    const __bf16 *v = static_cast<const __bf16 *>(a.v) + base;
    const int64_t row0 = (int64_t)t.tile * kBq;
    const int ntiles = (int)((min(row0 + kBq, a.S) - 1) / T) + 1;
    const int ring = wave * 2 * kTile;

    const TileOffsets<8, kBq> qoff = make_tile_offsets<8, SwzA, kBq>(a.ss, wave, lane);
    qoff.fill(lds + kQ, static_cast<const __bf16 *>(a.q) + base, a.ss, row0, a.S, wave);
    const TileOffsets<1, T> toff = make_tile_offsets<1, SwzA, T>(a.ss, 0, lane);
    constexpr int kFills = TileOffsets<1, T>::kInstr;
    auto fill_k = [&](int jt, int to) { toff.fill(lds + to, k, a.ss, (int64_t)jt * T, a.S, 0); };
    auto fill_v = [&](int jt, int to) { toff.fill(lds + to + kTile, v, a.ss, (int64_t)jt * T, a.S, 0); };
    if (wave < ntiles) {
        fill_k(wave, ring);
        fill_v(wave, ring);
    }
    __builtin_amdgcn_sched_barrier(0);                // addresses and accumulators are set up while the loads are on their way
    const LaneAddr la = make_lane_addr(lane);
    const float c = a.scale * kLog2e;
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // pieces of a row operand lie at address ^ (kc << 5), of a transposed one at address ^ (cb << 6)
    const uint32_t own = (uint32_t)(uintptr_t)(lds + ring);
    uint32_t q_row = (uint32_t)(uintptr_t)(lds + kQ) + (uint32_t)la.row_op[0], k_row = own + (uint32_t)la.row_op[0];
    uint32_t v_lo = own + (uint32_t)la.tr_op[0][0], v_hi = own + (uint32_t)la.tr_op[0][1];
    asm volatile("" : "+v"(q_row), "+v"(k_row), "+v"(v_lo), "+v"(v_hi));
    f32x16 accO[2][4];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            accO[b][cb] = zero;
            asm volatile("" : "+v"(accO[b][cb]));
        }
    float m[2] = {-INFINITY, -INFINITY}, mc[2] = {-INFINITY, -INFINITY}, lsum[2] = {0.f, 0.f};
    if (wave < ntiles) wait_fills_but<2 * kFills>();
    else wait_fills();
    __builtin_amdgcn_s_barrier();                     // the Q rows are complete
    asm volatile("" ::: "memory");

    // Of the two waves of a SIMD the older one is served first and would end its keys a fifth of the sweep ahead; from here on the
    // younger one is, so that they end together and neither works alone (without : with, us: S = 8192 H = 4 79.1 : 76.7, S = 6000 H = 4
    // 49.8 : 47.7, S = 12000 H = 3 134.7 : 131.0, S = 4096 H = 4 27.4 : 27.4; the place, between a third and a half of the sweep, matters by 0.5 %).
    const int even_out = ntiles * 7 / 16;

    // one key tile against the row blocks from `F` on (the tile past the first block's diagonal is the second's alone)
    auto tile_step = [&](auto firstc, int jt) {
        constexpr int F = decltype(firstc)::value;
        const int jn = jt + kFwdWaves;
        const bool first = jt == wave;
        if (wave >= 4 && jt >= even_out) __builtin_amdgcn_s_setprio(1);
        uint32_t qa = q_row, ka = k_row, va = v_lo, vb = v_hi;
        int to = ring;
        asm volatile("" : "+v"(qa), "+v"(ka), "+v"(va), "+v"(vb), "+s"(to));   // the other addresses are formed where they are used
        wait_fills_but<kFills>();                     // K has landed; V, queued behind it, may still be on its way
        f32x16 s[2];
        {
            KqSlot<2 - F> kq[3];
            auto issue = [&](auto n, KqSlot<2 - F> &slot) {
                constexpr int kc = decltype(n)::value;
                lds_issue_b128<0>(slot.k, ka ^ (kc << 5));
                static_for<F, 2>([&](auto b) { lds_issue_b128<8192 * decltype(b)::value>(slot.q[decltype(b)::value - F], qa ^ (kc << 5)); });
            };
            lds_pipeline_prologue<8, 2, 3 - F>(kq, issue);
            lds_pipeline_body<8, 2, 3 - F>(kq, issue, [&](auto n, KqSlot<2 - F> &slot) {
                constexpr int kc = decltype(n)::value;
#pragma unroll
                for (int b = F; b < 2; ++b) s[b] = mfma32(slot.k, slot.q[b - F], kc == 0 ? zero : s[b]);
            });
        }
        if (jn < ntiles) {                            // K is used up: the next K tile comes while V is worked
            fill_k(jn, to);
            wait_fills_but<kFills>();
        } else {
            wait_fills();
        }
        TrSlot vring[3];
        auto v_issue = [&](auto n, TrSlot &slot) {
            constexpr int kj = decltype(n)::value / 4, cb = decltype(n)::value % 4;
            lds_issue_tr<kj * 4096 + kTile>(slot, va ^ (cb << 6), vb ^ (cb << 6));
        };
        lds_pipeline_prologue<8, 2, 2>(vring, v_issue);
        bf16x8 pB[2][2];
#pragma unroll
        for (int b = F; b < 2; ++b) {
            const int64_t i0 = row0 + 32 * b;
            if ((int64_t)jt * T >= i0) {              // diagonal tile: mask keys j > i
                int thr = l32 - 4 * half;
                asm volatile("" : "+v"(thr));
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (8 * (e >> 2) + (e & 3) > thr) s[b][e] = -INFINITY;
            }
            // against the running maximum as it stands (see attn_fwd_bf16_kernel); the first tile has none yet
            float psum0 = INFINITY, psum1 = 0.f;
            auto exponentials = [&]() __attribute__((always_inline)) {
                psum0 = psum1 = 0.f;
#pragma unroll
                for (int e = 0; e < 16; e += 2) {
                    const f32x2 two = {__builtin_amdgcn_exp2f(fmaf(s[b][e], c, -mc[b])), __builtin_amdgcn_exp2f(fmaf(s[b][e + 1], c, -mc[b]))};
                    psum0 += two[0];
                    psum1 += two[1];
                    const bf16x2 r = __builtin_convertvector(two, bf16x2);
                    pB[b][e >> 3][e & 7] = r[0];
                    pB[b][e >> 3][(e & 7) + 1] = r[1];
                }
            };
            if (!first) exponentials();
            if (__builtin_amdgcn_ballot_w64(!(psum0 + psum1 <= kRescaleAbove)) != 0) {
                float mb = fmaxf(fmaxf(s[b][0], s[b][1]), s[b][2]);
#pragma unroll
                for (int e = 3; e < 15; e += 2) mb = fmaxf(fmaxf(mb, s[b][e]), s[b][e + 1]);
                mb = fmaxf(mb, s[b][15]);
                const float m_new = finite_max(m[b], max_across_halves(mb));
                if (!first) {
                    const float corr = __builtin_amdgcn_exp2f((m[b] - m_new) * c);
                    lsum[b] *= corr;
#pragma unroll
                    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                        for (int e = 0; e < 16; ++e) accO[b][cb][e] *= corr;
                }
                m[b] = m_new;
                mc[b] = scaled_max(m_new, c);
                exponentials();
            }
            lsum[b] += psum0 + psum1;
        }
        lds_pipeline_body<8, 2, 2>(vring, v_issue, [&](auto n, TrSlot &slot) {
            constexpr int kj = decltype(n)::value / 4, cb = decltype(n)::value % 4;
#pragma unroll
            for (int b = F; b < 2; ++b) accO[b][cb] = mfma32(tr_operand(slot), pB[b][kj], accO[b][cb]);
        });
        if (jn < ntiles) fill_v(jn, to);
    };
    const int last_both = (int)(row0 / T);            // tiles past it hold no key of the first block's rows
    int jt = wave;
#pragma clang loop unroll(disable)
    for (; jt <= last_both; jt += kFwdWaves) tile_step(IntC<0>{}, jt);
    if (jt < ntiles) tile_step(IntC<1>{}, jt);

    // the waves' parts of a block of rows meet in LDS, one block after the other; those of the first take the place of the wave's own buffer
    LDS_AS f32x4 *pieces = (LDS_AS f32x4 *)lds;
    LDS_AS f32x2 *stats = (LDS_AS f32x2 *)(lds + kStats);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int64_t i = row0 + 32 * b + l32;
        const float ltot = add_across_halves(lsum[b]);
        if (b == 1) __syncthreads();                  // every wave has read the first block's
#pragma unroll
        for (int e = 0; e < 16; ++e)
            pieces[(wave * 16 + e) * 64 + lane] = f32x4{accO[b][e >> 2][4 * (e & 3)], accO[b][e >> 2][4 * (e & 3) + 1],
                                                        accO[b][e >> 2][4 * (e & 3) + 2], accO[b][e >> 2][4 * (e & 3) + 3]};
        if (half == 0) stats[wave * 32 + l32] = f32x2{mc[b], ltot};
        __syncthreads();
        merge_waves(a, pieces, stats, base, ((int64_t)t.b * a.H + t.h) * a.S, i, wave, l32, half, lane);
    }
}

}  // namespace

hipError_t launch_attn_fwd_bf16(const AttnArgs &a, hipStream_t st)
{
    const int64_t heads = (int64_t)a.H * a.B;
    const TileChoice &c = fwd_plan(a.S, heads);
    const int order = tile_order(c.rows, c.order);
    const int64_t blocks = order_grid((a.S + c.rows - 1) / c.rows, heads, order);
    if (blocks > kMaxBlocks)
        return launch_fewer_heads(a, sizeof(__bf16), blocks, kMaxBlocks, [&](const AttnArgs &part) { return launch_attn_fwd_bf16(part, st); });
    switch (c.rows) {
    case 32: {
        const int parts = a.o_out == a.q ? 1 : column_parts(blocks);         // in place of Q: another part may not have read it yet
        auto launch = [&](auto kernel) { return launch_blocks(kernel, blocks * parts, st, a, Divisor(heads * parts), Divisor(a.H)); };
        return parts == 4 ? launch(attn_fwd_bf16_short_kernel<4>) : parts == 2 ? launch(attn_fwd_bf16_short_kernel<2>)
                                                                              : launch(attn_fwd_bf16_short_kernel<1>);
    }
    case 64: return launch_blocks(attn_fwd_bf16_own_kernel, blocks, st, a, Divisor(heads), Divisor(a.H));
    case 128: return launch_blocks(attn_fwd_bf16_kernel<4>, blocks, st, a, order);
    default: return c.waves == 4 ? launch_attn_fwd_bf16_long(a, order, blocks, st) : launch_blocks(attn_fwd_bf16_kernel<8>, blocks, st, a, order);
    }
}

}  // namespace memo

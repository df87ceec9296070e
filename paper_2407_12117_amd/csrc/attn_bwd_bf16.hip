// bf16 causal attention backward for gfx950 (CDNA4), head dim 128, on v_mfma_f32_16x16x32_bf16.
//
// What is computed (Section 2.1.3 of the paper): with P = exp(S - LSE) re-formed from Q, K and the
// logsumexp of the forward, dV = P^T dO, dP = dO V^T, dS = P (dP - D), dK = scale dS^T Q,
// dQ = scale dS K, D_i = dO_i . O_i.  Two kernels: a key-stationary one for dK, dV and a
// query-stationary one for dQ; no atomics, so the gradients are bit-reproducible.  S and dP are
// formed in both (7 contractions for the method's 5): the alternative, one kernel that adds its dQ
// partials to global memory, needs 16 KB of fp32 atomic adds per 32-query step of a 256-key
// workgroup, and this chip retires those at 1.4 TB/s: 2.5 times slower than the dQ kernel they
// would replace.
//
// Why this MFMA shape: the chip is power-limited on random data and the 16x16x32 instruction
// spends less energy per flop than the 32x32x16 one (an MFMA-only loop sustains about an eighth
// more flops per second with it); the wave tiles, and with them the bytes read from LDS per flop,
// are what a 32x32x16 version has.  The backward kernels have no per-row reductions, so the
// smaller accumulator blocks cost no extra vector arithmetic (measured against a 32x32x16 version
// of both kernels: 7 to 10 % faster on N(0,1) inputs).
//
// Operand conventions of the 16x16x32 MFMA, D = A(16xK32) * B(K32x16), lane = 16*g4 + l16:
//   A : lane holds row l16, k = 8*g4 .. 8*g4+7      (8 bf16)
//   B : lane holds col l16, k = 8*g4 .. 8*g4+7      (8 bf16)
//   D : lane holds col l16, rows 4*g4 + r for register r (4 fp32)
// As in the forward kernel every score block is produced so that its fp32 D registers, rounded
// to bf16, are directly the B operand of the next contraction: two D blocks stacked along the
// rows give a lane the 8 contraction slots  e <-> row 16*(e/4) + 4*g4 + e%4  of a 32-row chunk,
// and the matching A operand is two transposed LDS reads (ds_read_b64_tr_b16) of rows
// 4*g4 .. 4*g4+3 and 16 + 4*g4 .. of that chunk.  LDS tiles are rows of 256 bytes (64 per K/V tile
// of the dQ kernel, 32 per Q/dO tile of the dK/dV kernel) with the SwzB chunk swizzle
// (bf16_tiles.h); all operand reads are issued by hand ahead of their MFMAs.
#include "bf16_tiles.h"

namespace memo {
namespace {

constexpr int kDqWaves = 8;
constexpr f32x4 kZero4 = {0.f, 0.f, 0.f, 0.f};

// sum over the G groups of piece e of group member m (wave g * M + m), pieces as [wave][16][lane]
template <int G, int M>
__device__ __forceinline__ f32x4 sum_pieces(const LDS_AS f32x4 *pieces, int m, int e, int lane)
{
    f32x4 sum = pieces[(m * 16 + e) * 64 + lane];
#pragma unroll
    for (int g = 1; g < G; ++g) {
        const f32x4 x = pieces[((g * M + m) * 16 + e) * 64 + lane];
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[r] += x[r];
    }
    return sum;
}

// ============================================================================ backward: dQ
// 256 rows of longer sequences go out in four waves (attn_bwd_long_bf16.hip); this is for shorter ones and smaller workgroups.
// Workgroup: 8 waves, 32 query rows per wave (two blocks of 16); keys/values streamed in tiles
// of 64 through a double-buffered LDS ring filled asynchronously (one barrier per tile).
//   S^T = K Q^T, dP^T = V dO^T - D   (A = K / V rows from LDS, B = Q^T / dO^T from registers)
//   dS^T = exp(S^T - LSE) dP^T        (lane = query, registers = keys)
//   dQ^T += K^T dS^T                  (A = K^T, transposed LDS read; B = dS^T from registers)
// A tile is worked in halves of 32 keys so that the element-wise work of one half can run
// under the MFMAs of the other wave of the SIMD.
// Smaller workgroups for short sequences, as in the forward (attn_bf16.hip): QG query groups of 32 rows and
// 8 / QG key groups, each with its own ring of T-row tiles, their dQ added up at the end.  Rates of 256 / 128 / 64
// rows on a full chip (S = 128K, H = 4): 1383 / 1319 / 1138 TFLOP/s of its three contractions.  (32 rows with the
// keys in eight, V in registers and Q in LDS: 704, ahead of 64 rows only below S = 2000 and never in
// the joint launch below; not kept.)
template <int QG, int T>
struct DqShape {
    static constexpr int KS = kDqWaves / QG, kTile = T * 256;     // bytes of one K or V tile
    static constexpr int kStage = 2 * kTile, kGroup = 2 * kStage, kLds = KS * kGroup;
    static_assert(KS == 1 || kLds == 8 * 16384, "the sum over the key groups lays eight accumulator sets over the ring");
};

template <int QG, int T, typename Find>       // find(number of tiles): the workgroup's work
__device__ __forceinline__ void dq_rows(const AttnArgs &a, LDS_AS unsigned char *lds, Find &&find)
{
    using Shape = DqShape<QG, T>;
    constexpr int KS = Shape::KS, kTile = Shape::kTile, kStage = Shape::kStage, kGroup = Shape::kGroup;
    constexpr int kBq = 32 * QG, kBk = T;
    // lds: [key group][buf][K|V] tiles

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wq = wave % QG, grp = wave / QG;        // query group, key group
    const int64_t nqt = (a.S + kBq - 1) / kBq;
    const PairId t = find(nqt);                       // one query tile
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh;
    const __bf16 *q = static_cast<const __bf16 *>(a.q) + base;
    const __bf16 *k = static_cast<const __bf16 *>(a.k) + base;
    const __bf16 *v = static_cast<const __bf16 *>(a.v) + base;
    const __bf16 *g = static_cast<const __bf16 *>(a.d_o) + base;
    const int64_t stat = ((int64_t)t.b * a.H + t.h) * a.S;
    const LdsAddr16 ad = make_lds_addr16(lds + grp * kGroup, lane);
    const float c = a.scale * kLog2e;

    const int64_t row0 = t.first * kBq, i0w = row0 + 32 * wq;
    const int64_t last_row = min(row0 + kBq, a.S) - 1;
    const int ntiles = (int)(last_row / kBk) + 1, nsteps = (ntiles + KS - 1) / KS;
    // step n of a key group works tile KS * n + grp
    // K and V rows have the same strides: one set of per-lane offsets serves both fills
    const TileOffsets<QG, T> toff = make_tile_offsets<QG, SwzB, T>(a.ss, wq, lane);
    auto fill = [&](int off, int jt) {
        LDS_AS unsigned char *dst = lds + grp * kGroup + off;
        fill_tile_at<SwzB>(dst, toff, k, a.ss, (int64_t)jt * kBk, a.S, wq, lane);
        fill_tile_at<SwzB>(dst + kTile, toff, v, a.ss, (int64_t)jt * kBk, a.S, wq, lane);
    };
    // Workgroups whose key groups all need the same Q and dO rows bring them in once, as whole rows, in the place of the buffers that the
    // second tiles take: to each wave's registers straight from memory, 64 bytes of a row at a time, they cost a unit 5000 cycles.
    constexpr bool kStaged = QG < 8;
    constexpr int kBlocks = kStage / (32 * 256);      // 32-row blocks in one such buffer
    static_assert(!kStaged || KS * kBlocks >= 2 * QG, "room for the Q and dO rows");
    auto staged = [&](int block) { return lds + block / kBlocks * kGroup + kStage + block % kBlocks * 32 * 256; };
    if constexpr (kStaged) {
        const TileOffsets<8, 32> qoff = make_tile_offsets<8, SwzB, 32>(a.ss, wave, lane);
#pragma unroll
        for (int blk = 0; blk < QG; ++blk) {
            qoff.fill(staged(2 * blk), q, a.ss, row0 + 32 * blk, a.S, wave);
            qoff.fill(staged(2 * blk + 1), g, a.ss, row0 + 32 * blk, a.S, wave);
        }
    }
    if (grp < ntiles) fill(0, grp);

    // Q^T and dO^T as B operands: lane = query 16*qt + l16, 8 head-dim values per 32-wide k step
    bf16x8 qB[2][4], gB[2][4];
    float lse2[2];
    f32x4 neg_d[2];               // -D_i in all four registers: dP^T starts from it
    int64_t iq[2];
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
        const int64_t i = i0w + 16 * qt + l16;
        iq[qt] = i < a.S ? i : a.S - 1;               // rows past S are computed and never stored
        if constexpr (!kStaged) {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                qB[qt][kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(q + iq[qt] * a.ss + 32 * kk + 8 * g4));
                gB[qt][kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(g + iq[qt] * a.ss + 32 * kk + 8 * g4));
            }
        }
        lse2[qt] = a.lse[stat + iq[qt]] * kLog2e;
        const float nd = -a.delta[stat + iq[qt]];
        neg_d[qt] = f32x4{nd, nd, nd, nd};
    }
    f32x4 accQ[8][2];             // dQ^T: [head-dim block of 16][query block]; lane = query, rows = head dim
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) accQ[dt][qt] = kZero4;
    const int wave_first_tile_masked = min((int)((i0w + 31) / kBk) + 1, ntiles);   // tiles >= this are fully masked
    const int wave_first_diag = (int)(i0w / kBk);                     // tiles >= this need the mask
    if constexpr (kStaged) {
        wait_fills();
        __syncthreads();          // the Q and dO rows are complete; the first step's barrier is what their place waits for
        const uint32_t at = ad.row16[0] - (uint32_t)(uintptr_t)(lds + grp * kGroup);
        static_for<0, 8>([&](auto n) {
            constexpr int qt = decltype(n)::value / 4, kk = decltype(n)::value % 4;
            lds_issue_b128<4096 * qt>(qB[qt][kk], (uint32_t)(uintptr_t)staged(2 * wq) + (at ^ (kk << 6)));
            lds_issue_b128<4096 * qt>(gB[qt][kk], (uint32_t)(uintptr_t)staged(2 * wq + 1) + (at ^ (kk << 6)));
        });
        static_for<0, 8>([&](auto n) {
            lds_wait<0>(qB[decltype(n)::value / 4][decltype(n)::value % 4]);
            lds_wait<0>(gB[decltype(n)::value / 4][decltype(n)::value % 4]);
        });
    }

    auto tile_step = [&](auto bufc, int jt) {
        constexpr int BUF = decltype(bufc)::value;
        constexpr int kOff = BUF * kStage, vOff = kOff + kTile;
        constexpr int nOff = (BUF ^ 1) * kStage;
        wait_fills();
        __syncthreads();          // tile jt is complete; nobody still reads the other buffer
        const int jn = jt + KS;
        if (jn < ntiles) fill(nOff, jn);
        if (jt >= wave_first_tile_masked) return;
        const bool diag = jt >= wave_first_diag;
        static_for<0, T / 32>([&](auto hc) {
            constexpr int h = decltype(hc)::value;    // keys 32*h .. 32*h+31 of the tile: key blocks 2h, 2h+1
            f32x4 s[2][2], dp[2][2];                  // [key block of the half][query block]
            {
                // item n = (k step n/4, key block (n/2)%2, K or V = n%2): one row operand, two MFMAs
                bf16x8 ring[3];
                auto issue = [&](auto n, bf16x8 &slot) {
                    constexpr int kk = decltype(n)::value / 4, kt = (decltype(n)::value / 2) % 2, isv = decltype(n)::value % 2;
                    lds_issue_b128<(2 * h + kt) * 4096 + (isv ? vOff : kOff)>(slot, ad.row16[kk]);
                };
                lds_pipeline_prologue<16, 2, 1>(ring, issue);
                lds_pipeline_body<16, 2, 1>(ring, issue, [&](auto n, bf16x8 &slot) {
                    constexpr int kk = decltype(n)::value / 4, kt = (decltype(n)::value / 2) % 2, isv = decltype(n)::value % 2;
#pragma unroll
                    for (int qt = 0; qt < 2; ++qt) {
                        if constexpr (isv) dp[kt][qt] = mfma16(slot, gB[qt][kk], kk == 0 ? neg_d[qt] : dp[kt][qt]);
                        else s[kt][qt] = mfma16(slot, qB[qt][kk], kk == 0 ? kZero4 : s[kt][qt]);
                    }
                });
            }
            // dQ^T += K^T dS^T over the 32 keys of the half: item n = head-dim block dt, one transposed
            // operand (two reads), two MFMAs; the first operands are requested before the VALU work
            TrSlot kring[3];
            auto k_issue = [&](auto n, TrSlot &slot) {
                constexpr int dt = decltype(n)::value;
                lds_issue_tr_pair<h * 8192 + kOff>(slot, ad.tr16[dt]);
            };
            lds_pipeline_prologue<8, 2, 2>(kring, k_issue);
            if (diag) {           // mask keys beyond the query, behind a wave-uniform branch
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                    for (int qt = 0; qt < 2; ++qt) {
                        // key offset in the tile 32h + 16kt + 4g4 + r is visible iff <= query offset
                        const int thr = (int)(i0w + 16 * qt + l16 - (int64_t)jt * kBk) - (32 * h + 16 * kt + 4 * g4);
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (r > thr) s[kt][qt][r] = -INFINITY;
                    }
            }
            bf16x8 dsB[2];
#pragma unroll
            for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float p = __builtin_amdgcn_exp2f(fmaf(s[kt][qt][r], c, -lse2[qt]));
                        s[kt][qt][r] = p * dp[kt][qt][r];           // dS (dp already holds dP - D_i)
                    }
                dsB[qt] = pack44(s[0][qt], s[1][qt]);
            }
            lds_pipeline_body<8, 2, 2>(kring, k_issue, [&](auto n, TrSlot &slot) {
                constexpr int dt = decltype(n)::value;
#pragma unroll
                for (int qt = 0; qt < 2; ++qt) accQ[dt][qt] = mfma16(tr_operand(slot), dsB[qt], accQ[dt][qt]);
            });
        });
    };
    for (int n = 0; n < nsteps; n += 2) {
        tile_step(IntC<0>{}, grp + KS * n);
        if (n + 1 < nsteps) tile_step(IntC<1>{}, grp + KS * (n + 1));
    }
    __bf16 *dq = static_cast<__bf16 *>(a.dq) + base + (i0w + l16) * a.ss + 4 * g4;
    if constexpr (KS == 1) {
#pragma unroll
        for (int qt = 0; qt < 2; ++qt)
            if (i0w + 16 * qt + l16 < a.S) {
#pragma unroll
                for (int dt = 0; dt < 8; ++dt) store4(dq + 16 * qt * a.ss + 16 * dt, accQ[dt][qt], a.scale);
            }
    } else {
        // piece 8 qt + dt of every wave goes through LDS; each wave adds up 16/KS pieces of its rows over the key groups
        LDS_AS f32x4 *pieces = (LDS_AS f32x4 *)lds;
        __syncthreads();          // every wave has left the last LDS buffer
#pragma unroll
        for (int qt = 0; qt < 2; ++qt)
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) pieces[(wave * 16 + 8 * qt + dt) * 64 + lane] = accQ[dt][qt];
        __syncthreads();
#pragma unroll
        for (int n = 0; n < 16 / KS; ++n) {
            const int e = grp * (16 / KS) + n, qt = e >> 3, dt = e & 7;
            const f32x4 sum = sum_pieces<KS, QG>(pieces, wq, e, lane);
            if (i0w + 16 * qt + l16 < a.S) store4(dq + 16 * qt * a.ss + 16 * dt, sum, a.scale);
        }
    }
}

// ============================================================================ backward: dK, dV
// 256 keys of longer sequences go out in four waves (attn_bwd_long_bf16.hip); this is for shorter ones and smaller workgroups.
// Workgroup (KG = 8): 8 waves, 256 key rows whose K and V stay in LDS for the workgroup's lifetime (128 KB);
// queries streamed in tiles of 32 through a double-buffered ring (Q and dO rows, 16 KB per stage,
// one barrier per tile): LDS is full to the byte (160 KB).  The bytes streamed per (query, key) pair
// are (Q + dO bytes per query) / (keys per workgroup): 256 resident keys halve the L2 -> LDS and the
// HBM traffic of a 128-key workgroup for the same work per wave and step.
// Wave w owns key rows 32*w .. 32*w+31 and all 32 queries of every tile, as 2 x 2 blocks of 16, and
// runs all four contractions on its block, so nothing passes between waves:
//   S = Q K^T - LSE/scale, dP = dO V^T - D   (both operands from LDS; lane = key, registers = queries;
//                                             -LSE_i/scale and -D_i are the initial accumulators)
//   P = exp2(scale log2e S), dS = P dP
//   dV^T += dO^T P,  dK^T += Q^T dS  (A = transposed LDS reads over the tile's 32 queries,
//                                     B = P / dS from registers; lane = key, rows = head dim)
// No atomics, no reduction across waves: every wave writes the dK and dV rows of its own keys.
// Smaller workgroups for short sequences: KG = 4 or 2 key blocks, and 8 / KG query groups that take every
// 8 / KG-th query tile through rings of their own; their dV, then their dK, are added up through LDS at the end.
// Rates of 256 / 128 / 64 keys on a full chip (S = 128K, H = 4): 1264 / 1237 / 1186 TFLOP/s of its four contractions.
// The row statistics do not pass through LDS (there is no room left): see "Row statistics" below.
constexpr int kBq = 32;
constexpr int kStageBytes = 2 * kBq * 256;            // Q rows, then dO rows
constexpr int kKvBlockBytes = 2 * 32 * 256;           // per wave: its 32 K rows, then its 32 V rows

struct QuadSlot { bf16x8 a0, a1, b0, b1; };

template <int N>
__device__ __forceinline__ void lds_wait(QuadSlot &x)
{
    static_assert(N >= 0 && N <= 15, "lgkmcnt range");
    asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(x.a0), "+v"(x.a1), "+v"(x.b0), "+v"(x.b1) : "n"(N));
}

template <int KG>
struct DkdvShape {
    static constexpr int QS = 8 / KG;
    static constexpr int kGroup = 2 * kStageBytes, kKvOff = QS * kGroup;
    static constexpr int kLds = kKvOff + KG * kKvBlockBytes;      // 160, 128, 160 KB for KG = 8, 4, 2
    static_assert(QS == 1 || kLds >= 8 * 16384, "the sum over the query groups lays eight accumulator sets over it");
};

template <int KG, typename Find>
__device__ __forceinline__ void dkdv_rows(const AttnArgs &a, LDS_AS unsigned char *lds, Find &&find)
{
    using Shape = DkdvShape<KG>;
    constexpr int QS = Shape::QS, kKvOff = Shape::kKvOff, kBwdBk = 32 * KG;
    // lds: [query group][stage][Q|dO] tiles, then [key block][K|V] rows

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave % KG, grp = wave / KG;        // key block, query group
    const int64_t nkt = (a.S + kBwdBk - 1) / kBwdBk;
    const PairId t = find(nkt);                       // one key tile
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh;
    const __bf16 *q = static_cast<const __bf16 *>(a.q) + base;
    const __bf16 *g = static_cast<const __bf16 *>(a.d_o) + base;
    const float *lse = a.lse + ((int64_t)t.b * a.H + t.h) * a.S;
    const float *dlt = a.delta + ((int64_t)t.b * a.H + t.h) * a.S;
    const int nit = (int)((a.S + kBq - 1) / kBq);
    const float c = a.scale * kLog2e, neg_inv_scale = -1.f / a.scale;
    // a 32-row ring tile is eight fill instructions, 8 / KG per wave of the query group
    constexpr int NF = 8 / KG;
    const TileOffsets<KG, kBq> toff = make_tile_offsets<KG, SwzB, kBq>(a.ss, wk, lane);
    const int64_t tile_step_bytes = kBq * a.ss * 2;
    LDS_AS unsigned char *ring_base = lds + grp * Shape::kGroup;
    const LdsAddr16 ad = make_lds_addr16(ring_base, lane);

    // The tile walks the query tiles downwards from the last one to its diagonal: the workgroups of an XCD then read the same
    // Q/dO rows at about the same time.
    const int64_t col0 = t.first * kBwdBk, j0w = col0 + 32 * wk;
    const int it0 = (int)(col0 / kBq);                // the tile's first query tile (its diagonal)
    // the sweep's query tiles it_first, it_first - 1, ...: query group grp takes the positions grp, grp + QS, ...
    const int it_first = nit - 1, npos = nit - it0, nsteps = (npos + QS - 1) / QS;
    {   // resident K and V rows (rows past S repeat row S-1, never stored): 32-row pieces, 8 waves x 4 rows
        const __bf16 *kp = static_cast<const __bf16 *>(a.k) + base;
        const __bf16 *vp = static_cast<const __bf16 *>(a.v) + base;
        int ln = lane;            // opaque copy: these addresses are formed here, once per sweep, not kept in registers
        asm volatile("" : "+v"(ln));
#pragma unroll
        for (int blk = 0; blk < KG; ++blk) {
            fill_ragged_tile<8, SwzB, 32>(lds + kKvOff + blk * kKvBlockBytes, kp, a.ss, col0 + 32 * blk, a.S, wave, ln);
            fill_ragged_tile<8, SwzB, 32>(lds + kKvOff + blk * kKvBlockBytes + 8192, vp, a.ss, col0 + 32 * blk, a.S, wave, ln);
        }
    }
    auto fill_tile = [&](LDS_AS unsigned char *dst, const __bf16 *src, int64_t r0) {
        fill_tile_at<SwzB>(dst, toff, src, a.ss, r0, a.S, wk, lane);
    };
    if (grp < npos) {
        fill_tile(ring_base, q, (int64_t)(it_first - grp) * kBq);
        fill_tile(ring_base + kBq * 256, g, (int64_t)(it_first - grp) * kBq);
    }

    f32x4 accV[8][2], accK[8][2];                     // dV^T, dK^T: [head-dim block][key block]; lane = key
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) accV[dt][kt] = accK[dt][kt] = kZero4;

    // Row statistics.  The accumulator registers of lane 16*g4 + l16 stand for queries 4*g4 .. 4*g4+3 of a
    // 16-query block, so the lane needs -LSE_i/scale and -D_i of those four queries as the initial value
    // of S and dP: sixteen values per step.  Fetching them as such (from global memory or through LDS)
    // returns 64 bytes per lane and step to the registers, which costs the step 6 %.  Instead lane l
    // loads ONE value per block and statistic, that of query 4*(l/16) + l%4, and a 4x4x1 fp32 MFMA
    // (sixteen independent 4x4 outer products, block = l/4) spreads it: with B = the scaling constant in
    // every lane, register r of lane l receives A of lane 4*(l/4) + r, which is query 4*(l/16) + r.
    // The product is one fp32 multiplication, the same rounding as a v_mul.  Rows past S: LSE = +inf
    // makes their P exactly zero.
    const int stat_lane = 4 * g4 + (lane & 3);
    struct RawStats { float l[2], d[2]; };
    auto load_stats = [&](int it) {
        RawStats r;
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
            const int64_t row = (int64_t)it * kBq + 16 * qt + stat_lane;
            r.l[qt] = row < a.S ? lse[row] : INFINITY;
            r.d[qt] = row < a.S ? dlt[row] : 0.f;
        }
        return r;
    };
    f32x4 nl[2], nd[2];           // -LSE_i/scale and -D_i of the tile about to be worked
    auto spread_stats = [&](const RawStats &r) {
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
            nl[qt] = __builtin_amdgcn_mfma_f32_4x4x1f32(r.l[qt], neg_inv_scale, kZero4, 0, 0, 0);
            nd[qt] = __builtin_amdgcn_mfma_f32_4x4x1f32(r.d[qt], -1.f, kZero4, 0, 0, 0);
        }
    };
    RawStats raw = load_stats(it_first - min(grp, npos - 1));

    uint32_t kv_row[4];                               // this wave's K rows; its V rows are 8192 bytes further
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) kv_row[kk] = ad.row16[kk] + (uint32_t)(kKvOff - grp * Shape::kGroup + wk * kKvBlockBytes);
    const uint32_t (&q_row)[4] = ad.row16;            // query rows of ring stage 0 (Q part)
    const uint32_t (&q_tr)[8] = ad.tr16;

    auto tile_step = [&](auto bufc, int pos) {
        constexpr int BUF = decltype(bufc)::value;
        constexpr int qOff = BUF * kStageBytes, gOff = qOff + kBq * 256;
        constexpr int nOff = (BUF ^ 1) * kStageBytes;
        wait_fills();
        __syncthreads();          // tile `it` is complete; the other stage is free
        const int it = it_first - pos, itn = it - QS;
        const bool more = pos + QS < npos;
        const int64_t rn = (int64_t)itn * kBq;        // first query of the group's next tile (if there is one)
        const int64_t i0 = (int64_t)it * kBq;         // first query of the tile
        const RawStats raw_now = raw;
        if (more) raw = load_stats(itn);              // four registers, used a whole step from now
        // else there is no tile for this group, or all 32 queries precede this wave's keys
        const bool active = pos < npos && i0 + 31 >= j0w;
        // A full next tile is fetched by fill instructions queued one at a time between the
        // MFMAs below; the ragged last tile (and a wave with nothing to compute) queues them here.
        const bool spread = more && active && rn + kBq <= a.S;
        if (more && !spread) {
            fill_tile(ring_base + nOff, q, rn);
            fill_tile(ring_base + nOff + kBq * 256, g, rn);
        }
        const char *nq = reinterpret_cast<const char *>(q) + (int64_t)itn * tile_step_bytes;
        const char *ng = reinterpret_cast<const char *>(g) + (int64_t)itn * tile_step_bytes;
        auto fill_part = [&](auto pc) {
            constexpr int part = decltype(pc)::value;
            if (!spread) return;
            fill_full_tile_part(ring_base + nOff + (part / NF) * kBq * 256, toff, part % NF, part < NF ? nq : ng, wk);
        };
        if (active) {
            spread_stats(raw_now);
            const bool diag = i0 < j0w + 31;
            f32x4 s[2][2], dp[2][2];                  // [query block][key block]; register r = query 16*qt + 4*g4 + r
            {
                // item n = (k step n/2, S or dP = n%2): the Q (dO) rows of both query blocks and the
                // K (V) rows of both key blocks, four MFMAs
                QuadSlot ring[2];
                auto issue = [&](auto n, QuadSlot &slot) {
                    constexpr int kk = decltype(n)::value / 2, which = decltype(n)::value % 2;
                    lds_issue_b128<(which ? gOff : qOff)>(slot.a0, q_row[kk]);
                    lds_issue_b128<(which ? gOff : qOff) + 4096>(slot.a1, q_row[kk]);
                    lds_issue_b128<(which ? 8192 : 0)>(slot.b0, kv_row[kk]);
                    lds_issue_b128<(which ? 8192 : 0) + 4096>(slot.b1, kv_row[kk]);
                };
                lds_pipeline_prologue<8, 1, 4>(ring, issue);
                lds_pipeline_body<8, 1, 4>(ring, issue, [&](auto n, QuadSlot &slot) {
                    constexpr int kk = decltype(n)::value / 2, which = decltype(n)::value % 2;
                    if constexpr (which == 0) {
                        s[0][0] = mfma16(slot.a0, slot.b0, kk == 0 ? nl[0] : s[0][0]);
                        s[0][1] = mfma16(slot.a0, slot.b1, kk == 0 ? nl[0] : s[0][1]);
                        s[1][0] = mfma16(slot.a1, slot.b0, kk == 0 ? nl[1] : s[1][0]);
                        s[1][1] = mfma16(slot.a1, slot.b1, kk == 0 ? nl[1] : s[1][1]);
                    } else {
                        dp[0][0] = mfma16(slot.a0, slot.b0, kk == 0 ? nd[0] : dp[0][0]);
                        dp[0][1] = mfma16(slot.a0, slot.b1, kk == 0 ? nd[0] : dp[0][1]);
                        dp[1][0] = mfma16(slot.a1, slot.b0, kk == 0 ? nd[1] : dp[1][0]);
                        dp[1][1] = mfma16(slot.a1, slot.b1, kk == 0 ? nd[1] : dp[1][1]);
                    }
                    // 2 NF fills spread over the eight items
                    constexpr int done = decltype(n)::value + 1;
                    if constexpr (done * 2 * NF % 8 == 0) fill_part(IntC<done * 2 * NF / 8 - 1>{});
                });
            }
            // item n < 8: dV^T head-dim block n, A = dO^T; n >= 8: dK^T block n - 8, A = Q^T
            TrSlot tring[3];
            auto t_issue = [&](auto n, TrSlot &slot) {
                constexpr int dt = decltype(n)::value % 8;
                constexpr int off = decltype(n)::value < 8 ? gOff : qOff;
                lds_issue_tr_pair<off>(slot, q_tr[dt]);
            };
            lds_pipeline_prologue<16, 2, 2>(tring, t_issue);
            if (diag) {           // the causal mask, behind a wave-uniform branch
#pragma unroll
                for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt) {
                        // query offset 16qt + 4g4 + r of the tile is visible to key j iff it is >= j - i0
                        const int thr = (int)(j0w + 16 * kt + l16 - i0) - (16 * qt + 4 * g4);
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (r < thr) s[qt][kt][r] = -INFINITY;
                    }
            }
#pragma unroll
            for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float p = __builtin_amdgcn_exp2f(s[qt][kt][r] * c);   // s already holds S - LSE_i/scale
                        s[qt][kt][r] = p;
                        dp[qt][kt][r] = p * dp[qt][kt][r];                          // dp already holds dP - D_i
                    }
            bf16x8 pB[2], dsB[2];
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                pB[kt] = pack44(s[0][kt], s[1][kt]);
                dsB[kt] = pack44(dp[0][kt], dp[1][kt]);
            }
            lds_pipeline_body<16, 2, 2>(tring, t_issue, [&](auto n, TrSlot &slot) {
                constexpr int dt = decltype(n)::value % 8;
#pragma unroll
                for (int kt = 0; kt < 2; ++kt) {
                    if constexpr (decltype(n)::value < 8) accV[dt][kt] = mfma16(tr_operand(slot), pB[kt], accV[dt][kt]);
                    else accK[dt][kt] = mfma16(tr_operand(slot), dsB[kt], accK[dt][kt]);
                }
            });
        }
    };
    for (int n = 0; n < nsteps; n += 2) {
        tile_step(IntC<0>{}, QS * n + grp);
        if (n + 1 < nsteps) tile_step(IntC<1>{}, QS * (n + 1) + grp);
    }

    int g4e = g4;                 // opaque copy: the output addresses are formed here, once per sweep, not kept in registers
    asm volatile("" : "+v"(g4e));
    __bf16 *dv = static_cast<__bf16 *>(a.dv) + base + (j0w + l16) * a.ss + 4 * g4e;
    __bf16 *dk = static_cast<__bf16 *>(a.dk) + base + (j0w + l16) * a.ss + 4 * g4e;
    if constexpr (QS == 1) {
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
            if (j0w + 16 * kt + l16 < a.S) {
#pragma unroll
                for (int dt = 0; dt < 8; ++dt) {
                    store4(dv + 16 * kt * a.ss + 16 * dt, accV[dt][kt], 1.f);
                    store4(dk + 16 * kt * a.ss + 16 * dt, accK[dt][kt], a.scale);
                }
            }
    } else {
        // first dV, then dK: piece 8 kt + dt of every wave goes through LDS and each wave adds up 16/QS
        // pieces of its key block over the query groups
        LDS_AS f32x4 *pieces = (LDS_AS f32x4 *)lds;
        auto combine = [&](f32x4 (&acc)[8][2], __bf16 *out, float mul) {
            __syncthreads();      // every wave has left what lies there
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int dt = 0; dt < 8; ++dt) pieces[(wave * 16 + 8 * kt + dt) * 64 + lane] = acc[dt][kt];
            __syncthreads();
#pragma unroll
            for (int n = 0; n < 16 / QS; ++n) {
                const int e = grp * (16 / QS) + n, kt = e >> 3, dt = e & 7;
                const f32x4 sum = sum_pieces<QS, KG>(pieces, wk, e, lane);
                if (j0w + 16 * kt + l16 < a.S) store4(out + 16 * kt * a.ss + 16 * dt, sum, mul);
            }
        };
        combine(accV, dv, 1.f);
        combine(accK, dk, a.scale);
    }
}

// both gradients in one launch (joint_slot)
template <int KG, int QG, int T>
__global__ __launch_bounds__(512, 2) void attn_bwd_both_bf16_kernel(AttnArgs a, uint32_t key_tiles, Divisor heads, Divisor H)
{
    constexpr int kLds = DkdvShape<KG>::kLds > DqShape<QG, T>::kLds ? DkdvShape<KG>::kLds : DqShape<QG, T>::kLds;
    static_assert(KG == QG, "a position stands for a key tile or a query tile of as many rows");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kLds];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;
    const auto [pos, hb] = heads(blockIdx.x);
    const JointSlot slot = joint_slot(key_tiles, pos);
    const auto [b, h] = H(hb);
    const PairId t = {(int64_t)slot.rank, -1, (int)h, (int)b};
    if (slot.key) dkdv_rows<KG>(a, lds, [&](int64_t) { return t; });
    else dq_rows<QG, T>(a, lds, [&](int64_t nqt) { return PairId{nqt - 1 - t.first, -1, t.h, t.b}; });
}

// the same of 256 rows, with the workgroup id decoded as in the launches of one gradient: a tile found by Divisor moved the
// loops by half to one per cent (S = 90000 H = 4 23280 : 23516 us).  In the shorter launches above that costs as much where they last longest (64 rows,
// S = 3001 H = 4 46.2 : 46.6) and gains 1 to 2 % where they are short (S = 334 H = 24 14.5 : 14.2, S = 1657 H = 8 29.5 : 29.2), half a per cent on average.
__global__ __launch_bounds__(512, 2) void attn_bwd_both_long_bf16_kernel(AttnArgs a, uint32_t dkdv_blocks)
{
    constexpr int kLds = DkdvShape<8>::kLds > DqShape<8, 64>::kLds ? DkdvShape<8>::kLds : DqShape<8, 64>::kLds;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kLds];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;
    if (blockIdx.x < dkdv_blocks)
        dkdv_rows<8>(a, lds, [&](int64_t nkt) { return decode_block(a, blockIdx.x, nkt, kLongestFirst, false); });
    else
        dq_rows<8, 64>(a, lds, [&](int64_t nqt) { return decode_block(a, blockIdx.x - dkdv_blocks, nqt, kLongestFirst, true); });
}

// ============================================================================ backward, 32-row workgroups
// For short sequences: 32 keys (or query rows) per workgroup, the other side of the sweep in eight.  Every wave works all 32
// rows against 32-row tiles of its own, one buffer each, so there is no barrier in the sweep; a half of the buffer
// is refilled as soon as it is used up.  The sums meet in LDS at the end.  Twice the fill traffic of 64-row workgroups, and
// sweeps of half the steps: ahead where the longest sweep, not the work, is what a launch takes (own_us, launch_plan.h).  us with the
// D_i launch, 64-row workgroups : these: S = 256 H = 2 10.4 : 7.3, S = 640 H = 2 15.1 : 9.9, S = 1000 H = 4 20.0 : 14.9, S = 1500 H = 4 25.9 : 19.8,
// S = 2500 H = 2 37.3 : 24.4; but S = 2000 with 6 heads 33.3 : 40.5, S = 8192 H = 4 227 : 252.
// A start is bound by the 144 KB that eight waves fetch through a unit's 64 B per cycle (dQ: Q and dO once to the LDS, not to every wave's
// registers) with the set-up behind it, an end by 128 KB through the LDS per sum.  What Q and dO through the LDS and the set-up behind the loads gave, columns in one part: S = 256 H = 2
// 10.5 -> 9.5, S = 1000 H = 4 15.0 -> 14.7, S = 1536 H = 2 18.1 -> 17.6.  Tried at the end without gain: dK's pieces put while dV's are added up,
// barriers that do not wait for stores.
// CS: the output columns of a tile go to so many workgroups where units would be idle (column_parts, launch_plan.h): S = 640 H = 2 11.6 -> 9.9.
constexpr int kOwnTile = 32 * 256, kOwnRing = 8 * 2 * kOwnTile;

// piece of every wave -> its sum in the wave that owns the piece (two of sixteen for NB = 8 blocks of columns): out(block of rows, block of
// columns, sum).  A wave's pieces take the place of its own ring, so that the first sum needs no barrier before them.
template <bool kFirst, int NB, typename Out>
__device__ __forceinline__ void sum_over_waves(LDS_AS unsigned char *lds, const f32x4 (&acc)[NB][2], int wave, int lane, Out &&out)
{
    LDS_AS f32x4 *pieces = (LDS_AS f32x4 *)lds;
    if (!kFirst) __syncthreads(); // every wave has read the sum before
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int dt = 0; dt < NB; ++dt) pieces[(wave * 16 + NB * b + dt) * 64 + lane] = acc[dt][b];
    __syncthreads();
    constexpr int kOwn = NB >= 4 ? NB / 4 : 1;
    if (kOwn * wave >= 2 * NB) return;                // fewer pieces than waves
    f32x4 x[kOwn][8];
#pragma unroll
    for (int n = 0; n < kOwn; ++n)
#pragma unroll
        for (int g = 0; g < 8; ++g) x[n][g] = pieces[(g * 16 + kOwn * wave + n) * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);                // all reads are on their way before the first is waited for
#pragma unroll
    for (int n = 0; n < kOwn; ++n) {
        f32x4 sum = x[n][0];
#pragma unroll
        for (int g = 1; g < 8; ++g)
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[r] += x[n][g][r];
        const int e = kOwn * wave + n;
        out(e / NB, e % NB, sum);
    }
}

template <int CS>
__device__ __forceinline__ void dkdv_own_rows(const AttnArgs &a, LDS_AS unsigned char *lds, const TileId t, int part)
{
    constexpr int NB = 8 / CS;                        // blocks of 16 columns of dK and dV that the workgroup forms
    // lds: [wave][Q|dO] tiles, then the K and V rows
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nit = (int)((a.S + 31) / 32);
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh;
    const __bf16 *q = static_cast<const __bf16 *>(a.q) + base, *g = static_cast<const __bf16 *>(a.d_o) + base;
    const float *lse = a.lse + ((int64_t)t.b * a.H + t.h) * a.S, *dlt = a.delta + ((int64_t)t.b * a.H + t.h) * a.S;
    const float c = a.scale * kLog2e, neg_inv_scale = -1.f / a.scale;
    const int it0 = t.tile;                           // key tile and first query tile: the diagonal
    LDS_AS unsigned char *ring = lds + wave * 2 * kOwnTile;
    const TileOffsets<8, 32> koff = make_tile_offsets<8, SwzB, 32>(a.ss, wave, lane);
    koff.fill(lds + kOwnRing, static_cast<const __bf16 *>(a.k) + base, a.ss, (int64_t)it0 * 32, a.S, wave);
    koff.fill(lds + kOwnRing + kOwnTile, static_cast<const __bf16 *>(a.v) + base, a.ss, (int64_t)it0 * 32, a.S, wave);
    const OwnTileFill fill(a.ss, lane);
    // a tile past the last one is an empty buffer: its fills are still counted by the waits
    auto fill_q = [&](int it) { fill(ring, q, a.ss, (int64_t)it * 32, it < nit ? a.S : (int64_t)it * 32); };
    auto fill_g = [&](int it) { fill(ring + kOwnTile, g, a.ss, (int64_t)it * 32, it < nit ? a.S : (int64_t)it * 32); };
    // row statistics: one value per lane, spread by a 4x4x1 MFMA (see dkdv_rows)
    const int stat_lane = 4 * g4 + (lane & 3);
    float raw_l[2], raw_d[2];
    auto load_stats = [&](int it) {
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
            const int64_t row = (int64_t)it * 32 + 16 * qt + stat_lane;
            raw_l[qt] = row < a.S ? lse[row] : INFINITY;
            raw_d[qt] = row < a.S ? dlt[row] : 0.f;
        }
    };
    int it = it0 + wave;
    load_stats(min(it, nit - 1));
    fill_q(it);
    fill_g(it);
    __builtin_amdgcn_sched_barrier(0);                // addresses and accumulators are set up while the loads are on their way
    const LdsAddr16 ad = make_lds_addr16(ring, lane);
    const uint32_t kv_base = (uint32_t)(kOwnRing - wave * 2 * kOwnTile);
    uint32_t tr[NB];              // the workgroup's blocks of the transposed operands
#pragma unroll
    for (int dt = 0; dt < NB; ++dt) tr[dt] = ad.tr16[dt] ^ (uint32_t)(part * NB << 5);
    f32x4 accV[NB][2], accK[NB][2];                   // dV^T, dK^T: [head-dim block][key block]; lane = key
#pragma unroll
    for (int dt = 0; dt < NB; ++dt)
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
            accV[dt][kt] = accK[dt][kt] = kZero4;
            asm volatile("" : "+v"(accV[dt][kt]), "+v"(accK[dt][kt]));
        }
    wait_fills_but<16>();
    __builtin_amdgcn_s_barrier();                     // the K and V rows are complete
    asm volatile("" ::: "memory");

    // S before dP, dK before dV: Q is needed first and used up first, dO half a step later, so that the fill of either
    // half of the buffer has the work on the other one to hide under
#pragma clang loop unroll(disable)
    for (; it < nit; it += 8) {
        f32x4 nl[2], nd[2];       // -LSE_i/scale and -D_i
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
            nl[qt] = __builtin_amdgcn_mfma_f32_4x4x1f32(raw_l[qt], neg_inv_scale, kZero4, 0, 0, 0);
            nd[qt] = __builtin_amdgcn_mfma_f32_4x4x1f32(raw_d[qt], -1.f, kZero4, 0, 0, 0);
        }
        f32x4 s[2][2], dp[2][2];                      // [query block][key block]; register r = query 16*qt + 4*g4 + r
        {
            // item n = k step n: the Q (dO) rows of both query blocks and the K (V) rows of both key blocks
            auto contract = [&](auto whichc, f32x4 (&x)[2][2], const f32x4 (&init)[2]) {
                constexpr int off = decltype(whichc)::value * kOwnTile;
                QuadSlot slots[2];
                auto issue = [&](auto n, QuadSlot &slot) {
                    lds_issue_b128<off>(slot.a0, ad.row16[decltype(n)::value]);
                    lds_issue_b128<off + 4096>(slot.a1, ad.row16[decltype(n)::value]);
                    lds_issue_b128<off>(slot.b0, ad.row16[decltype(n)::value] + kv_base);
                    lds_issue_b128<off + 4096>(slot.b1, ad.row16[decltype(n)::value] + kv_base);
                };
                lds_pipeline_prologue<4, 1, 4>(slots, issue);
                lds_pipeline_body<4, 1, 4>(slots, issue, [&](auto n, QuadSlot &slot) {
                    constexpr int kk = decltype(n)::value;
                    x[0][0] = mfma16(slot.a0, slot.b0, kk == 0 ? init[0] : x[0][0]);
                    x[0][1] = mfma16(slot.a0, slot.b1, kk == 0 ? init[0] : x[0][1]);
                    x[1][0] = mfma16(slot.a1, slot.b0, kk == 0 ? init[1] : x[1][0]);
                    x[1][1] = mfma16(slot.a1, slot.b1, kk == 0 ? init[1] : x[1][1]);
                });
            };
            wait_fills_but<8>();  // Q has landed; dO, queued behind it, may still be on its way
            contract(IntC<0>{}, s, nl);
            wait_fills();
            if (it + 8 < nit) load_stats(it + 8);
            contract(IntC<1>{}, dp, nd);
        }
        TrSlot tring[3];
        auto t_issue = [&](auto n, TrSlot &slot) {
            constexpr int dt = decltype(n)::value % NB;
            lds_issue_tr_pair<(decltype(n)::value < NB ? 0 : kOwnTile)>(slot, tr[dt]);
        };
        lds_pipeline_prologue<2 * NB, 2, 2>(tring, t_issue);
        if (it == it0) {          // the causal mask: query 16qt + 4g4 + r sees key 16kt + l16 iff it is not before it
#pragma unroll
            for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (r < 16 * kt + l16 - (16 * qt + 4 * g4)) s[qt][kt][r] = -INFINITY;
        }
        if (it == nit - 1) {      // rows past S were read as zero, and zero times an infinite key is NaN: their LSE of +inf does not do
            const int left = (int)(a.S - (int64_t)it * 32);
#pragma unroll
            for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (r >= left - (16 * qt + 4 * g4)) s[qt][0][r] = s[qt][1][r] = -INFINITY;
        }
#pragma unroll
        for (int qt = 0; qt < 2; ++qt)
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float p = __builtin_amdgcn_exp2f(s[qt][kt][r] * c);   // s already holds S - LSE_i/scale
                    s[qt][kt][r] = p;
                    dp[qt][kt][r] = p * dp[qt][kt][r];                          // dp already holds dP - D_i
                }
        bf16x8 pB[2], dsB[2];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
            pB[kt] = pack44(s[0][kt], s[1][kt]);
            dsB[kt] = pack44(dp[0][kt], dp[1][kt]);
        }
        lds_pipeline_body<2 * NB, 2, 2>(tring, t_issue, [&](auto n, TrSlot &slot) {
            constexpr int dt = decltype(n)::value % NB;
            if constexpr (decltype(n)::value == NB) fill_q(it + 8);   // Q is used up
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                if constexpr (decltype(n)::value < NB) accK[dt][kt] = mfma16(tr_operand(slot), dsB[kt], accK[dt][kt]);
                else accV[dt][kt] = mfma16(tr_operand(slot), pB[kt], accV[dt][kt]);
            }
        });
        fill_g(it + 8);
    }
    wait_fills();                 // the empty ones too: they write LDS

    const int64_t j0 = (int64_t)it0 * 32 + l16;
    const int64_t first = base + j0 * a.ss + 16 * NB * part + 4 * g4;
    __bf16 *dv = static_cast<__bf16 *>(a.dv) + first, *dk = static_cast<__bf16 *>(a.dk) + first;
    auto store = [&](__bf16 *out, float mul) {
        return [=, &a](int kt, int dt, const f32x4 &sum) {
            if (j0 + 16 * kt < a.S) store4(out + 16 * kt * a.ss + 16 * dt, sum, mul);
        };
    };
    sum_over_waves<true>(lds, accV, wave, lane, store(dv, 1.f));
    sum_over_waves<false>(lds, accK, wave, lane, store(dk, a.scale));
}

template <int CS>
__device__ __forceinline__ void dq_own_rows(const AttnArgs &a, LDS_AS unsigned char *lds, const TileId t, int part)
{
    constexpr int NB = 8 / CS;                        // blocks of 16 columns of dQ that the workgroup forms
    // lds: [wave][K|V] tiles, then the Q and dO rows
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh;
    const __bf16 *q = static_cast<const __bf16 *>(a.q) + base, *g = static_cast<const __bf16 *>(a.d_o) + base;
    const __bf16 *k = static_cast<const __bf16 *>(a.k) + base, *v = static_cast<const __bf16 *>(a.v) + base;
    const int64_t stat = ((int64_t)t.b * a.H + t.h) * a.S;
    const float c = a.scale * kLog2e;
    const int ntiles = t.tile + 1;                    // the last one is the diagonal
    const int64_t i0 = (int64_t)t.tile * 32 + l16;
    float lse2[2], nd[2];
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
        const int64_t i = i0 + 16 * qt < a.S ? i0 + 16 * qt : a.S - 1;          // rows past S are computed and never stored
        lse2[qt] = a.lse[stat + i];
        nd[qt] = a.delta[stat + i];
    }
    const int ring = wave * 2 * kOwnTile;
    const TileOffsets<8, 32> qoff = make_tile_offsets<8, SwzB, 32>(a.ss, wave, lane);
    qoff.fill(lds + kOwnRing, q, a.ss, (int64_t)t.tile * 32, a.S, wave);
    qoff.fill(lds + kOwnRing + kOwnTile, g, a.ss, (int64_t)t.tile * 32, a.S, wave);
    const TileOffsets<1, 32> toff = make_tile_offsets<1, SwzB, 32>(a.ss, 0, lane);
    // a tile past the last one is an empty buffer: its fills are still counted by the waits
    auto fill_k = [&](int jt) { toff.fill(lds + ring, k, a.ss, (int64_t)jt * 32, jt < ntiles ? a.S : (int64_t)jt * 32, 0); };
    auto fill_v = [&](int jt) { toff.fill(lds + ring + kOwnTile, v, a.ss, (int64_t)jt * 32, jt < ntiles ? a.S : (int64_t)jt * 32, 0); };
    fill_v(wave);
    fill_k(wave);
    __builtin_amdgcn_sched_barrier(0);                // addresses and accumulators are set up while the loads are on their way
    const LdsAddr16 ad = make_lds_addr16(lds + ring, lane);
    uint32_t tr[NB];              // the workgroup's blocks of the transposed operand
#pragma unroll
    for (int dt = 0; dt < NB; ++dt) tr[dt] = ad.tr16[dt] ^ (uint32_t)(part * NB << 5);
    f32x4 accQ[NB][2];            // dQ^T: [head-dim block of 16][query block]; lane = query, rows = head dim
#pragma unroll
    for (int dt = 0; dt < NB; ++dt)
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
            accQ[dt][qt] = kZero4;
            asm volatile("" : "+v"(accQ[dt][qt]));
        }
    wait_fills_but<16>();
    __builtin_amdgcn_s_barrier();                     // the Q and dO rows are complete
    asm volatile("" ::: "memory");
    // Q^T and dO^T as B operands: lane = query 16*qt + l16, 8 head-dim values per 32-wide k step
    bf16x8 qB[2][4], gB[2][4];
    static_for<0, 8>([&](auto n) {
        constexpr int qt = decltype(n)::value / 4, kk = decltype(n)::value % 4;
        lds_issue_b128<4096 * qt>(gB[qt][kk], ad.row16[kk] + (uint32_t)(kOwnRing + kOwnTile - ring));
        lds_issue_b128<4096 * qt>(qB[qt][kk], ad.row16[kk] + (uint32_t)(kOwnRing - ring));
    });
    static_for<0, 8>([&](auto n) {
        lds_wait<0>(gB[decltype(n)::value / 4][decltype(n)::value % 4]);
        lds_wait<0>(qB[decltype(n)::value / 4][decltype(n)::value % 4]);
    });
    f32x4 neg_d[2];
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
        lse2[qt] *= kLog2e;
        neg_d[qt] = f32x4{-nd[qt], -nd[qt], -nd[qt], -nd[qt]};
    }

#pragma clang loop unroll(disable)
    for (int jt = wave; jt < ntiles; jt += 8) {
        int l = l16;              // opaque: the masks of the diagonal are formed there, not in front of the loop
        asm volatile("" : "+v"(l));
        // dP before S: V is needed first and used up first, K follows
        f32x4 s[2][2], dp[2][2];                      // [key block][query block]
        {
            // item n = (k step n/2, key block n%2): one row operand, two MFMAs
            auto contract = [&](auto offc, f32x4 (&x)[2][2], const bf16x8 (&b)[2][4], const f32x4 (&init)[2]) {
                bf16x8 slots[3];
                auto issue = [&](auto n, bf16x8 &slot) {
                    lds_issue_b128<(decltype(n)::value % 2) * 4096 + decltype(offc)::value>(slot, ad.row16[decltype(n)::value / 2]);
                };
                lds_pipeline_prologue<8, 2, 1>(slots, issue);
                lds_pipeline_body<8, 2, 1>(slots, issue, [&](auto n, bf16x8 &slot) {
                    constexpr int kk = decltype(n)::value / 2, kt = decltype(n)::value % 2;
#pragma unroll
                    for (int qt = 0; qt < 2; ++qt) x[kt][qt] = mfma16(slot, b[qt][kk], kk == 0 ? init[qt] : x[kt][qt]);
                });
            };
            const f32x4 zeros[2] = {kZero4, kZero4};
            wait_fills_but<8>();
            contract(IntC<kOwnTile>{}, dp, gB, neg_d);
            fill_v(jt + 8);
            wait_fills_but<8>();
            contract(IntC<0>{}, s, qB, zeros);
        }
        TrSlot kring[3];
        auto k_issue = [&](auto n, TrSlot &slot) { lds_issue_tr_pair<0>(slot, tr[decltype(n)::value]); };
        lds_pipeline_prologue<NB, 2, 2>(kring, k_issue);
        if (jt == ntiles - 1) {
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (r > 16 * qt + l - (16 * kt + 4 * g4)) s[kt][qt][r] = -INFINITY;
        }
        bf16x8 dsB[2];
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float p = __builtin_amdgcn_exp2f(fmaf(s[kt][qt][r], c, -lse2[qt]));
                    s[kt][qt][r] = p * dp[kt][qt][r];               // dS (dp already holds dP - D_i)
                }
            dsB[qt] = pack44(s[0][qt], s[1][qt]);
        }
        lds_pipeline_body<NB, 2, 2>(kring, k_issue, [&](auto n, TrSlot &slot) {
            constexpr int dt = decltype(n)::value;
#pragma unroll
            for (int qt = 0; qt < 2; ++qt) accQ[dt][qt] = mfma16(tr_operand(slot), dsB[qt], accQ[dt][qt]);
        });
        fill_k(jt + 8);
    }
    wait_fills();                 // the empty ones too: they write LDS
    __bf16 *dq = static_cast<__bf16 *>(a.dq) + base + i0 * a.ss + 16 * NB * part + 4 * g4;
    sum_over_waves<true>(lds, accQ, wave, lane, [=, &a](int qt, int dt, const f32x4 &sum) {
        if (i0 + 16 * qt < a.S) store4(dq + 16 * qt * a.ss + 16 * dt, sum, a.scale);
    });
}

template <int CS>
__global__ __launch_bounds__(512, 2) void attn_bwd_own_bf16_kernel(AttnArgs a, uint32_t key_tiles, Divisor heads, Divisor H)
{
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kOwnRing + 2 * kOwnTile];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;
    load_args_at_once(a);
    asm volatile("" ::"s"(a.d_o), "s"(a.delta));
    const auto [pos, hbp] = heads(blockIdx.x);        // CS parts of a head beside each other
    const int part = (int)(hbp % CS);
    const JointSlot slot = joint_slot(key_tiles, pos);
    const TileId t = head_of(hbp / CS, slot.key ? (int)slot.rank : (int)((a.S + 31) / 32) - 1 - (int)slot.rank, H);
    if (slot.key) dkdv_own_rows<CS>(a, lds, t, part);
    else dq_own_rows<CS>(a, lds, t, part);
}

// dkdv, dq: which of the gradients to launch; both in one launch where the plan says so
hipError_t launch_main(const AttnArgs &a, bool dkdv, bool dq, hipStream_t st)
{
    const int64_t heads = (int64_t)a.H * a.B;
    const BwdPlan p = bwd_plan(a.S, heads);
    const bool joint = p.joint || p.rows < 256;       // one kernel for both kinds of workgroup
    const int64_t tiles = (a.S + p.rows - 1) / p.rows;
    const int64_t nk = order_grid(tiles, heads, p.k_order), nq = order_grid(tiles, heads, p.q_order);
    const int64_t most = joint ? nk + nq : std::max(nk, nq);          // whatever is asked for, so that the parts are the same
    if (most > kMaxBlocks)
        return launch_fewer_heads(a, sizeof(__bf16), most, kMaxBlocks, [&](const AttnArgs &part) { return launch_main(part, dkdv, dq, st); });
    hipError_t e = hipSuccess;
    if (!joint) {
        if (dkdv) e = launch_attn_bwd_dkdv_bf16_long(a, p.k_order, nk, st);
        if (dq && e == hipSuccess) e = launch_attn_bwd_dq_bf16_long(a, p.q_order, nq, st);
        return e;
    }
    if (dkdv && dq && !p.joint) {
        e = launch_main(a, true, false, st);
        return e == hipSuccess ? launch_main(a, false, true, st) : e;
    }
    auto launch = [&](auto kernel, int parts = 1) {
        return launch_blocks(kernel, (dkdv + dq) * tiles * heads * parts, st, a, dkdv ? (uint32_t)tiles : 0u, Divisor(heads * parts), Divisor(a.H));
    };
    switch (p.rows) {
    case 32:
        // a dQ that takes the place of Q or dO is not split: another part may not have read them yet
        switch (dq_in_place(a) ? 1 : column_parts(2 * tiles * heads)) {
        case 4: return launch(attn_bwd_own_bf16_kernel<4>, 4);
        case 2: return launch(attn_bwd_own_bf16_kernel<2>, 2);
        default: return launch(attn_bwd_own_bf16_kernel<1>);
        }
    case 64: return launch(attn_bwd_both_bf16_kernel<2, 2, 32>);
    case 128: return launch(attn_bwd_both_bf16_kernel<4, 4, 64>);
    default:
        if (p.waves == 4) return launch_attn_bwd_both_bf16_long(a, dkdv ? nk : 0, (dkdv + dq) * tiles * heads, st);
        return launch_blocks(attn_bwd_both_long_bf16_kernel, (dkdv + dq) * tiles * heads, st, a, dkdv ? (uint32_t)nk : 0u);
    }
}

}  // namespace

// D_i preprocess, then dK, dV and dQ: in one launch of 32-, 64-, 128- or 256-row workgroups, or, where whole rounds
// of folded pairs are cheaper, the key-stationary kernel and then the query-stationary one.  The single launch
// fills the chip where neither kernel does alone (S = 2000, 6 heads: 32.4 + 27.6 -> 33.0 us with 64-row workgroups,
// 207 as two launches of 256-row pairs in eight waves) and lets the dQ tiles run in the tail of the dK/dV ones (S = 25000 H = 4 1943 -> 1739 us,
// 70000 H = 4 13004 -> 12669).  256 rows go out in four waves (attn_bwd_long_bf16.hip), in joint launches of up to 3072 rows in eight; two launches win at
// whole rounds from S = 32K on (S = 32768 H = 4 2741 joint, 2694 as two; 50000 H = 5 8434, 8377).
// A joint launch goes out in two parts, with the same bits, where dQ takes the place of Q or dO, which all key-stationary
// workgroups read, and where an event between the stages is asked for.
hipError_t launch_attn_bwd_bf16(const AttnArgs &a, hipStream_t st)
{
    hipError_t e = record_stage(a, 0, st);
    if (e != hipSuccess) return e;
    if ((e = launch_attn_delta(a, true, st)) != hipSuccess) return e;
    if ((e = record_stage(a, 1, st)) != hipSuccess) return e;
    if (!a.stage_events && !dq_in_place(a)) return launch_main(a, true, true, st);
    if ((e = launch_main(a, true, false, st)) != hipSuccess) return e;
    if ((e = record_stage(a, 2, st)) != hipSuccess) return e;
    if ((e = launch_main(a, false, true, st)) != hipSuccess) return e;
    return record_stage(a, 3, st);
}

}  // namespace memo

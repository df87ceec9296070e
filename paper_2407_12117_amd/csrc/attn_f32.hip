// fp32 causal attention forward/backward for gfx950 (Section 2.1.3 of the paper: exact
// softmax attention computed tile by tile with per-row running state, intermediates
// re-formed in the backward).  This is the full-precision path: fp32 operands on the matrix
// cores (v_mfma_f32_16x16x4_f32: fp32 products and sums), no rounding of the probabilities.
//
// What bounds it: the fp32 matrix rate, 256 flops per cycle and compute unit (157 TFLOP/s), the same as the
// vector units'; but one MFMA instruction does 32 cycles of that work from two registers, where the
// vector form needs an LDS read per multiply-add and lane.  An earlier VALU version of these kernels ran at 5 to
// 7 TFLOP/s, bound by its scalar LDS reads.  LDS and fill traffic are light here (16 KB of operands per 2048
// MFMA cycles), so small workgroups cost nothing per flop and the tiles are chosen to spread the work.
//
// Operand conventions of the 16x16x4 MFMA, D = A(16xK4) * B(K4x16), lane = 16*g4 + l16:
//   A : lane holds row l16, k = g4;  B : lane holds col l16, k = g4;
//   D : lane holds col l16, rows 4*g4 + r for register r
// A contraction over the head dim takes the k slots in the order {16c + 4*g4 + j} for step (c, j), so that
// one 16-byte read per lane feeds four MFMAs.  As in the bf16 kernels the score tile is produced so that
// its D registers are directly the B operand of the next contraction: step r contracts over the tile rows
// 4*g4 + r, and the matching A operand (the tile transposed) is row 4*g4 + r at 16-byte piece l16 of each 256-byte
// half h, which serves the four output blocks of that half: block 4h + e stands for dim 64h + 4*row + e.
// LDS rows are D floats; the 16-byte piece c of row r lies at c ^ SwzB(r) (low four bits), conflict-free for both
// reads as in the bf16 tiles.
//
// Workgroup: 8 waves = G row groups of 16 owned rows x 8/G groups that share out the streamed rows (16 per
// tile, a double-buffered ring per group, one barrier per step) and are combined through LDS at the end.
#include "bf16_tiles.h"

namespace memo {
namespace {

constexpr int kF32Waves = 8, kT = 16;                 // waves per workgroup; rows of a streamed tile
constexpr f32x4 kZero4 = {0.f, 0.f, 0.f, 0.f};
constexpr float kF32RescaleAbove = 1099511627776.f;   // 2^40, as in the bf16 forward

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int D, int G>
struct F32Shape {
    static constexpr int kParts = kF32Waves / G;      // groups that share out the streamed rows
    static constexpr bool kOwn = G == 1;              // every wave has a ring of its own: one stage, no barrier
    static constexpr int kTile = kT * D * 4, kFills = kTile / 1024 / G;       // bytes; fill instructions per wave
    static constexpr int kStage = 2 * kTile, kGroup = (kOwn ? 1 : 2) * kStage, kRing = kParts * kGroup;
    static constexpr int kPieces = D / 16;            // f32x4 per lane of one accumulator set
    static_assert(kRing >= kF32Waves * kPieces * 1024 && kRing <= 128 * 1024, "the combination lays the accumulators over the ring");
};

// two workgroups per compute unit where LDS has room for them and 128 registers hold a wave
template <int D, int G> constexpr int kFwdWavesPerSimd = F32Shape<D, G>::kRing <= 65536 ? 4 : 2;
template <int D, int G> constexpr int kBwdWavesPerSimd = D == 64 && G > 1 ? 4 : 2;

// fill of the 16-row tile at rows r0.. by the G waves of a group (rows past S repeat row S-1)
template <int D, int G>
__device__ __forceinline__ void f32_fill(LDS_AS unsigned char *tile, const float *src, int64_t ss, int64_t r0, int64_t S,
                                         int w, int lane)
{
    constexpr int rows = 256 / D, n_instr = kT / rows / G;        // rows per instruction, instructions per wave
    static_assert(n_instr >= 1, "more waves than instructions");
#pragma unroll
    for (int n = 0; n < n_instr; ++n) {
        const int row = rows * (n_instr * w + n) + lane / (D / 4), pos = lane % (D / 4);
        const int piece = pos ^ SwzB::f(row);
        const int64_t rg = r0 + row < S ? r0 + row : S - 1;
        __builtin_amdgcn_global_load_lds((const GLB_AS void *)(src + rg * ss + piece * 4),
                                         (LDS_AS void *)(tile + (n_instr * w + n) * 1024), 16, 0, 0);
    }
}

// LDS addresses of a lane's operand reads within a tile (bf16_tiles.h has the hand-issued pipeline they go through):
//   row[c % 4] + 256 (c / 4)   row-major operand: row l16, floats 16c + 4*g4 ..
//   tr[r] + 256 h              transposed operand: row 4*g4 + r, floats 64h + 4*l16 ..
struct F32Addr { uint32_t row[4], tr[4]; };
template <int D>
__device__ __forceinline__ F32Addr f32_addr(const LDS_AS unsigned char *base, int l16, int g4)
{
    F32Addr ad;
    const uint32_t b = (uint32_t)(uintptr_t)base;
#pragma unroll
    for (int c = 0; c < 4; ++c) ad.row[c] = b + (uint32_t)(l16 * D * 4 + (((4 * c + g4) ^ SwzB::f(l16)) << 4));
#pragma unroll
    for (int r = 0; r < 4; ++r) ad.tr[r] = b + (uint32_t)((4 * g4 + r) * D * 4 + ((l16 ^ SwzB::f(4 * g4 + r)) << 4));
    return ad;
}

struct F32Pair { f32x4 x, y; };
template <int N>
__device__ __forceinline__ void lds_wait(F32Pair &p)
{
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(p.x), "+v"(p.y) : "n"(N));
}

template <int D>
__device__ __forceinline__ void f32_load_row(f32x4 (&dst)[D / 16], const float *row, int g4)
{
#pragma unroll
    for (int c = 0; c < D / 16; ++c) dst[c] = *reinterpret_cast<const f32x4 *>(row + 16 * c + 4 * g4);
}

constexpr int kDepth = 3;         // operand reads in flight ahead of their MFMAs

// acc^T[dim][col] += tile^T x (tile rows 4*g4 + r), tile OFF bytes past `at`: item n = (r = n / (D/64), h = n % (D/64)),
// one read, four MFMAs.  f32_outer_issue asks for the first operands ahead of the element-wise work.
template <int D, int OFF>
struct F32Outer {
    static constexpr int H = D / 64, N = 4 * H;
    f32x4 ring[kDepth + 1];
    const F32Addr &ad;
    uint32_t at;
    __device__ __forceinline__ F32Outer(const F32Addr &addr, uint32_t off) : ad(addr), at(off)
    {
        lds_pipeline_prologue<N, kDepth, 1>(ring, [&](auto n, f32x4 &slot) { issue(n, slot); });
    }
    template <typename I>
    __device__ __forceinline__ void issue(I, f32x4 &slot)
    {
        lds_issue_b128<OFF + 256 * (I::value % H)>(slot, ad.tr[I::value / H] + at);
    }
    __device__ __forceinline__ void run(f32x4 (&acc)[D / 16], const f32x4 &x)
    {
        lds_pipeline_body<N, kDepth, 1>(ring, [&](auto n, f32x4 &slot) { issue(n, slot); }, [&](auto n, f32x4 &slot) {
            constexpr int r = decltype(n)::value / H, h = decltype(n)::value % H;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[4 * h + e] = mfma4(slot[e], x[r], acc[4 * h + e]);
        });
    }
};

// s += (rows of tile 0) x b0 and dp += (rows of tile 1) x b1 over the head dim: item c, two reads, eight MFMAs
template <int D>
__device__ __forceinline__ void f32_two_scores(f32x4 &s, f32x4 &dp, const F32Addr &ad, uint32_t at, const f32x4 (&b0)[D / 16],
                                               const f32x4 (&b1)[D / 16])
{
    constexpr int kTile = kT * D * 4;
    F32Pair ring[2];
    auto issue = [&](auto n, F32Pair &slot) {
        constexpr int c = decltype(n)::value;
        lds_issue_b128<256 * (c / 4)>(slot.x, ad.row[c % 4] + at);
        lds_issue_b128<kTile + 256 * (c / 4)>(slot.y, ad.row[c % 4] + at);
    };
    lds_pipeline_prologue<D / 16, 1, 2>(ring, issue);
    lds_pipeline_body<D / 16, 1, 2>(ring, issue, [&](auto n, F32Pair &slot) {
        constexpr int c = decltype(n)::value;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            s = mfma4(slot.x[j], b0[c][j], s);
            dp = mfma4(slot.y[j], b1[c][j], dp);
        }
    });
}

// Accumulator piece 4h + r of a lane: the four consecutive dims 64h + 16*g4 + 4r .. of its column.
template <int D>
__device__ __forceinline__ f32x4 f32_piece(const f32x4 (&acc)[D / 16], int p)
{
    const int h = p >> 2, r = p & 3;
    return f32x4{acc[4 * h][r], acc[4 * h + 1][r], acc[4 * h + 2][r], acc[4 * h + 3][r]};
}

template <int D, int G>
__global__ __launch_bounds__(512, (kFwdWavesPerSimd<D, G>)) void attn_fwd_f32_kernel(AttnArgs a)
{
    using Shape = F32Shape<D, G>;
    constexpr int KS = Shape::kParts, NP = Shape::kPieces;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[Shape::kRing + kF32Waves * 16 * 8];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;     // [key group][buf][K|V] tiles, then (c m, sum) per wave and row
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wq = wave % G, grp = wave / G;
    const PairId t = decode_block(a, blockIdx.x, (a.S + 16 * G - 1) / (16 * G), kLongestFirst, true);
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh;
    const float *k = static_cast<const float *>(a.k) + base, *v = static_cast<const float *>(a.v) + base;
    const int64_t row0 = t.first * 16 * G, i0w = row0 + 16 * wq, i = i0w + l16;
    const int ntiles = (int)((min(row0 + 16 * G, a.S) - 1) / kT) + 1;
    const float c = a.scale * kLog2e;
    LDS_AS unsigned char *ring = lds + grp * Shape::kGroup;
    auto fill_k = [&](int buf, int jt) { f32_fill<D, G>(ring + buf * Shape::kStage, k, a.ss, (int64_t)jt * kT, a.S, wq, lane); };
    auto fill_v = [&](int buf, int jt) {
        f32_fill<D, G>(ring + buf * Shape::kStage + Shape::kTile, v, a.ss, (int64_t)jt * kT, a.S, wq, lane);
    };
    if (grp < ntiles) {
        fill_k(0, grp);
        fill_v(0, grp);
    }
    const F32Addr ad = f32_addr<D>(ring, l16, g4);
    f32x4 q[D / 16], acc[D / 16];
    f32_load_row<D>(q, static_cast<const float *>(a.q) + base + (i < a.S ? i : a.S - 1) * a.ss, g4);
#pragma unroll
    for (int n = 0; n < D / 16; ++n) acc[n] = kZero4;
    float mc = -INFINITY, lsum = 0.f;                 // running maximum (times c) and sum of this lane's keys
    const int diag = (int)(i0w / kT);                 // tiles past this one are fully masked for the wave

    for (int jt = grp, n = 0; n * KS < ntiles; ++n, jt += KS) {
        const bool more = jt + KS < ntiles;
        if constexpr (Shape::kOwn) {
            wait_fills_but<Shape::kFills>();          // K has landed; V, queued behind it, may still be on its way
        } else {
            wait_fills();
            __syncthreads();      // tile jt is complete; nobody still reads the other buffer
            if (more) {
                fill_k((n + 1) & 1, jt + KS);
                fill_v((n + 1) & 1, jt + KS);
            }
        }
        if (jt > diag || jt >= ntiles) continue;
        const uint32_t at = Shape::kOwn ? 0u : (uint32_t)((n & 1) * Shape::kStage);
        f32x4 s = kZero4, s1 = kZero4;                // two chains
        {
            f32x4 kring[kDepth + 1];
            auto issue = [&](auto m, f32x4 &slot) {
                constexpr int cc = decltype(m)::value;
                lds_issue_b128<256 * (cc / 4)>(slot, ad.row[cc % 4] + at);
            };
            lds_pipeline_prologue<D / 16, kDepth, 1>(kring, issue);
            lds_pipeline_body<D / 16, kDepth, 1>(kring, issue, [&](auto m, f32x4 &slot) {
                constexpr int cc = decltype(m)::value;
                s = mfma4(slot[0], q[cc][0], s);
                s1 = mfma4(slot[1], q[cc][1], s1);
                s = mfma4(slot[2], q[cc][2], s);
                s1 = mfma4(slot[3], q[cc][3], s1);
            });
        }
        if constexpr (Shape::kOwn) {
            if (more) {
                fill_k(0, jt + KS);                   // K is used up
                wait_fills_but<Shape::kFills>();
            } else {
                wait_fills();
            }
        }
        F32Outer<D, Shape::kTile> pv(ad, at);         // the first V operands: their latency hides behind the softmax
        s += s1;
        if (jt == diag) {         // key 4*g4 + r of the tile is visible to query l16 iff it is <= l16
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (4 * g4 + r > l16) s[r] = -INFINITY;
        }
        // against the running maximum as it stands: it only has to keep the exponentials in range (as in the bf16 forward)
        f32x4 p;
        auto exponentials = [&]() {
#pragma unroll
            for (int r = 0; r < 4; ++r) p[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c, -mc));
        };
        exponentials();
        if (__builtin_amdgcn_ballot_w64(!(p[0] + p[1] + p[2] + p[3] <= kF32RescaleAbove)) != 0) {
            float m = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])) * c;
            m = fmaxf(m, __shfl_xor(m, 16));
            m = fmaxf(m, __shfl_xor(m, 32));
            const float m_new = fmaxf(mc, m);         // finite: key 0 of a processed tile is visible to every row
            const float corr = __builtin_amdgcn_exp2f(mc - m_new);
            mc = m_new;
            lsum *= corr;
#pragma unroll
            for (int e = 0; e < D / 16; ++e) acc[e] *= corr;
            exponentials();
        }
        lsum += (p[0] + p[1]) + (p[2] + p[3]);
        pv.run(acc, p);                               // O^T += V^T P^T
        if constexpr (Shape::kOwn)
            if (more) fill_v(0, jt + KS);
    }
    lsum += __shfl_xor(lsum, 16);
    lsum += __shfl_xor(lsum, 32);

    LDS_AS f32x4 *pieces = (LDS_AS f32x4 *)lds;
    LDS_AS f32x2 *stats = (LDS_AS f32x2 *)(lds + Shape::kRing);
    __syncthreads();              // every wave has left the last LDS buffer
#pragma unroll
    for (int p = 0; p < NP; ++p) pieces[(wave * NP + p) * 64 + lane] = f32_piece<D>(acc, p);
    if (g4 == 0) stats[wave * 16 + l16] = f32x2{mc, lsum};
    __syncthreads();
    float top = -INFINITY, total = 0.f, weight[KS];
    f32x2 st[KS];
#pragma unroll
    for (int g = 0; g < KS; ++g) {
        st[g] = stats[(g * G + wq) * 16 + l16];
        top = fmaxf(top, st[g][0]);
    }
#pragma unroll
    for (int g = 0; g < KS; ++g) {
        weight[g] = __builtin_amdgcn_exp2f(st[g][0] - top);       // a group without a tile: m = -inf, weight zero
        total += weight[g] * st[g][1];
    }
    if (i >= a.S) return;
    float *o = static_cast<float *>(a.o_out) + base + i * a.ss + 16 * g4;
    const float inv = 1.f / total;
    for (int p = grp; p < NP; p += KS) {
        f32x4 sum = kZero4;
#pragma unroll
        for (int g = 0; g < KS; ++g) sum += weight[g] * pieces[((g * G + wq) * NP + p) * 64 + lane];
        *reinterpret_cast<f32x4 *>(o + 64 * (p >> 2) + 4 * (p & 3)) = sum * inv;
    }
    if (grp == 0 && g4 == 0) a.lse[((int64_t)t.b * a.H + t.h) * a.S + i] = (top + __builtin_amdgcn_logf(total)) * kLn2;
}

// Adds up the accumulators of the row group's waves and writes mul times them: out points at the lane's row.
template <int D, int G>
__device__ __forceinline__ void f32_combine(LDS_AS unsigned char *lds, const f32x4 (&acc)[D / 16], float *out, bool live, float mul,
                                            int w, int grp, int lane)
{
    using Shape = F32Shape<D, G>;
    constexpr int NP = Shape::kPieces, KS = Shape::kParts;
    LDS_AS f32x4 *pieces = (LDS_AS f32x4 *)lds;
    __syncthreads();              // every wave has left what lies there
#pragma unroll
    for (int p = 0; p < NP; ++p) pieces[((grp * G + w) * NP + p) * 64 + lane] = f32_piece<D>(acc, p);
    __syncthreads();
    for (int p = grp; p < NP; p += KS) {
        f32x4 sum = kZero4;
#pragma unroll
        for (int g = 0; g < KS; ++g) sum += pieces[((g * G + w) * NP + p) * 64 + lane];
        if (live) *reinterpret_cast<f32x4 *>(out + 64 * (p >> 2) + 4 * (p & 3)) = sum * mul;
    }
}

// dQ_i = scale * sum_{j<=i} dS_ij k_j, dS_ij = P_ij (dO_i.v_j - D_i), P_ij = exp(s_ij - LSE_i); rows = queries
template <int D, int G>
__device__ __forceinline__ void f32_dq_rows(const AttnArgs &a, LDS_AS unsigned char *lds, uint32_t id)
{
    using Shape = F32Shape<D, G>;
    constexpr int KS = Shape::kParts;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wq = wave % G, grp = wave / G;
    const PairId t = decode_block(a, id, (a.S + 16 * G - 1) / (16 * G), kLongestFirst, true);
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh, stat = ((int64_t)t.b * a.H + t.h) * a.S;
    const float *k = static_cast<const float *>(a.k) + base, *v = static_cast<const float *>(a.v) + base;
    const int64_t row0 = t.first * 16 * G, i0w = row0 + 16 * wq, i = i0w + l16, iq = i < a.S ? i : a.S - 1;
    const int ntiles = (int)((min(row0 + 16 * G, a.S) - 1) / kT) + 1;
    const float c = a.scale * kLog2e;
    LDS_AS unsigned char *ring = lds + grp * Shape::kGroup;
    auto fill_k = [&](int buf, int jt) { f32_fill<D, G>(ring + buf * Shape::kStage, k, a.ss, (int64_t)jt * kT, a.S, wq, lane); };
    auto fill_v = [&](int buf, int jt) {
        f32_fill<D, G>(ring + buf * Shape::kStage + Shape::kTile, v, a.ss, (int64_t)jt * kT, a.S, wq, lane);
    };
    if (grp < ntiles) {
        fill_k(0, grp);
        fill_v(0, grp);
    }
    const F32Addr ad = f32_addr<D>(ring, l16, g4);
    f32x4 q[D / 16], go[D / 16], acc[D / 16];
    f32_load_row<D>(q, static_cast<const float *>(a.q) + base + iq * a.ss, g4);
    f32_load_row<D>(go, static_cast<const float *>(a.d_o) + base + iq * a.ss, g4);
    const float lse2 = a.lse[stat + iq] * kLog2e, nd = -a.delta[stat + iq];
#pragma unroll
    for (int n = 0; n < D / 16; ++n) acc[n] = kZero4;
    const int diag = (int)(i0w / kT);
    for (int jt = grp, n = 0; n * KS < ntiles; ++n, jt += KS) {
        wait_fills();
        const bool more = jt + KS < ntiles;
        if constexpr (!Shape::kOwn) {
            __syncthreads();      // tile jt is complete; nobody still reads the other buffer
            if (more) {
                fill_k((n + 1) & 1, jt + KS);
                fill_v((n + 1) & 1, jt + KS);
            }
        }
        if (jt > diag || jt >= ntiles) continue;
        const uint32_t at = Shape::kOwn ? 0u : (uint32_t)((n & 1) * Shape::kStage);
        f32x4 s = kZero4, dp = {nd, nd, nd, nd};      // keys 4*g4 + r x query l16
        f32_two_scores<D>(s, dp, ad, at, q, go);
        if constexpr (Shape::kOwn)
            if (more) fill_v(0, jt + KS);             // V is used up
        F32Outer<D, 0> kds(ad, at);
        if (jt == diag) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (4 * g4 + r > l16) s[r] = -INFINITY;
        }
        f32x4 ds;
#pragma unroll
        for (int r = 0; r < 4; ++r) ds[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c, -lse2)) * dp[r];
        kds.run(acc, ds);                             // dQ^T += K^T dS^T
        if constexpr (Shape::kOwn)
            if (more) fill_k(0, jt + KS);
    }
    f32_combine<D, G>(lds, acc, static_cast<float *>(a.dq) + base + iq * a.ss + 16 * g4, i < a.S, a.scale, wq, grp, lane);
}

// dV_j = sum_{i>=j} P_ij dO_i,  dK_j = scale * sum_{i>=j} dS_ij q_i; rows = keys, K and V rows in registers
template <int D, int G>
__device__ __forceinline__ void f32_dkdv_rows(const AttnArgs &a, LDS_AS unsigned char *lds, uint32_t id)
{
    using Shape = F32Shape<D, G>;
    constexpr int QS = Shape::kParts;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wk = wave % G, grp = wave / G;
    const PairId t = decode_block(a, id, (a.S + 16 * G - 1) / (16 * G), kLongestFirst, false);
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh, stat = ((int64_t)t.b * a.H + t.h) * a.S;
    const float *q = static_cast<const float *>(a.q) + base, *g = static_cast<const float *>(a.d_o) + base;
    const int64_t col0 = t.first * 16 * G, j0w = col0 + 16 * wk, j = j0w + l16, jk = j < a.S ? j : a.S - 1;
    const int it0 = (int)(col0 / kT), ntiles = (int)((a.S + kT - 1) / kT);
    const float c = a.scale * kLog2e;
    LDS_AS unsigned char *ring = lds + grp * Shape::kGroup;
    auto fill_q = [&](int buf, int it) { f32_fill<D, G>(ring + buf * Shape::kStage, q, a.ss, (int64_t)it * kT, a.S, wk, lane); };
    auto fill_g = [&](int buf, int it) {
        f32_fill<D, G>(ring + buf * Shape::kStage + Shape::kTile, g, a.ss, (int64_t)it * kT, a.S, wk, lane);
    };
    auto load_stats = [&](int it, f32x4 &l, f32x4 &d) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {                 // rows past S: LSE = +inf makes their P exactly zero
            const int64_t row = (int64_t)it * kT + 4 * g4 + r;
            l[r] = row < a.S ? a.lse[stat + row] : INFINITY;
            d[r] = row < a.S ? a.delta[stat + row] : 0.f;
        }
    };
    const F32Addr ad = f32_addr<D>(ring, l16, g4);
    f32x4 lse_n = kZero4, dl_n = kZero4;
    if (it0 + grp < ntiles) {
        fill_q(0, it0 + grp);
        fill_g(0, it0 + grp);
        load_stats(it0 + grp, lse_n, dl_n);
    }
    f32x4 kr[D / 16], vr[D / 16], dk[D / 16], dv[D / 16];
    f32_load_row<D>(kr, static_cast<const float *>(a.k) + base + jk * a.ss, g4);
    f32_load_row<D>(vr, static_cast<const float *>(a.v) + base + jk * a.ss, g4);
#pragma unroll
    for (int n = 0; n < D / 16; ++n) dk[n] = dv[n] = kZero4;
    const int diag = (int)(j0w / kT);                 // tiles before this one precede all of the wave's keys
    for (int it = it0 + grp, n = 0; it0 + n * QS < ntiles; ++n, it += QS) {
        wait_fills();
        const bool more = it + QS < ntiles;
        const f32x4 lse = lse_n, dl = dl_n;
        if constexpr (!Shape::kOwn) {
            __syncthreads();      // tile `it` is complete; nobody still reads the other buffer
            if (more) {
                fill_q((n + 1) & 1, it + QS);
                fill_g((n + 1) & 1, it + QS);
            }
        }
        if (more) load_stats(it + QS, lse_n, dl_n);
        if (it < diag || it >= ntiles) continue;
        const uint32_t at = Shape::kOwn ? 0u : (uint32_t)((n & 1) * Shape::kStage);
        f32x4 s = kZero4, dp;                         // queries 4*g4 + r x key l16
#pragma unroll
        for (int r = 0; r < 4; ++r) dp[r] = -dl[r];
        f32_two_scores<D>(s, dp, ad, at, kr, vr);
        F32Outer<D, Shape::kTile> gp(ad, at);
        if (it == diag) {         // query 4*g4 + r of the tile sees key l16 iff it is >= l16
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (4 * g4 + r < l16) s[r] = -INFINITY;
        }
        f32x4 p, ds;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            p[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c, -lse[r] * kLog2e));
            ds[r] = p[r] * dp[r];
        }
        gp.run(dv, p);                                // dV^T += dO^T P
        if constexpr (Shape::kOwn)
            if (more) fill_g(0, it + QS);             // dO is used up
        F32Outer<D, 0> qds(ad, at);
        qds.run(dk, ds);                              // dK^T += Q^T dS
        if constexpr (Shape::kOwn)
            if (more) fill_q(0, it + QS);
    }
    f32_combine<D, G>(lds, dv, static_cast<float *>(a.dv) + base + jk * a.ss + 16 * g4, j < a.S, 1.f, wk, grp, lane);
    f32_combine<D, G>(lds, dk, static_cast<float *>(a.dk) + base + jk * a.ss + 16 * g4, j < a.S, a.scale, wk, grp, lane);
}

// One launch for the gradients asked for: first the dkdv_blocks key-stationary workgroups, then the query-stationary ones.
template <int D, int G>
__global__ __launch_bounds__(512, (kBwdWavesPerSimd<D, G>)) void attn_bwd_f32_kernel(AttnArgs a, uint32_t dkdv_blocks)
{
    __shared__ __attribute__((aligned(1024))) unsigned char smem[F32Shape<D, G>::kRing];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;
    if (blockIdx.x < dkdv_blocks) f32_dkdv_rows<D, G>(a, lds, blockIdx.x);
    else f32_dq_rows<D, G>(a, lds, blockIdx.x - dkdv_blocks);
}

// D_i = sum_c dO_ic O_ic.  16 lanes per row, 16 rows per 256-thread workgroup.
template <typename T, int D>
__global__ __launch_bounds__(256) void attn_delta_kernel(AttnArgs a)
{
    const int tid = threadIdx.x, r = tid / 16, part = tid % 16;
    const int h = blockIdx.y, b = blockIdx.z;
    const int64_t i = (int64_t)blockIdx.x * 16 + r;
    const int64_t base = (int64_t)b * a.sb + (int64_t)h * a.sh;
    float sum = 0.f;
    if (i < a.S) {
        const T *o = static_cast<const T *>(a.o_in) + base + i * a.ss;
        const T *g = static_cast<const T *>(a.d_o) + base + i * a.ss;
        constexpr int per = D / 16;
#pragma unroll
        for (int c = 0; c < per; ++c)
            sum += static_cast<float>(o[part * per + c]) * static_cast<float>(g[part * per + c]);
    }
    sum += __shfl_xor(sum, 1);
    sum += __shfl_xor(sum, 2);
    sum += __shfl_xor(sum, 4);
    sum += __shfl_xor(sum, 8);
    if (i < a.S && part == 0) a.delta[((int64_t)b * a.H + h) * a.S + i] = sum;
}

inline dim3 row_grid(const AttnArgs &a, int rows)
{
    return dim3((unsigned)((a.S + rows - 1) / rows), (unsigned)a.H, (unsigned)a.B);
}

template <int D, int G>
hipError_t launch_fwd_f32(const AttnArgs &a, hipStream_t st)
{
    const int64_t blocks = order_grid((a.S + 16 * G - 1) / (16 * G), (int64_t)a.H * a.B, kLongestFirst);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    attn_fwd_f32_kernel<D, G><<<dim3((unsigned)blocks), 64 * kF32Waves, 0, st>>>(a);
    return hipGetLastError();
}

// dkdv, dq: which of the two to launch
template <int D, int G>
hipError_t launch_bwd_f32(const AttnArgs &a, bool dkdv, bool dq, hipStream_t st)
{
    const int64_t n = order_grid((a.S + 16 * G - 1) / (16 * G), (int64_t)a.H * a.B, kLongestFirst);
    if (2 * n > 0x7fffffffLL) return hipErrorInvalidValue;
    attn_bwd_f32_kernel<D, G><<<dim3((unsigned)(n * (dkdv + dq))), 64 * kF32Waves, 0, st>>>(a, dkdv ? (uint32_t)n : 0u);
    return hipGetLastError();
}

// Costs per 2^20 pairs as in the bf16 kernels (fitted to S = 300 .. 16000, 1 to 8 heads): {head dim 64, head dim 128} x {16, 32 rows}.
// 16-row workgroups fill the chip first, 32-row ones run 5 to 25 % faster per pair once it is full.
constexpr TileChoice kF32Fwd[2][2] = {
    {{16, kLongestFirst, 835.0, 4.0}, {32, kLongestFirst, 664.0, 4.0}},
    {{16, kLongestFirst, 1400.0, 5.0}, {32, kLongestFirst, 1264.0, 5.0}},
};
constexpr TileChoice kF32Dkdv[2][2] = {
    {{16, kLongestFirst, 1445.0, 0.0}, {32, kLongestFirst, 1233.0, 0.0}},
    {{16, kLongestFirst, 2563.0, 0.0}, {32, kLongestFirst, 2338.0, 0.0}},
};
constexpr TileChoice kF32Dq[2][2] = {
    {{16, kLongestFirst, 1084.0, 0.0}, {32, kLongestFirst, 925.0, 0.0}},
    {{16, kLongestFirst, 1922.0, 0.0}, {32, kLongestFirst, 1753.0, 0.0}},
};

}  // namespace

hipError_t launch_attn_fwd_f32(const AttnArgs &a, hipStream_t st)
{
    const bool wide = a.d == 128;
    const bool small = cheapest_tiles(kF32Fwd[wide], a.S, (int64_t)a.H * a.B) == 0;
    if (wide) return small ? launch_fwd_f32<128, 1>(a, st) : launch_fwd_f32<128, 2>(a, st);
    return small ? launch_fwd_f32<64, 1>(a, st) : launch_fwd_f32<64, 2>(a, st);
}

hipError_t launch_attn_delta(const AttnArgs &a, bool is_bf16, hipStream_t st)
{
    const dim3 grid = row_grid(a, 16);
    if (is_bf16) {
        if (a.d == 64)
            attn_delta_kernel<__hip_bfloat16, 64><<<grid, 256, 0, st>>>(a);
        else
            attn_delta_kernel<__hip_bfloat16, 128><<<grid, 256, 0, st>>>(a);
    } else {
        if (a.d == 64)
            attn_delta_kernel<float, 64><<<grid, 256, 0, st>>>(a);
        else
            attn_delta_kernel<float, 128><<<grid, 256, 0, st>>>(a);
    }
    return hipGetLastError();
}

hipError_t launch_attn_bwd_f32(const AttnArgs &a, hipStream_t st)
{
    const bool wide = a.d == 128;
    const int64_t hb = (int64_t)a.H * a.B;
    const bool small = both_us(kF32Dkdv[wide][0], kF32Dq[wide][0], a.S, hb) < both_us(kF32Dkdv[wide][1], kF32Dq[wide][1], a.S, hb);
    auto launch = [&](bool dkdv, bool dq) {
        if (wide) return small ? launch_bwd_f32<128, 1>(a, dkdv, dq, st) : launch_bwd_f32<128, 2>(a, dkdv, dq, st);
        return small ? launch_bwd_f32<64, 1>(a, dkdv, dq, st) : launch_bwd_f32<64, 2>(a, dkdv, dq, st);
    };
    hipError_t e = record_stage(a, 0, st);
    if (e != hipSuccess) return e;
    if ((e = launch_attn_delta(a, false, st)) != hipSuccess) return e;
    if ((e = record_stage(a, 1, st)) != hipSuccess) return e;
    if (!a.stage_events) return launch(true, true);
    if ((e = launch(true, false)) != hipSuccess) return e;
    if ((e = record_stage(a, 2, st)) != hipSuccess) return e;
    if ((e = launch(false, true)) != hipSuccess) return e;
    return record_stage(a, 3, st);
}

}  // namespace memo

// Workgroups of 16 rows of the fp32 attention kernels on fp32 matrix instructions (attn_f32.hip), which the kernels on fp16 ones (attn_f32_split.hip) take
// for what they cannot work.
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
// Workgroup: 16 owned rows, 8 waves that share out the streamed rows: every wave has tiles of 16 of them to itself, so there is
// no barrier in the sweep, and the waves' parts are combined through LDS at the end.  One buffer per wave: a half of
// it is refilled as soon as it is used up, while the other half is worked.  (32 owned rows, two waves to a tile and a
// barrier per step halve the fill traffic, and were ahead on a full chip while the fills computed 64-bit addresses; with
// buffer fills they lose everywhere: S = 5000, H = 4, d = 128 forward 260 against 225 us, backward 808 against 781.)
#pragma once
#include "bf16_tiles.h"

namespace memo {
namespace {

constexpr int kF32Waves = 8, kT = 16;                 // waves per workgroup; rows of a streamed tile
constexpr f32x4 kZero4 = {0.f, 0.f, 0.f, 0.f};
constexpr float kF32RescaleAbove = 1099511627776.f;   // 2^40, as in the bf16 forward
constexpr float kLowest = -3.402823466e38f;           // the lowest finite fp32

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int D>
struct F32Shape {
    static constexpr int kTile = kT * D * 4, kFills = kTile / 1024;       // bytes; fill instructions
    static constexpr int kStage = 2 * kTile, kRing = kF32Waves * kStage;
    static constexpr int kPieces = D / 16;            // f32x4 per lane of one accumulator set
    static constexpr int kSet = kStage / 1024;        // a wave's pieces lie in its own buffer, this many apart from the next wave's
    static_assert(kPieces <= kSet && kRing <= 128 * 1024, "the combination lays the accumulators over the ring");
};

// head dim 64: LDS has room for two workgroups per compute unit, and 128 registers hold a wave
template <int D> constexpr int kWavesPerSimd = D == 64 ? 4 : 2;

// Fill of the 16-row tile at rows r0..  The tile is a buffer that ends with row S - 1: rows past it are
// out of range and read as zero (every consumer masks them).  A lane's offset within an instruction's rows never
// changes; the next instruction is kRows rows on and, the swizzle being linear in the bits of the row, one XOR away.
// (With a 64-bit address and a clamped row per instruction: S = 3000 d = 128 H = 4 forward 114 us, 96 without.)
// FAR: rows so far apart (2^26 floats) that 16 of them leave a buffer's 4 GiB; full addresses, rows past S repeat row S-1.
constexpr int64_t kFarStride = (int64_t)1 << 26;
template <int D, bool FAR>
struct F32Fill {
    static constexpr int kRows = 256 / D, kInstr = kT / kRows;        // rows per instruction, instructions
    uint32_t row_off, piece_off;

    __device__ __forceinline__ F32Fill(int64_t ss, int lane)
    {
        const int row = lane / (D / 4), pos = lane % (D / 4);
        row_off = (uint32_t)row * (uint32_t)ss * 4;
        piece_off = (uint32_t)(pos ^ SwzB::f(row)) * 16;
    }
    template <int kCount>         // instructions first ..
    __device__ __forceinline__ void some(int first, LDS_AS unsigned char *tile, const float *src, int64_t ss, int64_t r0, int64_t S, int lane) const
    {
        if constexpr (FAR) {
#pragma unroll
            for (int n = first; n < first + kCount; ++n) {
                const int row = kRows * n + lane / (D / 4), piece = lane % (D / 4) ^ SwzB::f(row);
                const int64_t rg = r0 + row < S ? r0 + row : S - 1;
                __builtin_amdgcn_global_load_lds((const GLB_AS void *)(src + rg * ss + piece * 4),
                                                 (LDS_AS void *)(tile + n * 1024), 16, 0, 0);
            }
        } else {
#ifdef __HIP_DEVICE_COMPILE__      // the host pass does not know the 16-byte form of the builtin
            const int rows = (int)max((int64_t)0, min((int64_t)kT, S - r0));
            const uint32_t bytes = rows > 0 ? (uint32_t)(rows - 1) * (uint32_t)ss * 4 + D * 4 : 0;
            const __amdgpu_buffer_rsrc_t b = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(src + r0 * ss), 0, bytes, 0x00020000);
#pragma unroll
            for (int n = first; n < first + kCount; ++n)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(b, (LDS_AS void *)(tile + n * 1024), 16,
                                                         row_off + (piece_off ^ (uint32_t)(SwzB::f(kRows * n) * 16)) +
                                                             (uint32_t)(kRows * n) * (uint32_t)ss * 4, 0, 0, 0);
#endif
        }
    }
    __device__ __forceinline__ void operator()(LDS_AS unsigned char *tile, const float *src, int64_t ss, int64_t r0, int64_t S, int lane) const
    {
        some<kInstr>(0, tile, src, ss, r0, S, lane);
    }
    // The rows that all waves of a workgroup need, brought in once by all of them: a wave issues instruction `wave`, if there is one.  With
    // each wave loading them straight to its registers, 64 bytes of a row at a time and behind the fills of its own tiles, a workgroup's
    // start was bound by 8 times those bytes through the unit's 64 B per cycle, and no wave began before its second tile had
    // landed; the row pointers also cost registers (head dim 64 backward: 5 spilled, now none).  Forward and backward, us, before -> now:
    // S = 1024 H = 1 d = 64 33.4 -> 32.1, S = 3000 H = 4 d = 128 388 -> 372 (workgroups of many tiles gain least: S = 20000 H = 2 d = 128 1 %).
    // Head dim 64, where another workgroup of the unit can cover a start, does without where that is faster (f32_fwd_shares_rows and
    // f32_bwd_shares_rows, launch_plan.h).
    __device__ __forceinline__ void shared(LDS_AS unsigned char *tile, const float *src, int64_t ss, int64_t r0, int64_t S, int lane, int wave) const
    {
        if (wave < kInstr) some<1>(wave, tile, src, ss, r0, S, lane);
    }
};

// LDS addresses of a lane's operand reads within a tile (bf16_tiles.h has the hand-issued pipeline they go through):
//   row[c % 4] + 256 (c / 4)   row-major operand: row l16, floats 16c + 4*g4 ..
//   tr[r] + 256 h              transposed operand: row 4*g4 + r, floats 64h + 4*l16 .. (of these the workgroup's part)
struct F32Addr { uint32_t row[4], tr[4]; };
template <int D, int CS>
__device__ __forceinline__ F32Addr f32_addr(const LDS_AS unsigned char *base, int l16, int g4, int part)
{
    F32Addr ad;
    const uint32_t b = (uint32_t)(uintptr_t)base;
#pragma unroll
    for (int c = 0; c < 4; ++c) ad.row[c] = b + (uint32_t)(l16 * D * 4 + (((4 * c + g4) ^ SwzB::f(l16)) << 4));
#pragma unroll
    for (int r = 0; r < 4; ++r) ad.tr[r] = b + (uint32_t)((4 * g4 + r) * D * 4 + ((l16 ^ SwzB::f(4 * g4 + r)) << 4) + 16 / CS * part);
    return ad;
}

struct F32Pair { f32x4 x, y; };
template <int N>
__device__ __forceinline__ void lds_wait(F32Pair &p)
{
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(p.x), "+v"(p.y) : "n"(N));
}

// exp(scale s - lse), the probability of a raw score.  The product is rounded before the subtraction, as the forward rounds it
// for its logsumexp: inside an fma the exact product of a score of 1e20 (a masked key) is 1e12 away from that logsumexp.
__device__ __forceinline__ float f32_prob(float s, float scale, float lse)
{
#pragma clang fp contract(off)
    return __builtin_amdgcn_exp2f((s * scale - lse) * kLog2e);
}

// A lane's row of a shared tile that lies `off` bytes from the buffer that ad is for: floats 16c + 4*g4 ..
template <int D, int OFF = 0>
__device__ __forceinline__ void f32_issue_row(f32x4 (&dst)[D / 16], const F32Addr &ad, uint32_t off)
{
    static_for<0, D / 16>([&](auto n) {
        constexpr int c = decltype(n)::value;
        lds_issue_b128<OFF + 256 * (c / 4)>(dst[c], ad.row[c % 4] + off);
    });
}
template <int D>
__device__ __forceinline__ void f32_wait_row(f32x4 (&dst)[D / 16])
{
    static_for<0, D / 16>([&](auto n) { lds_wait<0>(dst[decltype(n)::value]); });
}

// The same row straight from memory to the registers of each wave.
template <int D>
__device__ __forceinline__ void f32_load_row(f32x4 (&dst)[D / 16], const float *row, int g4)
{
#pragma unroll
    for (int c = 0; c < D / 16; ++c) dst[c] = *reinterpret_cast<const f32x4 *>(row + 16 * c + 4 * g4);
}

// The end of the shared fills: `queued` says that this wave has queued its own first two tiles behind them.
template <int D>
__device__ __forceinline__ void f32_shared_rows_complete(bool queued)
{
    if (queued) wait_fills_but<2 * F32Shape<D>::kFills>();
    else wait_fills();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

constexpr int kDepth = 3;         // operand reads in flight ahead of their MFMAs

// CS workgroups share out the output columns of a tile (column_parts, launch_plan.h): block e of a half is in part e / (4 / CS), and a
// workgroup has kBlocks = D / 16 / CS accumulators.
template <int CS> struct F32Cols { float x[4 / CS]; };
template <> struct F32Cols<1> { f32x4 x; };
template <> struct F32Cols<2> { f32x2 x; };
template <int N, int CS>
__device__ __forceinline__ void lds_wait(F32Cols<CS> &c)
{
    if constexpr (CS == 4) asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(c.x[0]) : "n"(N));
    else asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(c.x) : "n"(N));
}
template <int OFF, int CS>
__device__ __forceinline__ void lds_issue_cols(F32Cols<CS> &dst, uint32_t addr)
{
    static_assert(OFF >= 0 && OFF < 65536, "LDS immediate offset");
    if constexpr (CS == 1) lds_issue_b128<OFF>(dst.x, addr);
    else if constexpr (CS == 2) asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(dst.x) : "v"(addr), "n"(OFF) : "memory");
    else asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(dst.x[0]) : "v"(addr), "n"(OFF) : "memory");
}

// acc^T[dim][col] += tile^T x (tile rows 4*g4 + r), tile OFF bytes into the buffer: item n = (r = n / (D/64), h = n % (D/64)),
// one read, 4 / CS MFMAs.  The constructor asks for the first operands ahead of the element-wise work.
template <int D, int OFF, int CS>
struct F32Outer {
    static constexpr int H = D / 64, N = 4 * H, E = 4 / CS;
    F32Cols<CS> ring[kDepth + 1];
    const F32Addr &ad;
    __device__ __forceinline__ F32Outer(const F32Addr &addr) : ad(addr)
    {
        lds_pipeline_prologue<N, kDepth, 1>(ring, [&](auto n, F32Cols<CS> &slot) { issue(n, slot); });
    }
    template <typename I>
    __device__ __forceinline__ void issue(I, F32Cols<CS> &slot)
    {
        lds_issue_cols<OFF + 256 * (I::value % H)>(slot, ad.tr[I::value / H]);
    }
    __device__ __forceinline__ void run(f32x4 (&acc)[D / 16 / CS], const f32x4 &x)
    {
        lds_pipeline_body<N, kDepth, 1>(ring, [&](auto n, F32Cols<CS> &slot) { issue(n, slot); }, [&](auto n, F32Cols<CS> &slot) {
            constexpr int r = decltype(n)::value / H, h = decltype(n)::value % H;
#pragma unroll
            for (int e = 0; e < E; ++e) acc[E * h + e] = mfma4(slot.x[e], x[r], acc[E * h + e]);
        });
    }
};

// A score is added up in four chains, two over each half of the head dim, in the forward and in the backward alike.  The
// logsumexp fits the scores of the backward only if their bits are those of the forward, and a longer chain rounds more often:
// relative error of dV against 64 bits at S = 1500, d = 64, scores of +-40: two chains in the forward and one in the backward
// 4.5e-6, two in both 1.28e-6, four in both 1.18e-6 (O: 7.2e-7, 7.2e-7, 5.2e-7).  The first two are added up under the MFMAs of
// the others.  Forward at S = 5000, H = 4, d = 128: two chains 229 us, four as here 234, four at a time 240.
template <int D>
struct F32Chains {
    f32x4 chain[2] = {kZero4, kZero4}, first;
    template <int C>              // item C of the head dim: 16 floats
    __device__ __forceinline__ void add(const f32x4 &a, const f32x4 &b)
    {
        constexpr bool second_half = C == D / 32;
        f32x4 x, y;
        if constexpr (second_half) {
            x = chain[0], y = chain[1];
            chain[0] = chain[1] = kZero4;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) chain[j % 2] = mfma4(a[j], b[j], chain[j % 2]);
        if constexpr (second_half) {
            first = x + y;
            asm volatile("" : "+v"(first));           // formed here, not at the end
        }
    }
    __device__ __forceinline__ f32x4 sum() const { return first + (chain[0] + chain[1]); }
};

// s = (rows of tile 0) x b0 and dp += (rows of tile 1) x b1 over the head dim: item c, two reads, eight MFMAs
template <int D>
__device__ __forceinline__ void f32_two_scores(f32x4 &s, f32x4 &dp, const F32Addr &ad, const f32x4 (&b0)[D / 16],
                                               const f32x4 (&b1)[D / 16])
{
    constexpr int kTile = kT * D * 4;
    F32Pair ring[2];
    F32Chains<D> scores;
    auto issue = [&](auto n, F32Pair &slot) {
        constexpr int c = decltype(n)::value;
        lds_issue_b128<256 * (c / 4)>(slot.x, ad.row[c % 4]);
        lds_issue_b128<kTile + 256 * (c / 4)>(slot.y, ad.row[c % 4]);
    };
    lds_pipeline_prologue<D / 16, 1, 2>(ring, issue);
    lds_pipeline_body<D / 16, 1, 2>(ring, issue, [&](auto n, F32Pair &slot) {
        constexpr int c = decltype(n)::value;
        scores.template add<c>(slot.x, b0[c]);
#pragma unroll
        for (int j = 0; j < 4; ++j) dp = mfma4(slot.y[j], b1[c][j], dp);
    });
    s = scores.sum();
}

// Accumulator piece p = h * 4/CS + i of a lane, four values: blocks e of rows r = CS * i .. of half h, which are the dims
// 64h + 16*g4 + 4r + 4/CS * part + e of its column (CS = 1: four consecutive ones).
template <int D, int CS>
__device__ __forceinline__ f32x4 f32_piece(const f32x4 (&acc)[D / 16 / CS], int p)
{
    constexpr int E = 4 / CS;
    f32x4 x;
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = acc[E * (p / E) + k % E][CS * (p % E) + k / E];
    return x;
}

// out: the lane's column at dim 16*g4 + 4/CS * part
template <int CS>
__device__ __forceinline__ void f32_store_piece(float *out, int p, const f32x4 &x)
{
    constexpr int E = 4 / CS;
    float *at = out + 64 * (p / E) + 4 * CS * (p % E);
    if constexpr (CS == 1) {
        *reinterpret_cast<f32x4 *>(at) = x;
    } else if constexpr (CS == 2) {
        *reinterpret_cast<f32x2 *>(at) = f32x2{x[0], x[1]};
        *reinterpret_cast<f32x2 *>(at + 4) = f32x2{x[2], x[3]};
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) at[4 * k] = x[k];
    }
}

template <int D> constexpr int kF32FwdLds = F32Shape<D>::kRing + F32Shape<D>::kTile + kF32Waves * 16 * 8;
template <int D> constexpr int kF32BwdLds = F32Shape<D>::kRing + 2 * F32Shape<D>::kTile;

// lds: [wave][K|V] tiles, the Q rows, (maximum, sum) per wave and row
template <int D, bool FAR, int CS, bool SHARED>
__device__ __forceinline__ void f32_fwd_rows(const AttnArgs &a, LDS_AS unsigned char *lds, const TileId t, int part)
{
    using Shape = F32Shape<D>;
    constexpr int KS = kF32Waves, NP = Shape::kPieces / CS;
    constexpr int kStats = Shape::kRing + Shape::kTile;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh;
    const float *k = static_cast<const float *>(a.k) + base, *v = static_cast<const float *>(a.v) + base;
    const int64_t row0 = (int64_t)t.tile * kT, i = row0 + l16;
    const int ntiles = t.tile + 1;                    // the last one is the diagonal
    const float c = a.scale * kLog2e;
    LDS_AS unsigned char *ring = lds + wave * Shape::kStage;
    const F32Fill<D, FAR> fill(a.ss, lane);
    auto fill_k = [&](int jt) { fill(ring, k, a.ss, (int64_t)jt * kT, a.S, lane); };
    auto fill_v = [&](int jt) { fill(ring + Shape::kTile, v, a.ss, (int64_t)jt * kT, a.S, lane); };
    if constexpr (SHARED) fill.shared(lds + Shape::kRing, static_cast<const float *>(a.q) + base, a.ss, row0, a.S, lane, wave);
    if (wave < ntiles) {
        fill_k(wave);
        fill_v(wave);
    }
    __builtin_amdgcn_sched_barrier(0);                // addresses and accumulators are set up while the loads are on their way
    const F32Addr ad = f32_addr<D, CS>(ring, l16, g4, part);
    f32x4 q[D / 16], acc[D / 16 / CS];                // rows past S are computed and never stored
    if constexpr (!SHARED) f32_load_row<D>(q, static_cast<const float *>(a.q) + base + (i < a.S ? i : a.S - 1) * a.ss, g4);
#pragma unroll
    for (int n = 0; n < D / 16 / CS; ++n) acc[n] = kZero4;
    if constexpr (SHARED) {
        f32_shared_rows_complete<D>(wave < ntiles);
        f32_issue_row<D>(q, ad, (uint32_t)(Shape::kRing - wave * Shape::kStage));
        f32_wait_row<D>(q);
    }
    float m = -INFINITY, lsum = 0.f;                  // running maximum and sum of this lane's keys

    for (int jt = wave; jt < ntiles; jt += KS) {
        const bool more = jt + KS < ntiles;
        wait_fills_but<Shape::kFills>();              // K has landed; V, queued behind it, may still be on its way
        F32Chains<D> scores;
        {
            f32x4 kring[kDepth + 1];
            auto issue = [&](auto m, f32x4 &slot) {
                constexpr int cc = decltype(m)::value;
                lds_issue_b128<256 * (cc / 4)>(slot, ad.row[cc % 4]);
            };
            lds_pipeline_prologue<D / 16, kDepth, 1>(kring, issue);
            lds_pipeline_body<D / 16, kDepth, 1>(kring, issue, [&](auto m, f32x4 &slot) {
                scores.template add<decltype(m)::value>(slot, q[decltype(m)::value]);
            });
        }
        if (more) {
            fill_k(jt + KS);      // K is used up
            wait_fills_but<Shape::kFills>();
        } else {
            wait_fills();
        }
        F32Outer<D, Shape::kTile, CS> pv(ad);         // the first V operands: their latency hides behind the softmax
        f32x4 s = scores.sum();
        if (jt == ntiles - 1) {         // key 4*g4 + r of the tile is visible to query l16 iff it is <= l16
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (4 * g4 + r > l16) s[r] = -INFINITY;
        }
        // against the running maximum as it stands: it only has to keep the exponentials in range (as in the bf16 forward).
        // The difference comes before the scale: exact for the maximum itself, however large (a row of masked keys only)
        f32x4 p;
        auto exponentials = [&]() {
#pragma unroll
            for (int r = 0; r < 4; ++r) p[r] = __builtin_amdgcn_exp2f((s[r] - m) * c);
        };
        exponentials();
        if (__builtin_amdgcn_ballot_w64(!(p[0] + p[1] + p[2] + p[3] <= kF32RescaleAbove)) != 0) {
            float mt = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
            mt = fmaxf(mt, __shfl_xor(mt, 16));
            mt = fmaxf(mt, __shfl_xor(mt, 32));
            // finite also where a row sees nothing but scores of -inf in the tile: they weigh zero then
            const float m_new = fmaxf(fmaxf(m, mt), kLowest);
            const float corr = __builtin_amdgcn_exp2f((m - m_new) * c);
            m = m_new;
            lsum *= corr;
#pragma unroll
            for (int e = 0; e < D / 16 / CS; ++e) acc[e] *= corr;
            exponentials();
        }
        lsum += (p[0] + p[1]) + (p[2] + p[3]);
        pv.run(acc, p);                               // O^T += V^T P^T
        if (more) fill_v(jt + KS);
    }
    lsum += __shfl_xor(lsum, 16);
    lsum += __shfl_xor(lsum, 32);

    LDS_AS f32x4 *pieces = (LDS_AS f32x4 *)lds;
    LDS_AS f32x2 *stats = (LDS_AS f32x2 *)(lds + kStats);
#pragma unroll
    for (int p = 0; p < NP; ++p) pieces[(wave * Shape::kSet + p) * 64 + lane] = f32_piece<D, CS>(acc, p);
    if (g4 == 0) stats[wave * 16 + l16] = f32x2{m, lsum};
    __syncthreads();
    float top = -INFINITY, total = 0.f, weight[KS];
    f32x2 st[KS];
#pragma unroll
    for (int g = 0; g < KS; ++g) {
        st[g] = stats[g * 16 + l16];
        top = fmaxf(top, st[g][0]);
    }
#pragma unroll
    for (int g = 0; g < KS; ++g) {
        weight[g] = __builtin_amdgcn_exp2f((st[g][0] - top) * c); // a group without a tile: m = -inf, weight zero
        total += weight[g] * st[g][1];
    }
    if (i >= a.S) return;
    float *o = static_cast<float *>(a.o_out) + base + i * a.ss + 16 * g4 + 4 / CS * part;
    const float inv = 1.f / total;
    for (int p = wave; p < NP; p += KS) {
        f32x4 sum = kZero4;
#pragma unroll
        for (int g = 0; g < KS; ++g) sum += weight[g] * pieces[(g * Shape::kSet + p) * 64 + lane];
        f32_store_piece<CS>(o, p, sum * inv);
    }
    if (wave == 0 && g4 == 0 && part == 0) {
#pragma clang fp contract(off)    // the rounded product, as in f32_prob
        a.lse[((int64_t)t.b * a.H + t.h) * a.S + i] = top * a.scale + __builtin_amdgcn_logf(total) * kLn2;
    }
}

// Adds up the accumulators of the eight waves and writes mul times them: out points at the lane's row.
template <int D, int CS, bool kFirst>
__device__ __forceinline__ void f32_combine(LDS_AS unsigned char *lds, const f32x4 (&acc)[D / 16 / CS], float *out, bool live, float mul,
                                            int wave, int lane)
{
    using Shape = F32Shape<D>;
    constexpr int NP = Shape::kPieces / CS, KS = kF32Waves;
    LDS_AS f32x4 *pieces = (LDS_AS f32x4 *)lds;
    if (!kFirst) __syncthreads(); // every wave has read the sum before
#pragma unroll
    for (int p = 0; p < NP; ++p) pieces[(wave * Shape::kSet + p) * 64 + lane] = f32_piece<D, CS>(acc, p);
    __syncthreads();
    for (int p = wave; p < NP; p += KS) {
        f32x4 sum = kZero4;
#pragma unroll
        for (int g = 0; g < KS; ++g) sum += pieces[(g * Shape::kSet + p) * 64 + lane];
        if (live) f32_store_piece<CS>(out, p, sum * mul);
    }
}

// dQ_i = scale * sum_{j<=i} dS_ij k_j, dS_ij = P_ij (dO_i.v_j - D_i), P_ij = exp(s_ij - LSE_i); rows = queries
template <int D, bool FAR, int CS, bool SHARED>
__device__ __forceinline__ void f32_dq_rows(const AttnArgs &a, LDS_AS unsigned char *lds, const TileId t, int part)
{
    using Shape = F32Shape<D>;
    constexpr int KS = kF32Waves;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh, stat = ((int64_t)t.b * a.H + t.h) * a.S;
    const float *k = static_cast<const float *>(a.k) + base, *v = static_cast<const float *>(a.v) + base;
    const int64_t i = (int64_t)t.tile * kT + l16, iq = i < a.S ? i : a.S - 1;
    const int ntiles = t.tile + 1;                    // the last one is the diagonal
    LDS_AS unsigned char *ring = lds + wave * Shape::kStage;
    const F32Fill<D, FAR> fill(a.ss, lane);
    auto fill_k = [&](int jt) { fill(ring, k, a.ss, (int64_t)jt * kT, a.S, lane); };
    auto fill_v = [&](int jt) { fill(ring + Shape::kTile, v, a.ss, (int64_t)jt * kT, a.S, lane); };
    const float lse = a.lse[stat + iq], nd = -a.delta[stat + iq];
    if constexpr (SHARED) {
        fill.shared(lds + Shape::kRing, static_cast<const float *>(a.q) + base, a.ss, (int64_t)t.tile * kT, a.S, lane, wave);
        fill.shared(lds + Shape::kRing + Shape::kTile, static_cast<const float *>(a.d_o) + base, a.ss, (int64_t)t.tile * kT, a.S, lane, wave);
    }
    if (wave < ntiles) {
        fill_k(wave);
        fill_v(wave);
    }
    __builtin_amdgcn_sched_barrier(0);                // addresses and accumulators are set up while the loads are on their way
    const F32Addr ad = f32_addr<D, CS>(ring, l16, g4, part);
    f32x4 q[D / 16], go[D / 16], acc[D / 16 / CS];
    if constexpr (!SHARED) {
        f32_load_row<D>(q, static_cast<const float *>(a.q) + base + iq * a.ss, g4);
        f32_load_row<D>(go, static_cast<const float *>(a.d_o) + base + iq * a.ss, g4);
    }
#pragma unroll
    for (int n = 0; n < D / 16 / CS; ++n) acc[n] = kZero4;
    if constexpr (SHARED) {
        f32_shared_rows_complete<D>(wave < ntiles);
        f32_issue_row<D>(q, ad, (uint32_t)(Shape::kRing - wave * Shape::kStage));
        f32_issue_row<D, Shape::kTile>(go, ad, (uint32_t)(Shape::kRing - wave * Shape::kStage));
        f32_wait_row<D>(q);
        f32_wait_row<D>(go);
    }
    for (int jt = wave; jt < ntiles; jt += KS) {
        const bool more = jt + KS < ntiles;
        wait_fills();
        f32x4 s, dp = {nd, nd, nd, nd};               // keys 4*g4 + r x query l16
        f32_two_scores<D>(s, dp, ad, q, go);
        if (more) fill_v(jt + KS);                    // V is used up
        F32Outer<D, 0, CS> kds(ad);
        if (jt == ntiles - 1) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (4 * g4 + r > l16) s[r] = -INFINITY;
        }
        f32x4 ds;
#pragma unroll
        for (int r = 0; r < 4; ++r) ds[r] = f32_prob(s[r], a.scale, lse) * dp[r];
        kds.run(acc, ds);                             // dQ^T += K^T dS^T
        if (more) fill_k(jt + KS);
    }
    f32_combine<D, CS, true>(lds, acc, static_cast<float *>(a.dq) + base + iq * a.ss + 16 * g4 + 4 / CS * part, i < a.S, a.scale, wave, lane);
}

// dV_j = sum_{i>=j} P_ij dO_i,  dK_j = scale * sum_{i>=j} dS_ij q_i; rows = keys, K and V rows in registers
template <int D, bool FAR, int CS, bool SHARED>
__device__ __forceinline__ void f32_dkdv_rows(const AttnArgs &a, LDS_AS unsigned char *lds, const TileId t, int part)
{
    using Shape = F32Shape<D>;
    constexpr int QS = kF32Waves;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh, stat = ((int64_t)t.b * a.H + t.h) * a.S;
    const float *q = static_cast<const float *>(a.q) + base, *g = static_cast<const float *>(a.d_o) + base;
    const int64_t col0 = (int64_t)t.tile * kT, j = col0 + l16, jk = j < a.S ? j : a.S - 1;
    const int it0 = t.tile, ntiles = (int)((a.S + kT - 1) / kT);
    LDS_AS unsigned char *ring = lds + wave * Shape::kStage;
    const F32Fill<D, FAR> fill(a.ss, lane);
    auto fill_q = [&](int it) { fill(ring, q, a.ss, (int64_t)it * kT, a.S, lane); };
    auto fill_g = [&](int it) { fill(ring + Shape::kTile, g, a.ss, (int64_t)it * kT, a.S, lane); };
    auto load_stats = [&](int it, f32x4 &l, f32x4 &d) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {                 // rows past S: LSE = +inf makes their P exactly zero
            const int64_t row = (int64_t)it * kT + 4 * g4 + r;
            l[r] = row < a.S ? a.lse[stat + row] : INFINITY;
            d[r] = row < a.S ? a.delta[stat + row] : 0.f;
        }
    };
    f32x4 lse_n = kZero4, dl_n = kZero4;
    if (it0 + wave < ntiles) load_stats(it0 + wave, lse_n, dl_n);
    if constexpr (SHARED) {
        fill.shared(lds + Shape::kRing, static_cast<const float *>(a.k) + base, a.ss, col0, a.S, lane, wave);
        fill.shared(lds + Shape::kRing + Shape::kTile, static_cast<const float *>(a.v) + base, a.ss, col0, a.S, lane, wave);
    }
    if (it0 + wave < ntiles) {
        fill_q(it0 + wave);
        fill_g(it0 + wave);
    }
    __builtin_amdgcn_sched_barrier(0);                // addresses and accumulators are set up while the loads are on their way
    const F32Addr ad = f32_addr<D, CS>(ring, l16, g4, part);
    f32x4 kr[D / 16], vr[D / 16], dk[D / 16 / CS], dv[D / 16 / CS];
    if constexpr (!SHARED) {
        f32_load_row<D>(kr, static_cast<const float *>(a.k) + base + jk * a.ss, g4);
        f32_load_row<D>(vr, static_cast<const float *>(a.v) + base + jk * a.ss, g4);
    }
#pragma unroll
    for (int n = 0; n < D / 16 / CS; ++n) dk[n] = dv[n] = kZero4;
    if constexpr (SHARED) {
        f32_shared_rows_complete<D>(it0 + wave < ntiles);
        f32_issue_row<D>(kr, ad, (uint32_t)(Shape::kRing - wave * Shape::kStage));
        f32_issue_row<D, Shape::kTile>(vr, ad, (uint32_t)(Shape::kRing - wave * Shape::kStage));
        f32_wait_row<D>(kr);
        f32_wait_row<D>(vr);
    }
    for (int it = it0 + wave; it < ntiles; it += QS) {
        const bool more = it + QS < ntiles;
        wait_fills();
        const f32x4 lse = lse_n, dl = dl_n;
        if (more) load_stats(it + QS, lse_n, dl_n);
        f32x4 s, dp;                                  // queries 4*g4 + r x key l16
#pragma unroll
        for (int r = 0; r < 4; ++r) dp[r] = -dl[r];
        f32_two_scores<D>(s, dp, ad, kr, vr);
        F32Outer<D, Shape::kTile, CS> gp(ad);
        if (it == it0) {         // query 4*g4 + r of the tile sees key l16 iff it is >= l16
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (4 * g4 + r < l16) s[r] = -INFINITY;
        }
        if (it == ntiles - 1) {   // rows past S were read as zero, and zero times an infinite key is NaN: their LSE of +inf does not do
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if ((int64_t)it * kT + 4 * g4 + r >= a.S) s[r] = -INFINITY;
        }
        f32x4 p, ds;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            p[r] = f32_prob(s[r], a.scale, lse[r]);
            ds[r] = p[r] * dp[r];
        }
        gp.run(dv, p);                                // dV^T += dO^T P
        if (more) fill_g(it + QS);                    // dO is used up
        F32Outer<D, 0, CS> qds(ad);
        qds.run(dk, ds);                              // dK^T += Q^T dS
        if (more) fill_q(it + QS);
    }
    f32_combine<D, CS, true>(lds, dv, static_cast<float *>(a.dv) + base + jk * a.ss + 16 * g4 + 4 / CS * part, j < a.S, 1.f, wave, lane);
    f32_combine<D, CS, false>(lds, dk, static_cast<float *>(a.dk) + base + jk * a.ss + 16 * g4 + 4 / CS * part, j < a.S, a.scale, wave, lane);
}

}  // namespace
}  // namespace memo

// Token-wise recomputation of the first saved tensors of a layer (Section 4.1 of the paper:
// the stored layer input is what "input_norm", "q", "k", "v" are rebuilt from): LayerNorm over
// the hidden dimension and the projection that follows it, both restricted to a row range
// [row_begin, row_end) so that only the dropped tokens are recomputed.  Each output row depends
// on its own input row only and is accumulated in a fixed order, so a row recomputed in any
// range is bit-identical to the same row of a full pass.
#include "bf16_tiles.h"

namespace memo {
namespace {

// ---------------------------------------------------------------------------- LayerNorm
// One wave per row, 8 consecutive elements per lane and 512-element chunk; fp32 statistics in two
// passes over the registers (mean, then centred sum of squares).  HBM-bound: 2*h*2 bytes per row.
constexpr int kLnMaxChunks = 16;            // h <= 8192

template <int NCH>                          // h = 512 * NCH: the row lives in 8 * NCH registers per lane
__global__ __launch_bounds__(256) void layernorm_rows_bf16_kernel(const __bf16 *x, const __bf16 *gamma,
                                                                  const __bf16 *beta, __bf16 *y, int64_t row_begin,
                                                                  int64_t row_end, int h, float eps)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = row_begin + (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= row_end) return;
    constexpr int nch = NCH;
    const __bf16 *xr = x + row * h;
    float v[NCH][8];
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        if (c < nch) {
            const bf16x8 raw = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(xr + c * 512 + lane * 8));
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                v[c][e] = (float)raw[e];
                sum += v[c][e];
            }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    const float mean = sum / (float)h;
    float sq = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c)
        if (c < nch)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float dlt = v[c][e] - mean;
                sq = fmaf(dlt, dlt, sq);
            }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
    const float rstd = 1.0f / sqrtf(sq / (float)h + eps);
    __bf16 *yr = y + row * h;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        if (c < nch) {
            const bf16x8 gm = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(gamma + c * 512 + lane * 8));
            const bf16x8 bt = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(beta + c * 512 + lane * 8));
            bf16x8 out;
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                f32x2 two = {fmaf((v[c][e] - mean) * rstd, (float)gm[e], (float)bt[e]),
                             fmaf((v[c][e + 1] - mean) * rstd, (float)gm[e + 1], (float)bt[e + 1])};
                bf16x2 r = __builtin_convertvector(two, bf16x2);
                out[e] = r[0];
                out[e + 1] = r[1];
            }
            *reinterpret_cast<u32x4 *>(yr + c * 512 + lane * 8) = __builtin_bit_cast(u32x4, out);
        }
    }
}

// ---------------------------------------------------------------------------- projection
// out[token, feature] = sum_c a[token, c] * w[feature, c] + bias[feature]   (w as [N, K], K contiguous)
// Workgroup: 8 waves as WM x WN, a wave's tile TB x FB blocks of 16 tokens x 16 features:
// D[feature, token] = W_rows * A_rows^T on v_mfma_f32_16x16x32_bf16, so a lane holds one token and 4
// consecutive features per accumulator.  K is streamed in chunks of 64 through LDS, token rows and weight
// rows in rings of their own (ST and SW chunks deep).  A workgroup works several tiles, one after the other, and
// the stream of chunks does not stop between them: the next tile's first chunks arrive under the last MFMAs and the
// stores of the one before.
//
// What bounds it: a 256 x 256 tile is worked at the rate the MFMAs sustain under the power limit, within a tenth; short
// launches are bound by how few tiles there are, so that the tile shrinks with the work (launch_plan.h), and the smallest
// by the latency of a chunk: barrier, operand reads, MFMAs.  Steps of the 256 x 256 shape at 138937 x 4096 -> 1536:
// one barrier, the fills and the wait for the operands in front of every chunk's MFMAs 1531 us; operands and fills a
// chunk ahead as described at `phase` 1370; stream not stopped between tiles, 16-byte stores 1309.
//
// Operand conventions of the 16x16x32 MFMA, D = A(16xK32) * B(K32x16), lane = 16*g4 + l16:
//   A : lane holds row l16, k = 8*g4 .. 8*g4+7;  B : lane holds col l16, k = 8*g4 .. 8*g4+7;
//   D : lane holds col l16, rows 4*g4 + r for register r (4 fp32).
// Row 4*g + r of feature block 2p + j is feature 32p + 8g + 4j + r, so that a lane's accumulators of two blocks are 8
// consecutive features: one 16-byte store.
// Every shape adds up K in the same order with the same instruction, so a row's result does not depend on
// the shape that computed it.
//
// An LDS row is one chunk of one matrix row, 128 or 256 bytes; its 16-byte piece c sits at position c ^ tok_swz(r)
// (token rows) or c ^ wgt_swz(r) (weight rows, read in the order above).  Both keep the reads on distinct banks.
template <int RB> __device__ __forceinline__ int tok_swz(int r) { return RB == 128 ? (r >> 1) & 7 : r & 15; }
template <int RB> __device__ __forceinline__ int wgt_swz(int r)
{
    return RB == 128 ? ((r >> 2) & 6) | ((r >> 1) & 1) : ((r >> 1) & 12) | (r & 3);
}

template <int WM_, int WN_, int TB_, int FB_, int ST_, int SW_, int KPH_>
struct LinShape {
    static constexpr int WM = WM_, WN = WN_, TB = TB_, FB = FB_;   // waves and 16-blocks per wave along tokens, features
    static constexpr int ST = ST_, SW = SW_;                       // ring depths in chunks
    static constexpr int KPH = KPH_, RB = 128 * KPH;               // 32-wide k steps of half a chunk; bytes of a chunk's row
    static constexpr int BM = 16 * WM * TB, BN = 16 * WN * FB;
    static constexpr int kTokTile = BM * RB, kWgtTile = BN * RB, kWgtOff = ST * kTokTile;
    static constexpr int kLds = ST * kTokTile + SW * kWgtTile;
    static constexpr int NT = kTokTile / 8192, NW = kWgtTile / 8192;   // fill instructions per wave and chunk
    static_assert(WM * WN == 8 && BM % 64 == 0 && BN % 64 == 0 && FB % 2 == 0 && kLds <= 160 * 1024, "workgroup shape");
    // the waits count fills in issue order: tokens run at most one chunk ahead of the weights, and what the first chunk
    // of a tile needs was queued before the stores of the tile before it
    static_assert(SW >= 2 && ST >= 3 && (ST == SW || ST == SW + 1), "ring depths");
};

// One operand's sequence of chunks over the tiles of a workgroup, as a buffer whose base is the tile's first row:
// rows past the end of the matrix are out of the buffer's range and read as zero (their results are never stored).
// Behind the last chunk the buffer is empty: the fills are still issued, so that every wait counts the same.  The range check
// subtracts the scalar offset from the buffer's size, so that an empty buffer's stays zero (a larger one would wrap and let
// the fill read).
struct ChunkStream {
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t tile;                // the tile that is being fetched
    int chunk;                    // its next chunk
    uint32_t off, step;           // the chunk's byte offset in a row; from one chunk to the next
};

template <typename Sh>
__global__ __launch_bounds__(512, 2) void linear_rows_bf16_kernel(const __bf16 *a, const __bf16 *w, const __bf16 *bias,
                                                                            __bf16 *out, int64_t row_begin, int64_t row_end,
                                                                            int K, int N, uint32_t ntiles)
{
    constexpr int TB = Sh::TB, FB = Sh::FB, KPH = Sh::KPH, RB = Sh::RB, NT = Sh::NT, NW = Sh::NW, ST = Sh::ST, SW = Sh::SW;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[Sh::kLds];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;   // [token ring][weight ring]

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % Sh::WM, wn = wave / Sh::WM;
    const uint32_t ntn = (uint32_t)(N + Sh::BN - 1) / Sh::BN;
    // Workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2.  Every XCD works through a
    // contiguous range of (token tile, feature tile) pairs, its workgroups side by side, with the feature tile
    // running fastest: the workgroups that share a token tile then run on one XCD close
    // in time, and the token rows are fetched from HBM once instead of once per feature tile.
    const uint32_t xcd = blockIdx.x % 8, per = ntiles / 8, rem = ntiles % 8;
    const uint32_t stride = gridDim.x / 8 + (xcd < gridDim.x % 8 ? 1 : 0);      // workgroups of this XCD
    const uint32_t tile0 = xcd * per + (xcd < rem ? xcd : rem) + blockIdx.x / 8;
    const uint32_t tile_end = (xcd + 1) * per + (xcd + 1 < rem ? xcd + 1 : rem);
    if (tile0 >= tile_end) return;
    const int nchunks = K / (RB / 2);                 // K is a multiple of 128

    // operand read addresses: piece 4*ks + g4 of this lane's row
    uint32_t tok_addr[2 * KPH], wgt_addr[2 * KPH];
#pragma unroll
    for (int ks = 0; ks < 2 * KPH; ++ks) {
        const int wrow = 8 * (l16 >> 2) + (l16 & 3);
        tok_addr[ks] = (uint32_t)(uintptr_t)lds + (uint32_t)((16 * TB * wm + l16) * RB + (((4 * ks + g4) ^ tok_swz<RB>(l16)) << 4));
        wgt_addr[ks] = (uint32_t)(uintptr_t)lds + (uint32_t)(Sh::kWgtOff + (16 * FB * wn + wrow) * RB + (((4 * ks + g4) ^ wgt_swz<RB>(wrow)) << 4));
    }
    // fills: instruction n of this wave covers the 1024 / RB tile rows from (wave + 8 n) * 1024 / RB on; the swizzles do
    // not depend on n, so one offset register per operand serves them all
    constexpr int kPieces = RB / 16;
    const int frow = (64 / kPieces) * wave + lane / kPieces, fpiece = lane % kPieces;
    const uint32_t tok_off = (uint32_t)frow * (uint32_t)K * 2 + (uint32_t)(fpiece ^ tok_swz<RB>(frow)) * 16;
    const uint32_t wgt_off = (uint32_t)frow * (uint32_t)K * 2 + (uint32_t)(fpiece ^ wgt_swz<RB>(frow)) * 16;
    uint32_t fill_step = (uint32_t)K * (2 * 8192 / RB);         // bytes between the rows of instructions n and n + 1
    const uint32_t row_bytes = (uint32_t)K * 2;
    auto start = [&](ChunkStream &s, uint32_t tile, const __bf16 *rows_at, int rows) {
        s.rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16 *>(rows_at), 0, (uint32_t)rows * row_bytes, 0x00020000);
        s.tile = tile;
        s.chunk = 0;
        s.off = 0;
        s.step = rows > 0 ? RB : 0;
    };
    auto tok_tile = [&](ChunkStream &s, uint32_t tile) {
        const RowWindow r = row_window(row_begin, row_end, tile / ntn, Sh::BM, tile < tile_end);
        start(s, tile, a + r.first * K, r.rows);
    };
    auto wgt_tile = [&](ChunkStream &s, uint32_t tile) {
        const RowWindow r = row_window(0, N, tile % ntn, Sh::BN, tile < tile_end);
        start(s, tile, w + r.first * K, r.rows);
    };
    ChunkStream ts, ws;
    tok_tile(ts, tile0);
    wgt_tile(ws, tile0);
    int tslot = 0, wslot = 0;                         // ring slots the next chunks go to
    auto next = [](int slot, int depth) { return slot + 1 == depth ? 0 : slot + 1; };
    auto fill_tok = [&](int n) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ts.rsrc, (LDS_AS void *)(lds + tslot * Sh::kTokTile + (wave + 8 * n) * 1024), 16,
                                                 tok_off + n * fill_step, ts.off, 0, 0);
    };
    auto fill_wgt = [&](int n) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ws.rsrc, (LDS_AS void *)(lds + Sh::kWgtOff + wslot * Sh::kWgtTile + (wave + 8 * n) * 1024), 16,
                                                 wgt_off + n * fill_step, ws.off, 0, 0);
    };
    auto tok_done = [&]() {       // the chunk's fills are queued: on to the next one
        tslot = next(tslot, ST);
        ts.off += ts.step;
        if (++ts.chunk == nchunks) tok_tile(ts, ts.tile + stride);
    };
    auto wgt_done = [&]() {
        wslot = next(wslot, SW);
        ws.off += ws.step;
        if (++ws.chunk == nchunks) wgt_tile(ws, ws.tile + stride);
    };

    f32x4 acc[FB][TB];                               // [feature block of 16][token block of 16]
    auto clear = [&]() {
#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
#pragma unroll
            for (int t = 0; t < TB; ++t) acc[fb][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    };

    // Chunk g (counted over all tiles) is worked in two phases of KPH k steps.  Sync point g lies in its second one, when
    // every operand of chunk g is in registers: chunk g + 1 has landed, and the slots of chunk g are free for the
    // weights of chunk g + SW (queued behind the sync point) and the tokens of chunk g + ST (queued in the next phase).
    // Behind it the operands of chunk g + 1 are read between the MFMAs of chunk g, so neither a
    // fill nor an LDS read is waited for unless it takes longer than the MFMAs above it.
    bf16x8 xa[2][KPH * FB], xb[2][KPH * TB];          // two operand sets
    constexpr int kReads = KPH * (TB + FB), kMfmas = KPH * TB * FB;
    uint32_t ra = 0, rb = 0;                          // ring offsets of the chunk being read
    auto read = [&](auto setc, auto ks0c, auto rc) {
        constexpr int set = decltype(setc)::value, r = decltype(rc)::value % (TB + FB);
        constexpr int s = decltype(rc)::value / (TB + FB), ks = decltype(ks0c)::value + s, fb = r - TB;
        if constexpr (r < TB) lds_issue_b128<r * 16 * RB>(xb[set][s * TB + r], tok_addr[ks] + rb);
        else lds_issue_b128<((fb / 2) * 32 + (fb % 2) * 4) * RB>(xa[set][s * FB + fb], wgt_addr[ks] + ra);
    };
    auto wait_reads = [&](auto setc) {
        constexpr int set = decltype(setc)::value;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < KPH * FB; ++i) {
            bf16x8 &x = xa[set][i];
            asm volatile("" : "+v"(x));
        }
#pragma unroll
        for (int i = 0; i < KPH * TB; ++i) {
            bf16x8 &x = xb[set][i];
            asm volatile("" : "+v"(x));
        }
    };
    // In flight behind the chunk a sync point needs: younger fills, and the stores of a tile that was finished since
    constexpr int kBehind = (ST - 2) * NT + (SW - 2) * NW, kStores = TB * FB / 2;
    static_assert(kBehind + kStores <= 63, "vmcnt range");
    constexpr int kNever = -2;
    int stores_at = kNever;       // the sync point in front of which a whole tile's stores were issued
    auto arrive = [&](int g) {
        asm volatile("s_cmp_eq_u32 %0, %1\n\ts_cbranch_scc1 .Lstores%=\n\ts_waitcnt vmcnt(%2)\n.Lstores%=:\n\ts_waitcnt vmcnt(%3)"
                     :: "s"(g), "s"(stores_at), "n"(kBehind), "n"(kBehind + kStores) : "memory", "scc");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // one phase: MFMAs of operand set `set`, the reads of the other set (k steps from ks0), the sync point (SYNC) and
    // the fills dealt out between them
    auto phase = [&](auto setc, auto ks0c, auto syncc, int g) {
        constexpr int set = decltype(setc)::value;
        constexpr bool sync = decltype(syncc)::value != 0;
        constexpr int first = kMfmas >= 32 && sync ? kMfmas / 4 : 0;            // MFMAs before the sync point
        constexpr int span = kMfmas >= 32 ? kMfmas / 2 : (kMfmas + 1) / 2;
        constexpr int nfills = sync ? NW : NT;
        static_for<0, kMfmas>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            if constexpr (sync && m == first) {
                arrive(g);
                ra = (ra + Sh::kWgtTile == SW * Sh::kWgtTile) ? 0 : ra + Sh::kWgtTile;
                rb = (rb + Sh::kTokTile == ST * Sh::kTokTile) ? 0 : rb + Sh::kTokTile;
            }
            if constexpr (m >= first) {
                static_for<0, kReads>([&](auto rc) {
                    if constexpr (first + decltype(rc)::value * span / kReads == m) read(IntC<set ^ 1>{}, ks0c, rc);
                });
                static_for<0, nfills>([&](auto nc) {
                    constexpr int n = decltype(nc)::value;
                    if constexpr (first + n * (kMfmas - first) / nfills == m) {
                        if constexpr (sync) fill_wgt(n);
                        else fill_tok(n);
                    }
                });
            }
            constexpr int s = m / (TB * FB), fb = m % (TB * FB) / TB, t = m % TB;
            acc[fb][t] = mfma16(xa[set][s * FB + fb], xb[set][s * TB + t], acc[fb][t]);
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (sync) wgt_done();
        else tok_done();
        wait_reads(IntC<set ^ 1>{});
    };

    // acc[fb][t][r] is token m0 + 16 (TB wm + t) + l16, feature n0 + 16 FB wn + 32 (fb / 2) + 8 g4 + 4 (fb % 2) + r.
    // True if every store of the tile was issued (a tile at the edge leaves some out)
    auto finish = [&](uint32_t tile) {
        const int64_t m0 = row_begin + (int64_t)(tile / ntn) * Sh::BM + 16 * TB * wm;
        const int f0 = (int)(tile % ntn) * Sh::BN + 16 * FB * wn;
        const bool whole = m0 + 16 * TB <= row_end && f0 + 16 * FB <= N;
        int ln = lane;            // opaque copy: the addresses are formed here, once per tile, not kept in registers
        asm volatile("" : "+v"(ln));
        const int l16 = ln & 15, g4 = ln >> 4;
        __bf16 *obase = out + (m0 + l16) * N + f0 + 8 * g4;
#pragma unroll
        for (int p = 0; p < FB / 2; ++p) {
            if (f0 + 32 * p >= N) continue;           // N is a multiple of 32: a pair of blocks is whole or absent
            float b8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (bias) {                               // by scalar loads: a vector load would wait for the fills queued before it
                const __attribute__((address_space(4))) uint32_t *bp =
                    (const __attribute__((address_space(4))) uint32_t *)(bias + f0 + 32 * p);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t lo = g4 & 1 ? bp[4 + i] : bp[i], hi = g4 & 1 ? bp[12 + i] : bp[8 + i];
                    const uint32_t two = g4 & 2 ? hi : lo;
                    b8[2 * i] = __builtin_bit_cast(float, two << 16);
                    b8[2 * i + 1] = __builtin_bit_cast(float, two & 0xffff0000u);
                }
            }
#pragma unroll
            for (int t = 0; t < TB; ++t) {
                const f32x4 &x = acc[2 * p][t], &y = acc[2 * p + 1][t];
                const bf16x8 r = pack44(f32x4{x[0] + b8[0], x[1] + b8[1], x[2] + b8[2], x[3] + b8[3]},
                                        f32x4{y[0] + b8[4], y[1] + b8[5], y[2] + b8[6], y[3] + b8[7]});
                if (whole || m0 + 16 * t + l16 < row_end)
                    *reinterpret_cast<u32x4 *>(obase + (int64_t)(16 * t) * N + 32 * p) = __builtin_bit_cast(u32x4, r);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        return whole;
    };

    // the fills of sync points -ST .. -2, then sync point -1
#pragma unroll
    for (int s = -ST; s < 0; ++s) {
        if (s == -1) arrive(-1);
        if (s + SW >= 0) {
#pragma unroll
            for (int n = 0; n < NW; ++n) fill_wgt(n);
            wgt_done();
        }
        if (s < -1) {             // the tokens of sync point -1 follow in the first phase
#pragma unroll
            for (int n = 0; n < NT; ++n) fill_tok(n);
            tok_done();
        }
    }
    static_for<0, kReads>([&](auto rc) { read(IntC<0>{}, IntC<0>{}, rc); });
    wait_reads(IntC<0>{});
    int g = 0;
#pragma clang loop unroll(disable)
    for (uint32_t tile = tile0; tile < tile_end; tile += stride) {
        clear();
        const int tile_chunks = g + nchunks;
#pragma clang loop unroll(disable)
        do {
            asm volatile("" : "+s"(fill_step));       // the fill offsets are formed where they are used, not kept in registers
            phase(IntC<0>{}, IntC<KPH>{}, IntC<0>{}, g);
            phase(IntC<1>{}, IntC<0>{}, IntC<1>{}, g);
            ++g;
        } while (g < tile_chunks);
        stores_at = finish(tile) ? g : kNever;
    }
    wait_fills();                 // the empty fills behind the last chunk write LDS too: none may outlive the workgroup
}

}  // namespace

hipError_t launch_layernorm_rows_bf16(const void *x, const void *gamma, const void *beta, void *y, int64_t row_begin,
                                      int64_t row_end, int h, float eps, hipStream_t st)
{
    const int64_t rows = row_end - row_begin;
    if (rows <= 0) return hipSuccess;
    const int64_t blocks = (rows + 3) / 4;
    if (blocks > 0x7fffffffLL || h % 512 || h / 512 > kLnMaxChunks) return hipErrorInvalidValue;
    const __bf16 *xp = static_cast<const __bf16 *>(x), *gp = static_cast<const __bf16 *>(gamma);
    const __bf16 *bp = static_cast<const __bf16 *>(beta);
    __bf16 *yp = static_cast<__bf16 *>(y);
    const dim3 grid((unsigned)blocks);
    switch (h / 512) {
#define MEMO_LN_CASE(n) \
    case n: layernorm_rows_bf16_kernel<n><<<grid, 256, 0, st>>>(xp, gp, bp, yp, row_begin, row_end, h, eps); break;
        MEMO_LN_CASE(1) MEMO_LN_CASE(2) MEMO_LN_CASE(3) MEMO_LN_CASE(4) MEMO_LN_CASE(5) MEMO_LN_CASE(6)
        MEMO_LN_CASE(7) MEMO_LN_CASE(8) MEMO_LN_CASE(9) MEMO_LN_CASE(10) MEMO_LN_CASE(11) MEMO_LN_CASE(12)
        MEMO_LN_CASE(13) MEMO_LN_CASE(14) MEMO_LN_CASE(15) MEMO_LN_CASE(16)
#undef MEMO_LN_CASE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename Sh>
hipError_t launch_linear(const __bf16 *a, const __bf16 *w, const __bf16 *bias, __bf16 *out, int64_t row_begin, int64_t row_end,
                         int K, int N, hipStream_t st)
{
    const int64_t tiles = ((row_end - row_begin + Sh::BM - 1) / Sh::BM) * ((N + Sh::BN - 1) / Sh::BN);
    if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    const int64_t resident = kXcds * kChunk;          // one workgroup per compute unit
    linear_rows_bf16_kernel<Sh><<<dim3((unsigned)std::min(tiles, resident)), 512, 0, st>>>(a, w, bias, out, row_begin, row_end, K, N,
                                                                                          (uint32_t)tiles);
    return hipGetLastError();
}

// The shape of the least estimated time (all give the same bits).  us before (256 x 256 always) -> now: 75 rows
// 1024 -> 384 28.1 -> 5.9, 300 rows 4096 -> 1536 92 -> 15.0, 1000 rows 93 -> 22, 3075 rows 5120 -> 1920 117 -> 55,
// 20000 rows 4096 -> 1536 253 -> 193.
hipError_t launch_linear_rows_bf16(const void *a, const void *w, const void *bias, void *out, int64_t row_begin,
                                   int64_t row_end, int K, int N, hipStream_t st)
{
    const int64_t rows = row_end - row_begin;
    if (rows <= 0) return hipSuccess;
    // 256 rows of either operand must span < 4 GiB (32-bit per-lane offsets)
    if ((int64_t)256 * K * 2 >= (1LL << 32)) return hipErrorInvalidValue;
    const __bf16 *ap = static_cast<const __bf16 *>(a), *wp = static_cast<const __bf16 *>(w), *bp = static_cast<const __bf16 *>(bias);
    __bf16 *op = static_cast<__bf16 *>(out);
    const LinChoice &c = lin_plan(rows, K, N);
    switch (c.bm * 1000 + c.bn) {
    case 64064: return launch_linear<LinShape<4, 2, 1, 2, 5, 5, 2>>(ap, wp, bp, op, row_begin, row_end, K, N, st);
    case 128064: return launch_linear<LinShape<4, 2, 2, 2, 3, 3, 2>>(ap, wp, bp, op, row_begin, row_end, K, N, st);
    case 128128: return launch_linear<LinShape<4, 2, 2, 4, 3, 2, 2>>(ap, wp, bp, op, row_begin, row_end, K, N, st);
    case 192128: return launch_linear<LinShape<4, 2, 3, 4, 4, 4, 1>>(ap, wp, bp, op, row_begin, row_end, K, N, st);
    case 256128: return launch_linear<LinShape<4, 2, 4, 4, 3, 3, 1>>(ap, wp, bp, op, row_begin, row_end, K, N, st);
    default: return launch_linear<LinShape<2, 4, 8, 4, 3, 2, 1>>(ap, wp, bp, op, row_begin, row_end, K, N, st);
    }
}

}  // namespace memo

// fp32 causal attention forward/backward for gfx950 (Section 2.1.3 of the paper: exact
// softmax attention computed tile by tile with per-row running state, intermediates
// re-formed in the backward).  This is the full-precision path: fp32 operands on the matrix
// cores (v_mfma_f32_16x16x4_f32: fp32 products and sums), no rounding of the probabilities.
//
// What bounds it: the fp32 matrix rate, 256 flops per cycle and compute unit (157 TFLOP/s), the same as the
// vector units'; but one MFMA instruction does 32 cycles of that work from two registers, where the
// vector form needs an LDS read per multiply-add and lane.  An earlier VALU version of these kernels ran at 5 to
// 7 TFLOP/s, bound by its scalar LDS reads; these reach 116 (forward) and 122 (backward, of its seven contractions) at
// S = 5000, B = 2, H = 4, d = 128.  Where units would be idle a tile's output columns go to two or four workgroups, which halves or quarters
// the second contractions of the longest tile, the one that such a launch takes (us, one part : as they go out, with the D_i launch: S = 1024 H = 1 d = 64
// forward 12.7 : 10.4, backward 24.6 : 21.5; d = 128 20.7 : 17.5 and 39.8 : 34.0).
#include "attn_f32_rows.h"

namespace memo {
namespace {

template <int D, bool FAR, int CS, bool SHARED>
__global__ __launch_bounds__(512, kWavesPerSimd<D>) void attn_fwd_f32_kernel(AttnArgs a, Divisor heads, Divisor H)
{
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kF32FwdLds<D>];
    if constexpr (SHARED) load_args_at_once(a);
    const auto [rank, hbp] = heads(blockIdx.x);       // CS parts of a head beside each other
    f32_fwd_rows<D, FAR, CS, SHARED>(a, (LDS_AS unsigned char *)smem, head_of(hbp / CS, (int)((a.S + kT - 1) / kT) - 1 - (int)rank, H), (int)(hbp % CS));
}

// One launch for the gradients asked for: first the key-stationary workgroups (key_ranks tiles of every head), then the query-stationary
// ones.  Longest first, except where all of them are resident at once, two per unit (head dim 64): then a unit gets the key tile
// of a rank and the query tile of the same rank, and the query tiles go shortest first to even that out
// (S = 2000, H = 2: 66 us both longest first).
template <int D, bool FAR, int CS, bool SHARED>
__global__ __launch_bounds__(512, kWavesPerSimd<D>) void attn_bwd_f32_kernel(AttnArgs a, uint32_t key_ranks, Divisor heads, Divisor H)
{
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kF32BwdLds<D>];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;     // [wave] two tiles, then the two rows that all waves need
    if constexpr (SHARED) {
        load_args_at_once(a);
        asm volatile("" ::"s"(a.d_o), "s"(a.delta));
    }
    const bool resident = D == 64 && gridDim.x <= 2 * kXcds * kChunk;
    const uint32_t key_blocks = key_ranks * heads.d;
    if (blockIdx.x < key_blocks) {
        const auto [rank, hbp] = heads(blockIdx.x);
        f32_dkdv_rows<D, FAR, CS, SHARED>(a, lds, head_of(hbp / CS, (int)rank, H), (int)(hbp % CS));
    } else {
        const auto [rank, hbp] = heads(blockIdx.x - key_blocks);
        f32_dq_rows<D, FAR, CS, SHARED>(a, lds, head_of(hbp / CS, resident ? (int)rank : (int)((a.S + kT - 1) / kT) - 1 - (int)rank, H), (int)(hbp % CS));
    }
}

// x of the lane that DPP control `Ctrl` names, added
template <int Ctrl>
__device__ __forceinline__ float add_dpp(float x)
{
    return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), Ctrl, 0xf, 0xf, true));
}

// D_i = sum_c dO_ic O_ic.  16 lanes per row, 16 rows per 256-thread workgroup.  Bound by memory at long sequences (5.7 TB/s at 1.3 million rows) and
// by its start at short ones: one fetch of arguments and one of the rows, O and dO together, and the 16 lanes added up
// by lane moves.  (With dO asked for when O had come and exchanges through the LDS the backward took, us, before -> now: bf16 S = 640
// H = 2 10.1 -> 9.85, S = 2000 with 6 heads 34.3 -> 34.0; fp32 S = 1024 H = 1 23.2 -> 22.9.)
template <typename T, int D>
__global__ __launch_bounds__(256) void attn_delta_kernel(AttnArgs a)
{
    asm volatile("" ::"s"(a.o_in), "s"(a.d_o), "s"(a.delta), "s"(a.S), "s"(a.sb), "s"(a.ss), "s"(a.sh), "s"(a.H));
    constexpr int kPer = D / 16, kLoads = kPer * (int)sizeof(T) / 16;
    const int tid = threadIdx.x, r = tid / 16, part = tid % 16;
    const int h = blockIdx.y, b = blockIdx.z;
    const int64_t i = (int64_t)blockIdx.x * 16 + r;
    const int64_t first = (int64_t)b * a.sb + (int64_t)h * a.sh + i * a.ss + part * kPer;
    float sum = 0.f;
    if (i < a.S) {
        const u32x4 *o = reinterpret_cast<const u32x4 *>(static_cast<const T *>(a.o_in) + first);
        const u32x4 *g = reinterpret_cast<const u32x4 *>(static_cast<const T *>(a.d_o) + first);
        u32x4 ov[kLoads], gv[kLoads];
#pragma unroll
        for (int n = 0; n < kLoads; ++n) {
            ov[n] = o[n];
            gv[n] = g[n];
        }
        __builtin_amdgcn_sched_barrier(0);            // all loads are on their way before the first is waited for
#pragma unroll
        for (int c = 0; c < kPer; ++c) {
            // scalars before the bit cast: applied to a vector's element it reads element 0 with this compiler (as in split_halves)
            uint32_t x, y;
            if constexpr (sizeof(T) == 4) {
                x = ov[c / 4][c % 4];
                y = gv[c / 4][c % 4];
            } else {                                  // bf16: the upper half of an fp32
                x = c % 2 ? ov[c / 8][c % 8 / 2] & 0xffff0000u : ov[c / 8][c % 8 / 2] << 16;
                y = c % 2 ? gv[c / 8][c % 8 / 2] & 0xffff0000u : gv[c / 8][c % 8 / 2] << 16;
            }
            sum += __builtin_bit_cast(float, x) * __builtin_bit_cast(float, y);
        }
    }
    sum = add_dpp<0xb1>(sum);     // the lane beside
    sum = add_dpp<0x4e>(sum);     // the pair beside
    sum = add_dpp<0x141>(sum);    // the other four of eight, mirrored
    sum = add_dpp<0x140>(sum);    // the other eight of sixteen
    if (i < a.S && part == 0) a.delta[((int64_t)b * a.H + h) * a.S + i] = sum;
}

inline dim3 row_grid(const AttnArgs &a, int rows)
{
    return dim3((unsigned)((a.S + rows - 1) / rows), (unsigned)a.H, (unsigned)a.B);
}

template <int D, bool FAR>
hipError_t launch_fwd_f32(const AttnArgs &a, hipStream_t st)
{
    const int64_t blocks = order_grid((a.S + kT - 1) / kT, (int64_t)a.H * a.B, kLongestFirst);
    if (blocks > kMaxBlocks)
        return launch_fewer_heads(a, sizeof(float), blocks, kMaxBlocks, [&](const AttnArgs &part) { return launch_fwd_f32<D, FAR>(part, st); });
    const int64_t heads = (int64_t)a.H * a.B;
    auto launch = [&](auto kernel, int parts) { return launch_blocks(kernel, blocks * parts, st, a, Divisor(heads * parts), Divisor(a.H)); };
    if constexpr (!FAR) {
        const int parts = a.o_out == a.q ? 1 : column_parts(blocks);         // in place of Q: another part may not have read it yet
        if (parts == 4) return launch(attn_fwd_f32_kernel<D, FAR, 4, true>, 4);
        if (parts == 2) return launch(attn_fwd_f32_kernel<D, FAR, 2, true>, 2);
        if constexpr (D == 64)
            if (!f32_fwd_shares_rows(blocks / heads, heads)) return launch(attn_fwd_f32_kernel<D, FAR, 1, false>, 1);
    }
    return launch(attn_fwd_f32_kernel<D, FAR, 1, true>, 1);
}

// dkdv, dq: which of the two to launch
template <int D, bool FAR>
hipError_t launch_bwd_f32(const AttnArgs &a, bool dkdv, bool dq, hipStream_t st)
{
    const int64_t heads = (int64_t)a.H * a.B, tiles = (a.S + kT - 1) / kT, blocks = tiles * heads * (dkdv + dq);
    if (blocks > kMaxBlocks)
        return launch_fewer_heads(a, sizeof(float), blocks, kMaxBlocks, [&](const AttnArgs &part) { return launch_bwd_f32<D, FAR>(part, dkdv, dq, st); });
    auto launch = [&](auto kernel, int parts) {
        return launch_blocks(kernel, blocks * parts, st, a, dkdv ? (uint32_t)tiles : 0u, Divisor(heads * parts), Divisor(a.H));
    };
    if constexpr (!FAR) {
        // a dQ that takes the place of Q or dO is not split: another part may not have read them yet
        const int parts = dq_in_place(a) ? 1 : column_parts(2 * tiles * heads);
        if (parts == 4) return launch(attn_bwd_f32_kernel<D, FAR, 4, true>, 4);
        if (parts == 2) return launch(attn_bwd_f32_kernel<D, FAR, 2, true>, 2);
        if constexpr (D == 64)
            if (!f32_bwd_shares_rows(tiles)) return launch(attn_bwd_f32_kernel<D, FAR, 1, false>, 1);
    }
    return launch(attn_bwd_f32_kernel<D, FAR, 1, true>, 1);
}

// whether the kernels of attn_f32_split.hip take the launch
bool splits(const AttnArgs &a)
{
    return a.ss < kSplitStride && a.S < kSplitRows && f32_splits(a.S, (int64_t)a.H * a.B, a.d);
}

}  // namespace

hipError_t launch_attn_fwd_f32(const AttnArgs &a, hipStream_t st)
{
    if (splits(a)) return launch_attn_fwd_f32_split(a, st);
    if (a.ss >= kFarStride) return a.d == 128 ? launch_fwd_f32<128, true>(a, st) : launch_fwd_f32<64, true>(a, st);
    return a.d == 128 ? launch_fwd_f32<128, false>(a, st) : launch_fwd_f32<64, false>(a, st);
}

hipError_t launch_attn_delta(const AttnArgs &a, bool is_bf16, hipStream_t st)
{
    const dim3 grid = row_grid(a, 16);
    if (is_bf16) attn_delta_kernel<__bf16, 128><<<grid, 256, 0, st>>>(a);
    else if (a.d == 64) attn_delta_kernel<float, 64><<<grid, 256, 0, st>>>(a);
    else attn_delta_kernel<float, 128><<<grid, 256, 0, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_attn_bwd_f32(const AttnArgs &a, hipStream_t st)
{
    auto launch = [&](bool dkdv, bool dq) {
        if (splits(a)) return launch_attn_bwd_f32_split(a, dkdv, dq, st);
        if (a.ss >= kFarStride) return a.d == 128 ? launch_bwd_f32<128, true>(a, dkdv, dq, st) : launch_bwd_f32<64, true>(a, dkdv, dq, st);
        return a.d == 128 ? launch_bwd_f32<128, false>(a, dkdv, dq, st) : launch_bwd_f32<64, false>(a, dkdv, dq, st);
    };
    hipError_t e = record_stage(a, 0, st);
    if (e != hipSuccess) return e;
    if ((e = launch_attn_delta(a, false, st)) != hipSuccess) return e;
    if ((e = record_stage(a, 1, st)) != hipSuccess) return e;
    if (!a.stage_events && !dq_in_place(a)) return launch(true, true);
    if ((e = launch(true, false)) != hipSuccess) return e;
    if ((e = record_stage(a, 2, st)) != hipSuccess) return e;
    if ((e = launch(false, true)) != hipSuccess) return e;
    return record_stage(a, 3, st);
}

}  // namespace memo

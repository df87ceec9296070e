// Internal interface between the C-ABI front end (memo_api.cpp) and the gfx950 kernels.
// Not installed; the public contract is include/memo.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <initializer_list>

namespace memo {

// One attention problem as the kernels see it.  Element (b, s, h, c) of q/k/v/o/d_o/dq/dk/dv
// is at b*sb + s*ss + h*sh + c (elements); lse and delta are [B,H,S] fp32.
struct AttnArgs {
    const void *q, *k, *v;
    const void *o_in;     // backward: forward output
    const void *d_o;      // backward: dL/dO
    void *o_out;          // forward: output
    void *dq, *dk, *dv;   // backward outputs
    float *lse;           // forward: written; backward: read
    float *delta;         // backward workspace: D_i = sum_c dO_ic O_ic, [B,H,S]
    int32_t B, H, d;
    int64_t S;
    float scale;
    int64_t sb, ss, sh;
    hipEvent_t *stage_events;   // backward only, nullable: 4 events recorded between the stages
};

// One copy of `rows` swapped rows between device and pinned host memory, one contiguous block.  Asked for as a linear copy, a large block goes to a copy engine that
// is free at the time of the call, and the stream keeps it: with some copies already queued on other streams these are engines that move 16 GB/s for the
// 57 of the link (a layer's step of 32K tokens with 192 MiB each way, passes rotating over three pairs of streams: 11.4 to 15 ms for 7.2).
// Asked for as rows it takes the engine of its direction, from any stream, at the link's rate.  Both forms take as long by themselves: 64 KiB 10.5 us,
// 1 MiB 27 us, 192 MiB 3.53 ms, 5 GiB 93.9 ms, for rows of 1 KiB to 16 MiB; rows of 256 bytes take 4.6 ms for 192 MiB, and a block of 4 KiB takes 9 us for 5.
// The engine of the way out is also the one with which the driver clears freed device memory: for 28 ms per GiB after a hipFree a copy shares it (16 MiB
// 0.5 ms for 0.3, 1 GiB 51 GB/s for 57), which a linear copy does not.
// The whole block has to go as rows: a few bytes left to a linear copy are moved by a kernel, which beside a launch that fills the chip waits for one of its workgroups
// to end (four copies of 64 MiB and 1 KiB beside dK/dV of 256K tokens: 41 ms for 4.7).  So the rows are the token rows where these are of 1 to 64 KiB and a multiple of 16, else
// of 4 KiB where that divides the block.  Other blocks, those below 256 KiB or off 16 bytes, host memory that is not pinned (128 MiB out 7.5 ms, as rows 235) and
// what the runtime does not take as rows stay linear.  Any other failure is the call's.
inline hipError_t copy_swapped(void *dst, const void *src, int64_t rows, size_t row_bytes, hipMemcpyKind kind, hipStream_t st)
{
    const size_t bytes = (size_t)rows * row_bytes, width = row_bytes >= 1024 && row_bytes <= 65536 && row_bytes % 16 == 0 ? row_bytes : 4096;
    const bool aligned = ((reinterpret_cast<uintptr_t>(dst) | reinterpret_cast<uintptr_t>(src)) & 15u) == 0;
    if (aligned && bytes % width == 0 && bytes >= 256 * 1024) {
        const hipError_t before = hipPeekAtLastError();
        hipPointerAttribute_t host{};
        hipError_t e = hipPointerGetAttributes(&host, kind == hipMemcpyDeviceToHost ? dst : src);
        if (e == hipSuccess && host.type == hipMemoryTypeHost) {
            e = hipMemcpy2DAsync(dst, width, src, width, width, bytes / width, kind, st);
            if (e != hipErrorInvalidValue && e != hipErrorInvalidPitchValue && e != hipErrorNotSupported) return e;
        }
        if (e != hipSuccess && before == hipSuccess) (void)hipGetLastError();    // the refusal's own; an error that the caller has not read yet stays one
    }
    return hipMemcpyAsync(dst, src, bytes, kind, st);
}

inline hipError_t record_stage(const AttnArgs &a, int idx, hipStream_t st)
{
    return a.stage_events ? hipEventRecord(a.stage_events[idx], st) : hipSuccess;
}

// dQ may take the place of Q or of dO (all have one layout): a query-stationary workgroup reads only the rows it
// writes later, so that it is enough to work all key-stationary ones first
inline bool dq_in_place(const AttnArgs &a) { return a.dq == a.q || a.dq == a.d_o; }

// Works a problem of more workgroups than one launch takes (max_blocks) as problems of fewer heads: some batch entries at a
// time, or some heads of a single one.  launch(part) may split its part again.  On the host, so that no kernel has to know
// (an offset of the workgroup id as a kernel argument moved the loops of the long backward by one instruction: 2.5 % at
// S = 1M).
template <typename Launch>
hipError_t launch_fewer_heads(const AttnArgs &a, size_t element_bytes, int64_t blocks, int64_t max_blocks, Launch &&launch)
{
    const int64_t heads = (int64_t)a.B * a.H, per = heads / ((blocks + max_blocks - 1) / max_blocks);
    if (heads == 1) return hipErrorInvalidValue;
    const bool by_batch = a.B > 1;
    const int32_t n = by_batch ? a.B : a.H;
    const int64_t want = by_batch ? per / a.H : per;
    const int32_t step = want < 1 ? 1 : (int32_t)want;
    for (int32_t i = 0; i < n; i += step) {
        AttnArgs part = a;
        (by_batch ? part.B : part.H) = step < n - i ? step : n - i;
        const int64_t bytes = i * (by_batch ? a.sb : a.sh) * (int64_t)element_bytes, rows = i * (by_batch ? (int64_t)a.H : 1) * a.S;
        for (const void **p : {&part.q, &part.k, &part.v, &part.o_in, &part.d_o})
            if (*p) *p = static_cast<const char *>(*p) + bytes;
        for (void **p : {&part.o_out, &part.dq, &part.dk, &part.dv})
            if (*p) *p = static_cast<char *>(*p) + bytes;
        part.lse += rows;
        if (part.delta) part.delta += rows;
        const hipError_t e = launch(part);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// fp32 path (fp32 matrix instructions, fp32 throughout), d in {64, 128}
hipError_t launch_attn_fwd_f32(const AttnArgs &a, hipStream_t st);
hipError_t launch_attn_bwd_f32(const AttnArgs &a, hipStream_t st);

// the same on fp16 matrix instructions, every fp32 operand as the sum of two fp16 ones; rows less than kSplitStride floats apart, S below kSplitRows
inline constexpr int64_t kSplitStride = (int64_t)1 << 25, kSplitRows = (int64_t)1 << 28;
hipError_t launch_attn_fwd_f32_split(const AttnArgs &a, hipStream_t st);
hipError_t launch_attn_bwd_f32_split(const AttnArgs &a, bool dkdv, bool dq, hipStream_t st);     // which of the gradients

// bf16 path (bf16 MFMA contractions, fp32 accumulation and softmax), d = 128
hipError_t launch_attn_fwd_bf16(const AttnArgs &a, hipStream_t st);
hipError_t launch_attn_fwd_bf16_long(const AttnArgs &a, int order, int64_t blocks, hipStream_t st);      // 256-row workgroups
hipError_t launch_attn_bwd_bf16(const AttnArgs &a, hipStream_t st);
hipError_t launch_attn_bwd_dkdv_bf16_long(const AttnArgs &a, int order, int64_t blocks, hipStream_t st); // dK, dV by 256-key workgroups
hipError_t launch_attn_bwd_dq_bf16_long(const AttnArgs &a, int order, int64_t blocks, hipStream_t st);   // dQ by 256-row workgroups
hipError_t launch_attn_bwd_both_bf16_long(const AttnArgs &a, int64_t dkdv_blocks, int64_t blocks, hipStream_t st);   // single tiles of both kinds, dK and dV's first

// D_i = sum_c dO_ic * O_ic for either dtype (is_bf16 selects the element type)
hipError_t launch_attn_delta(const AttnArgs &a, bool is_bf16, hipStream_t st);

// Token-wise recomputation (bf16): LayerNorm of rows [row_begin,row_end) of x [S,h] and the
// projection out[rows, N] = a[rows, K] * w[N, K]^T + bias over the same kind of row range.
hipError_t launch_layernorm_rows_bf16(const void *x, const void *gamma, const void *beta, void *y,
                                      int64_t row_begin, int64_t row_end, int h, float eps, hipStream_t st);
hipError_t launch_linear_rows_bf16(const void *a, const void *w, const void *bias, void *out,
                                   int64_t row_begin, int64_t row_end, int K, int N, hipStream_t st);

}  // namespace memo

// fp32 causal attention forward and backward for gfx950 on fp16 matrix instructions: every fp32 operand goes into them as the sum of two fp16 numbers, h = x rounded to
// fp16 and l = x - h rounded to fp16 (24 bits in all), and a product is h h + h l + l h, added up in fp32.  For launches that fill the chip; smaller ones, and
// what cannot be split so, are worked by the fp32 matrix instructions (attn_f32.hip, attn_f32_rows.h), which take 512 cycles for a block of 32 x 32 x 16 where these take 96.
//
// Precision.  What is left out of a product (l l, and the rounding of l) is about 2^-24 of it, as is an fp32 rounding, and an accumulator is rounded once for 16 terms
// instead of four: relative error of a sum of 128 products of N(0,1) numbers 1.39e-7 in one accumulator and 1.1e-7 in two, as the scores are formed here, against
// 2.05e-7 of one and 1.5e-7 of two on fp32 instructions; of 4096 products 7.1e-7 against 1.15e-6.  fp16's range is kept by powers of two:
//  * a workgroup's own 32 rows: one per row, from the row's largest magnitude;
//  * streamed tensors: one per workgroup, from the largest magnitude of that tensor's rows at the workgroup's place (kRowTop); also where they lie in fp16's range by themselves
//    (N(0,1) numbers without a scale are 3 to 5 % faster, but l has no bits below 2^-24, and columns much smaller than the others, alone in a product because the other
//    tensor is zero there, lose theirs; output of S = 1300 H = 4 with every other column of K smaller, by 1: 1.39e-7, 2^8 1.51e-7, 2^10 1.64e-7, 2^12 4.1e-7);
//  * probabilities: against the running maximum (forward), times 2^15 (backward); dS: one per output row, brought down when the row's largest dS asks for it.
// Whether a streamed row fits its scale is checked: its largest magnitude, scaled, must be at least 1/2 (l is then exact to 2^-24 of it), or the row zero; one that
// overflows makes NaN.  A workgroup that met a row that does not fit, or whose result is not finite, writes nothing and works its rows with the fp32 instructions.
// (Three bf16 parts need no scales, but six products and 44 vector instructions for a split of eight values: forward S = 5000 H = 4 B = 2 d = 128 331 us, this 242.)
//
// Workgroup: 32 rows, eight waves.  A wave works steps of 32 streamed rows of its own, so there is no barrier in the sweep.  As row operand (scores, dP) streamed rows
// come through a ring in LDS, 16 columns a slot (from memory straight to the lanes of a row operand a unit takes in 16 B per cycle, by way of LDS 64); as transposed
// operand (output, gradients) straight to registers, kVec consecutive columns a lane, which the output blocks are numbered after.  The split of an operand goes between the
// MFMAs of the one before it.
//
// Errors against 64 bits (relative, root mean square; O, lse, dQ, dK, dV), fp32 instructions -> this: S = 1400 H = 2 d = 64 1.67e-7 3.7e-8 3.7e-7 4.6e-7 4.2e-7 -> 1.58e-7 3.1e-8
// 3.3e-7 3.7e-7 3.3e-7; S = 1292 H = 3 d = 128 1.81e-7 4.7e-8 4.3e-7 5.0e-7 4.3e-7 -> 1.68e-7 4.2e-8 3.7e-7 4.0e-7 3.5e-7; S = 5000 d = 64 2.2e-7 5.1e-8 4.6e-7 7.0e-7 6.9e-7 ->
// 1.9e-7 4.4e-8 4.0e-7 5.3e-7 5.0e-7; scores ten times those of N(0,1), S = 3000 d = 64, 5.8e-7 5.7e-8 1.7e-6 1.7e-6 1.3e-6 -> 5.6e-7 5.3e-8 1.4e-6 1.5e-6 1.1e-6.
//
// What bounds it: vector issue.  A step of the forward (d = 128) has 48 MFMAs (1536 cycles) and 580 vector instructions (3180 cycles of issue: v_fma_mix, which
// makes l, and exponentials take 8 and 16), two waves share a SIMD, and a wave waits a third of its time.  Without the splits 14 % less, without fills 10, without the
// other loads 8, without operand reads 4.  v_dot2c (x - h in one instruction) runs on the matrix core.
// us, fp32 instructions -> this, d = 128: S = 3000 H = 4 forward 97 -> 53, backward 309 -> 166; S = 5000 H = 4 B = 2 486 -> 244 and 1628 -> 799; d = 64 S = 3000 H = 4 49 -> 34 and
// 156 -> 94.
#include "attn_f32_rows.h"

namespace memo {
namespace {

constexpr int kWaves = 8, kRows = 32, kStep = 32;     // waves of a workgroup, its rows; streamed rows of a wave's step
constexpr f32x16 kZero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
// What is split is brought high in fp16's range, so that l has its bits down to 2^-24 of it.  The forward's probabilities: times kWeightUp against the running
// maximum, which is brought up to date before they pass kMostP; the backward's, at most 1: times kProbUp.  By a multiplication, which is exact: in the exponent, five more
// make its rounding that of a larger number (error of the output 6 % and of the logsumexp 25 % up).
constexpr float kWeightUp = 32.f, kMostP = 1024.f, kProbUp = 32768.f;
// Streamed rows are brought to 2^8 by the workgroup's own rows of the tensor, which leaves 2^7 and more for larger rows and 2^8 for smaller ones (us of S = 3000 H = 4 d = 128 with one row of dO
// a hundred times the others: backward 169, brought to 2^10 316 and on fp32 instructions 298; one row of V: forward 56, 159, 99; tensors whose rows no scale fits: 120 and 355 for 101 and 292).
constexpr int kRowTop = 8, kOwnTop = 12;

__device__ __forceinline__ float as_float(uint32_t u) { return __builtin_bit_cast(float, u); }
__device__ __forceinline__ uint32_t as_bits(float x) { return __builtin_bit_cast(uint32_t, x); }

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x16 mfma_half(f16x8 a, f16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }

// x = h + l, eight values a lane
struct Split { f16x8 h, l; };

// The split of eight values as vector instructions, to be dealt out between MFMAs.  SCALED: times `scale` first.  TRACK: top becomes the largest magnitude.
template <bool SCALED, bool TRACK> constexpr int kSplitOps = 4 * (3 + 2 * SCALED + TRACK);
struct SplitJob {
    float x[8], top;
    uint32_t h[4], l[4];
    template <bool SCALED, bool TRACK, int I>
    __device__ __forceinline__ void op(float scale)
    {
        constexpr int per = kSplitOps<SCALED, TRACK> / 4, p = I / per, k = I % per + (SCALED ? 0 : 2);
        float &a = x[2 * p], &b = x[2 * p + 1];
        if constexpr (k == 0) a *= scale;
        if constexpr (k == 1) b *= scale;
        if constexpr (k == 2) asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(h[p]) : "v"(a), "v"(b));
        if constexpr (k == 3) asm("v_fma_mixlo_f16 %0, %1, 1.0, -%2 op_sel_hi:[0,0,1]" : "=v"(l[p]) : "v"(a), "v"(h[p]));
        if constexpr (k == 4) asm("v_fma_mixhi_f16 %0, %1, 1.0, -%2 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "+v"(l[p]) : "v"(b), "v"(h[p]));
        if constexpr (k == 5) top = fmaxf(fmaxf(fabsf(a), fabsf(b)), top);
    }
    __device__ __forceinline__ Split result() const
    {
        const u32x4 a = {h[0], h[1], h[2], h[3]}, c = {l[0], l[1], l[2], l[3]};
        return {__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, c)};
    }
    template <bool SCALED = false>
    __device__ __forceinline__ Split at_once(float scale = 1.f)
    {
        static_for<0, kSplitOps<SCALED, false>>([&](auto i) { op<SCALED, false, decltype(i)::value>(scale); });
        asm volatile("s_nop 1" : "+v"(l[0]), "+v"(l[1]), "+v"(l[2]), "+v"(l[3]));         // see product()
        return result();
    }
};
__device__ __forceinline__ void take(SplitJob &job, const f32x4 &a, const f32x4 &b)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) job.x[e] = e < 4 ? a[e] : b[e - 4];
}
__device__ __forceinline__ Split split8(const f32x16 &x, int first, float mul = 1.f)
{
    SplitJob job;
#pragma unroll
    for (int e = 0; e < 8; ++e) job.x[e] = x[first + e] * mul;
    return job.at_once();
}

// The products, those of the second operand's l first, so that its registers come free: h l, then l l where it is formed (LOW), l h, h h.  The first one never
// reads the first operand's l: an MFMA right behind the v_fma_mixhi that writes half of such a register reads the old half (dK of S = 504 d = 64 was 9e-5 off with
// l l in front), and the compiler does not know the instruction inside an asm; SplitJob::at_once waits.
// l l is left out but from the scores and the output of head dim 64, whose sums are short: output of S = 750 H = 4 1.58e-7 off without, 1.51e-7 with, 1.52e-7 on fp32 instructions.
template <int D> constexpr bool kLow = D == 64;
template <bool LOW> constexpr int kProducts = LOW ? 4 : 3;
template <bool LOW, int P> constexpr bool kLastOfLow = P == (LOW ? 1 : 0);             // of the second operand's l
template <bool LOW, int P>
__device__ __forceinline__ f32x16 product(const Split &a, const Split &b, const f32x16 &c)
{
    if constexpr (P == 0) return mfma_half(a.h, b.l, c);
    else if constexpr (LOW && P == 1) return mfma_half(a.l, b.l, c);
    else if constexpr (P + 1 < kProducts<LOW>) return mfma_half(a.l, b.h, c);
    else return mfma_half(a.h, b.h, c);
}

// Streamed rows, 32 a step.  As row operand (lane: row l32, 8 of 16 columns) they pass through a wave's own ring in LDS, an operand a slot, as rows of
// 64 bytes whose 16-byte piece p lies at p ^ (row / 4 % 4); a lane of half h reads the pieces 2 h and 2 h + 1.  As transposed operand (lane: D / 32 columns from 8 of 16 rows) straight to registers.
constexpr int kSlot = kStep * 64;

template <int D>
struct Streams {
    static constexpr int kVec = D / 32;               // consecutive columns of a lane in a transposed operand: kVec l32 ..
    uint32_t fill_off, tr_off, ss4, row_at;
    int64_t ss;
    LDS_AS unsigned char *ring;
    __device__ __forceinline__ Streams(LDS_AS unsigned char *own_ring, int64_t stride, int lane)
    {
        const int l32 = lane & 31, half = lane >> 5;
        ss = stride;
        ss4 = (uint32_t)stride * 4;
        fill_off = (uint32_t)(lane / 4) * ss4 + (uint32_t)((lane % 4) ^ (lane / 16)) * 16;
        tr_off = (uint32_t)(4 * half) * ss4 + 4 * kVec * l32;
        ring = own_ring;
        row_at = (uint32_t)(uintptr_t)own_ring + (uint32_t)(l32 * 64 + ((2 * half ^ (l32 >> 2)) & 3) * 16);
    }
    // rows 32 step .. of src, which ends with row S - 1: rows past it read as zero
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const float *src, int64_t step, int64_t S) const
    {
        const int64_t r0 = step * kStep, left = S - r0;
        const int rows = left < 0 ? 0 : left > kStep ? kStep : (int)left;
        const uint32_t bytes = rows > 0 ? (uint32_t)(rows - 1) * ss4 + D * 4 : 0;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(src + (rows > 0 ? r0 * ss : 0)), 0, bytes, 0x00020000);
    }
    __device__ __forceinline__ void fill(int slot, __amdgpu_buffer_rsrc_t b, int c) const
    {
#ifdef __HIP_DEVICE_COMPILE__      // the host pass does not know the 16-byte form of the builtin
#pragma unroll
        for (int i = 0; i < 2; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(b, (LDS_AS void *)(ring + slot * kSlot + i * 1024), 16, fill_off + (uint32_t)(16 * i) * ss4 + 64 * c, 0, 0, 0);
#endif
    }
    struct Rows { f32x4 x[2]; };
    template <int SLOT>
    __device__ __forceinline__ void read(Rows &r) const
    {
        lds_issue_b128<SLOT * kSlot>(r.x[0], row_at);
        lds_issue_b128<SLOT * kSlot>(r.x[1], row_at ^ 16);
    }
    // group G of 16 rows: slot e is row 16 G + 8 (e / 4) + 4 half + e % 4
    struct Tr { uint32_t x[8][kVec]; };
    template <int G>
    __device__ __forceinline__ void load(Tr &r, __amdgpu_buffer_rsrc_t b) const
    {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t at = tr_off + (16 * G + e / 4 * 8 + e % 4) * ss4;
            if constexpr (kVec == 4) {
                const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(b, at, 0, 0);
#pragma unroll
                for (int c = 0; c < 4; ++c) r.x[e][c] = v[c];
            } else {
                const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(b, at, 0, 0);
#pragma unroll
                for (int c = 0; c < 2; ++c) r.x[e][c] = v[c];
            }
        }
    }
};
template <typename Tr>
__device__ __forceinline__ void take(SplitJob &job, const Tr &raw, int c)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) job.x[e] = as_float(raw.x[e][c]);
}
// reads queued after the wanted ones may still be on their way
template <int LATER, typename Rows>
__device__ __forceinline__ void wait_rows(Rows &r) { asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(r.x[0]), "+v"(r.x[1]) : "n"(LATER)); }

// x of the lane that DPP control `Ctrl` names, or x where that is larger
template <int Ctrl>
__device__ __forceinline__ float max_dpp(float x)
{
    return fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), Ctrl, 0xf, 0xf, true)));
}

// The power of two that brings a magnitude to 2^TO .. 2^(TO + 1); one for zero, for what is not finite any.
template <int TO>
__device__ __forceinline__ float scale_for(float top)
{
    if (top == 0.f) return 1.f;
    const int e = (int)(as_bits(top) >> 23) & 255;
    const int to = 127 + 127 + TO - e;
    return as_float((uint32_t)(to < 1 ? 1 : to > 254 ? 254 : to) << 23);
}
__device__ __forceinline__ float inverse(float power_of_two) { return as_float((254u << 23) - as_bits(power_of_two)); }

// The 32 rows that all waves need, each scaled by a power of two of its own and split once: operand n (16 columns) as [plane][lane].
template <int D>
struct Planes {
    static constexpr int kItems = D / 16, kBytes = kItems * 2 * 1024, kLanes = D / 8;      // lanes of a row
    template <int C, int PART>     // part 0: l, 1: h of operand C, tensor by tensor; at: this lane's place in the first
    static __device__ __forceinline__ void read(Split &x, uint32_t at) { lds_issue_b128<C * 2 * 1024 + (1 - PART) * 1024>(PART == 0 ? x.l : x.h, at); }
    struct Own { f32x4 x[2]; };    // eight floats of the row tid / kLanes
    static __device__ __forceinline__ void load(Own &own, const float *src, int64_t ss, int64_t r0, int64_t S)
    {
        const int tid = threadIdx.x, r = tid / kLanes % kRows;
        const int64_t i = r0 + r, row = i < S ? i : S - 1;
        const f32x4 *p = reinterpret_cast<const f32x4 *>(src + row * ss + 8 * (tid % kLanes));
        own.x[0] = p[0];
        own.x[1] = p[1];
    }
    static __device__ __forceinline__ float row_top(const Own &own)
    {
        float m = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(own.x[e / 4][e % 4]));
        m = max_dpp<0xb1>(m);
        m = max_dpp<0x4e>(m);
        m = max_dpp<0x141>(m);
        if constexpr (kLanes == 16) m = max_dpp<0x140>(m);
        return m;
    }
    // scales: one a row
    static __device__ __forceinline__ void put(LDS_AS unsigned char *at, LDS_AS float *scales, const Own &own)
    {
        const int tid = threadIdx.x, r = tid / kLanes, c = tid % kLanes;
        if (r >= kRows) return;
        const float scale = scale_for<kOwnTop>(row_top(own));
        SplitJob job;
        take(job, own.x[0], own.x[1]);
        const Split s = job.at_once<true>(scale);
        LDS_AS f16x8 *q = (LDS_AS f16x8 *)(at + c / 2 * 2 * 1024) + c % 2 * 32 + r;
        q[0] = s.h;
        q[64] = s.l;
        if (c == 0) scales[r] = scale;
    }
    // the largest magnitude among a wave's rows
    static __device__ __forceinline__ float wave_top(const Own &own)
    {
        float m = row_top(own);
        if constexpr (kLanes == 8) m = max_dpp<0x140>(m);
        m = fmaxf(m, __shfl_xor(m, 16));
        return fmaxf(m, __shfl_xor(m, 32));
    }
};

// N MFMAs, behind each its share of the next operand's split (JOB) and what extra() puts there
template <int N, bool JOB, bool TRACK, typename Mfma, typename Extra>
__device__ __forceinline__ void mfmas(SplitJob &job, float scale, Mfma &&mfma, Extra &&extra)
{
    static_for<0, N>([&](auto jc) {
        constexpr int j = decltype(jc)::value, ops = kSplitOps<true, TRACK>;
        mfma(jc);
        __builtin_amdgcn_sched_barrier(0);
        extra(jc);
        if constexpr (JOB) static_for<j * ops / N, (j + 1) * ops / N>([&](auto i) { job.template op<true, TRACK, decltype(i)::value>(scale); });
        __builtin_amdgcn_sched_barrier(0);
    });
}

// The row operands of a step: K tensors of D / 16, through SLOTS slots.  When operand n starts, its own split is there, and the reads of the
// rows of n + 1 and of its own planes l, h are there or on their way, in this order.
template <int D, int K, int SLOTS>
struct RowItems {
    using St = Streams<D>;
    using P = Planes<D>;
    static constexpr int kPer = D / 16, kAll = K * kPer;
    typename St::Rows raw[2];     // of even and odd operands
    Split a, y;
    SplitJob job;
    float scale[K];               // of the streamed tensors
    uint64_t bad = 0;             // lanes that met a row whose largest magnitude, scaled, is below 1/2 and not zero: its l is not exact enough; or out of fp16's range

    // rows of operand n (kAll and kAll + 1: the next step's first two)
    template <int N>
    __device__ __forceinline__ void read_rows(const St &st)
    {
        constexpr int n = N % kAll;
        st.template read<n % SLOTS>(raw[n % 2]);
    }
    __device__ __forceinline__ void check(float top)
    {
        const float t = max_across_halves(top);
        bad |= __builtin_amdgcn_ballot_w64(!(t >= 0.5f && t < 65504.f) && t != 0.f);
    }
    __device__ __forceinline__ void first(const St &st, uint32_t plane_at)
    {
        read_rows<0>(st);
        read_rows<1>(st);
        P::template read<0, 0>(y, plane_at);
        P::template read<0, 1>(y, plane_at);
        wait_rows<4>(raw[0]);
        first_job();
        static_for<0, kSplitOps<true, true>>([&](auto i) { job.template op<true, true, decltype(i)::value>(scale[0]); });
        a = job.result();
    }
    __device__ __forceinline__ void first_job()
    {
        take(job, raw[0].x[0], raw[0].x[1]);
        job.top = 0.f;
    }
    __device__ __forceinline__ void keep()            // reads queued for a step that does not follow: their registers are taken up to here
    {
        asm volatile("s_waitcnt lgkmcnt(0) ; %0 %1 %2 %3" : "+v"(raw[1].x[0]), "+v"(raw[1].x[1]), "+v"(y.h), "+v"(y.l));
    }
    // start(n): in front of operand n, whose successor's rows have left their slot; done(n): behind it;  last(job): whether there is an operand
    // to split behind the last one, and which
    template <typename Start, typename Mfma, typename Done, typename Last>
    __device__ __forceinline__ void run(const St &st, uint32_t plane_at, float last_scale, Start &&start, Mfma &&mfma, Done &&done, Last &&last)
    {
        static_for<0, kAll>([&](auto nc) {
            constexpr int n = decltype(nc)::value;
            constexpr bool more = n + 1 < kAll, more2 = n + 2 < kAll;
            if constexpr (more) wait_rows<2>(raw[(n + 1) % 2]);
            start(nc);
            if constexpr (more) {
                take(job, raw[(n + 1) % 2].x[0], raw[(n + 1) % 2].x[1]);
                if constexpr ((n + 1) % kPer == 0) {
                    check(job.top);
                    job.top = 0.f;
                }
            } else {
                check(job.top);
                last(job);
            }
            constexpr bool ahead = more || decltype(last(job))::value;
            __builtin_amdgcn_sched_barrier(0);
            constexpr bool low = n < kPer && kLow<D>;
            constexpr int products = kProducts<low>;
            auto mf = [&](auto pc) __attribute__((always_inline)) {
                constexpr int p = decltype(pc)::value;
                if constexpr (p == 0) asm volatile("s_waitcnt lgkmcnt(1)" : "+v"(y.l));
                if constexpr (p == products - 2) asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(y.h) : "n"((more2 ? 2 : 0) + (more ? 1 : 0)));
                mfma(nc, pc, IntC<low>{}, a, y);
            };
            auto extra = [&](auto jc) __attribute__((always_inline)) {
                constexpr int j = decltype(jc)::value;
                if constexpr (more2 && j == 0) read_rows<n + 2>(st);
                if constexpr (more && kLastOfLow<low, j>) P::template read<n + 1, 0>(y, plane_at);
                if constexpr (more && j == products - 1) P::template read<n + 1, 1>(y, plane_at);
            };
            if constexpr (more) mfmas<products, true, true>(job, scale[(n + 1) / kPer], mf, extra);
            else mfmas<products, ahead, false>(job, last_scale, mf, extra);
            if constexpr (ahead) a = job.result();
            done(nc);
        });
    }
    // the same reads for the next step's first operands, behind MFMA J of the last two blocks of a step's last transposed operand.  BUT: loads and
    // fills queued behind the second operand's
    template <int BUT, int LEFT, int J>               // LEFT: blocks left, 1 or 0
    __device__ __forceinline__ void first_of_next(const St &st, uint32_t plane_at)
    {
        if constexpr (LEFT == 1 && J == 0) {
            wait_fills_but<BUT>();
            read_rows<kAll>(st);
        }
        if constexpr (LEFT == 0 && J == 0) {
            read_rows<kAll + 1>(st);
            P::template read<0, 0>(y, plane_at);
        }
        if constexpr (LEFT == 0 && J == 2) P::template read<0, 1>(y, plane_at);
    }
};

// Product P of operand N of the scores: h h of the even and of the odd operands and the smaller products add up by themselves.  Forward and backward in the same way: the
// logsumexp fits the scores of the backward only if these are the forward's (gradients of scores of +-20 with one of the two on fp32 instructions: 1.4e-6 off, on the same 9e-7).
// (h h in one sum: output of S = 977 d = 128 1.80e-7 off, in two 1.66e-7, on fp32 instructions 1.73e-7.)
template <bool LOW, int N, int P>
__device__ __forceinline__ void score(f32x16 &even, f32x16 &odd, f32x16 &small, const Split &a, const Split &b)
{
    if constexpr (P < kProducts<LOW> - 1) small = product<LOW, P>(a, b, N == 0 && P == 0 ? kZero16 : small);
    else if constexpr (N % 2 == 0) even = product<LOW, P>(a, b, N == 0 ? kZero16 : even);
    else odd = product<LOW, P>(a, b, N == 1 ? kZero16 : odd);
}

// acc^T += tile^T x of one group of 16 rows: block c holds the columns kVec row + c; block 0 is split already.
// next(job): whether there is an operand to split with the last block, and which (NEXT_ROW: a row operand)
template <bool NEXT_ROW, bool LOW, int NB, typename Tr, typename Next, typename Extra>
__device__ __forceinline__ void outer(f32x16 (&acc)[NB], const Tr &raw, const Split &b, Split &a, SplitJob &job, float scale, float next_scale, Next &&next, Extra &&extra)
{
    static_for<0, NB>([&](auto cc) {
        constexpr int c = decltype(cc)::value;
        constexpr bool JOB = c < NB - 1 || decltype(next(job))::value;
        if constexpr (c < NB - 1) take(job, raw, c + 1);
        else next(job);
        __builtin_amdgcn_sched_barrier(0);
        auto mf = [&](auto pc) __attribute__((always_inline)) { acc[c] = product<LOW, decltype(pc)::value>(a, b, acc[c]); };
        auto ex = [&](auto jc) __attribute__((always_inline)) { extra(cc, jc); };
        mfmas<kProducts<LOW>, JOB, NEXT_ROW && c == NB - 1>(job, c < NB - 1 ? scale : next_scale, mf, ex);
        if constexpr (JOB) a = job.result();
    });
}

template <int D>
struct Shape {
    static constexpr int kBlocks = D / 32, kPieces = D / 8, kPerWave = kPieces / kWaves;
    static constexpr int kPieceBytes = kWaves * kPieces * 1024;
    static constexpr int kFwdSlots = D / 16, kBwdSlots = 4;
    // behind planes and rings, over which the pieces are laid: [wave][row] (maximum, sum) or factors, [tensor][row] scales, [wave][tensor] largest magnitudes
    static constexpr int kFwdStats = std::max(Planes<D>::kBytes + kWaves * kFwdSlots * kSlot, kPieceBytes), kFwdScales = kFwdStats + kWaves * kRows * 8;
    static constexpr int kBwdStats = std::max(2 * Planes<D>::kBytes + kWaves * kBwdSlots * kSlot, kPieceBytes), kBwdScales = kBwdStats + kWaves * kRows * 4;
    static constexpr int kScaleBytes = 2 * kRows * 4 + kWaves * 2 * 4, kFwdLds = kFwdScales + kScaleBytes, kBwdLds = kBwdScales + kScaleBytes;
};
// piece p of the accumulators, four consecutive columns of the lane's row l32, and the first of them
template <int D>
__device__ __forceinline__ f32x4 piece_of(const f32x16 (&acc)[D / 32], int p)
{
    if constexpr (D == 128) return f32x4{acc[0][p], acc[1][p], acc[2][p], acc[3][p]};
    else return f32x4{acc[0][2 * p], acc[1][2 * p], acc[0][2 * p + 1], acc[1][2 * p + 1]};
}
template <int D>
__device__ __forceinline__ int piece_column(int p, int half)
{
    if constexpr (D == 128) return 4 * (8 * (p / 4) + 4 * half + p % 4);
    else return 2 * (8 * (p / 2) + 4 * half + 2 * (p % 2));
}

// Puts a wave's accumulators down, and adds up this wave's share of the pieces (wave, wave + 8) over the waves, times weight[wave]
template <int D>
__device__ __forceinline__ void add_up(LDS_AS unsigned char *lds, const f32x16 (&acc)[D / 32], f32x4 (&out)[Shape<D>::kPerWave], const float (&weight)[kWaves], int wave, int lane)
{
    using S = Shape<D>;
    LDS_AS f32x4 *pieces = (LDS_AS f32x4 *)lds;
    __syncthreads();              // every wave has left what lies there
#pragma unroll
    for (int p = 0; p < S::kPieces; ++p) pieces[(wave * S::kPieces + p) * 64 + lane] = piece_of<D>(acc, p);
    __syncthreads();
#pragma unroll
    for (int n = 0; n < S::kPerWave; ++n) {
        out[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int g = 0; g < kWaves; ++g) out[n] += weight[g] * pieces[(g * S::kPieces + wave + n * kWaves) * 64 + lane];
    }
}
template <int D>
__device__ __forceinline__ void put(float *row, const f32x4 (&out)[Shape<D>::kPerWave], int wave, int half)
{
#pragma unroll
    for (int n = 0; n < Shape<D>::kPerWave; ++n) *reinterpret_cast<f32x4 *>(row + piece_column<D>(wave + n * kWaves, half)) = out[n];
}
// the pieces times mul; whether one of them is not a number
template <int D>
__device__ __forceinline__ bool finish(f32x4 (&out)[Shape<D>::kPerWave], float mul)
{
    float sum = 0.f;
#pragma unroll
    for (int n = 0; n < Shape<D>::kPerWave; ++n) {
        out[n] *= mul;
#pragma unroll
        for (int r = 0; r < 4; ++r) sum = fmaf(out[n][r], 0.f, sum);      // infinity too
    }
    return sum != sum;
}

// four values of a quad of lanes, in each of them
template <int R>
__device__ __forceinline__ float of_quad(uint32_t u)
{
    const int x = __builtin_amdgcn_mov_dpp((int)u, 0x55 * R, 0xf, 0xf, true);
    return __builtin_bit_cast(float, x);
}

// The scales of the two streamed tensors, from the largest magnitudes of the workgroup's own rows of them, which put_tops leaves in LDS.  Rows
// of down to 2^-9 and up to 2^7 times that can then be split.
__device__ __forceinline__ void put_tops(LDS_AS float *tops, float a, float b, int wave, int lane)
{
    if (lane == 0) {
        tops[2 * wave] = a;
        tops[2 * wave + 1] = b;
    }
}
__device__ __forceinline__ void streamed_scales(const LDS_AS float *tops, float &a, float &b)
{
    float ta = tops[0], tb = tops[1];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
        ta = fmaxf(ta, tops[2 * w]);
        tb = fmaxf(tb, tops[2 * w + 1]);
    }
    a = as_float(__builtin_amdgcn_readfirstlane(as_bits(scale_for<kRowTop>(ta))));
    b = as_float(__builtin_amdgcn_readfirstlane(as_bits(scale_for<kRowTop>(tb))));
}
// Scales whose products stay far inside fp32, whatever they meet
__device__ __forceinline__ bool far_scale(float s) { return !(s >= 0x1p-42f && s <= 0x1p42f); }

// Of the two waves of a SIMD the older one is served first and would end its steps ahead; from here on the younger one is, so that they end together and neither works alone
// (us without : with, forward S = 5000 H = 4 B = 2 d = 128 250 : 244, S = 12000 H = 2 d = 64 222 : 214, backward 812 : 799 and 624 : 610; served first from the start on, 250, 221, 816, 622;
// from 1/4 of the sweep to 1/2 within 1 %, forward S = 3000 H = 4 d = 128 51.7 at 1/4, 51.3 at 3/8, 52.9 at 7/16, 54.2 at 1/2).
__device__ __forceinline__ void even_out(int wave, int step, int steps)
{
    if (wave >= kWaves / 2 && step >= steps * 3 / 8) __builtin_amdgcn_s_setprio(1);
}

constexpr int64_t kNone = (int64_t)1 << 40;           // a step past the end of any sequence

// false: some value or row cannot be split (see RowItems::bad, far_scale), nothing has been written
template <int D>
__device__ __forceinline__ bool fwd_rows(const AttnArgs &a, LDS_AS unsigned char *lds, const TileId t)
{
    using S = Shape<D>;
    using P = Planes<D>;
    using Tr = typename Streams<D>::Tr;
    constexpr int NB = S::kBlocks, SL = S::kFwdSlots;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh;
    const float *k = static_cast<const float *>(a.k) + base, *v = static_cast<const float *>(a.v) + base;
    const int64_t row0 = (int64_t)t.tile * kRows, i = row0 + l32;
    const int steps = t.tile + 1;                     // the last one is the diagonal
    const Streams<D> st(lds + P::kBytes + wave * SL * kSlot, a.ss, lane);
    LDS_AS f32x2 *stats = (LDS_AS f32x2 *)(lds + S::kFwdStats);
    LDS_AS float *scales = (LDS_AS float *)(lds + S::kFwdScales), *tops = scales + 2 * kRows;
    typename P::Own own, own_k, own_v;
    P::load(own, static_cast<const float *>(a.q) + base, a.ss, row0, a.S);
    P::load(own_k, k, a.ss, row0, a.S);
    P::load(own_v, v, a.ss, row0, a.S);
    __builtin_amdgcn_sched_barrier(0);
    {
        const __amdgpu_buffer_rsrc_t kb = st.buffer(k, wave < steps ? wave : kNone, a.S);
#pragma unroll
        for (int n = 0; n < SL; ++n) st.fill(n, kb, n);
    }
    const uint32_t plane_at = (uint32_t)(uintptr_t)lds + lane * 16;
    P::put(lds, scales, own);
    put_tops(tops, P::wave_top(own_k), P::wave_top(own_v), wave, lane);
    f32x16 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = kZero16;
    float m = -INFINITY, lsum = 0.f;                  // m in scaled units
    wait_fills();                 // also the first step's: the counts in the loop are those of a step behind another
    __syncthreads();
    float scale_k, scale_v;
    streamed_scales(tops, scale_k, scale_v);
    const float scale_q = scales[l32], unscale = inverse(scale_q) * inverse(scale_k);
    const float c = a.scale * kLog2e * unscale;
    bool bad = far_scale(scale_q) || far_scale(scale_k) || far_scale(scale_v);
    if (wave < steps) {
        RowItems<D, 1, SL> rows;
        rows.scale[0] = scale_k;
        rows.first(st, plane_at);
        const float low_v = 0.5f * inverse(scale_v);
        // the rows of a transposed group as RowItems::check: by one column of each lane, by all of them if that one does not tell
        auto check = [&](const Tr &tr) __attribute__((always_inline)) {
            uint32_t some = ~0u;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint64_t high = __builtin_amdgcn_ballot_w64(fabsf(as_float(tr.x[e][0])) >= low_v);
                some = min(some, min((uint32_t)high, (uint32_t)(high >> 32)));
            }
            if (__builtin_expect(some == 0, 0)) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float top = 0.f;
#pragma unroll
                    for (int x = 0; x < Streams<D>::kVec; ++x) top = fmaxf(top, fabsf(as_float(tr.x[e][x])));
                    const uint64_t high = __builtin_amdgcn_ballot_w64(top >= low_v), any = __builtin_amdgcn_ballot_w64(top != 0.f);
                    if (((uint32_t)high == 0 && (uint32_t)any != 0) || (high >> 32 == 0 && any >> 32 != 0)) rows.bad = ~0ull;
                }
            }
        };
#pragma clang loop unroll(disable)
        for (int step = wave; step < steps && !rows.bad; step += kWaves) {
            even_out(wave, step, steps);
            const __amdgpu_buffer_rsrc_t kn = st.buffer(k, step + kWaves < steps ? step + kWaves : kNone, a.S), vb = st.buffer(v, step, a.S);
            Tr tr[2];
            st.template load<0>(tr[0], vb);
            __builtin_amdgcn_sched_barrier(0);
            f32x16 s, s1, small;
            rows.run(st, plane_at, scale_v,
                [&](auto nc) __attribute__((always_inline)) {
                    constexpr int n = decltype(nc)::value;
                    if constexpr (n == 0) st.fill(0, kn, 0);
                    if constexpr (n + 1 < SL) st.fill(n + 1, kn, n + 1);
                    if constexpr (n + 2 < SL) wait_fills_but<16 + 2 * (SL - 1)>();
                },
                [&](auto nc, auto pc, auto lowc, const Split &x, const Split &y) __attribute__((always_inline)) {
                    score<decltype(lowc)::value, decltype(nc)::value, decltype(pc)::value>(s, s1, small, x, y);
                },
                [&](auto) __attribute__((always_inline)) {},
                [&](SplitJob &job) __attribute__((always_inline)) { take(job, tr[0], 0); return IntC<1>{}; });
            check(tr[0]);
            s += s1;
            s += small;
            if (step == steps - 1) {      // key 8 (e / 4) + 4 half + e % 4 of the step is visible to query l32 iff it is <= l32
                const int thr = l32 - 4 * half;
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (8 * (e / 4) + e % 4 > thr) s[e] = -INFINITY;
            }
            f32x16 p;
            float sum[2];
            auto exponentials = [&]() __attribute__((always_inline)) {
                sum[0] = sum[1] = 0.f;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    p[e] = __builtin_amdgcn_exp2f((s[e] - m) * c);
                    sum[e % 2] += p[e];
                }
            };
            exponentials();
            if (__builtin_amdgcn_ballot_w64(!(sum[0] + sum[1] <= kMostP)) != 0) {
                float mt = fmaxf(s[0], s[1]);
#pragma unroll
                for (int e = 2; e < 16; ++e) mt = fmaxf(mt, s[e]);
                // finite also where a row sees nothing but scores of -inf in the step: they weigh zero then
                const float m_new = fmaxf(fmaxf(m, max_across_halves(mt)), kLowest);
                const float corr = __builtin_amdgcn_exp2f((m - m_new) * c);
                m = m_new;
                lsum *= corr;
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b] *= corr;
                exponentials();
                rows.bad |= __builtin_amdgcn_ballot_w64(!(sum[0] + sum[1] <= kMostP));
            }
            lsum += sum[0] + sum[1];
            const Split pB[2] = {split8(p, 0, kWeightUp), split8(p, 8, kWeightUp)};
            __builtin_amdgcn_sched_barrier(0);
            st.template load<1>(tr[1], vb);
            outer<false, kLow<D>>(acc, tr[0], pB[0], rows.a, rows.job, scale_v, scale_v, [&](SplitJob &job) __attribute__((always_inline)) { take(job, tr[1], 0); return IntC<1>{}; },
                      [](auto, auto) {});
            check(tr[1]);
            outer<true, kLow<D>>(acc, tr[1], pB[1], rows.a, rows.job, scale_v, scale_k,
                [&](SplitJob &job) __attribute__((always_inline)) {
                    wait_rows<0>(rows.raw[0]);
                    rows.first_job();
                    return IntC<1>{};
                },
                [&](auto cc, auto jc) __attribute__((always_inline)) {
                    constexpr int left = NB - 1 - decltype(cc)::value;
                    if constexpr (left < 2) rows.template first_of_next<8 + 2 * (SL - 2), left, decltype(jc)::value>(st, plane_at);
                });
        }
        rows.keep();
        bad |= rows.bad != 0;
    }
    wait_fills();                 // the empty ones too: they write LDS
    lsum = add_across_halves(lsum);
    if (half == 0) stats[wave * kRows + l32] = f32x2{m, lsum};
    __syncthreads();
    float weight[kWaves], top = -INFINITY, total = 0.f;
    f32x2 of[kWaves];
#pragma unroll
    for (int g = 0; g < kWaves; ++g) {
        of[g] = stats[g * kRows + l32];
        top = fmaxf(top, of[g][0]);
    }
#pragma unroll
    for (int g = 0; g < kWaves; ++g) {
        weight[g] = __builtin_amdgcn_exp2f((of[g][0] - top) * c);         // a wave without a step: m = -inf, weight zero
        total += weight[g] * of[g][1];
    }
    f32x4 out[S::kPerWave];
    add_up<D>(lds, acc, out, weight, wave, lane);
    bad |= finish<D>(out, inverse(scale_v * kWeightUp) / total);
    if (__syncthreads_or(bad)) return false;
    if (i >= a.S) return true;
    put<D>(static_cast<float *>(a.o_out) + base + i * a.ss, out, wave, half);
    if (wave == 0 && half == 0) {
#pragma clang fp contract(off)    // the score rounded by itself, as in f32_prob
        a.lse[((int64_t)t.b * a.H + t.h) * a.S + i] = __builtin_fmaf(__builtin_amdgcn_logf(total), kLn2, top * unscale * a.scale);
    }
    return true;
}

// dS of a step, 16 values a lane of one output row (query or key), times a power of two of that row's own: what brings the largest so far to 2^10 .. 2^15.
template <int NB>
__device__ __forceinline__ void scale_ds(f32x16 &ds, float &factor, f32x16 (&acc)[NB])
{
    float top = 0.f;
#pragma unroll
    for (int e = 0; e < 16; e += 2) top = fmaxf(fmaxf(fabsf(ds[e]), fabsf(ds[e + 1])), top);
    top = max_across_halves(top);
    if (__builtin_amdgcn_ballot_w64(top * factor > 32768.f) != 0) {
        const float to = top * factor > 32768.f ? scale_for<10>(top) : factor, corr = to / factor;
        factor = to;
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b] *= corr;
    }
    ds *= factor;
}

template <int D>
__device__ __forceinline__ bool dq_rows(const AttnArgs &a, LDS_AS unsigned char *lds, const TileId t)
{
    using S = Shape<D>;
    using P = Planes<D>;
    using Tr = typename Streams<D>::Tr;
    constexpr int NB = S::kBlocks, SL = S::kBwdSlots, kPer = D / 16, kAll = 2 * kPer;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh, stat = ((int64_t)t.b * a.H + t.h) * a.S;
    const float *k = static_cast<const float *>(a.k) + base, *v = static_cast<const float *>(a.v) + base;
    const int64_t row0 = (int64_t)t.tile * kRows, i = row0 + l32, iq = i < a.S ? i : a.S - 1;
    const int steps = t.tile + 1;                     // the last one is the diagonal
    const Streams<D> st(lds + 2 * P::kBytes + wave * SL * kSlot, a.ss, lane);
    LDS_AS float *factors = (LDS_AS float *)(lds + S::kBwdStats), *scales = (LDS_AS float *)(lds + S::kBwdScales), *tops = scales + 2 * kRows;
    typename P::Own own_q, own_g, own_k, own_v;
    P::load(own_q, static_cast<const float *>(a.q) + base, a.ss, row0, a.S);
    P::load(own_g, static_cast<const float *>(a.d_o) + base, a.ss, row0, a.S);
    P::load(own_k, k, a.ss, row0, a.S);
    P::load(own_v, v, a.ss, row0, a.S);
    const float lse = a.lse[stat + iq], delta = a.delta[stat + iq];
    __builtin_amdgcn_sched_barrier(0);
    __amdgpu_buffer_rsrc_t kb = st.buffer(k, wave < steps ? wave : kNone, a.S);
#pragma unroll
    for (int n = 0; n < SL; ++n) st.fill(n, kb, n);
    const uint32_t plane_at = (uint32_t)(uintptr_t)lds + lane * 16;
    P::put(lds, scales, own_q);
    P::put(lds + P::kBytes, scales + kRows, own_g);
    put_tops(tops, P::wave_top(own_k), P::wave_top(own_v), wave, lane);
    f32x16 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = kZero16;
    float factor = 0x1p120f;      // any dS but zero brings it down
    wait_fills();                 // also the first step's: the counts in the loop are those of a step behind another
    __syncthreads();
    float scale_k, scale_v;
    streamed_scales(tops, scale_k, scale_v);
    const float scale_q = scales[l32], scale_g = scales[kRows + l32], s_scale = inverse(scale_q) * inverse(scale_k) * a.scale, nd = -delta * scale_g * scale_v;
    bool bad = far_scale(scale_q) || far_scale(scale_g) || far_scale(scale_k) || far_scale(scale_v);
    if (wave < steps) {
        RowItems<D, 2, SL> rows;
        rows.scale[0] = scale_k;
        rows.scale[1] = scale_v;
        rows.first(st, plane_at);
#pragma clang loop unroll(disable)
        for (int step = wave; step < steps && !rows.bad; step += kWaves) {
            even_out(wave, step, steps);
            const __amdgpu_buffer_rsrc_t kn = st.buffer(k, step + kWaves < steps ? step + kWaves : kNone, a.S), vb = st.buffer(v, step, a.S);
            Tr tr[2];
            f32x16 s, s1, small, dp;
            rows.run(st, plane_at, scale_k,
                [&](auto nc) __attribute__((always_inline)) {
                    constexpr int n = decltype(nc)::value;
                    static_for<n == 0 ? 0 : n + 1, n + 1 < kAll ? n + 2 : 0>([&](auto xc) __attribute__((always_inline)) {
                        constexpr int x = decltype(xc)::value + SL;    // takes the place of the rows of x - SL
                        st.fill(x % SL, x < kPer ? kb : x < kAll ? vb : kn, x % kPer);
                    });
                    if constexpr (n + 2 < kAll) wait_fills_but<(n == 0 ? 16 : n == 1 ? 8 : 0) + 2 * (SL - 1)>();
                    if constexpr (n == kAll - 3) st.template load<0>(tr[0], kb);
                },
                [&](auto nc, auto pc, auto lowc, const Split &x, const Split &y) __attribute__((always_inline)) {
                    constexpr int n = decltype(nc)::value, p = decltype(pc)::value;
                    constexpr bool low = decltype(lowc)::value;
                    if constexpr (n < kPer) score<low, n, p>(s, s1, small, x, y);
                    else dp = product<low, p>(x, y, dp);
                },
                [&](auto nc) __attribute__((always_inline)) {
                    if constexpr (decltype(nc)::value == kPer - 1) {
                        s += s1;
                        s += small;
                        if (step == steps - 1) {
                            const int thr = l32 - 4 * half;
#pragma unroll
                            for (int e = 0; e < 16; ++e)
                                if (8 * (e / 4) + e % 4 > thr) s[e] = -INFINITY;
                        }
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            s[e] = f32_prob(s[e], s_scale, lse);
                            dp[e] = nd;
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                },
                [&](SplitJob &job) __attribute__((always_inline)) { take(job, tr[0], 0); return IntC<1>{}; });
            s *= dp;
            scale_ds(s, factor, acc);
            const Split dsB[2] = {split8(s, 0), split8(s, 8)};
            __builtin_amdgcn_sched_barrier(0);
            st.template load<1>(tr[1], kb);
            outer<false, false>(acc, tr[0], dsB[0], rows.a, rows.job, scale_k, scale_k, [&](SplitJob &job) __attribute__((always_inline)) { take(job, tr[1], 0); return IntC<1>{}; },
                      [](auto, auto) {});
            outer<true, false>(acc, tr[1], dsB[1], rows.a, rows.job, scale_k, scale_k,
                [&](SplitJob &job) __attribute__((always_inline)) {
                    wait_rows<0>(rows.raw[0]);
                    rows.first_job();
                    return IntC<1>{};
                },
                [&](auto cc, auto jc) __attribute__((always_inline)) {
                    constexpr int left = NB - 1 - decltype(cc)::value;
                    if constexpr (left < 2) rows.template first_of_next<16 + 2 * (SL - 2), left, decltype(jc)::value>(st, plane_at);
                });
            kb = kn;
        }
        rows.keep();
        bad |= rows.bad != 0;
    }
    wait_fills();                 // the empty ones too: they write LDS
    if (half == 0) factors[wave * kRows + l32] = 1.f / factor;
    __syncthreads();
    float weight[kWaves];
#pragma unroll
    for (int g = 0; g < kWaves; ++g) weight[g] = factors[g * kRows + l32] * a.scale;
    f32x4 out[S::kPerWave];
    add_up<D>(lds, acc, out, weight, wave, lane);
    bad |= finish<D>(out, inverse(scale_g) * inverse(scale_v) * inverse(scale_k));
    if (__syncthreads_or(bad)) return false;
    if (i < a.S) put<D>(static_cast<float *>(a.dq) + base + i * a.ss, out, wave, half);
    return true;
}

template <int D>
__device__ __forceinline__ bool dkdv_rows(const AttnArgs &a, LDS_AS unsigned char *lds, const TileId t)
{
    using S = Shape<D>;
    using P = Planes<D>;
    using Tr = typename Streams<D>::Tr;
    constexpr int NB = S::kBlocks, SL = S::kBwdSlots, kPer = D / 16, kAll = 2 * kPer;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t base = (int64_t)t.b * a.sb + (int64_t)t.h * a.sh, stat = ((int64_t)t.b * a.H + t.h) * a.S;
    const float *q = static_cast<const float *>(a.q) + base, *g = static_cast<const float *>(a.d_o) + base;
    const int64_t col0 = (int64_t)t.tile * kRows, j = col0 + l32;
    const int first = t.tile, steps = (int)((a.S + kStep - 1) / kStep);
    const Streams<D> st(lds + 2 * P::kBytes + wave * SL * kSlot, a.ss, lane);
    LDS_AS float *factors = (LDS_AS float *)(lds + S::kBwdStats), *scales = (LDS_AS float *)(lds + S::kBwdScales), *tops = scales + 2 * kRows;
    typename P::Own own_k, own_v, own_q, own_g;
    P::load(own_k, static_cast<const float *>(a.k) + base, a.ss, col0, a.S);
    P::load(own_v, static_cast<const float *>(a.v) + base, a.ss, col0, a.S);
    P::load(own_q, q, a.ss, col0, a.S);
    P::load(own_g, g, a.ss, col0, a.S);
    __builtin_amdgcn_sched_barrier(0);
    __amdgpu_buffer_rsrc_t qb = st.buffer(q, first + wave < steps ? first + wave : kNone, a.S);
#pragma unroll
    for (int n = 0; n < SL; ++n) st.fill(n, qb, n);
    const uint32_t plane_at = (uint32_t)(uintptr_t)lds + lane * 16;
    P::put(lds, scales, own_k);
    P::put(lds + P::kBytes, scales + kRows, own_v);
    put_tops(tops, P::wave_top(own_q), P::wave_top(own_g), wave, lane);
    const uint32_t stat_bytes = (uint32_t)min(a.S * 4, (int64_t)0x7fffffff);
    const __amdgpu_buffer_rsrc_t lse_buf = __builtin_amdgcn_make_buffer_rsrc(a.lse + stat, 0, stat_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t dlt_buf = __builtin_amdgcn_make_buffer_rsrc(a.delta + stat, 0, stat_bytes, 0x00020000);
    f32x16 dk[NB], dv[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) dk[b] = dv[b] = kZero16;
    float factor = 0x1p120f;      // any dS but zero brings it down
    wait_fills();                 // also the first step's: the counts in the loop are those of a step behind another
    __syncthreads();
    float scale_q, scale_g;
    streamed_scales(tops, scale_q, scale_g);
    const float scale_k = scales[l32], scale_v = scales[kRows + l32], s_scale = inverse(scale_k) * inverse(scale_q) * a.scale, d_scale = -scale_g * scale_v;
    bool bad = far_scale(scale_q) || far_scale(scale_g) || far_scale(scale_k) || far_scale(scale_v);
    if (first + wave < steps) {
        RowItems<D, 2, SL> rows;
        rows.scale[0] = scale_q;
        rows.scale[1] = scale_g;
        rows.first(st, plane_at);
#pragma clang loop unroll(disable)
        for (int step = first + wave; step < steps && !rows.bad; step += kWaves) {
            even_out(wave, step - first, steps - first);
            const __amdgpu_buffer_rsrc_t qn = st.buffer(q, step + kWaves < steps ? step + kWaves : kNone, a.S), gb = st.buffer(g, step, a.S);
            f32x16 s, s1, small, dp;
            uint32_t ul[4], ud[4];                    // of query 8 x + 4 half + lane % 4
            rows.run(st, plane_at, scale_g,
                [&](auto nc) __attribute__((always_inline)) {
                    constexpr int n = decltype(nc)::value;
                    static_for<n == 0 ? 0 : n + 1, n + 1 < kAll ? n + 2 : 0>([&](auto xc) __attribute__((always_inline)) {
                        constexpr int x = decltype(xc)::value + SL;    // takes the place of the rows of x - SL
                        st.fill(x % SL, x < kPer ? qb : x < kAll ? gb : qn, x % kPer);
                    });
                    if constexpr (n + 2 < kAll) wait_fills_but<(n < 2 ? 32 : n >= kPer - 2 && n <= kPer ? 8 : 0) + 2 * (SL - 1)>();
                    if constexpr (n == kPer - 3) {
#pragma unroll
                        for (int x = 0; x < 4; ++x) {
                            const int at = (step * kStep + 8 * x + 4 * half + (lane & 3)) * 4;
                            ul[x] = __builtin_amdgcn_raw_buffer_load_b32(lse_buf, at, 0, 0);
                            ud[x] = __builtin_amdgcn_raw_buffer_load_b32(dlt_buf, at, 0, 0);
                        }
                    }
                },
                [&](auto nc, auto pc, auto lowc, const Split &x, const Split &y) __attribute__((always_inline)) {
                    constexpr int n = decltype(nc)::value, p = decltype(pc)::value;
                    constexpr bool low = decltype(lowc)::value;
                    if constexpr (n < kPer) score<low, n, p>(s, s1, small, x, y);
                    else dp = product<low, p>(x, y, dp);
                },
                [&](auto nc) __attribute__((always_inline)) {
                    if constexpr (decltype(nc)::value == kPer - 1) {
                        s += s1;
                        s += small;
                        const int64_t i0 = (int64_t)step * kStep;
                        if (step == first || i0 + kStep > a.S) {       // query 8 (e / 4) + 4 half + e % 4 of the step sees key l32 iff it is >= l32
                            const int thr = (step == first ? l32 : 0) - 4 * half, end = (int)min(a.S - i0, (int64_t)kStep) - 4 * half;
#pragma unroll
                            for (int e = 0; e < 16; ++e)
                                if (8 * (e / 4) + e % 4 < thr || 8 * (e / 4) + e % 4 >= end) s[e] = -INFINITY;
                        }
                        static_for<0, 16>([&](auto ec) __attribute__((always_inline)) {
                            constexpr int e = decltype(ec)::value;
                            s[e] = f32_prob(s[e], s_scale, of_quad<e % 4>(ul[e / 4]));
                            dp[e] = of_quad<e % 4>(ud[e / 4]) * d_scale;
                        });
                        __builtin_amdgcn_sched_barrier(0);
                    }
                },
                [&](SplitJob &) __attribute__((always_inline)) { return IntC<0>{}; });
            Tr tr;
            st.template load<0>(tr, gb);
            __builtin_amdgcn_sched_barrier(0);
            dp *= s;
            Split b[2] = {split8(s, 0, kProbUp), split8(s, 8, kProbUp)};
            static_for<0, 4>([&](auto uc) __attribute__((always_inline)) {
                constexpr int u = decltype(uc)::value;                 // dV over the two groups, then dK
                if constexpr (u == 2) {
                    scale_ds(dp, factor, dk);
                    b[0] = split8(dp, 0);
                    b[1] = split8(dp, 8);
                }
                const float scale = u < 2 ? scale_g : scale_q;
                take(rows.job, tr, 0);
                rows.a = rows.job.template at_once<true>(scale);
                __builtin_amdgcn_sched_barrier(0);
                outer<u == 3, false>(u < 2 ? dv : dk, tr, b[u % 2], rows.a, rows.job, scale, scale_q,
                    [&](SplitJob &job) __attribute__((always_inline)) {
                        if constexpr (u == 3) {
                            wait_rows<0>(rows.raw[0]);
                            rows.first_job();
                        }
                        return IntC<u == 3>{};
                    },
                    [&](auto cc, auto jc) __attribute__((always_inline)) {
                        constexpr int left = NB - 1 - decltype(cc)::value;
                        if constexpr (u < 3 && left == 0 && decltype(jc)::value == 0) st.template load<(u + 1) % 2>(tr, u == 0 ? gb : qb);
                        if constexpr (u == 3 && left < 2) rows.template first_of_next<32 + 2 * (SL - 2), left, decltype(jc)::value>(st, plane_at);
                    });
            });
            qb = qn;
        }
        rows.keep();
        bad |= rows.bad != 0;
    }
    wait_fills();                 // the empty ones too: they write LDS
    if (half == 0) factors[wave * kRows + l32] = 1.f / factor;
    f32x4 ov[S::kPerWave], ok[S::kPerWave];
    const float one[kWaves] = {1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f};
    add_up<D>(lds, dv, ov, one, wave, lane);
    float weight[kWaves];
#pragma unroll
    for (int g = 0; g < kWaves; ++g) weight[g] = factors[g * kRows + l32] * a.scale;
    add_up<D>(lds, dk, ok, weight, wave, lane);
    bad |= finish<D>(ov, inverse(scale_g * kProbUp));
    bad |= finish<D>(ok, inverse(scale_g) * inverse(scale_v) * inverse(scale_q));
    if (__syncthreads_or(bad)) return false;
    if (j >= a.S) return true;
    put<D>(static_cast<float *>(a.dv) + base + j * a.ss, ov, wave, half);
    put<D>(static_cast<float *>(a.dk) + base + j * a.ss, ok, wave, half);
    return true;
}

template <int D>
__global__ __launch_bounds__(512, 2) void attn_fwd_f32_split_kernel(AttnArgs a, Divisor heads, Divisor H)
{
    __shared__ __attribute__((aligned(1024))) unsigned char smem[std::max(Shape<D>::kFwdLds, kF32FwdLds<D>)];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;
    load_args_at_once(a);
    const TileId t = decode_tile(blockIdx.x, (int)((a.S + kRows - 1) / kRows), heads, H);
    if (fwd_rows<D>(a, lds, t)) return;
#pragma clang loop unroll(disable)
    for (int tile = 2 * t.tile; tile < 2 * t.tile + 2 && (int64_t)tile * kT < a.S; ++tile) {
        __syncthreads();
        f32_fwd_rows<D, false, 1, true>(a, lds, {tile, t.h, t.b}, 0);
    }
}

// both gradients in one launch (joint_slot)
template <int D>
__global__ __launch_bounds__(512, 2) void attn_bwd_f32_split_kernel(AttnArgs a, uint32_t key_tiles, Divisor heads, Divisor H)
{
    __shared__ __attribute__((aligned(1024))) unsigned char smem[std::max(Shape<D>::kBwdLds, kF32BwdLds<D>)];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;
    load_args_at_once(a);
    asm volatile("" ::"s"(a.d_o), "s"(a.delta));
    const auto [pos, hb] = heads(blockIdx.x);
    const JointSlot slot = joint_slot(key_tiles, pos);
    const TileId t = head_of(hb, slot.key ? (int)slot.rank : (int)((a.S + kRows - 1) / kRows) - 1 - (int)slot.rank, H);
    if (slot.key ? dkdv_rows<D>(a, lds, t) : dq_rows<D>(a, lds, t)) return;
#pragma clang loop unroll(disable)
    for (int tile = 2 * t.tile; tile < 2 * t.tile + 2 && (int64_t)tile * kT < a.S; ++tile) {
        __syncthreads();
        if (slot.key) f32_dkdv_rows<D, false, 1, true>(a, lds, {tile, t.h, t.b}, 0);
        else f32_dq_rows<D, false, 1, true>(a, lds, {tile, t.h, t.b}, 0);
    }
}

}  // namespace

hipError_t launch_attn_fwd_f32_split(const AttnArgs &a, hipStream_t st)
{
    const int64_t heads = (int64_t)a.H * a.B, blocks = (a.S + kRows - 1) / kRows * heads;
    if (blocks > kMaxBlocks)
        return launch_fewer_heads(a, sizeof(float), blocks, kMaxBlocks, [&](const AttnArgs &part) { return launch_attn_fwd_f32_split(part, st); });
    return launch_blocks(a.d == 128 ? attn_fwd_f32_split_kernel<128> : attn_fwd_f32_split_kernel<64>, blocks, st, a, Divisor(heads), Divisor(a.H));
}

hipError_t launch_attn_bwd_f32_split(const AttnArgs &a, bool dkdv, bool dq, hipStream_t st)
{
    const int64_t heads = (int64_t)a.H * a.B, tiles = (a.S + kRows - 1) / kRows, blocks = tiles * heads * (dkdv + dq);
    if (blocks > kMaxBlocks)
        return launch_fewer_heads(a, sizeof(float), blocks, kMaxBlocks, [&](const AttnArgs &part) { return launch_attn_bwd_f32_split(part, dkdv, dq, st); });
    return launch_blocks(a.d == 128 ? attn_bwd_f32_split_kernel<128> : attn_bwd_f32_split_kernel<64>, blocks, st, a, dkdv ? (uint32_t)tiles : 0u,
                         Divisor(heads), Divisor(a.H));
}

}  // namespace memo

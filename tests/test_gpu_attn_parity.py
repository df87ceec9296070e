"""GPU parity: the HIP attention path vs the fp64 oracle, element by element, through the
C-ABI.  Sizes here are ones the dense oracle finishes in seconds; they span several tiles
(256-row query tiles and 64-row key tiles in the forward and dQ kernels, 256-row key tiles and 32-row
query tiles in the dK/dV kernel) and ragged tails."""
import math

import numpy as np
import pytest
import torch

from paper_2407_12117_amd import binding as mb
from paper_2407_12117_amd import synth
import shape_cases as shapes
from gpu_util import LSE_MAX_ABS_BF16, assert_close, gpu_fwd_bwd, to_f64

pytestmark = pytest.mark.gpu


def _dense_case(oracle, B, S, H, d, dtype, seed, scale=None, scaled=False):
    print(f"[case] dense B={B} S={S} H={H} d={d} {dtype} seed={seed}", flush=True)
    scale = synth.default_scale(d) if scale is None else scale
    q, k, v, g = synth.attn_inputs(B, S, H, d, dtype, seed)
    o, lse, dq, dk, dv = gpu_fwd_bwd(*(t.cuda() for t in (q, k, v, g)), scale)
    qf, kf, vf, gf = (to_f64(t) for t in (q, k, v, g))
    ro, rlse = oracle.attn_fwd(qf, kf, vf, scale)
    rdq, rdk, rdv = oracle.attn_bwd(qf, kf, vf, gf, scale)
    assert_close("O", to_f64(o), ro, dtype)
    lse_err = np.abs(to_f64(lse) - rlse).max()
    assert lse_err <= (LSE_MAX_ABS_BF16 if dtype == "bf16" else 1e-4), f"LSE max_abs={lse_err:.3e}"
    assert_close("dQ", to_f64(dq), rdq, dtype, scaled)
    assert_close("dK", to_f64(dk), rdk, dtype, scaled)
    assert_close("dV", to_f64(dv), rdv, dtype, scaled)


def test_c1_fp32_dense(oracle):
    c = synth.CONFIGS["C1"]
    _dense_case(oracle, c["B"], c["S"], c["H"], c["d"], "f32", synth.config_seed("C1"))


@pytest.mark.parametrize("B,S,H,d", [(2, 333, 3, 64), (1, 257, 2, 128), (1, 1, 1, 64), (2, 31, 1, 128)])
def test_fp32_ragged_and_small(oracle, B, S, H, d):
    _dense_case(oracle, B, S, H, d, "f32", 7 + S)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("S,heads", [(15, 2), (17, 70), (128, 3), (289, 24), (289, 64), (500, 100), (1025, 2)])
def test_fp32_every_workgroup_shape(oracle, S, heads, d):
    # few and many workgroups (all of them resident at once or not), lengths on and off their 16-row tiles, fewer tiles
    # than the waves that share them out
    _dense_case(oracle, 1, S, heads, d, "f32", 900 + S + heads)


def test_fp32_padded_rows(oracle):
    B, S, H, d = 2, 150, 3, 64
    print("[case] fp32 padded rows", flush=True)
    scale = synth.default_scale(d)
    q, k, v, g = synth.attn_inputs(B, S, H, d, "f32", 21)

    def padded(values=None):
        buf = torch.zeros(B, S, H, d + 12, device="cuda")[..., :d]
        if values is not None:
            buf.copy_(values)
        return buf

    qd, kd, vd, gd = (padded(x) for x in (q, k, v, g))
    o, lse = mb.memo_attn_fwd(qd, kd, vd, scale, o=padded())
    dq, dk, dv = mb.memo_attn_bwd(qd, kd, vd, o, lse, gd, scale, dq=padded(), dk=padded(), dv=padded())
    torch.cuda.synchronize()
    qf, kf, vf, gf = (to_f64(x) for x in (q, k, v, g))
    ro, rlse = oracle.attn_fwd(qf, kf, vf, scale)
    for name, got, ref in zip(("O", "LSE", "dQ", "dK", "dV"), (o, lse, dq, dk, dv),
                              (ro, rlse) + tuple(oracle.attn_bwd(qf, kf, vf, gf, scale))):
        assert_close(name, to_f64(got), ref, "f32")


@pytest.mark.parametrize("S", [1, 2, 31, 32, 33, 63, 64, 65, 97, 127, 128, 129, 200, 255, 256, 257, 287, 289, 383, 385, 511, 513, 777])
def test_bf16_small_and_ragged(oracle, S):
    _dense_case(oracle, 2, S, 2, 128, "bf16", 100 + S)


@pytest.mark.parametrize("B,S,H", [(1, 2048, 2), (2, 1024, 3), (1, 3000, 1)])
def test_bf16_multi_tile(oracle, B, S, H):
    _dense_case(oracle, B, S, H, 128, "bf16", 300 + S)


def test_bf16_many_query_tiles_dense(oracle):
    # every element compared over a long sweep of one head, with a ragged tail: the 32-row forward (eight waves that
    # take up to 65 key tiles each) and the 64-row joint backward (four query groups of up to 129 query tiles
    # each beside dQ workgroups of four key groups)
    _dense_case(oracle, 1, 16461, 1, 128, "bf16", 333)


@pytest.mark.parametrize("S", [289, 513, 700])
@pytest.mark.parametrize("heads", [2, 24, 32, 48, 64, 100, 160])
def test_bf16_every_workgroup_shape(oracle, S, heads):
    # how a launch is cut into workgroups (32 to 256 rows each, keys or queries split over up to eight
    # wave groups, single tiles or pairs) depends on the length and the number of heads: few heads take the
    # small tiles, many the large ones.  Scaled bar: among this many heads some |dV| exceeds 4 (dV of the
    # first keys sums dO over rows that see little else), where half a bf16 ulp is 2^-6 = 1.6e-2 of the
    # unscaled bar's 2e-2; the relative bar is the plain one
    _dense_case(oracle, 1, S, heads, 128, "bf16", 7000 + S + heads, scaled=True)


@pytest.mark.parametrize("S,heads", shapes.FWD_64_EDGES)
def test_bf16_forward_64_row_edges(oracle, S, heads):
    # the 64-row forward with one row, one block of rows, one more and all but one in the last tile, whose second block
    # sees a key tile that the first does not
    _dense_case(oracle, 1, S, heads, 128, "bf16", 9000 + S, scaled=True)


@pytest.mark.parametrize("B,H", [(1, 1), (3, 1), (1, 7), (5, 3), (2, 13)])
def test_bf16_short_forward_batches_and_heads(oracle, B, H):
    # 32-row workgroups: which head and batch entry a workgroup id stands for, for divisors that are a power of two, one
    # and neither; nine tiles, of which the first eight leave waves without a key tile
    _dense_case(oracle, B, 257, H, 128, "bf16", 9500 + 16 * B + H)


@pytest.mark.parametrize("S,heads", shapes.BWD_32_EDGES)
def test_bf16_backward_32_row_edges(oracle, S, heads):
    _dense_case(oracle, 1, S, heads, 128, "bf16", 9100 + S)


@pytest.mark.parametrize("S,heads", list(shapes.BWD_LONG_SHAPES))
def test_bf16_ragged_lengths_of_256_row_workgroups(oracle, S, heads):
    # whole rounds of pairs (an even and an odd number of tiles, so that a pair may be one tile), one tile at a time, and both in
    # one backward: the first, a middle and the last head compared in full
    print(f"[case] ragged 256-row S={S} H={heads}", flush=True)
    scale = synth.default_scale(128)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(S)
    q, k, v, g = (torch.randn((1, S, heads, 128), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4))
    got = gpu_fwd_bwd(q, k, v, g, scale)
    for h in (0, heads // 2 - 1, heads - 1):
        qf, kf, vf, gf = (to_f64(t[:, :, h:h + 1]) for t in (q, k, v, g))
        ro, rlse = oracle.attn_fwd(qf, kf, vf, scale)
        assert_close("O", to_f64(got[0][:, :, h:h + 1]), ro, "bf16")
        assert np.abs(to_f64(got[1][:, h:h + 1]) - rlse).max() <= LSE_MAX_ABS_BF16
        for name, x, r in zip(("dQ", "dK", "dV"), got[2:], oracle.attn_bwd(qf, kf, vf, gf, scale)):
            assert_close(name, to_f64(x[:, :, h:h + 1]), r, "bf16", scaled=True)


def test_bf16_scale_below_the_usual_one(oracle):
    _dense_case(oracle, 1, 500, 2, 128, "bf16", 41, scale=0.06)


def test_bf16_scale_above_the_usual_one(oracle):
    # scale 0.2 > 1/sqrt(128): peaked softmax, gradients of magnitude > 4, where half a bf16 ulp
    # alone exceeds 2e-2: the absolute bar scales with max|ref| (gpu_util), the relative one stays
    _dense_case(oracle, 1, 500, 2, 128, "bf16", 41, scale=0.2, scaled=True)


@pytest.mark.parametrize("log2_per_tile", [3.0, 12.0, 500.0])
def test_bf16_forward_with_scores_climbing_along_the_keys(oracle, log2_per_tile):
    # The forward keeps a running maximum that it brings up to date only when a row sum shows a score
    # far above it (2^40).  Here every score grows with the key index by `log2_per_tile` binary orders
    # of magnitude per 64-key tile: 3 and 12 let the exponentials run up to 2^40 between updates, 500
    # forces an update (and the rescaling of everything accumulated so far) on every tile.
    # Forward only: with a common offset this large in K, dQ and dK are differences of nearly equal
    # sums, which the bf16 rounding of dS alone moves by several per cent in any implementation.
    B, S, H, d = 1, 1100, 2, 128
    scale = synth.default_scale(d)
    q, k, v, _ = synth.attn_inputs(B, S, H, d, "bf16", 77)
    slope = log2_per_tile / 64.0 / (scale * math.log2(math.e))        # growth of q.k per key
    q = (0.05 * q.float() + 1.0).to(torch.bfloat16)                     # q.k = sum_c k_c, nearly
    k = (0.05 * k.float() + (slope / d) * torch.arange(S, dtype=torch.float32).view(1, S, 1, 1)).to(torch.bfloat16)
    print(f"[case] climbing scores, {log2_per_tile} binary orders per tile", flush=True)
    o, lse = mb.memo_attn_fwd(q.cuda(), k.cuda(), v.cuda(), scale)
    ro, rlse = oracle.attn_fwd(to_f64(q), to_f64(k), to_f64(v), scale)
    assert_close("O", to_f64(o), ro, "bf16")
    # the logsumexp itself grows to thousands here: fp32 holds it to a relative 2^-24 or so
    assert np.abs(to_f64(lse) - rlse).max() <= LSE_MAX_ABS_BF16 * max(1.0, np.abs(rlse).max())


def test_bf16_nan_in_one_key_row_reaches_what_depends_on_it():
    # a NaN in key row j of head 0: o, lse, dq of query rows i >= j are non-finite (they see the key),
    # rows before the 256-row block of j are bit-identical to the clean run (inside the block a masked
    # zero probability may still meet the NaN in a contraction); every dk, dv row of that head is
    # reached through some query row i >= j; head 1 is untouched
    B, S, H, d, j = 1, 700, 2, 128, 389
    q, k, v, g = (t.cuda() for t in synth.attn_inputs(B, S, H, d, "bf16", 123))
    scale = synth.default_scale(d)
    clean = gpu_fwd_bwd(q, k, v, g, scale)
    k2 = k.clone()
    k2[0, j, 0, 5] = float("nan")
    o, lse, dq, dk, dv = gpu_fwd_bwd(q, k2, v, g, scale)
    for name, t, c, tok in (("o", o, clean[0], 1), ("lse", lse, clean[1], 2), ("dq", dq, clean[2], 1)):
        sl = lambda x, a, b, h: x[0, a:b, h] if tok == 1 else x[0, h, a:b]
        assert torch.isnan(sl(t, j, S, 0).float()).all(), f"{name}: rows that see the NaN key must be NaN"
        assert torch.equal(sl(t, 0, j // 256 * 256, 0), sl(c, 0, j // 256 * 256, 0)), f"{name}: rows before the NaN key's block changed"
        assert torch.equal(sl(t, 0, S, 1), sl(c, 0, S, 1)), f"{name}: the other head changed"
    for name, t, c in (("dk", dk, clean[3]), ("dv", dv, clean[4])):
        assert torch.isnan(t[0, :, 0].float()).all(), f"{name}: every key row of the head is reached"
        assert torch.equal(t[0, :, 1], c[0, :, 1]), f"{name}: the other head changed"


def test_bf16_strided_views_of_a_packed_qkv(oracle):
    # q, k, v as slices of one [B,S,3,H,d] buffer: stride_s = 3*H*d
    B, S, H, d = 1, 640, 2, 128
    print(f"[case] packed qkv S={S}", flush=True)
    scale = synth.default_scale(d)
    q, k, v, g = synth.attn_inputs(B, S, H, d, "bf16", 55)
    packed = torch.stack((q, k, v), dim=2).cuda()
    pg = torch.zeros_like(packed)
    pg[:, :, 0] = g.cuda()
    qd, kd, vd, gd = packed[:, :, 0], packed[:, :, 1], packed[:, :, 2], pg[:, :, 0]
    out = torch.zeros_like(packed)
    o, lse = mb.memo_attn_fwd(qd, kd, vd, scale, o=out[:, :, 0])
    grads = torch.zeros_like(packed)
    dq, dk, dv = mb.memo_attn_bwd(qd, kd, vd, o, lse, gd, scale, dq=grads[:, :, 0], dk=grads[:, :, 1],
                                  dv=grads[:, :, 2])
    torch.cuda.synchronize()
    qf, kf, vf, gf = (to_f64(t) for t in (q, k, v, g))
    ro, _ = oracle.attn_fwd(qf, kf, vf, scale)
    rdq, rdk, rdv = oracle.attn_bwd(qf, kf, vf, gf, scale)
    assert_close("O", to_f64(o), ro, "bf16")
    assert_close("dQ", to_f64(dq), rdq, "bf16")
    assert_close("dK", to_f64(dk), rdk, "bf16")
    assert_close("dV", to_f64(dv), rdv, "bf16")
    # the untouched slots of the packed output buffers stay zero
    assert out[:, :, 1:].abs().max().item() == 0.0


@pytest.mark.parametrize("seed", [0, 1, 2])
def test_bf16_random_shapes_and_row_padding(oracle, seed):
    # shapes drawn at random (batch 1..2, heads 1..3, lengths on no tile edge in particular), rows
    # of 128 values inside rows of 128, 136 or 192: all eight tensors share the padded layout
    rng = np.random.default_rng(seed)
    scale = synth.default_scale(128)
    for case in range(5):
        B, H = int(rng.integers(1, 3)), int(rng.integers(1, 4))
        S = int(rng.choice([rng.integers(1, 70), rng.integers(70, 600), rng.integers(600, 2200)]))
        pad = int(rng.choice([0, 8, 64]))
        print(f"[case] random shape seed={seed} B={B} S={S} H={H} pad={pad}", flush=True)

        def padded(values=None):
            buf = torch.zeros(B, S, H, 128 + pad, dtype=torch.bfloat16, device="cuda")[..., :128]
            if values is not None:
                buf.copy_(values)
            return buf

        q, k, v, g = synth.attn_inputs(B, S, H, 128, "bf16", 5000 + 10 * seed + case)
        qd, kd, vd, gd = (padded(x) for x in (q, k, v, g))
        o, lse = mb.memo_attn_fwd(qd, kd, vd, scale, o=padded())
        dq, dk, dv = mb.memo_attn_bwd(qd, kd, vd, o, lse, gd, scale, dq=padded(), dk=padded(), dv=padded())
        torch.cuda.synchronize()
        qf, kf, vf, gf = (to_f64(x) for x in (q, k, v, g))
        ro, rlse = oracle.attn_fwd(qf, kf, vf, scale)
        rdq, rdk, rdv = oracle.attn_bwd(qf, kf, vf, gf, scale)
        assert_close("O", to_f64(o), ro, "bf16")
        assert np.abs(to_f64(lse) - rlse).max() <= LSE_MAX_ABS_BF16
        assert_close("dQ", to_f64(dq), rdq, "bf16")
        assert_close("dK", to_f64(dk), rdk, "bf16")
        assert_close("dV", to_f64(dv), rdv, "bf16")


def test_bf16_constant_values_give_constant_output():
    # rows of the softmax sum to one: V = 1 -> O = 1 (bf16 rounding of P allows 2^-8)
    B, S, H, d = 1, 1500, 2, 128
    q, k, _, _ = synth.attn_inputs(B, S, H, d, "bf16", 77)
    v = torch.ones_like(q)
    o, _ = mb.memo_attn_fwd(q.cuda(), k.cuda(), v.cuda(), synth.default_scale(d))
    torch.cuda.synchronize()
    assert (o.float() - 1.0).abs().max().item() <= 2 ** -7


def test_bf16_causality():
    # changing keys / values after position p leaves O[:p], LSE[:p] bit-identical
    B, S, H, d, p = 1, 700, 1, 128, 300
    q, k, v, _ = (t.cuda() for t in synth.attn_inputs(B, S, H, d, "bf16", 88))
    scale = synth.default_scale(d)
    o1, l1 = mb.memo_attn_fwd(q, k, v, scale)
    k2, v2 = k.clone(), v.clone()
    k2[:, p:] += 3.0
    v2[:, p:] -= 2.0
    o2, l2 = mb.memo_attn_fwd(q, k2, v2, scale)
    torch.cuda.synchronize()
    assert torch.equal(o1[:, :p], o2[:, :p]) and torch.equal(l1[:, :, :p], l2[:, :, :p])
    assert not torch.equal(o1[:, p:], o2[:, p:])


def test_bf16_is_deterministic():
    B, S, H, d = 1, 900, 2, 128
    q, k, v, g = (t.cuda() for t in synth.attn_inputs(B, S, H, d, "bf16", 99))
    a = gpu_fwd_bwd(q, k, v, g, synth.default_scale(d))
    b = gpu_fwd_bwd(q, k, v, g, synth.default_scale(d))
    for x, y in zip(a, b):
        assert torch.equal(x, y)


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_rows_far_apart(d):
    # rows 2^26 floats apart take the fills with full addresses: the same bits as a contiguous copy
    S, ss = 19, 1 << 26
    scale = synth.default_scale(d)
    q, k, v, g = (t.cuda() for t in synth.attn_inputs(1, S, 1, d, "f32", seed=77))
    o, lse = mb.memo_attn_fwd(q, k, v, scale)
    grads = mb.memo_attn_bwd(q, k, v, o, lse, g, scale)
    buf = torch.zeros((S - 1) * ss + 8 * d, dtype=torch.float32, device="cuda")
    far = [torch.as_strided(buf, (1, S, 1, d), (S * ss, ss, d, 1), n * d) for n in range(8)]
    for dst, src in zip(far, (q, k, v, g)):
        dst.copy_(src)
    _, lse_far = mb.memo_attn_fwd(far[0], far[1], far[2], scale, o=far[4])
    mb.memo_attn_bwd(far[0], far[1], far[2], far[4], lse_far, far[3], scale, dq=far[5], dk=far[6], dv=far[7])
    assert torch.equal(far[4], o) and torch.equal(lse_far, lse)
    for got, ref in zip(far[5:], grads):
        assert torch.equal(got, ref)


def _key_mask_case(oracle, S, H, d, dtype, value, tile, scaled=False):
    # a key mask carried in a head-dim column: q is 1 there, k is `value` at the masked keys and 0 elsewhere.  Head h masks
    # the h-th tile of `tile` keys (past tile 0, so that every row keeps some key), modulo the tiles there are: every wave
    # of every workgroup shape gets a first tile of which a row sees nothing else
    print(f"[case] key mask {value} S={S} H={H} d={d} {dtype} tile={tile}", flush=True)
    scale = synth.default_scale(d)
    q, k, v, g = synth.attn_inputs(1, S, H, d, dtype, 40 + S)
    q[..., 0], k[..., 0] = 1.0, 0.0
    for h in range(H):
        first = tile * (1 + h % ((S - 1) // tile))
        k[:, first:first + tile, h, 0] = value
    got = gpu_fwd_bwd(*(t.cuda() for t in (q, k, v, g)), scale)
    qf, kf, vf, gf = (to_f64(t) for t in (q, k, v, g))
    ref = oracle.attn_fwd(qf, kf, vf, scale) + tuple(oracle.attn_bwd(qf, kf, vf, gf, scale))
    for name, x, r in zip(("O", "LSE", "dQ", "dK", "dV"), got, ref):
        x = to_f64(x)
        if name == "dQ":          # its mask column is zero times an infinity
            x, r = x[..., 1:], r[..., 1:]
        if name == "LSE":
            assert np.abs(x - r).max() <= LSE_MAX_ABS_BF16
        else:
            assert_close(name, x, r, dtype, scaled and name != "O")


# S is a whole number of tiles, masks from "never" to values whose products with the scale lose whole powers of two to rounding
@pytest.mark.parametrize("value", [-math.inf, float(np.finfo(np.float32).min), -1e20, -1e9])
@pytest.mark.parametrize("d", [64, 128])
def test_fp32_masked_first_tiles(oracle, d, value):
    _key_mask_case(oracle, 288, 9, d, "f32", value, 16)


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_rows_without_a_key(oracle, d):
    # the first 20 keys masked: rows 0 .. 19 see nothing.  -inf: those rows are NaN, the others as if the keys were not there;
    # a finite mask leaves a uniform softmax over them, and a zero dO keeps them out of the gradients
    S, H, dead = 150, 2, 20
    print(f"[case] fp32 rows without a key d={d}", flush=True)
    scale = synth.default_scale(d)
    q, k, v, g = synth.attn_inputs(1, S, H, d, "f32", 77)
    q[..., 0], k[..., 0] = 1.0, 0.0
    g[:, :dead] = 0.0
    for value in (-math.inf, float(np.finfo(np.float32).min), -1e20):
        k[:, :dead, :, 0] = value
        qd, kd, vd, gd = (t.cuda() for t in (q, k, v, g))
        o, lse = mb.memo_attn_fwd(qd, kd, vd, scale)
        live = [to_f64(t[:, dead:]) for t in (q, k, v, g)]
        ro, rlse = oracle.attn_fwd(*live[:3], scale)
        assert_close("O", to_f64(o[:, dead:]), ro, "f32")
        assert np.abs(to_f64(lse[:, :, dead:]) - rlse).max() <= 1e-4
        if value == -math.inf:
            assert torch.isnan(o[:, :dead]).all() and torch.isneginf(lse[:, :, :dead]).all()
            continue
        assert torch.isfinite(o[:, :dead]).all()
        dq, dk, dv = mb.memo_attn_bwd(qd, kd, vd, o, lse, gd, scale)
        rdq, rdk, rdv = oracle.attn_bwd(*live, scale)
        assert_close("dQ", to_f64(dq[:, dead:, :, 1:]), rdq[..., 1:], "f32")
        assert_close("dK", to_f64(dk[:, dead:]), rdk, "f32")
        assert_close("dV", to_f64(dv[:, dead:]), rdv, "f32")
        for name, x in (("dQ", dq[..., 1:]), ("dK", dk), ("dV", dv)):
            assert (x[:, :dead] == 0).all(), f"{name}: a row without a key is touched by its zero dO"


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_large_scores(oracle, d):
    # scores of +-40: the softmax is peaked, and an error e of a score is a relative error e of its probability.  Bound: a scaled
    # score below 2^6 is held to 2^-19 (half an ulp is 2^-19), its sum of d/4 products per chain and the logsumexp add about
    # as much again in the 2-norm; the forward must form the scores in the order of the backward for the two to cancel
    S, H = 1500, 2
    print(f"[case] fp32 large scores d={d}", flush=True)
    scale = synth.default_scale(d)
    q, k, v, g = synth.attn_inputs(1, S, H, d, "f32", 61)
    q = q * 10
    got = gpu_fwd_bwd(*(t.cuda() for t in (q, k, v, g)), scale)
    qf, kf, vf, gf = (to_f64(t) for t in (q, k, v, g))
    ref = oracle.attn_fwd(qf, kf, vf, scale)[:1] + tuple(oracle.attn_bwd(qf, kf, vf, gf, scale))
    for name, x, r in zip(("O", "dQ", "dK", "dV"), (got[0],) + got[2:], ref):
        rel = np.linalg.norm(to_f64(x) - r) / np.linalg.norm(r)
        print(f"  {name} rel {rel:.2e}", flush=True)
        assert rel <= 2 ** -19 + 2 ** -22, f"{name}: rel_l2={rel:.2e}"


# every shape of the forward; all lengths whole 32-row tiles
@pytest.mark.parametrize("value", [-math.inf, float(torch.finfo(torch.bfloat16).min), -1e20, -1e9])
@pytest.mark.parametrize("S,heads,tile", list(shapes.FWD_SHAPES))
def test_bf16_masked_first_tiles(oracle, S, heads, tile, value):
    _key_mask_case(oracle, S, heads, 128, "bf16", value, tile, scaled=True)


def test_bf16_rows_without_a_key(oracle):
    # keys 0 .. 19 at -inf: rows 0 .. 19 are NaN (their logsumexp too, or -inf), the others as if the keys were not there
    for S, H in ((300, 2), (320, 48), (352, 48), (700, 100)):
        print(f"[case] bf16 rows without a key S={S} H={H}", flush=True)
        dead, scale = 20, synth.default_scale(128)
        q, k, v, _ = synth.attn_inputs(1, S, H, 128, "bf16", 78)
        q[..., 0], k[..., 0] = 1.0, 0.0
        k[:, :dead, :, 0] = -math.inf
        o, lse = mb.memo_attn_fwd(q.cuda(), k.cuda(), v.cuda(), scale)
        ro, rlse = oracle.attn_fwd(*(to_f64(t[:, dead:]) for t in (q, k, v)), scale)
        assert_close("O", to_f64(o[:, dead:]), ro, "bf16")
        assert np.abs(to_f64(lse[:, :, dead:]) - rlse).max() <= LSE_MAX_ABS_BF16
        assert torch.isnan(o[:, :dead].float()).all() and not torch.isfinite(lse[:, :, :dead]).any()


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_masked_keys_before_a_ragged_end(oracle, d):
    # key rows of -inf meet the rows past S of the last query tile
    _key_mask_case(oracle, 300, 18, d, "f32", -math.inf, 16)


@pytest.mark.parametrize("S,heads", list(shapes.BWD_SHAPES))
def test_bf16_masked_keys_before_a_ragged_end(oracle, S, heads):
    # as above, in every joint shape of the backward
    _key_mask_case(oracle, S, heads, 128, "bf16", -math.inf, 32, scaled=True)


# one case for each workgroup shape of the backward, and the pair of launches of the longer sequences
@pytest.mark.parametrize("dtype,S,H,d", [("f32", 333, 2, 64), ("f32", 700, 40, 128), ("bf16", 300, 3, 128), ("bf16", 353, 48, 128),
                                         ("bf16", 513, 64, 128), ("bf16", 700, 160, 128), ("bf16", 8155, 16, 128)])
def test_outputs_in_place_of_inputs(dtype, S, H, d):
    print(f"[case] in place {dtype} S={S} H={H} d={d}", flush=True)
    scale = synth.default_scale(d)
    q, k, v, g = (t.cuda() for t in synth.attn_inputs(1, S, H, d, dtype, 31 + S))
    want = gpu_fwd_bwd(q, k, v, g, scale)
    # the forward writes o over q
    q2 = q.clone()
    o, lse = mb.memo_attn_fwd(q2, k, v, scale, o=q2)
    assert torch.equal(o, want[0]) and torch.equal(lse, want[1])
    # the backward writes dq over q, then over d_o, and dk over o
    for place in ("q", "d_o"):
        q2, g2, o2 = q.clone(), g.clone(), want[0].clone()
        got = mb.memo_attn_bwd(q2, k, v, o2, want[1], g2, scale, dq=q2 if place == "q" else g2, dk=o2)
        for name, x, y in zip(("dQ", "dK", "dV"), got, want[2:]):
            assert torch.equal(x, y), f"{name} differs with dQ in place of {place}"


@pytest.mark.parametrize("dtype,S,H,d", [("f32", 333, 2, 64), ("bf16", 300, 3, 128), ("bf16", 640, 2, 128), ("bf16", 353, 48, 128),
                                         ("bf16", 513, 64, 128), ("bf16", 700, 160, 128), ("bf16", 8155, 16, 128)])
def test_stage_events_do_not_change_the_gradients(dtype, S, H, d):
    print(f"[case] stage events {dtype} S={S} H={H} d={d}", flush=True)
    scale = synth.default_scale(d)
    q, k, v, g = (t.cuda() for t in synth.attn_inputs(1, S, H, d, dtype, 33 + S))
    o, lse = mb.memo_attn_fwd(q, k, v, scale)
    want = mb.memo_attn_bwd(q, k, v, o, lse, g, scale)
    events = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    got = mb.memo_attn_bwd(q, k, v, o, lse, g, scale, stage_events=events)
    torch.cuda.synchronize()
    for name, x, y in zip(("dQ", "dK", "dV"), got, want):
        assert torch.equal(x, y), f"{name} differs"
    assert all(a.elapsed_time(b) > 0 for a, b in zip(events, events[1:]))


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 128)])
def test_more_workgroups_than_one_launch_takes(dtype, d):
    # 8.45 million sequences of one token: with 512 threads a workgroup, more than the 2^32 threads of a HIP launch.  One token:
    # o = v, lse = scale q.k, dv = d_o, dq = dk = 0
    B, H = 65535, 129
    print(f"[case] {B * H} heads of one token {dtype}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    x = torch.randn((B, 1, H, d), generator=gen, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)
    o, lse = mb.memo_attn_fwd(x, x, x, 0.125)
    assert torch.equal(o, x)
    want = 0.125 * (x.float() ** 2).sum(3).permute(0, 2, 1)
    assert ((lse - want).abs() <= 1e-5 * want.clamp(min=1.0)).all()
    dq, dk, dv = mb.memo_attn_bwd(x, x, x, o, lse, x, 0.125)
    # dP - D cancels but for the order of its sums: sqrt(d) roundings of 2^-24 of |v|^2 < 400, times scale |k| < 1
    assert torch.equal(dv, x) and dq.float().abs().max() <= 3e-4 and dk.float().abs().max() <= 3e-4


def _far_rows(dtype, S, H, d, ss):
    # rows `ss` elements apart, eight tensors side by side in them, against contiguous copies: the same bits
    print(f"[case] rows far apart {dtype} S={S} H={H} d={d} stride {ss}", flush=True)
    scale = synth.default_scale(d)
    q, k, v, g = (t.cuda() for t in synth.attn_inputs(1, S, H, d, dtype, seed=78))
    o, lse = mb.memo_attn_fwd(q, k, v, scale)
    grads = mb.memo_attn_bwd(q, k, v, o, lse, g, scale)
    buf = torch.zeros((S - 1) * ss + 8 * H * d, dtype=q.dtype, device="cuda")
    far = [torch.as_strided(buf, (1, S, H, d), (S * ss, ss, d, 1), n * H * d) for n in range(8)]
    for dst, src in zip(far, (q, k, v, g)):
        dst.copy_(src)
    _, lse_far = mb.memo_attn_fwd(far[0], far[1], far[2], scale, o=far[4])
    mb.memo_attn_bwd(far[0], far[1], far[2], far[4], lse_far, far[3], scale, dq=far[5], dk=far[6], dv=far[7])
    assert torch.equal(far[4], o) and torch.equal(lse_far, lse)
    for got, ref in zip(far[5:], grads):
        assert torch.equal(got, ref)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("ss", [(1 << 25) + 4, (1 << 26) - 4])
def test_fp32_rows_almost_too_far_for_a_buffer(d, ss):
    # a 16-row tile spans 2 to 4 GiB: offsets above 2^31 in the fills
    _far_rows("f32", 35, 1, d, ss)


@pytest.mark.parametrize("S,heads", [(70, 1), (257, 48), (353, 48), (513, 64), (700, 160)])
def test_bf16_rows_as_far_apart_as_accepted(S, heads):
    # the largest row stride that is not refused: a 64-row tile spans 2 GiB, in every shape of both directions
    _far_rows("bf16", S, heads, 128, 1 << 24)


@pytest.mark.parametrize("B,S,H", [(1, 33, 1), (2, 255, 2), (1, 480, 4), (1, 1023, 2), (1, 1025, 2), (1, 2050, 1)])
def test_bf16_columns_in_parts(oracle, B, S, H):
    # launches that go out with the output columns in four, two and one parts, on both sides of either limit (64 and 128
    # workgroups), forward and backward; fewer tiles than waves among them
    _dense_case(oracle, B, S, H, 128, "bf16", 8100 + S)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,S,H", [(1, 17, 1), (2, 250, 2), (1, 513, 1), (1, 529, 2), (1, 1025, 1), (1, 2049, 1)])
def test_fp32_columns_in_parts(oracle, B, S, H, d):
    # the same for the 16-row workgroups of fp32
    _dense_case(oracle, B, S, H, d, "f32", 8200 + S)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,S,H", [(1, 1, 1), (1, 15, 2), (1, 15, 270), (2, 19, 70), (1, 129, 3)])
def test_fp32_rows_that_all_waves_share(oracle, B, S, H, d):
    # one to nine tiles of 16 rows, ragged last ones: waves that bring in rows for the others and have no tile of their own, with
    # the columns in four parts, in two and in one
    _dense_case(oracle, B, S, H, d, "f32", 8300 + S)


@pytest.mark.parametrize("S,H", [(257, 14), (257, 16), (2033, 2), (2049, 2), (4097, 1), (5120, 1), (5121, 1), (6003, 1)])
def test_fp32_rows_shared_and_not(oracle, S, H):
    # head dim 64 in one part, on both sides of the lengths and numbers of workgroups from which each wave brings in the workgroup's
    # rows for itself, forward and backward
    _dense_case(oracle, 1, S, H, 64, "f32", 8400 + S)

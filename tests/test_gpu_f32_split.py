"""The fp32 attention kernels on fp16 matrix instructions (csrc/attn_f32_split.hip) where they can go wrong: steps, rows and waves at their edges, magnitudes
that need a scale, rows that one scale does not fit, running maxima that climb, values that are not finite (both of these are worked again by the fp32 kernels)."""
import math

import numpy as np
import pytest
import torch

import shape_cases as shapes
from gpu_util import assert_close, gpu_fwd_bwd, to_f64
from paper_2407_12117_amd import binding as mb
from paper_2407_12117_amd import synth

pytestmark = pytest.mark.gpu

NAMES = ("O", "dQ", "dK", "dV")


@pytest.fixture(scope="module")
def oracle():
    from oracle import memo_oracle
    memo_oracle.build()
    return memo_oracle


def _inputs(S, H, d, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.randn((1, S, H, d), generator=gen, device="cuda") for _ in range(4)]


def _relative_errors(oracle, q, k, v, g, heads):
    scale = synth.default_scale(q.shape[-1])
    o, lse, dq, dk, dv = gpu_fwd_bwd(q, k, v, g, scale)
    worst = dict.fromkeys(NAMES, 0.0)
    for h in heads:
        one = [to_f64(t[:, :, h:h + 1]) for t in (q, k, v, g)]
        ro, rlse = oracle.attn_fwd(*one[:3], scale)
        for name, x, r in zip(NAMES, (o, dq, dk, dv), (ro,) + tuple(oracle.attn_bwd(*one, scale))):
            worst[name] = max(worst[name], float(np.linalg.norm(to_f64(x[:, :, h:h + 1]) - r) / np.linalg.norm(r)))
        assert np.abs(to_f64(lse[:, h:h + 1]) - rlse).max() <= 2e-6 * max(1.0, np.abs(rlse).max())
    print("  " + " ".join(f"{n} {e:.1e}" for n, e in worst.items()), flush=True)
    return worst


# Relative error of a sum of products of which each is off by at most 2^-22 (two parts of 12 bits each, the product of the two low ones left out) and that is
# rounded to 2^-24 some n / 16 times, with random signs: below 2^-22.  Probabilities are off by what their exponent is: three roundings of a number of up to 16
# (log2 of 1 / P here), each up to 2^-21 of it and 2^-22.4 in the mean square, so 2^-22.1 in all; the gradients go through two such sums and the probabilities, and
# through dP - D, whose terms of up to the same size are both off: 2 (2 * 2^-22 + 2^-22.1) < 2^-19.3 at most, 2^-20 with signs that do not agree.
REL = 2.0 ** -20


@pytest.mark.parametrize("S,H,d", shapes.F32_SPLIT_EDGES)
def test_edges(oracle, S, H, d):
    print(f"[case] fp32 split S={S} H={H} d={d}", flush=True)
    for name, e in _relative_errors(oracle, *_inputs(S, H, d, S), (0, H - 1)).items():
        assert e <= REL, f"{name}: {e:.2e}"


@pytest.mark.parametrize("factors", [(1e-3, 1e-3, 1e-3, 1e-6), (30.0, 0.05, 1e4, 1e-8), (1e-9, 1e9, 1e8, 1e-12)])
@pytest.mark.parametrize("S,H,d", shapes.F32_SPLIT_ONE)
def test_magnitudes(oracle, S, H, d, factors):
    # the same numbers times powers of ten: scores of the same size or smaller, everything else scaled
    print(f"[case] fp32 split times {factors} S={S} H={H} d={d}", flush=True)
    scaled = [t * f for t, f in zip(_inputs(S, H, d, 3), factors)]
    for name, e in _relative_errors(oracle, *scaled, (0,)).items():
        assert e <= REL, f"{name}: {e:.2e}"


@pytest.mark.parametrize("kind", ["spread", "far apart", "zero rows", "one large", "peaked"])
@pytest.mark.parametrize("S,H,d", shapes.F32_SPLIT_ONE)
def test_rows_of_different_magnitude(oracle, S, H, d, kind):
    # by row of the inputs: over 2^12, which one scale holds; over 2^40 and zero rows; a single large value; softmax over a few keys
    print(f"[case] fp32 split, {kind} S={S} H={H} d={d}", flush=True)
    q, k, v, g = _inputs(S, H, d, 5)
    gen = torch.Generator(device="cuda").manual_seed(8)
    bits = {"spread": 6, "far apart": 20}.get(kind)
    if bits:
        for t in (v, g):
            t *= torch.exp2((torch.rand((1, S, H, 1), generator=gen, device="cuda") * 2 - 1) * bits)
    elif kind == "zero rows":
        for t in (q, k, v, g):
            t[:, torch.rand(S, generator=gen, device="cuda") < 0.3] = 0.0
        v[:, 32:96] = 0.0
    elif kind == "one large":
        v[0, S // 2, 0, 3] = 1e9
        g[0, S // 3, 0, 5] = -1e12
    else:
        q *= 8.0
    # an error e of a score is a relative one of its probability: scores of up to 2^5.5 are off by up to 2^-19 / 2 (test_fp32_large_scores)
    bar = 2.0 ** -19 + 2.0 ** -22 if kind == "peaked" else REL
    for name, e in _relative_errors(oracle, q, k, v, g, (0,)).items():
        assert e <= bar, f"{name}: {e:.2e}"


@pytest.mark.parametrize("S,H,d", shapes.F32_SPLIT_ONE)
def test_rows_are_exact_by_themselves(oracle, S, H, d):
    # a row's precision does not depend on larger ones: queries that see only keys whose v is 2^-9 of the others', far behind them
    print(f"[case] fp32 split, small rows S={S} H={H} d={d}", flush=True)
    q, k, v, _ = _inputs(S, H, d, 9)
    v[:, : S // 2] *= 2.0 ** -9
    scale = synth.default_scale(d)
    o, _ = mb.memo_attn_fwd(q, k, v, scale)
    ro, _ = oracle.attn_fwd(*(to_f64(t[:, : S // 2, :1]) for t in (q, k, v)), scale)
    e = np.linalg.norm(to_f64(o[:, : S // 2, :1]) - ro, axis=-1) / np.linalg.norm(ro, axis=-1)
    assert e.max() <= 4 * REL, f"{e.max():.2e}"


@pytest.mark.parametrize("log2_per_step", [3.0, 60.0, -60.0])
@pytest.mark.parametrize("S,H,d", shapes.F32_SPLIT_ONE)
def test_scores_climbing_along_the_keys(oracle, S, H, d, log2_per_step):
    print(f"[case] fp32 split climbing {log2_per_step} S={S} H={H} d={d}", flush=True)
    scale = synth.default_scale(d)
    q, k, v, _ = _inputs(S, H, d, 10)
    q[..., 0] = 1.0
    k[..., 0] = (log2_per_step / 32.0 / (scale * math.log2(math.e)) * torch.arange(S, device="cuda", dtype=torch.float32))[None, :, None]
    o, lse = mb.memo_attn_fwd(q, k, v, scale)
    ro, rlse = oracle.attn_fwd(*(to_f64(t[:, :, :1]) for t in (q, k, v)), scale)
    # the scores are up to |lse| and rounded in 3 d / 16 accumulations of two chains, two sums and a product, each up to 2^-24 of them: sqrt(27) 2^-24 < 2^-21 of
    # them with random signs, and so the probabilities
    bar = 2.0 ** -21 * np.abs(rlse).max()
    assert np.abs(to_f64(lse[:, :1]) - rlse).max() <= bar + 2e-6
    assert np.abs(to_f64(o[:, :, :1]) - ro).max() <= 4 * bar + 2e-6


@pytest.mark.parametrize("value", [math.inf, -math.inf, math.nan, 3e38])
@pytest.mark.parametrize("where", ["q", "k", "v", "g"])
def test_values_that_no_scale_fits(oracle, where, value):
    # the same as the fp32 kernels give, which a launch too small for these takes: heads beside it as without it, and what it reaches
    S, H, d = shapes.F32_SPLIT_ONE[0]
    print(f"[case] fp32 split, {value} in {where} S={S} H={H} d={d}", flush=True)
    scale = synth.default_scale(d)
    tensors = dict(zip("qkvg", _inputs(S, H, d, 12)))
    clean = gpu_fwd_bwd(*tensors.values(), scale)
    tensors[where][0, 700, 1, 3] = value
    got = gpu_fwd_bwd(*tensors.values(), scale)
    for x, y in zip(clean, got):
        other = [h for h in range(H) if h != 1]
        assert torch.equal(x[:, :, other], y[:, :, other]) if x.dim() == 4 else torch.equal(x[:, other], y[:, other])
    if where in "kv" and not math.isfinite(value):
        assert not torch.isfinite(got[0][0, 700:, 1]).all(dim=-1).all() or value == -math.inf
    first = 700 // 32 * 32
    assert torch.equal(clean[0][0, :first, 1], got[0][0, :first, 1]) and torch.equal(clean[2][0, :first, 1], got[2][0, :first, 1])
    # one head and few rows go to the fp32 kernels: the rows that see the value first
    small = [t[:, :720, 1:2].contiguous() for t in tensors.values()]
    o, lse = mb.memo_attn_fwd(*small[:3], scale)
    a, b = o[0, 700:720, 0], got[0][0, 700:720, 1]
    assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.isinf(a), torch.isinf(b))
    fine = torch.isfinite(a)
    assert torch.allclose(a[fine], b[fine], rtol=1e-4, atol=1e-5)


@pytest.mark.parametrize("S,H,d", shapes.F32_SPLIT_ONE)
def test_layouts_and_places(S, H, d):
    # slices of a packed projection, dQ in place of Q and of dO, O in place of Q, and the gradients in two launches: the same bits
    print(f"[case] fp32 split, layouts S={S} H={H} d={d}", flush=True)
    scale = synth.default_scale(d)
    q, k, v, g = _inputs(S, H, d, 14)
    want = gpu_fwd_bwd(q, k, v, g, scale)
    packed = torch.stack((q, k, v, g), dim=2)
    outs = torch.zeros_like(packed)
    o, lse = mb.memo_attn_fwd(*(packed[:, :, n] for n in range(3)), scale, o=outs[:, :, 0])
    mb.memo_attn_bwd(*(packed[:, :, n] for n in range(3)), o, lse, packed[:, :, 3], scale, dq=outs[:, :, 1], dk=outs[:, :, 2], dv=outs[:, :, 3])
    for x, y in zip((o, lse, outs[:, :, 1], outs[:, :, 2], outs[:, :, 3]), want):
        assert torch.equal(x, y)
    q2 = q.clone()
    assert torch.equal(mb.memo_attn_fwd(q2, k, v, scale, o=q2)[0], want[0])
    for place in ("q", "g"):
        q2, g2 = q.clone(), g.clone()
        got = mb.memo_attn_bwd(q2, k, v, want[0], want[1], g2, scale, dq=q2 if place == "q" else g2)
        for x, y in zip(got, want[2:]):
            assert torch.equal(x, y)

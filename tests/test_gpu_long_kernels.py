"""The four-wave kernels of 256-row workgroups (csrc/attn_fwd_long_bf16.hip, csrc/attn_bwd_long_bf16.hip), and the eight-wave forward of shorter sequences, where they can go wrong: waves without
rows, of one row and of 63, one tile and several, both sweeps of a pair; a running maximum that is brought up to date in every tile, in
either block of keys and either direction; rows apart, batches; infinities and NaN."""
import math

import numpy as np
import pytest
import torch

import shape_cases as shapes
from gpu_util import LSE_MAX_ABS_BF16, assert_close, gpu_fwd_bwd, to_f64
from paper_2407_12117_amd import binding as mb
from paper_2407_12117_amd import synth

pytestmark = pytest.mark.gpu

SCALE = synth.default_scale(128)


@pytest.fixture(scope="module")
def oracle():
    from oracle import memo_oracle
    memo_oracle.build()
    return memo_oracle


def _inputs(S, heads, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.randn((1, S, heads, 128), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4)]


def _check_forward(oracle, q, k, v, o, lse, heads):
    for h in heads:
        ro, rlse = oracle.attn_fwd(*(to_f64(t[:, :, h:h + 1]) for t in (q, k, v)), SCALE)
        assert_close("O", to_f64(o[:, :, h:h + 1]), ro, "bf16")
        # the bar of unit-scale scores, and fp32's share of larger ones (their products and sums are rounded at 2^-24 of their size)
        bar = LSE_MAX_ABS_BF16 + 4e-6 * np.abs(rlse).max()
        assert np.abs(to_f64(lse[:, h:h + 1]) - rlse).max() <= bar


@pytest.mark.parametrize("S,heads", list(shapes.FWD_LONG_EDGES) + list(shapes.FWD_FOUR_WAVE_EDGES))
def test_forward_edges(oracle, S, heads):
    print(f"[case] long forward S={S} H={heads}", flush=True)
    q, k, v, _ = _inputs(S, heads, S)
    o, lse = mb.memo_attn_fwd(q, k, v, SCALE)
    _check_forward(oracle, q, k, v, o, lse, (0, heads // 2, heads - 1))


@pytest.mark.parametrize("S,heads", list(shapes.BWD_LONG_EDGES) + shapes.BWD_JOINT_EDGES)
def test_backward_edges(oracle, S, heads):
    print(f"[case] long backward S={S} H={heads}", flush=True)
    q, k, v, g = _inputs(S, heads, S)
    got = gpu_fwd_bwd(q, k, v, g, SCALE)
    for h in (0, heads - 1):
        refs = oracle.attn_bwd(*(to_f64(t[:, :, h:h + 1]) for t in (q, k, v, g)), SCALE)
        for name, x, r in zip(("dQ", "dK", "dV"), got[2:], refs):
            assert_close(name, to_f64(x[:, :, h:h + 1]), r, "bf16", scaled=True)


def _bits_of_rows_apart(B, S, heads, views):
    # the same bits as with contiguous tensors; views(): eight tensors of one layout, of which the last four are written
    gen = torch.Generator(device="cuda").manual_seed(S)
    data = [torch.randn((B, S, heads, 128), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4)]
    want = gpu_fwd_bwd(*data, SCALE)
    q, k, v, g, o, dq, dk, dv = views
    for dst, src in zip(views, data):
        dst.copy_(src)
    _, lse = mb.memo_attn_fwd(q, k, v, SCALE, o=o)
    mb.memo_attn_bwd(q, k, v, o, lse, g, SCALE, dq=dq, dk=dk, dv=dv)
    for x, y in zip((o, lse, dq, dk, dv), want):
        assert torch.equal(x, y)


@pytest.mark.parametrize("B,S,heads", list(shapes.LONG_LAYOUTS))
def test_batches_in_packed_rows(B, S, heads):
    # q, k, v and dO as slices of one [B, S, 5, H, d] buffer, the outputs as slices of another, whose last slot nobody writes
    print(f"[case] long kernels, packed B={B} S={S} H={heads}", flush=True)
    ins, outs = (torch.zeros((B, S, 5, heads, 128), device="cuda", dtype=torch.bfloat16) for _ in range(2))
    _bits_of_rows_apart(B, S, heads, [t[:, :, n] for t in (ins, outs) for n in range(4)])
    assert not outs[:, :, 4].any() and not ins[:, :, 4].any()


def test_rows_far_apart():
    # 2 MiB between rows: tiles of 64 rows that span 128 MiB, of tensors of 8 GiB
    S, heads, ss = 3905, 128, 1 << 20
    print(f"[case] long kernels, rows apart S={S} H={heads} stride {ss}", flush=True)
    buf = torch.zeros((S - 1) * ss + 8 * heads * 128, device="cuda", dtype=torch.bfloat16)
    _bits_of_rows_apart(1, S, heads, [torch.as_strided(buf, (1, S, heads, 128), (S * ss, ss, 128, 1), n * heads * 128) for n in range(8)])


@pytest.mark.parametrize("log2_per_tile", [12.0, 500.0, -500.0])
@pytest.mark.parametrize("S,heads", [(1025, 80), (1024, 160), (3521, 48), (3393, 68)])
def test_forward_with_scores_climbing_along_the_keys(oracle, S, heads, log2_per_tile):
    # every score moves with the key index by so many binary orders of magnitude per 64 keys (the first channel alone carries it)
    print(f"[case] long forward climbing {log2_per_tile} S={S} H={heads}", flush=True)
    q, k, v, _ = _inputs(S, heads, 5)
    slope = log2_per_tile / 64.0 / (SCALE * math.log2(math.e))
    q[..., 0] = 1.0
    k[..., 0] = (slope * torch.arange(S, device="cuda", dtype=torch.float32))[None, :, None].to(torch.bfloat16)
    o, lse = mb.memo_attn_fwd(q, k, v, SCALE)
    _check_forward(oracle, q, k, v, o, lse, (0, heads - 1))


@pytest.mark.parametrize("S,heads", list(shapes.FWD_LONG_SUMS))
def test_row_sums_grow_by_whole_tiles(S, heads):
    # 64 keys of weight 1, all others of 2^-23.25: a lane sums half of a row's keys, 32 and then 0.42 ulp of that with every 32 keys.  Added up block
    # by block all of it is lost (1.0e-7 of the sum per tile, 2.6e-5 at the end); by tiles of 64 keys 0.84 ulp becomes one: at most 0.17 ulp a tile, 2^-18 / 32 each.
    print(f"[case] long forward, row sums S={S} H={heads}", flush=True)
    q = torch.zeros((1, S, heads, 128), device="cuda", dtype=torch.bfloat16)
    k = torch.zeros_like(q)
    q[..., 0] = 1.0
    k[:, 64:, :, 0] = -23.25
    lse = to_f64(mb.memo_attn_fwd(q, k, torch.ones_like(q), math.log(2.0))[1])[0]
    keys = np.arange(1, S + 1)
    exact = np.log(np.minimum(keys, 64) + np.maximum(keys - 64, 0) * 2.0 ** -23.25)
    # one ulp for the sums of a row's last tile, and two of the logsumexp, which is at most 4.2.  Rows of the lower half sweep downwards: their running maximum
    # is that of the small weights, and the logsumexp is -23.25 ln 2 plus the logarithm of up to 2^30, an fp32 number of 2^-19 an ulp.
    bar = (0.17 * keys / 64 + 1.0) * 2.0 ** -23 + np.where(keys > S // 2, 2.0 ** -20, 2.0 ** -18)
    assert (np.abs(lse - exact) <= bar).all()


def test_rows_that_depend_on_what_is_not_finite():
    # what a key's rows reach: O and dQ of its queries and later ones, nothing before its 64-key tile
    S, heads, h, j = 3905, 128, 3, 2000
    print(f"[case] long kernels, NaN S={S} H={heads}", flush=True)
    q, k, v, g = _inputs(S, heads, 9)
    clean = gpu_fwd_bwd(q, k, v, g, SCALE)
    v[0, j, h, 5] = math.nan
    got = gpu_fwd_bwd(q, k, v, g, SCALE)
    first = j // 64 * 64
    assert torch.isnan(got[0][0, j:, h, 5]).all() and torch.isnan(got[2][0, j:, h]).all() and torch.isnan(got[3][0, j, h]).all()
    for x, y in zip(clean, got):
        other = torch.arange(heads, device="cuda") != h
        rows = (0, slice(None), other) if x.dim() == 4 else (0, other)
        assert torch.equal(x[rows], y[rows])
    assert torch.equal(clean[0][0, :first, h], got[0][0, :first, h]) and torch.equal(clean[2][0, :first, h], got[2][0, :first, h])


@pytest.mark.parametrize("S,heads", [(1025, 80), (3521, 48), (3393, 68)])
def test_masked_scores_of_minus_infinity(oracle, S, heads):
    # keys whose scores are all -inf weigh nothing, also where they are a wave's first tile
    print(f"[case] long forward, -inf S={S} H={heads}", flush=True)
    q, k, v, _ = _inputs(S, heads, 11)
    q[..., 0] = q[..., 0].abs() + 0.5
    hidden = torch.zeros(S, dtype=torch.bool, device="cuda")
    hidden[1:200] = True
    hidden[640:768] = True
    k[0, hidden, :, 0] = -math.inf
    o, lse = mb.memo_attn_fwd(q, k, v, SCALE)
    kf = k.clone()
    kf[0, hidden, :, 0] = -1e30
    for h in (0, heads - 1):
        ro, rlse = oracle.attn_fwd(*(to_f64(t[:, :, h:h + 1]) for t in (q, kf, v)), SCALE)
        assert_close("O", to_f64(o[:, :, h:h + 1]), ro, "bf16")
        assert np.abs(to_f64(lse[:, h:h + 1]) - rlse).max() <= LSE_MAX_ABS_BF16


def test_backward_with_scores_of_minus_infinity(oracle):
    # hidden keys get and give nothing: no gradient of their own, none in the others'.  The first channel of dQ, 0 times -inf, is left out
    S, heads = 3905, 128
    print(f"[case] long backward, -inf S={S} H={heads}", flush=True)
    q, k, v, g = _inputs(S, heads, 13)
    q[..., 0] = q[..., 0].abs() + 0.5
    hidden = torch.zeros(S, dtype=torch.bool, device="cuda")
    hidden[1:200] = True
    hidden[1024:1280] = True
    hidden[3900:] = True
    k[0, hidden, :, 0] = -math.inf
    _, _, dq, dk, dv = gpu_fwd_bwd(q, k, v, g, SCALE)
    assert not dk[0, hidden].any() and not dv[0, hidden].any()
    kf = k.clone()
    kf[0, hidden, :, 0] = -1e30
    for h in (0, heads - 1):
        refs = oracle.attn_bwd(*(to_f64(t[:, :, h:h + 1]) for t in (q, kf, v, g)), SCALE)
        for name, x, r, first in zip(("dQ", "dK", "dV"), (dq, dk, dv), refs, (1, 0, 0)):
            assert_close(name, to_f64(x[:, :, h:h + 1, first:]), r[..., first:], "bf16", scaled=True)

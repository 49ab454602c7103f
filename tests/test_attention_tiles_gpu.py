"""Decode attention where its passes change form: record counts around the
merge's rounds, tile counts around a wave's share, and K and V that are not
finite or not of one size.  Finite outputs are held to the per-element bound of
tests/attn_tolerance.py against the float64 oracle."""

import numpy as np
import pytest
import torch

from paper_2504_03775_amd import flowkv as fk
from tests.gpu_helpers import BM, LM
from tests.test_attention_gpu import bf16_to_f64, run_case, say
from workloads import Geometry, make_device_pool

pytestmark = pytest.mark.gpu


# one wave merges up to 8 records at head_dim 128 (16 at 64), a workgroup 32
# (64) a round
@pytest.mark.parametrize("dh,records", [(d, n) for d, ns in ((128, (1, 2, 7, 8, 9, 31, 32, 33, 65)),
                                                           (64, (1, 3, 15, 16, 17, 63, 64, 65)))
                                        for n in ns])
def test_merge_at_its_record_counts(dh, records):
    split = 16
    lens = [split * records, split * records - 5, max(1, split * records // 3)]
    say(f"merge: head_dim {dh}, {records} records")
    # a workgroup of one wave a head takes four: half a four, one and a half, whole ones
    for hq in (2, 6, 8):
        geom = Geometry("merge", 1, 3 if hq == 6 else 2, dh, 16, "bfloat16")
        run_case(geom, (LM, BM)[records % 2], sum(-(-t // 16) for t in lens) + 3, lens, hq,
                 900 + records, split, host_lens=bool(hq == 8))


# tiles of 32 tokens, four waves: shares of 0, 1 and 2 tiles, full and ragged
@pytest.mark.parametrize("dh,group", [(64, 1), (64, 8), (128, 2), (128, 8)])
@pytest.mark.parametrize("split", [0, 1024])
def test_tile_counts_of_a_wave(dh, group, split):
    geom = Geometry("tiles", 2, 2, dh, 7, "bfloat16")
    lens = [1, 31, 32, 33, 96, 97, 127, 128, 129, 160, 255, 256, 257]
    say(f"tiles: head_dim {dh}, group {group}, split {split}")
    run_case(geom, BM, sum(-(-t // 7) for t in lens) + 3, lens, 2 * group, 950 + dh + group, split)


@pytest.mark.parametrize("dh,group,split", [(128, 8, 0), (128, 8, 64), (128, 4, 0), (64, 2, 0)])
def test_values_that_are_not_finite(dh, group, split):
    """An infinite V gives an infinite output (of the heaviest token too, whose
    weight has zero lower parts), opposite infinities and NaN give NaN, and a
    score of -inf weighs nothing; the other dims are untouched."""
    T, bs = 150, 16
    geom = Geometry("inf", 1, 1, dh, bs, "bfloat16")
    B = -(-T // bs)
    t = make_device_pool(geom, BM, B, "cuda", 77)[0]     # (B, 1, 2, bs, 1, dh)
    q = torch.randn((1, group, dh), generator=torch.Generator("cuda").manual_seed(5),
                    device="cuda").to(torch.bfloat16)
    q[:, :, 3] = 1.0
    k, v = t[:, 0, 0, :, 0].reshape(-1, dh), t[:, 0, 1, :, 0].reshape(-1, dh)
    scores = bf16_to_f64(q[0]) @ bf16_to_f64(k).T[:, :T] / np.sqrt(dh)
    top, other = int(scores[0].argmax()), 40
    assert top != other
    for tok, dim, val in ((top, 5, np.inf), (other, 6, -np.inf), (top, 7, np.inf),
                          (other, 7, -np.inf), (90, 9, np.nan)):
        t[tok // bs, 0, 1, tok % bs, 0, dim] = val
    t[70 // bs, 0, 0, 70 % bs, 0, 3] = -np.inf           # score -inf: q there is 1
    pool = fk.KVPool(BM, [t])
    out = torch.full((1, group, dh), 3.0, device="cuda")
    ws = torch.empty(max(1, fk.flowkv_decode_attention_workspace(1, group, dh, T, split)),
                     dtype=torch.uint8, device="cuda")
    fk.flowkv_decode_attention(pool, 0, q, torch.arange(B, dtype=torch.int32, device="cuda")[None],
                               torch.tensor([T], dtype=torch.int32, device="cuda"), T,
                               1 / np.sqrt(dh), out, ws, split)
    got = out.cpu().numpy()[0].astype(np.float64)
    k, v = bf16_to_f64(t[:, 0, 0, :, 0].reshape(-1, dh))[:T], bf16_to_f64(
        t[:, 0, 1, :, 0].reshape(-1, dh))[:T]
    s = bf16_to_f64(q[0]) @ np.where(np.isinf(k), 0, k).T / np.sqrt(dh)
    s[:, 70] = -np.inf
    p = np.exp(s - s.max(1, keepdims=True))
    p /= p.sum(1, keepdims=True)
    with np.errstate(invalid="ignore"):
        want = np.stack([(p[h][:, None] * v).sum(0) for h in range(group)])
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(np.isposinf(got), np.isposinf(want))
    assert np.array_equal(np.isneginf(got), np.isneginf(want))
    fin = np.isfinite(want)
    assert fin.sum() == group * (dh - 4)
    # roundings of 2^-24 on sums of at most sum p |V| ~ 1, a score's own (2^-24 x
    # sum |q k| ~ 10) moving a weight by as much: about 20 x 2^-24, and four times that
    # as the bound
    assert np.abs(got[fin] - want[fin]).max() < 20 * 2.0 ** -24 * 4


@pytest.mark.parametrize("dh,group", [(64, 4), (128, 8)])
@pytest.mark.parametrize("host", [False, True])
def test_one_split_writes_every_output(dh, group, host):
    """Where no merge runs, a request without tokens still gets zeros, and a
    request's output is the one it has beside longer ones (which do merge, of
    one record)."""
    geom = Geometry("one", 1, 2, dh, 16, "bfloat16")
    pool = fk.KVPool(LM, make_device_pool(geom, LM, 64, "cuda", 31))
    lens = np.array([0, 256, 1, 100], np.int32)
    tab = torch.randperm(64, dtype=torch.int32, generator=torch.Generator().manual_seed(3)
                         ).reshape(4, 16).cuda()
    q = torch.randn((4, 2 * group, dh), generator=torch.Generator("cuda").manual_seed(4),
                    device="cuda").to(torch.bfloat16)
    outs = []
    for top in (256, 257):                  # one split of 256 tokens, then two
        out = torch.full((4, 2 * group, dh), float("nan"), device="cuda")
        ws = torch.empty(fk.flowkv_decode_attention_workspace(4, 2 * group, dh, top),
                         dtype=torch.uint8, device="cuda")
        fk.flowkv_decode_attention(pool, 0, q, tab, torch.as_tensor(lens, device="cuda"), top,
                                   0.1, out, ws, seq_lens_host=lens if host else None)
        outs.append(out.cpu())
    assert (outs[0][0] == 0).all()
    assert torch.equal(outs[0], outs[1])


def one_head_pool(T, dh, seed):
    """K and V views (tokens, dh) of a one-layer, one-KV-head pool, N(0, 1)."""
    geom = Geometry("one", 1, 1, dh, 16, "bfloat16")
    t = make_device_pool(geom, BM, -(-T // 16), "cuda", seed)[0]     # (B, 1, 2, 16, 1, dh)
    return fk.KVPool(BM, [t]), t


def attend(pool, q, T, scale, split, host):
    n, hq, dh = q.shape
    blocks = pool.num_blocks
    tab = torch.arange(blocks, dtype=torch.int32, device="cuda").repeat(n, 1)
    out = torch.full((n, hq, dh), 3.0, device="cuda")
    ws = torch.empty(max(1, fk.flowkv_decode_attention_workspace(n, hq, dh, T, split)),
                     dtype=torch.uint8, device="cuda")
    lens = np.full(n, T, np.int32)
    fk.flowkv_decode_attention(pool, 0, q, tab, torch.as_tensor(lens, device="cuda"), T, scale,
                               out, ws, split, seq_lens_host=lens if host else None)
    return out.cpu().numpy().astype(np.float64)


def put(t, kv, token, dim, val):
    t[token // 16, 0, kv, token % 16, 0, dim] = val


@pytest.mark.parametrize("dh,group", [(64, 1), (64, 8), (128, 2), (128, 4), (128, 8)])
@pytest.mark.parametrize("split", [0, 32, 64])
def test_values_far_larger_than_their_weights(dh, group, split):
    """A weight that is exactly 0 takes nothing of a V of 3e38, one of about
    2^-115 its share, and an infinite V stays infinite under the smallest
    weights.  The scores are K's first dim (q is its unit vector), in log2 units:
    0 for all other tokens, whose weights are then 1."""
    T = 100
    pool, t = one_head_pool(T, dh, 55)
    t[:, 0, 0, :, 0] = 0                                  # K
    q = torch.zeros((1, group, dh), dtype=torch.bfloat16, device="cuda")
    q[:, :, 0] = 1.0
    scale = np.float32(np.log(2.0))
    scores = np.zeros(T)
    for token, score, dim, val in ((37, -300, 4, 3e38), (60, -115, 5, 2.0 ** 127),
                                   (61, -109.5, 6, -2.0 ** 125), (70, -115, 9, np.inf),
                                   (20, -125, 10, -np.inf)):
        put(t, 0, token, 0, score)
        put(t, 1, token, dim, val)
        scores[token] = score
    v = bf16_to_f64(t[:, 0, 1, :, 0].reshape(-1, dh))[:T]
    w = np.exp2(scores * np.float64(scale * np.float32(np.log2(np.e))))
    w[37] = 0.0                                           # (2^-300 is no float32)
    with np.errstate(invalid="ignore"):
        want = (w[:, None] * v).sum(0) / w.sum()
    for host in (False, True):
        got = attend(pool, q, T, float(scale), split, host)[0]
        assert np.array_equal(np.isposinf(got), np.broadcast_to(np.isposinf(want), got.shape))
        assert np.array_equal(np.isneginf(got), np.broadcast_to(np.isneginf(want), got.shape))
        fin = np.isfinite(want)
        # sums of 100 terms of at most |V| ~ 4: 2^-24 x 100 x 4 / 100 a sum, four
        # sums; for the tiny weights' dims, exp2's argument (2^-24 x 115) and the
        # parts below bf16's smallest value (2 x 2^-133 of 2^-115)
        tol = np.full(dh, 16 * 2.0 ** -24)
        tol[[5, 6]] = np.abs(want[[5, 6]]) * 2.0 ** -16
        assert np.all(np.abs(got[:, fin] - want[fin]) <= tol[fin])


@pytest.mark.parametrize("dh,group", [(64, 2), (64, 8), (128, 1), (128, 4), (128, 8)])
def test_error_beside_a_float32_evaluation(dh, group):
    """The error against 64 bits over all outputs of a long request stays within
    1.6 times that of a float32 evaluation in the pass's own order, which rounds
    each 32-token tile's sum onto a wave's running sum once (numpy, tiles exact).
    An MFMA rounds inside its 32 products too, hence the margin: one MFMA per
    tile and sum measures 1.37-1.45 times, three onto one sum 1.73-2.16."""
    T, split = 16384, 1024
    pool, t = one_head_pool(T, dh, 57)
    q = torch.randn((1, group, dh), generator=torch.Generator("cuda").manual_seed(3),
                    device="cuda").to(torch.bfloat16)
    got = attend(pool, q, T, 1 / np.sqrt(dh), split, True)[0]
    k, v = (bf16_to_f64(t[:, 0, i, :, 0].reshape(-1, dh)) for i in (0, 1))
    s = bf16_to_f64(q[0]) @ k.T                           # (group, T)
    scale = np.float64(np.float32(1 / np.sqrt(dh)))
    p = np.exp(scale * s - (scale * s).max(1, keepdims=True))
    want = (p @ v) / p.sum(1, keepdims=True)
    arg = s.astype(np.float32) * np.float32(np.float32(scale) * np.float32(np.log2(np.e)))
    w = np.exp2(arg - arg.max(1, keepdims=True)).astype(np.float64)
    # waves take every fourth tile of a split
    tiles = np.einsum("gntx,ntxd->ngtd", w.reshape(group, -1, 32, 32),
                      v.reshape(-1, 32, 32, dh)).reshape(-1, group, 8, 4, dh)
    acc = np.zeros(tiles[:, :, 0].shape, np.float32)
    for i in range(8):
        acc = (acc + tiles[:, :, i]).astype(np.float32)
    f32 = acc.astype(np.float64).sum((0, 2)) / w.sum(1, keepdims=True)
    kernel, ideal = (np.linalg.norm(x - want) for x in (got, f32))
    say(f"head_dim {dh}, group {group}: {kernel / np.linalg.norm(want):.2e} against 64 bits, "
        f"{kernel / ideal:.2f} times a float32 evaluation's")
    assert kernel <= 1.6 * ideal



@pytest.mark.parametrize("dh,group", [(64, 2), (128, 4), (128, 8)])
@pytest.mark.parametrize("split", [0, 64])
@pytest.mark.parametrize("host", [False, True])
def test_scores_that_are_nan_reach_the_output(dh, group, split, host):
    """A NaN among a head's scores (a NaN in K or q, or a score of +inf, whose
    weight is inf - inf) gives NaN, whether it stands beside finite scores or
    fills a whole split; other heads and requests stay as they are."""
    T = 150
    q = torch.randn((1, group, dh), generator=torch.Generator("cuda").manual_seed(2),
                    device="cuda").to(torch.bfloat16)
    q[:, :, 3] = 1.0
    pool, t = one_head_pool(T, dh, 56)
    clean = attend(pool, q, T, 0.1, split, host)
    assert np.isfinite(clean).all()
    two = q.repeat(2, 1, 1)
    two[1, group - 1, 0] = float("nan")
    got = attend(pool, two, T, 0.1, split, host)
    assert np.array_equal(got[0], clean[0])
    assert np.array_equal(got[1, :-1], clean[0, :-1])
    assert np.isnan(got[1, -1]).all()
    for tokens, val in (((90,), np.nan), ((5,), np.inf), (range(64, 128), np.nan),
                        ((149,), np.inf)):
        pool, t = one_head_pool(T, dh, 56)
        for x in tokens:
            put(t, 0, x, 3, val)
        got = attend(pool, q, T, 0.1, split, host)
        assert np.isnan(got).all(), (tokens, val)


@pytest.mark.parametrize("dh,group", [(64, 2), (128, 8)])
@pytest.mark.parametrize("past", [0, 1], ids=["two-per-cu", "one-more"])
@pytest.mark.parametrize("host", [False, True])
def test_workgroups_around_two_per_cu(dh, group, past, host):
    """At most two workgroups per CU are launched with LDS added, so that no CU
    takes a third; one more split and they are not.  Splits of one tile on two
    KV heads; with the lengths on the host, beside requests that end early."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    geom = Geometry("spread", 1, 2, dh, 16, "bfloat16")
    lens = [32 * (cus - 3) + past, 1, 32, 5] if host else [32 * cus + past]
    say(f"spread: {lens}, {cus} CUs, host {host}")
    run_case(geom, BM, sum(-(-t // 16) for t in lens) + 3, lens, 2 * group, 970 + past, 32,
             host_lens=host)

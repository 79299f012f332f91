"""Selection of short sequences (N <= 16384: scores in the workspace, one workgroup per
row) against the passes that longer ones take, and against the oracle.

A causal block's eligible keys end with its own rows, so the blocks of a causal sequence of
n tokens select the same lists as the first blocks of any longer one: the same rows go
through both kinds of selection.  Scores are bit-identical in both, so rank and threshold
lists are equal; by mass, sums of the same fp32 terms in another order can move a cut whose
cumulative mass lies within an ulp or so of p (at most one row in fifty is allowed to)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_29494_amd as va
from paper_2603_29494_amd import synth

from selection_parity import check_rows

pytestmark = pytest.mark.gpu

LONG = 16384 + 64  # longer than any short sequence, whole blocks of 64


def dev(bits):
    return torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16).cuda()


@pytest.fixture(scope="module")
def long_layer(gpu):
    out = {}
    for D in (64, 128):
        q, k, _ = synth.planted_case(60 + D, 1, 2, 1, LONG, D)
        k[0, 0, 5::7] = k[0, 0, 5]        # exact ties
        out[D] = dev(q), dev(k)
    return out


CASES = [("topk", 0.15), ("topk", 1.0), ("topp", 0.9), ("topp", 1.0), ("mins", 0.7), ("mins", 0.0)]


@pytest.mark.parametrize("mode,param", CASES)
@pytest.mark.parametrize("n,P,D", [(1, 64, 64), (64, 64, 128), (1000, 16, 128), (1024, 64, 64),
                                   (1025, 64, 128), (4096, 64, 64), (4097, 64, 128),
                                   (16384, 64, 128), (16383, 64, 64)])
def test_short_equals_passes(long_layer, n, P, D, mode, param):
    q, k = long_layer[D]
    for keep_diag in (False, True):
        cap = va.max_count(LONG, P, True, mode, param, keep_diag)
        Np = (n + P - 1) // P
        whole = n // P  # blocks of P rows in both sequences (the ragged ones: the oracle, below)
        # the longer sequence selected only as far as the short one's whole blocks reach
        il, cl = va.select(q, k, P, mode, param, True, cap=cap, keep_diag=keep_diag)
        i_s, c_s = va.select(q[:, :, :n], k[:, :, :n], P, mode, param, True, cap=cap,
                             keep_diag=keep_diag)
        torch.cuda.synchronize()
        assert tuple(i_s.shape) == (1, 2, Np, cap)
        a, b = i_s[:, :, :whole], il[:, :, :whole]
        same = (a == b).all(-1) & (c_s[:, :, :whole] == cl[:, :, :whole])
        bad = int((~same).sum())
        assert bad == 0 or (mode == "topp" and param < 1.0 and bad * 50 <= same.numel()), bad
        del il, i_s
    assert va.check_lists(*va.select(q[:, :, :n], k[:, :, :n], P, mode, param, True), n) == 0


@pytest.mark.parametrize("N,P,Hq,mode,param,cap", [
    (1000, 1, 5, "topk", 0.1, None), (1000, 1, 5, "topp", 0.9, None),       # one wave per row
    (2500, 1, 2, "topk", 0.2, None), (2500, 1, 2, "topp", 0.95, 777),
    (2500, 1, 2, "mins", 2.0, 301),
    (700, 64, 2, "topp", 0.95, 130), (5000, 64, 2, "topp", 0.9, 401), (5000, 64, 2, "mins", 3.0, 1022),
    (1, 64, 2, "topk", 0.5, None), (1, 1, 3, "topp", 0.5, None), (1, 64, 2, "mins", 0.0, None),
    (8000, 64, 2, "topk", 0.3, None), (12345, 64, 2, "topk", 0.2, None), (12345, 128, 2, "topp", 0.9, None),
    (12345, 64, 2, "mins", 0.7, None), (12345, 128, 2, "topp", 0.95, 3001), (16383, 128, 1, "topp", 0.6, None),
    (16383, 128, 1, "mins", 2.0, 2222)])
def test_short_matches_oracle_with_caps(gpu, N, P, Hq, mode, param, cap):
    q, k, _ = synth.planted_case(N + P, 1, Hq, 1, N, 64, frac=0.03, logits=1.5)
    full = va.max_count(N, P, False, mode, param)
    cap = full if cap is None else cap
    ncl = torch.zeros(1, dtype=torch.int32, device="cuda")
    idx, cnt = va.select(dev(q), dev(k), P, mode, param, False, cap=cap, n_clamped=ncl)
    torch.cuda.synchronize()
    Np = (N + P - 1) // P
    r = np.random.Generator(np.random.PCG64(3))
    rows = np.sort(r.choice(Hq * Np, size=min(Hq * Np, 64), replace=False))
    om = {"topk": oracle.TOPK, "topp": oracle.TOPP, "mins": oracle.MINS}[mode]
    ih = idx.reshape(-1, cap).cpu().numpy()[rows]
    ch = cnt.reshape(-1).cpu().numpy()
    mism = check_rows(q, k, P, om, param, False, cap, ih, ch[rows], rows, compact=True)
    assert mism <= max(1, len(rows) // 20)
    if cap < full:
        # clamped: the blocks whose whole set has more than cap keys
        _, whole = va.select(dev(q), dev(k), P, mode, param, False, cap=full)
        assert int(ncl.item()) == int((whole > cap).sum()) > 0
        assert torch.equal(cnt, whole.clamp(max=cap))


@pytest.mark.parametrize("mode,param", CASES)
@pytest.mark.parametrize("n,P,D", [(1, 64, 64), (63, 64, 128), (1000, 16, 128), (1025, 64, 128),
                                   (4097, 64, 128), (8191, 48, 64), (8193, 64, 128), (16383, 64, 64)])
def test_short_last_blocks_match_oracle(long_layer, n, P, D, mode, param):
    """The ragged last block, whose rows another length does not share, and the one before it."""
    tq, tk = (x[:, :, :n].contiguous() for x in long_layer[D])
    q, k = (x.view(torch.int16).cpu().numpy().view(np.uint16) for x in (tq, tk))
    Np = (n + P - 1) // P
    rows = np.array([h * Np + i for h in range(2) for i in range(max(0, Np - 2), Np)])
    om = {"topk": oracle.TOPK, "topp": oracle.TOPP, "mins": oracle.MINS}[mode]
    for causal in (False, True):
        cap = va.max_count(n, P, causal, mode, param)
        idx, cnt = va.select(tq, tk, P, mode, param, causal, cap=cap)
        torch.cuda.synchronize()
        mism = check_rows(q, k, P, om, param, causal, cap, idx.reshape(-1, cap).cpu().numpy()[rows],
                          cnt.reshape(-1).cpu().numpy()[rows], rows, compact=True)
        assert mism <= 1


@pytest.mark.parametrize("bad", ["nan", "inf", "-inf", "huge"])
def test_short_lists_stay_valid_for_non_finite_scores(gpu, bad):
    N, P = 1500, 64
    q = synth.bits_to_f32(synth.random_bits(1, (1, 2, N, 128)))
    k = synth.bits_to_f32(synth.random_bits(2, (1, 2, N, 128)))
    k[0, :, 7::11] = {"nan": np.nan, "inf": np.inf, "-inf": -np.inf, "huge": 3e38}[bad]
    tq, tk = dev(synth.to_bf16_bits(q)), dev(synth.to_bf16_bits(k))
    for mode, param in CASES:
        idx, cnt = va.select(tq, tk, P, mode, param, False)
        torch.cuda.synchronize()
        assert va.check_lists(idx, cnt, N) == 0
        if mode == "topk":
            assert int(cnt.min()) == int(cnt.max()) == idx.shape[-1]


def test_short_rows_in_groups_and_small_workspace(gpu):
    """Score groups: a workspace that holds one row tile at a time gives the same lists as
    one that holds them all, and so does the one the size query asks for."""
    N, P = 3000, 16
    q, k, _ = synth.planted_case(77, 2, 4, 2, N, 128)
    tq, tk = dev(q), dev(k)
    cap = va.max_count(N, P, False, "topk", 0.1)
    want = va.select(tq, tk, P, "topk", 0.1, False, cap=cap)
    qp = -(-(2 * 4 * 188 * 256) // 256) * 256
    ld = -(-N // 32) * 32
    for tiles in (1, 3):
        ws = torch.full((qp + tiles * 64 * ld * 4,), 0xFF, dtype=torch.uint8, device="cuda")
        got = va.select(tq, tk, P, "topk", 0.1, False, cap=cap, workspace=ws)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("N,P,cap,params", [
    (700, 1, 128, 1.0), (1000, 64, 300, 1.0), (1000, 64, 301, [0.6, 1.0]), (3000, 64, 1024, [1.0, 0.6]),
    (3000, 64, 5, 1.0), (7000, 128, 4097, 1.0), (9000, 256, 4096, [1.0, 0.6]), (16384, 512, 16380, 1.0)])
def test_short_topp_of_one_is_clamped_to_cap(gpu, N, P, cap, params, causal):
    """p = 1 keeps every eligible key; a block with more than cap of them keeps its cap best (not
    the first by index) and is counted.  One case for every shape of the row kernel."""
    q, k, _ = synth.planted_case(N + cap, 1, 2, 1, N, 64, frac=0.03, logits=1.5)
    head = [params, params] if np.isscalar(params) else params
    Np = (N + P - 1) // P
    ncl = torch.zeros(1, dtype=torch.int32, device="cuda")
    idx, cnt = va.select(dev(q), dev(k), P, "topp", params, causal, cap=cap, n_clamped=ncl)
    torch.cuda.synchronize()
    L = np.minimum(N, (np.arange(Np) + 1) * P) if causal else np.full(Np, N)
    c = cnt.cpu().numpy()[0]
    clamped = 0
    some = np.unique(np.linspace(0, Np - 1, 12).astype(int))
    for h, p in enumerate(head):
        if p == 1.0:
            assert np.array_equal(c[h], np.minimum(L, cap))
            clamped += int((L > cap).sum())
        else:
            clamped += int((c[h] == cap).sum())
        rows = h * Np + some
        mism = check_rows(q, k, P, oracle.TOPP, p, causal, cap,
                          idx.reshape(-1, cap).cpu().numpy()[rows], c.reshape(-1)[rows], rows,
                          compact=True)
        assert mism <= 1
    assert int(ncl.item()) == clamped


@pytest.mark.parametrize("mode,param,Hq,N,P,D,causal,keep_diag,capdiv", [
    ("mins", 0.3, 12, 9001, 16, 64, False, False, 1), ("mins", 0.7, 28, 16384, 64, 128, True, False, 1),
    ("mins", float("inf"), 12, 9001, 16, 64, True, True, 1),
    ("topk", 0.4, 12, 8193, 12, 64, False, False, 1), ("topk", 0.1, 28, 16383, 32, 128, True, True, 1),
    ("topk", [0.02, 0.9, 0.5, 1.0], 4, 8000, 2, 64, False, False, 1),
    ("topp", 0.9, 12, 12345, 6, 64, False, False, 1), ("topp", 0.6, 28, 9000, 7, 128, True, True, 1),
    ("topp", [0.5, 1.0, 0.9, 0.99], 4, 8200, 1, 64, False, False, 5)])
def test_both_kinds_agree_where_the_passes_are_faster(gpu, mode, param, Hq, N, P, D, causal, keep_diag, capdiv):
    """Calls of up to 16384 tokens with so many blocks that the passes are faster: with the workspace
    of the size query they run (behind the pooled queries they leave a row's last phase, 3 or 4,
    where the short kind has a score), with one row tile's scores the short kind does.  Lists, counts and clamped blocks are equal; by mass, at most one
    block in fifty may differ (the same terms in another order)."""
    q, k, _ = synth.planted_case(N + P, 1, Hq, 2 if Hq == 4 else 4, N, D, frac=0.04, logits=2.0)
    k[0, 0, 5::7] = k[0, 0, 5]        # exact ties
    tq, tk = dev(q), dev(k)
    cap = max(1, va.max_count(N, P, causal, mode, param, keep_diag) // capdiv)
    Np = (N + P - 1) // P
    out = []
    big = va.workspace_bytes(tq, tk, P, causal, mode, cap)
    pooled = -(-(Hq * Np * D * 2) // 256) * 256
    tile = min(Np, 64) * (-(-N // 32) * 32) * 4
    for size in (big, pooled + tile):
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
        ncl = torch.zeros(1, dtype=torch.int32, device="cuda")
        idx, cnt = va.select(tq, tk, P, mode, param, causal, cap=cap, workspace=ws, n_clamped=ncl,
                             keep_diag=keep_diag)
        out.append((idx, cnt, ncl))
        torch.cuda.synchronize()
        assert (int(ws[pooled:pooled + 4].view(torch.int32)) in (3, 4)) == (size == big)
        del ws
    assert va.check_lists(out[0][0], out[0][1], N) == 0
    same = (out[0][0] == out[1][0]).all(-1) & (out[0][1] == out[1][1])
    bad = int((~same).sum())
    assert bad == 0 or (mode == "topp" and bad * 50 <= same.numel()), bad
    assert abs(int(out[0][2]) - int(out[1][2])) <= bad
    assert capdiv == 1 or int(out[0][2]) > 0

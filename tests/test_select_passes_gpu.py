"""Selection by the score passes (csrc/select.hip), at a length that the kernels for short
sequences do not take: every mode, cap, option and input that can go wrong there, against the
oracle (the index-set rule is in selection_parity.py).  The same properties are tested at
300 to 8192 tokens, where the short kernels run, in test_select_gpu.py."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_29494_amd as va
from paper_2603_29494_amd import synth

from selection_parity import check_rows

pytestmark = pytest.mark.gpu

N, P = 16500, 256                # above 16384 tokens; a ragged last block of 116 rows
NP = (N + P - 1) // P
OMODE = {"topk": oracle.TOPK, "topp": oracle.TOPP, "mins": oracle.MINS}


def dev(bits):
    return torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16).cuda()


def check(q, k, mode, param, causal, cap, idx, cnt, rows=None):
    rows = np.arange(q.shape[1] * NP) if rows is None else rows
    ih = idx.reshape(-1, cap).cpu().numpy()[rows]
    ch = cnt.reshape(-1).cpu().numpy()[rows]
    mism = check_rows(q, k, P, OMODE[mode], param, causal, cap, ih, ch, rows, compact=True)
    assert mism <= max(1, len(rows) // 20)


def check_heads(q, k, mode, params, causal, cap, idx, cnt):
    g = q.shape[1] // k.shape[1]
    for h, p in enumerate(params):
        check(np.ascontiguousarray(q[:, h:h + 1]), np.ascontiguousarray(k[:, h // g:h // g + 1]), mode,
              p, causal, cap, idx[:, h:h + 1], cnt[:, h:h + 1])


def run(tq, tk, mode, param, causal, cap=None, **kw):
    cap = va.max_count(N, P, causal, mode, param) if cap is None else cap
    ncl = torch.zeros(1, dtype=torch.int32, device="cuda")
    idx, cnt = va.select(tq, tk, P, mode, param, causal, cap=cap, n_clamped=ncl, **kw)
    torch.cuda.synchronize()
    return idx, cnt, cap, int(ncl.item())


@pytest.fixture(scope="module")
def layer(gpu):
    q, k, _ = synth.planted_case(21, 1, 2, 1, N, 64, frac=0.03, logits=1.5)
    return q, k, dev(q), dev(k)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("params", [1.0, [0.5, 1.0]])
@pytest.mark.parametrize("cap", [4096, 4097])
def test_topp_of_one_is_clamped_to_cap(layer, cap, params, causal):
    """p = 1 keeps every eligible key and so more than cap: such a block keeps its cap best and
    is counted, and no list reaches past its row (rows that start on 16 bytes, stored four
    entries at a time, and others)."""
    q, k, tq, tk = layer
    head = [params, params] if np.isscalar(params) else params
    pad = 4 * N
    store = torch.full((2 * NP * cap + pad,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    idx = store[:2 * NP * cap].view(1, 2, NP, cap)
    ncl = torch.zeros(1, dtype=torch.int32, device="cuda")
    _, cnt = va.select(tq, tk, P, "topp", params, causal, cap=cap, idx=idx, n_clamped=ncl)
    torch.cuda.synchronize()
    assert bool((store[2 * NP * cap:] == 0x5A5A5A5A).all())
    L = np.minimum(N, (np.arange(NP) + 1) * P) if causal else np.full(NP, N)
    c = cnt.cpu().numpy()[0]
    clamped = 0
    for h, p in enumerate(head):
        if p == 1.0:
            assert np.array_equal(c[h], np.minimum(L, cap))
            clamped += int((L > cap).sum())
        rows = np.array([h * NP + i for i in (0, 15, 16, 17, 40, NP - 1)])
        check(q, k, "topp", p, causal, cap, idx, cnt, rows)
    assert int(ncl.item()) == clamped + int((c[[h for h in (0, 1) if head[h] != 1.0]] == cap).sum())


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("mode,param", [("topk", 0.15), ("topk", 0.002), ("topk", 1.0), ("topp", 0.9),
                                        ("topp", 0.3), ("topp", 1.0), ("mins", 0.0), ("mins", 2.0),
                                        ("mins", float("inf"))])
def test_matches_oracle(layer, mode, param, causal):
    q, k, tq, tk = layer
    idx, cnt, cap, ncl = run(tq, tk, mode, param, causal)
    assert ncl == 0
    check(q, k, mode, param, causal, cap, idx, cnt)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("mode,param", [("topp", 0.9), ("topp", 0.99), ("mins", 0.6), ("mins", 2.0)])
@pytest.mark.parametrize("where", ["above", "median", "few", "one"])
def test_threshold_modes_with_caps(layer, where, mode, param, causal):
    """Caps above every count and below N (minS counts its keys by histogram, no block is clamped),
    at the median count (some blocks are clamped by a few keys, inside the last interval, others
    far above it: the second round), and far below all counts."""
    q, k, tq, tk = layer
    _, whole, _, _ = run(tq, tk, mode, param, causal)
    w = whole.cpu().numpy()
    top = int(w.max())
    cap = {"above": min(top + 3, N - 1), "median": int(np.median(w)) // 4 * 4, "few": 201, "one": 1}[where]
    idx, cnt, cap, ncl = run(tq, tk, mode, param, causal, cap=cap)
    assert ncl == int((w > cap).sum()) and (ncl > 0) == (where != "above" or cap < top)
    assert np.array_equal(cnt.cpu().numpy(), np.minimum(w, cap))
    check(q, k, mode, param, causal, cap, idx, cnt)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("mode,params", [("topk", [0.05, 0.1, 0.2, 0.4]), ("topp", [0.5, 0.8, 0.9, 0.99]),
                                         ("mins", [0.3, 0.6, 1.0, 2.0])])
def test_per_head_parameters(gpu, mode, params, causal):
    q, k, _ = synth.planted_case(31 + causal, 1, 4, 2, N, 64, frac=0.03, logits=1.5)
    tq, tk = dev(q), dev(k)
    full = va.max_count(N, P, causal, mode, params)
    for cap in (full,) if mode == "topk" else (full, full // 3):     # topK is never clamped
        idx, cnt, cap, ncl = run(tq, tk, mode, params, causal, cap=cap)
        assert (ncl > 0) == (cap < full)
        check_heads(q, k, mode, params, causal, cap, idx, cnt)


@pytest.mark.parametrize("sampled_high", [False, True])
@pytest.mark.parametrize("mode,param", [("topk", 0.1), ("topk", 0.6), ("topp", 0.8)])
def test_level0_interval_from_misleading_sample(gpu, mode, param, sampled_high):
    # Every 16th 32-key block is sampled for the first interval of a topK row.  Shifting only the
    # unsampled blocks' keys (or only the sampled ones) toward the queries' direction puts the true
    # cut above (or below) the estimate.
    rng = np.random.default_rng(41 + int(sampled_high))
    u = rng.standard_normal(128).astype(np.float32)
    u /= np.linalg.norm(u)
    q = rng.standard_normal((1, 2, N, 128)).astype(np.float32) + 2.0 * u
    k = rng.standard_normal((1, 2, N, 128)).astype(np.float32)
    sampled = ((np.arange(N) // 32) % 16) == 0
    k[:, :, sampled if sampled_high else ~sampled] += 3.0 * u
    qb, kb = synth.to_bf16_bits(q), synth.to_bf16_bits(k)
    idx, cnt, cap, _ = run(dev(qb), dev(kb), mode, param, False)
    check(qb, kb, mode, param, False, cap, idx, cnt)


@pytest.mark.parametrize("mode,param,cap", [("topk", 0.3, None), ("topp", 0.5, None), ("topp", 0.999, None),
                                            ("topp", 0.999, 700), ("mins", 0.0, None), ("mins", 0.0, 700)])
def test_tie_storm_zero_queries(gpu, mode, param, cap):
    # Q = 0: every score is exactly 0; the kept keys are the lowest indices.
    q = np.zeros((1, 2, N, 128), dtype=np.uint16)
    k = synth.random_bits(5, (1, 2, N, 128))
    idx, cnt, cap, ncl = run(dev(q), dev(k), mode, param, False, cap=cap)
    idx_o, cnt_o, ncl_o = oracle.select(q, k, P, OMODE[mode], param, False, cap)
    assert np.array_equal(cnt.cpu().numpy(), cnt_o) and ncl == ncl_o
    assert np.array_equal(idx.cpu().numpy(), idx_o)


@pytest.mark.parametrize("mode,param,cap", [("topk", 0.2, None), ("topk", 0.4, None), ("topp", 0.7, None),
                                            ("topp", 0.9, 5000), ("mins", 0.2, 3001)])
def test_partial_ties_from_duplicate_keys(gpu, mode, param, cap):
    # a third of the keys are one row: ties at the cut, more of them than the candidate buffer
    # holds, broken toward lower indices
    k = synth.random_bits(6, (1, 1, N, 128))
    k[0, 0, 1::3] = k[0, 0, 0]
    q = synth.random_bits(7, (1, 1, N, 128))
    idx, cnt, cap, _ = run(dev(q), dev(k), mode, param, False, cap=cap)
    check(q, k, mode, param, False, cap, idx, cnt)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("mode,param", [("topk", 0.1), ("topp", 0.8), ("mins", 0.5)])
def test_writer_paths_padding_diagonal_and_repeats(layer, mode, param, causal):
    """Lists of rows that start on 16 bytes (stored four entries at a time) and of others, padded
    and not, with the block's own rows kept, and of a second call: the same entries."""
    q, k, tq, tk = layer
    need = va.max_count(N, P, causal, mode, param, True)
    cap = need + (-need) % 4
    idx, cnt, _, _ = run(tq, tk, mode, param, causal, cap=cap)
    check(q, k, mode, param, causal, cap, idx, cnt, np.arange(0, 2 * NP, 7))
    again, cnt2, _, _ = run(tq, tk, mode, param, causal, cap=cap)
    assert torch.equal(idx, again) and torch.equal(cnt, cnt2)
    odd, cnt3, _, _ = run(tq, tk, mode, param, causal, cap=cap + 1)
    assert torch.equal(idx, odd[..., :cap]) and torch.equal(cnt, cnt3) and bool((odd[..., cap] == -1).all())
    for c in (cap, cap + 1):
        raw = torch.full((1, 2, NP, c), 0x7FFF7FFF, dtype=torch.int32, device="cuda")
        run(tq, tk, mode, param, causal, cap=c, idx=raw, unpadded=True)
        live = torch.arange(c, device="cuda").view(1, 1, 1, -1) < cnt.unsqueeze(-1)
        assert torch.equal(raw[..., :cap][live[..., :cap]], idx[live[..., :cap]])
        assert bool((raw[~live] == 0x7FFF7FFF).all())
    diag, cnt4, _, _ = run(tq, tk, mode, param, causal, cap=cap, keep_diag=True)
    want_idx, want_cnt = oracle.with_diagonal(idx.cpu().numpy(), cnt.cpu().numpy(), N, P, cap)
    assert np.array_equal(diag.cpu().numpy(), want_idx) and np.array_equal(cnt4.cpu().numpy(), want_cnt)


def test_topp_mass_beyond_fp32_exponent_range(gpu):
    # Scores spread over ~100 nats: the masses of the low keys take the exact power-of-two rescale.
    q, k, _ = synth.planted_case(750, 1, 2, 2, N, 128, frac=0.05, logits=3.0)
    kf = synth.bits_to_f32(k)
    r = np.random.Generator(np.random.PCG64(751))
    kf *= np.float32(24.0)
    kf[0, :, r.choice(N, 200, replace=False)] *= np.float32(3.0)
    k = synth.to_bf16_bits(kf)
    for h in range(2):
        s = oracle.pooled_scores(q, k, P, False, 0, h, 3)
        assert s.max() - s.min() > 90.0
    for p in (0.5, 0.99, 0.999999):
        idx, cnt, cap, _ = run(dev(q), dev(k), "topp", p, False)
        check(q, k, "topp", p, False, cap, idx, cnt)


@pytest.mark.parametrize("bad", ["nan", "inf", "-inf", "huge", "inf dimension"])
def test_lists_stay_valid_for_non_finite_scores(gpu, bad):
    """Valid lists, and nothing written outside them, whatever the scores: among them more keys
    scoring +infinity than a topK keeps ("inf dimension": the sign of one pooled value decides)."""
    q = synth.bits_to_f32(synth.random_bits(1, (1, 2, N, 128)))
    k = synth.bits_to_f32(synth.random_bits(2, (1, 2, N, 128)))
    if bad == "inf dimension":
        k[0, :, ::3, 0] = np.inf
    else:
        k[0, :, 7::11] = {"nan": np.nan, "inf": np.inf, "-inf": -np.inf, "huge": 3e38}[bad]
    tq, tk = dev(synth.to_bf16_bits(q)), dev(synth.to_bf16_bits(k))
    for mode, param in [("topk", 0.1), ("topk", 1.0), ("topp", 0.9), ("topp", 1.0), ("mins", 0.7), ("mins", 0.0)]:
        full = va.max_count(N, P, False, mode, param)
        for cap in (full, 1000) if mode != "topk" else (full, full + (-full) % 4):
            store = torch.full((2 * NP * cap + 4 * N,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
            idx, cnt, _, _ = run(tq, tk, mode, param, False, cap=cap, idx=store[:2 * NP * cap].view(1, 2, NP, cap))
            assert va.check_lists(idx, cnt, N) == 0, (mode, param, cap)
            assert bool((store[2 * NP * cap:] == 0x5A5A5A5A).all()), (mode, param, cap)

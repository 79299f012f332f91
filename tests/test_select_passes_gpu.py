"""Selection by the score passes (csrc/select.hip), at lengths that the kernels for short
sequences do not take: every mode, cap, option and input that can go wrong there, against the
oracle on sampled blocks (the index-set rule is in selection_parity.py)."""
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


def sampled_rows(Hq, n=24):
    """Blocks of all heads, the first and last of each among them."""
    r = np.random.Generator(np.random.PCG64(Hq))
    ends = [h * NP + i for h in range(Hq) for i in (0, NP - 1)]
    return np.unique(np.concatenate([ends, r.choice(Hq * NP, size=n, replace=False)]))


def check(q, k, mode, param, causal, cap, idx, cnt, rows=None, block=P, allowed=20):
    rows = sampled_rows(q.shape[1]) if rows is None else rows
    ih = idx.reshape(-1, cap).cpu().numpy()[rows]
    ch = cnt.reshape(-1).cpu().numpy()[rows]
    mism = check_rows(q, k, block, OMODE[mode], param, causal, cap, ih, ch, rows, compact=True)
    assert mism <= max(1, len(rows) // allowed)


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

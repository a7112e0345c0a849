"""Prefill grids: the order that keeps few (group, kv-head) pairs on an XCD at a time, its remainders, and
the plain order of small grids (up to 1024 workgroups, 2048 with 64-wide heads and more than 16 pairs an
XCD) and of pair counts that are no multiple of 8; prompts around the ends of key blocks and workgroup rows,
one and two row tiles per wave. Every row is compared with the oracle."""
import numpy as np
import pytest
import torch

import oracle
from workloads import make_prefill_workload

pytestmark = pytest.mark.gpu

CASES = [
    # (name, Hq, Hkv, d, prompt lengths, kv dtype)
    ("one-set", 16, 8, 128, [33, 64, 31], "bf16"),
    ("two-sets-odd-blocks", 16, 8, 64, [95, 1, 32, 65, 96, 17], "bf16"),
    ("two-sets-even-blocks", 8, 8, 128, [128, 127, 0, 63, 64, 3, 100], "bf16"),
    ("half-pairs", 16, 4, 128, [40, 16, 70, 8], "fp8"),
    # Ordered grids: one set of an XCD's pairs (at most 16, K and V up to 24 MiB), with an idle slot where they
    # are even; sets of 5 otherwise, with every remainder, odd and even row blocks.
    ("ordered-one-set", 64, 8, 128, [345, 337, 344], "bf16"),             # 3 pairs per XCD, 44 row blocks
    ("ordered-one-even-set", 32, 4, 128, [40, 16, 70, 8] * 8, "fp8"),     # 16 pairs, 10 row blocks
    ("ordered-two-tiles", 64, 8, 64, [385, 641, 400, 150, 700, 390], "bf16"),  # 6 pairs
    ("ordered-large-rest-1", 32, 8, 128, [1040, 1040, 1041, 1030, 1040, 1000], "bf16"),  # 6 pairs, above 24 MiB
    ("ordered-large-rest-4", 32, 8, 128, [700, 650, 697, 690, 690, 680, 701, 700, 690], "bf16"),  # 9 pairs
    ("ordered-rest-0", 16, 8, 64, [61, 1, 32, 64, 33] * 26, "bf16"),      # 130 pairs, 2 row blocks
    ("ordered-rest-2", 32, 8, 128, [128, 5, 64, 90] * 4 + [100], "bf16"),  # 17 pairs, 8 row blocks
    ("ordered-rest-3", 32, 8, 128, [5, 17, 33, 40, 0, 16] * 8, "bf16"),   # 48 pairs, 3 row blocks
    ("ordered-rest-4", 32, 8, 128, [112, 5, 64, 90] * 4 + [100, 3, 31], "fp8"),  # 19 pairs, 7 row blocks
    ("few-d64-plain", 32, 8, 64, [255, 240, 256, 249, 13], "bf16"),     # 5 pairs, 640: plain
    ("few-d64-over-the-line", 64, 8, 64, [255, 240, 256, 249, 13], "bf16"),  # 1280: one set
    ("many-d64-at-the-line", 8, 8, 64, [127, 65, 63, 0] * 32, "bf16"),    # 128 pairs, 2048: plain
    ("at-the-line", 8, 8, 128, [64, 63, 17, 0] * 32, "bf16"),             # 1024 workgroups: plain
    ("over-the-line", 8, 8, 128, [65, 63, 17, 0] * 17, "bf16"),           # 1088
    ("plain-order", 4, 2, 128, [50, 33, 130], "bf16"),                   # 6 pairs
    ("plain-order-nrep8", 8, 1, 64, [20, 45, 64], "bf16"),
    ("two-tiles", 16, 8, 128, [400, 385, 31, 800], "bf16"),              # 404 tokens a prompt
    ("two-tiles-nrep8", 32, 4, 128, [390, 417, 500, 400], "bf16"),
    ("two-tiles-plain", 6, 3, 64, [410, 390], "fp8"),
    ("two-tiles-mha", 8, 8, 64, [641, 129], "bf16"),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_every_row_of_every_order(case):
    import paper_2606_26997_amd as rp
    name, hq, hkv, d, lens, dt = case
    print(f"[case] prefill order {name}", flush=True)
    w = make_prefill_workload(num_q_heads=hq, num_kv_heads=hkv, head_dim=d, prefix_lens=lens, seed=len(name),
                              kv_dtype=dt)
    b = rp.PrefillBatch.from_workload(w)
    b.out.fill_(float("nan"))
    b.lse.fill_(float("nan"))
    b.prefill()
    torch.cuda.synchronize()
    ref, ref_lse = oracle.prefill_attention(w.q, w.k, w.v, w.prefix_offs, w.softmax_scale)
    out, lse = b.out.float().cpu().numpy().astype(np.float64), b.lse.cpu().numpy().astype(np.float64)
    # The bf16 output's own rounding (half an ulp of each exact value) plus the contract's bound.
    half_ulp = np.ldexp(1.0, np.frexp(np.abs(ref))[1] - 9)
    assert np.maximum(np.abs(out - ref) - half_ulp, 0).max() <= 1e-2
    assert np.linalg.norm(out - ref) <= 5e-3 * np.linalg.norm(ref)
    assert np.abs(lse - ref_lse).max() <= 1e-4


@pytest.mark.parametrize("two_tiles", [False, True], ids=["one-tile", "two-tiles"])
@pytest.mark.parametrize("nrep", [1, 2, 4, 8])
@pytest.mark.parametrize("d", [64, 128])
def test_page_rows_end_with_the_prompt(d, nrep, two_tiles):
    """bf16 rows that the attention writes into the pages: those of the page-write call, byte for byte, around
    the ends of a workgroup's rows and of one pass of its threads over them; no row past a prompt's end."""
    import paper_2606_26997_amd as rp
    print(f"[case] page rows d {d} nrep {nrep} two tiles {two_tiles}", flush=True)
    lens = [1, 7, 8, 9, 0, 15, 16, 17, 31, 32, 33, 47, 63, 64, 65, 127, 128, 129]
    if two_tiles:
        lens = [511, 513] * 30 + lens
        assert sum(lens) >= 384 * len(lens)
    w = make_prefill_workload(num_q_heads=2 * nrep, num_kv_heads=2, head_dim=d, prefix_lens=lens, seed=d + nrep)
    pools = []
    for call in ("prefill", "kv_write"):
        b = rp.PrefillBatch.from_workload(w)
        for x in (b.k_pages, b.v_pages):
            x.view(torch.int16).fill_(0x5555)
        getattr(b, call)()
        torch.cuda.synchronize()
        pools.append((b.k_pages.view(torch.int16).clone(), b.v_pages.view(torch.int16).clone()))
    assert (pools[1][0] == 0x5555).any()  # rows past the ends
    for x, y in zip(*pools):
        assert torch.equal(x, y)


def test_large_and_hidden_scores():
    """Scores that grow by far more than the lazy maximum's headroom from block to block, and a first key
    block whose scores are all hugely negative: the running maximum has to move at the right blocks."""
    import paper_2606_26997_amd as rp
    print("[case] prefill large scores", flush=True)
    w = make_prefill_workload(num_q_heads=4, num_kv_heads=2, head_dim=64, prefix_lens=[200, 130], seed=2)
    q, k = (torch.from_numpy(x.view(np.int16).copy()).view(torch.bfloat16) for x in (w.q, w.k))
    ramp = torch.ones(330)
    ramp[:200] = torch.linspace(-40, 40, 200)
    ramp[200:232] = -300.0
    q = (q.abs() + 0.5).to(torch.bfloat16)
    k = ((k.abs() * 0.05 + 1.0) * ramp.view(-1, 1, 1)).to(torch.bfloat16)
    bits = lambda x: x.view(torch.int16).numpy().view(np.uint16)
    w.q, w.k = bits(q), bits(k)
    b = rp.PrefillBatch.from_workload(w)
    b.prefill()
    torch.cuda.synchronize()
    ref, ref_lse = oracle.prefill_attention(w.q, w.k, w.v, w.prefix_offs, w.softmax_scale)
    out, lse = b.out.float().cpu().numpy().astype(np.float64), b.lse.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(out - ref) <= 5e-3 * np.linalg.norm(ref)
    # fp32 scores of magnitude up to 4000: an ulp is 2.4e-4, a dot product of 64 terms adds a few.
    assert np.abs(lse - ref_lse).max() <= 4e-3

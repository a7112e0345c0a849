"""Response units of the partial attention at the edges of a step (one, two or four pages, by head size
and KV type), for every head ratio, in the precision the partial results are kept in: the fp32 partials
are merged in fp64 and compared with the oracle, so that a lost term of the probabilities (bf16 alone
would be 2^-9 of each) cannot hide behind the bf16 rounding of the output."""
import copy

import numpy as np
import pytest
import torch

import oracle
from gpu_util import compare, run_hip, run_oracle
from workloads import make_workload

pytestmark = pytest.mark.gpu

# Tokens around the ends of one, two and four pages, the first piece boundary (256 tokens) and beyond it.
LENS = [1, 15, 16, 17, 31, 32, 33, 48, 49, 63, 64, 65, 80, 81, 255, 256, 257, 300]
SHAPES = [(nrep, d, dt) for nrep in (1, 2, 4, 8) for d in (64, 128) for dt in ("bf16", "fp8")]


def _merged_partials(b):
    """Output and lse of every query row from the planned workspace's fp32 partials, in fp64."""
    import paper_2606_26997_amd as rp
    b.plan()
    b.attn_parts()
    torch.cuda.synchronize()
    info = rp._binding.plan_layout(b.kv, b.attn_layout)
    S, Hq, d, n = b.q.shape[0], b.q.shape[1], b.q.shape[2], info.parts_per_row
    ws = b.workspace.cpu().numpy()
    po = ws[info.part_o:info.part_o + 4 * info.max_parts * d].view(np.float32).reshape(S, Hq, n, d).astype(np.float64)
    pl = ws[info.part_lse:info.part_lse + 4 * info.max_parts].view(np.float32).reshape(S, Hq, n).astype(np.float64)
    parts = b.plan_contents()["seq_parts"]
    out, lse = np.zeros((S, Hq, d)), np.zeros((S, Hq))
    for s in range(S):
        p, o = pl[s, :, :parts[s]], po[s, :, :parts[s]]
        lse[s] = np.logaddexp.reduce(p, axis=1)
        out[s] = (np.exp(p - lse[s][:, None])[:, :, None] * o).sum(1)
    return out, lse


@pytest.mark.parametrize("nrep,d,dt", SHAPES)
def test_partials_keep_fp32_precision(nrep, d, dt):
    import paper_2606_26997_amd as rp
    print(f"[case] steps nrep {nrep} d {d} {dt}", flush=True)
    hkv = 3  # not a power of two, and not the eight that the XCD order divides by
    wl = make_workload(num_q_heads=hkv * nrep, num_kv_heads=hkv, head_dim=d, seq_to_group=[0] * len(LENS),
                       prefix_lens=[0], resp_lens=LENS, seed=nrep + d, kv_dtype=dt)
    out, lse = _merged_partials(rp.DeviceBatch.from_workload(wl))
    ref, ref_lse = oracle.attention_for_workload(wl)
    absv = copy.copy(wl)
    absv.v_pages = wl.v_pages & (0x7F if dt == "fp8" else 0x7FFF)
    mag, _ = oracle.attention_for_workload(absv)  # sum p |v|
    # fp32 rounding relative to sum p |v|: the dot product (sqrt(128) roundings of sum |q k| sigma ~ 7), the
    # exponent's argument (at most 2^5) and the sums, about 1e-5 in all.
    assert np.abs(lse - ref_lse).max() <= 3e-5
    assert (np.abs(out - ref) / mag).max() <= 3e-5


def _staged(b):
    b.plan()
    b.attn_parts()
    b.combine_parts()


@pytest.mark.parametrize("staged", [False, True], ids=["one-launch", "staged"])
@pytest.mark.parametrize("nrep", [1, 2, 4, 8])
def test_infinite_and_nan_values_stay_in_their_column(nrep, staged):
    import paper_2606_26997_amd as rp
    print(f"[case] inf/nan nrep {nrep} staged {staged}", flush=True)
    wl = make_workload(num_q_heads=2 * nrep, num_kv_heads=2, head_dim=128, seq_to_group=[0, 0], prefix_lens=[0],
                       resp_lens=[40, 21], seed=5)
    page = int(wl.resp_block_table[0, 1])
    for col, bits in ((7, 0x7F80), (64, 0xFF80), (100, 0x7FC0)):
        wl.v_pages[page, 1, 3, col] = bits
    b = rp.DeviceBatch.from_workload(wl)
    _staged(b) if staged else b.attention()
    torch.cuda.synchronize()
    out = b.out.float().cpu().numpy()
    assert np.all(out[0, nrep:, 7] == np.inf) and np.all(out[0, nrep:, 64] == -np.inf)
    assert np.isnan(out[0, nrep:, 100]).all()
    out[0, nrep:, [7, 64, 100]] = 0
    assert np.isfinite(out).all()


@pytest.mark.parametrize("d,dt", [(64, "bf16"), (128, "bf16"), (64, "fp8"), (128, "fp8")])
@pytest.mark.parametrize("nrep", [4, 8])
def test_infinite_and_nan_values_leave_the_other_elements_alone(nrep, d, dt):
    """Every element whose values are finite keeps the bits it has without the infinite one: the fp32
    partials of the staged form, and the output of the one-launch form."""
    import paper_2606_26997_amd as rp
    print(f"[case] bits beside inf nrep {nrep} d {d} {dt}", flush=True)
    wl = make_workload(num_q_heads=2 * nrep, num_kv_heads=2, head_dim=d, seq_to_group=[0, 0], prefix_lens=[0],
                       resp_lens=[100, 21], seed=6, kv_dtype=dt)
    marked = copy.copy(wl)
    marked.v_pages = wl.v_pages.copy()
    page = int(wl.resp_block_table[0, 1])
    cols = {9: 0x7FC0, 50: 0x7F80} if dt == "bf16" else {9: 0x7F, 50: 0x7F}  # NaN, infinity; e4m3 has no infinity
    for c, bits in cols.items():
        marked.v_pages[page, 1, 3, c] = bits
    got = []
    for w in (wl, marked):
        b = rp.DeviceBatch.from_workload(w)
        b.workspace.fill_(0xFF)
        b.plan()
        b.attn_parts()
        torch.cuda.synchronize()
        info = rp._binding.plan_layout(b.kv, b.attn_layout)
        ws = b.workspace.cpu().numpy()
        po = ws[info.part_o:info.part_o + 4 * info.max_parts * d].view(np.uint32).reshape(-1, d)
        pl = ws[info.part_lse:info.part_lse + 4 * info.max_parts].view(np.uint32)
        b.attention()
        torch.cuda.synchronize()
        out = b.out.view(torch.int16).cpu().numpy().reshape(-1, d)
        got.append((po.copy(), pl.copy(), out, b.lse.cpu().numpy()))
    for x, y in zip(*got):
        keep = np.ones(x.shape, bool)
        if x.ndim == 2 and x.shape[1] == d:
            keep[:, list(cols)] = False
        assert np.array_equal(x[keep], y[keep])
    special = torch.from_numpy(got[1][2][nrep:2 * nrep]).view(torch.bfloat16).float().numpy()
    assert np.isnan(special[:, 9]).all()
    assert np.isinf(special[:, 50]).all() if dt == "bf16" else np.isnan(special[:, 50]).all()


@pytest.mark.parametrize("hkv,lens", [(1, [40] * 19), (2, [20] * 8), (8, [33] * 9), (3, [700, 16, 5])])
def test_fp8_unit_order_covers_every_unit(hkv, lens):
    """fp8 units are dealt eight items at a time; batches with a remainder of items, fewer than eight, and
    kv-head counts that divide nothing."""
    import paper_2606_26997_amd as rp
    from tests.gpu_util import compare, to_host_out
    print(f"[case] fp8 order hkv {hkv} items {len(lens)}", flush=True)
    wl = make_workload(num_q_heads=2 * hkv, num_kv_heads=hkv, head_dim=128, seq_to_group=[0] * len(lens),
                       prefix_lens=[18], resp_lens=lens, seed=hkv, kv_dtype="fp8")
    b = rp.DeviceBatch.from_workload(wl)
    b.workspace.fill_(0xFF)  # NaN partials: a unit left out shows
    _staged(b)
    out, lse = to_host_out(b)
    ref, ref_lse = oracle.attention_for_workload(wl)
    compare(out, lse, ref, ref_lse, "fp8", f"order-{hkv}")


# (Hq, Hkv, d, dtype, groups' prefix lengths, group of each sequence, response lengths): batches on both
# sides of the lines between one launch and three (64 sequences; the steps of 7 x 8 KiB of K and V that the
# tables take, at most 10, or 20 from four query rows per kv-head, and fewer for fp8 and 64-wide heads unless
# a group's rows need several passes over its prefix), pieces that end with the prefix, with a page and inside
# a step, empty prefixes and responses.
SMALL = [
    (4, 2, 64, "bf16", [128], [0] * 4, [32, 43, 54, 64]),
    (16, 8, 128, "bf16", [17, 0, 130], [0, 0, 1, 1, 2], [0, 1, 0, 16, 300]),
    (8, 8, 128, "bf16", [560, 1], [0, 1, 0], [559, 560, 3]),          # 70 pages
    (8, 8, 128, "bf16", [560, 1], [0, 1, 0], [559, 561, 3]),          # 71: three launches
    (6, 3, 64, "fp8", [40, 1200], [0, 1, 1, 0], [1000, 7, 33, 0]),    # 138 pages of 1 KiB
    (16, 2, 128, "fp8", [300, 90], [0] * 5 + [1] * 3, [5, 900, 64, 63, 65, 0, 129, 800]),
    (8, 1, 128, "bf16", [1000], [0, 0], [1200, 1]),                   # 20 steps, one pass: three launches
    (4, 2, 64, "bf16", [20, 33], [i % 2 for i in range(64)], [3 * i for i in range(64)]),
    (4, 2, 64, "bf16", [20, 33], [i % 2 for i in range(65)], [3 * i for i in range(65)]),  # three launches
    (8, 1, 128, "bf16", [1000], [0] * 8, [1200, 1, 0, 16, 700, 33, 15, 64]),  # 20 steps, four passes: one launch
    (4, 2, 64, "fp8", [480, 3], [0, 0], [1740, 5]),                   # 139 pages of 1 KiB, 5 steps: one launch
    (4, 2, 64, "fp8", [480, 3], [0, 0], [1800, 5]),                   # 143 pages, 6 steps: three
    (16, 2, 64, "fp8", [300, 90], [0] * 5 + [1] * 3, [5, 2400, 64, 63, 65, 0, 129, 800]),  # 7 steps, two passes: one
    (4, 2, 64, "bf16", [480, 3], [0, 0], [1290, 5]),                  # 111 pages of 2 KiB, 8 steps: one launch
    (4, 2, 64, "bf16", [480, 3], [0, 0], [1330, 5]),                  # 114 pages, 9 steps: three
]


@pytest.mark.parametrize("case", range(len(SMALL)))
def test_one_launch_and_staged_match_the_oracle_and_each_other(case):
    import paper_2606_26997_amd as rp
    from tests.gpu_util import compare, to_host_out
    hq, hkv, d, dt, P, s2g, L = SMALL[case]
    print(f"[case] small {case}", flush=True)
    wl = make_workload(num_q_heads=hq, num_kv_heads=hkv, head_dim=d, seq_to_group=s2g, prefix_lens=P, resp_lens=L,
                       seed=case, kv_dtype=dt)
    ref, ref_lse = oracle.attention_for_workload(wl)
    b = rp.DeviceBatch.from_workload(wl)
    b.workspace.fill_(0xFF)
    b.attention()
    out, lse = to_host_out(b)
    compare(out, lse, ref, ref_lse, dt, f"one call {case}")
    plan = b.plan_contents()
    _staged(b)
    out2, lse2 = to_host_out(b)
    compare(out2, lse2, ref, ref_lse, dt, f"staged {case}")
    fin = np.isfinite(ref_lse)
    assert np.abs(lse[fin] - lse2[fin]).max() <= 3e-5
    # The one call leaves the plan behind (pieces of equal length may be listed in any order).
    want = b.plan_contents()
    assert np.array_equal(plan["hdr"][:4], want["hdr"][:4])
    for key in ("grp_off", "prefix_items", "seq_parts"):
        assert np.array_equal(plan[key], want[key]), key
    order = lambda x: x[np.lexsort(x.T)]
    assert np.array_equal(order(plan["resp_items"]), order(want["resp_items"]))


@pytest.mark.parametrize("case", range(len(SMALL)))
def test_combine_after_the_one_call_gives_its_results_again(case):
    """rp_group_decode_attn leaves partial results that rp_combine_parts merges to the same bits, in the
    one-launch form too, for rows without keys and rows with NaN scores as well."""
    import paper_2606_26997_amd as rp
    hq, hkv, d, dt, P, s2g, L = SMALL[case]
    print(f"[case] combine again {case}", flush=True)
    wl = make_workload(num_q_heads=hq, num_kv_heads=hkv, head_dim=d, seq_to_group=s2g, prefix_lens=P, resp_lens=L,
                       seed=case, kv_dtype=dt)
    wl.q[-1, 1, 3] = 0x7FC0
    if dt == "bf16":
        wl.k_pages[wl.resp_block_table[0, 0], 0, 0, 5] = 0x7FC0  # one NaN key: NaN beside finite parts
    b = rp.DeviceBatch.from_workload(wl)
    b.workspace.fill_(0xFF)
    b.attention()
    out, lse = b.out.clone(), b.lse.clone()
    b.out.fill_(7.0)
    b.lse.fill_(7.0)
    b.combine_parts()
    torch.cuda.synchronize()
    assert torch.equal(torch.isnan(out), torch.isnan(b.out))
    assert torch.equal(out.nan_to_num(9.0).view(torch.int16), b.out.nan_to_num(9.0).view(torch.int16))
    assert torch.equal(lse.view(torch.int32), b.lse.view(torch.int32))


@pytest.mark.parametrize("below", [False, True], ids=["at-the-line", "below"])
@pytest.mark.parametrize("nrep,d,dt", [(1, 128, "bf16"), (2, 64, "bf16"), (4, 128, "fp8"), (8, 64, "fp8")])
def test_prefix_units_at_the_line_of_the_streaming_hint(nrep, d, dt, below):
    """128 MiB of prefixes in full chunks of 256 tokens, and one chunk less; one group of two passes."""
    print(f"[case] prefix stream line nrep {nrep} d {d} {dt} below {below}", flush=True)
    hkv = 8
    groups = (128 << 20) // (4 * 256 * hkv * 2 * d * (2 if dt == "bf16" else 1))  # 4 chunks each
    lens = [1024 - (37 * g) % 200 for g in range(groups)]
    if below:
        lens[-1] = 700
    members = [0] * (16 // nrep) + list(range(groups))
    wl = make_workload(num_q_heads=hkv * nrep, num_kv_heads=hkv, head_dim=d, seq_to_group=members, prefix_lens=lens,
                       resp_lens=[(5 * i) % 40 for i in range(len(members))], seed=d + nrep, kv_dtype=dt)
    _, out, lse = run_hip(wl, staged=True)
    ref, ref_lse, _ = run_oracle(wl)
    compare(out, lse, ref, ref_lse, dt)

"""fp8 append at every row of a page: kept scales, and raised ones whose requantised rows land on midpoints
between codes (ratios of 2, 1.5, 1.25, 7 and 1 + 2^-7), with all codes in the earlier rows; scales outside
the range that quotients by the inverse cover. Codes and scales equal the oracle's byte for byte, through
rp_kv_append (K and V) and rp_decode_qk_prep (V, which it appends unchanged)."""
import numpy as np
import pytest
import torch

import oracle
from tests.paged import bf16_bits
from workloads import make_qkprep_inputs, make_workload

pytestmark = pytest.mark.gpu

RATIOS = [0.5, 2.0, 1.5, 1.25, 7.0, 1.0078125]


@pytest.mark.parametrize("d,hkv", [(128, 8), (64, 3), (128, 1), (64, 8)])
@pytest.mark.parametrize("base", [1.0, 2.0 ** -110, 2.0 ** 90])
def test_every_row_and_ratio(d, hkv, base):
    import paper_2606_26997_amd as rp
    print(f"[case] fp8 append d {d} hkv {hkv} scale {base:g}", flush=True)
    rng = np.random.default_rng(d + hkv)
    lens = [16 * (i % 2) + r for i, r in enumerate(list(range(16)) * len(RATIOS))]
    S = len(lens)
    wl = make_workload(num_q_heads=2 * hkv, num_kv_heads=hkv, head_dim=d, seq_to_group=[0] * S, prefix_lens=[5],
                       resp_lens=lens, seed=7, append=True, kv_dtype="fp8")
    new = rng.standard_normal((2, S, hkv, d)).clip(-4, 4)
    for s, L in enumerate(lens):
        page, r = int(wl.resp_block_table[s, L // 16]), L % 16
        for pages, scale in ((wl.k_pages, wl.k_scale), (wl.v_pages, wl.v_scale)):
            codes = rng.integers(0, 0x7F, (hkv, 16, d)).astype(np.uint8) | (rng.integers(0, 2, (hkv, 16, d)) << 7).astype(np.uint8)
            pages[page, :, :r] = codes[:, :r]
            scale[page] = base
        new[:, s, :, 3] = 448.0 * RATIOS[s // 16]  # amax = 448 old ratio
    new = np.clip(new * base, -3e38, 3e38)
    wl.k_new[:], wl.v_new[:] = bf16_bits(new[0]), bf16_bits(new[1])
    kw = dict(k_pages=wl.k_pages, v_pages=wl.v_pages, k_scale=wl.k_scale, v_scale=wl.v_scale, kv_dtype="fp8",
              page_size=16, resp_lens=wl.resp_lens, resp_block_table=wl.resp_block_table)
    kp, vp, ks, vs = oracle.kv_append(**kw, k_new=wl.k_new, v_new=wl.v_new)
    b = rp.DeviceBatch.from_workload(wl)
    b.kv_append()
    torch.cuda.synchronize()
    for got, want in ((b.k_scale, ks), (b.v_scale, vs), (b.k_pages, kp), (b.v_pages, vp)):
        np.testing.assert_array_equal(got.cpu().numpy(), want)

    x = make_qkprep_inputs(num_seqs=S, num_q_heads=2 * hkv, num_kv_heads=hkv, head_dim=d, seed=1)
    b = rp.DeviceBatch.from_workload(wl)
    b.set_projections(x.q_in, x.k_in, wl.v_new, x.q_norm_w, x.k_norm_w)
    b.qk_prep()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(b.v_scale.cpu().numpy(), vs)
    np.testing.assert_array_equal(b.v_pages.cpu().numpy(), vp)


@pytest.mark.parametrize("d,hq,hkv", [(128, 16, 8), (128, 3, 3), (64, 8, 2), (64, 32, 32)])
def test_some_heads_of_a_wave_raise(d, hq, hkv):
    """A wave holds several (sequence, kv-head) rows and requantises the pages of those that raise their
    scale one after the other; here each K and V row of a head raises it or not by itself, none to all of them."""
    import paper_2606_26997_amd as rp
    print(f"[case] fp8 append mixed d {d} hq {hq} hkv {hkv}", flush=True)
    rng = np.random.default_rng(d + hq + hkv)
    lens = [r for r in range(16)] * 6
    S = len(lens)
    wl = make_workload(num_q_heads=hq, num_kv_heads=hkv, head_dim=d, seq_to_group=[0] * S, prefix_lens=[5],
                       resp_lens=lens, seed=9, append=True, kv_dtype="fp8")
    share = rng.choice([0.0, 0.2, 0.5, 1.0], (2, S, 1))  # of a sequence's rows that raise
    ratio = np.where(rng.random((2, S, hkv)) < share, rng.choice(RATIOS[1:], (2, S, hkv)), 0.5)
    base = np.exp2(rng.integers(-8, 8, (2, S, hkv)))
    new = rng.standard_normal((2, S, hkv, d)).clip(-4, 4)
    for s, L in enumerate(lens):
        page = int(wl.resp_block_table[s, 0])
        for i, (pages, scale) in enumerate(((wl.k_pages, wl.k_scale), (wl.v_pages, wl.v_scale))):
            pages[page, :, :L] = rng.integers(0, 0x7F, (hkv, L, d)) | (rng.integers(0, 2, (hkv, L, d)) << 7)
            scale[page] = base[i, s]
    new[..., 3] = 448.0 * ratio
    new *= base[..., None]
    wl.k_new[:], wl.v_new[:] = bf16_bits(new[0]), bf16_bits(new[1])
    x = make_qkprep_inputs(num_seqs=S, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, seed=1)
    kw = dict(k_pages=wl.k_pages, v_pages=wl.v_pages, k_scale=wl.k_scale, v_scale=wl.v_scale, kv_dtype="fp8",
              page_size=16, resp_lens=wl.resp_lens, resp_block_table=wl.resp_block_table)
    kp, vp, ks, vs = oracle.kv_append(**kw, k_new=wl.k_new, v_new=wl.v_new)
    b = rp.DeviceBatch.from_workload(wl)
    b.kv_append()
    torch.cuda.synchronize()
    for got, want in ((b.k_scale, ks), (b.v_scale, vs), (b.k_pages, kp), (b.v_pages, vp)):
        np.testing.assert_array_equal(got.cpu().numpy(), want)

    b = rp.DeviceBatch.from_workload(wl)
    b.set_projections(x.q_in, x.k_in, wl.v_new, x.q_norm_w, x.k_norm_w)
    b.qk_prep()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(b.v_scale.cpu().numpy(), vs)
    np.testing.assert_array_equal(b.v_pages.cpu().numpy(), vp)

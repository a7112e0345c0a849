"""fp8 page writes at the values where a quotient by the inverse scale could round otherwise than the
division: midpoints between codes, subnormal codes, equal mantissas, scales at the ends of their range,
zeros, infinities and NaN. Codes and scales equal the oracle's, byte for byte, from rp_prefill_kv_write and
from rp_prefill (one launch with the attention)."""
import numpy as np
import pytest
import torch

import oracle
from workloads import make_prefill_workload

pytestmark = pytest.mark.gpu


def _bits(x):
    return torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)


def _values(rng, n):
    """Rows of bf16 bits, one (page, kv-head) block of 16 x 128 each."""
    codes = np.array([oracle.e4m3_to_f64(np.array([c], np.uint8))[0] for c in range(0x7F)])
    mids = np.concatenate([(codes[1:] + codes[:-1]) / 2, codes])  # exact in bf16
    sign = lambda shape: rng.choice([-1.0, 1.0], shape)
    out = []
    for amax in (448.0, 3.5, 96.0, 320.0, 1.75, 1.0):  # scale 1, and amax mantissas of small odd parts
        x = rng.choice(mids * (amax / 448.0), (16, 128)) * sign((16, 128))
        x[3, 5] = amax
        out.append(_bits(x))
    for span in (4, 12, 30):  # ever more subnormal and zero codes
        out.append(_bits(np.exp2(rng.uniform(-span, 0, (16, 128))) * sign((16, 128))))
    out.append(_bits(rng.standard_normal((16, 128)) * np.exp(1.5 * rng.standard_normal((1, 128)))))
    out.append(_bits(np.zeros((16, 128))))
    out.append(rng.integers(0, 0x60, (16, 128)).astype(np.uint16))                 # bf16 subnormals: subnormal scale
    out.append((rng.integers(0x0080, 0x0700, (16, 128))).astype(np.uint16))        # tiny scale, beyond its plain range
    out.append((rng.integers(0x7E00, 0x7F80, (16, 128))).astype(np.uint16))        # largest scale
    while len(out) < n:
        out.append(_bits(rng.standard_normal((16, 128)) * rng.choice([0.5, 1.0, 7.0])))
    return np.stack(out[:n])


@pytest.mark.parametrize("lens", [[16] * 5, [70, 10], [400, 401]], ids=["pages", "ragged", "two-tiles"])
def test_codes_and_scales_match_the_division(lens):
    import paper_2606_26997_amd as rp
    print(f"[case] fp8 pages {lens}", flush=True)
    rng = np.random.default_rng(len(lens) + lens[0])
    hkv, d = 4, 128
    w = make_prefill_workload(num_q_heads=8, num_kv_heads=hkv, head_dim=d, prefix_lens=lens, seed=3, kv_dtype="fp8")
    T = int(w.prefix_offs[-1])
    for arr in (w.k, w.v):
        blocks = _values(rng, -(-T // 16) * hkv)
        rng.shuffle(blocks)
        arr[:] = blocks.reshape(-1, hkv, 16, d).transpose(0, 2, 1, 3).reshape(-1, hkv, d)[:T]
    kp, vp, ks, vs = oracle.prefill_kv_write(k_pages=w.k_pages, v_pages=w.v_pages, k_scale=w.k_scale,
                                             v_scale=w.v_scale, kv_dtype="fp8", page_size=16,
                                             prefix_block_table=w.prefix_block_table, prefix_offs=w.prefix_offs,
                                             k=w.k, v=w.v)
    for call in ("kv_write", "prefill"):
        b = rp.PrefillBatch.from_workload(w)
        getattr(b, call)()
        torch.cuda.synchronize()
        for got, want in ((b.k_scale, ks), (b.v_scale, vs), (b.k_pages, kp), (b.v_pages, vp)):
            np.testing.assert_array_equal(got.cpu().numpy(), want, err_msg=call)


def test_nan_and_infinity():
    import paper_2606_26997_amd as rp
    print("[case] fp8 pages nan/inf", flush=True)
    w = make_prefill_workload(num_q_heads=4, num_kv_heads=2, head_dim=64, prefix_lens=[32], seed=4, kv_dtype="fp8")
    nan_at = [(0, 0, 3, 0x7FC0), (5, 0, 63, 0xFFFF), (17, 1, 8, 0x7F81)]
    clean = w.k.copy()
    for t, h, c, bits in nan_at:
        w.k[t, h, c] = bits
        clean[t, h, c] = 0
    w.v[20, 0, 10] = 0x7F80  # the page's scale becomes infinite
    vfin = w.v.copy()
    vfin[20, 0, 10] = 0
    kp, vp, ks, vs = oracle.prefill_kv_write(k_pages=w.k_pages, v_pages=w.v_pages, k_scale=w.k_scale,
                                             v_scale=w.v_scale, kv_dtype="fp8", page_size=16,
                                             prefix_block_table=w.prefix_block_table, prefix_offs=w.prefix_offs,
                                             k=clean, v=vfin)
    p0, p1 = (int(p) for p in w.prefix_block_table[0, :2])
    for t, h, c, bits in nan_at:
        kp[(p0, p1)[t // 16], h, t % 16, c] = 0x7E | (0x80 if bits & 0x8000 else 0)
    vs[p1, 0] = np.inf  # finite / inf = 0 with the value's sign; inf / inf saturates, its sign is the division's
    signs = (w.v[16:32, 0] >> 15).astype(np.uint8) << 7
    vp[p1, 0] = signs
    vp[p1, 0, 4, 10] = 0x7E
    for call in ("kv_write", "prefill"):
        b = rp.PrefillBatch.from_workload(w)
        getattr(b, call)()
        torch.cuda.synchronize()
        v_pages = b.v_pages.cpu().numpy()
        v_pages[p1, 0, 4, 10] &= 0x7F
        for got, want in ((b.k_scale.cpu().numpy(), ks), (b.v_scale.cpu().numpy(), vs),
                          (b.k_pages.cpu().numpy(), kp), (v_pages, vp)):
            np.testing.assert_array_equal(got, want, err_msg=call)

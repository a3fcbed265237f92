"""GPU parity at the largest batch the calls take: decode runs one grid row per sequence, so
65535 is the largest, and prefill takes no more.
Short ragged contexts keep the caches small; sampled sequences, the first and the last
among them, are compared with the oracle at max|d| <= 2e-3 * max|O|."""
import numpy as np
import pytest
import torch

from oracle import hack_oracle as O

pytestmark = pytest.mark.gpu
TOL = 2e-3
B_MAX = 65535


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util
    return gpu_util


def _sampled(batch, extra, seed):
    g = np.random.default_rng(seed)
    fixed = [0, 1, 2, batch // 2, batch - 2, batch - 1]
    return sorted(set(fixed) | set(int(x) for x in g.integers(0, batch, extra)))


def test_decode_at_the_batch_limit():
    gu = _gpu()
    from paper_2502_03589_amd import hack as hk
    gu.announce(f"decode batch={B_MAX} lens U[0, 40] bits=2 pi=32 G=2")
    lens = np.random.default_rng(2024).integers(0, 41, B_MAX)
    lens[:3] = [0, 1, 40]
    lens[-1] = 33
    case = gu.Case(2024, B_MAX, 1, lens, 2, 32, group=2).quantize()
    out = hk.hack_attend_decode(case.layout, case.cache, torch.from_numpy(case.q).to(gu.DEV), case.lens_dev,
                                case.max_len)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    seqs_b = _sampled(B_MAX, 24, 1)
    seqs = case.oracle_seqs({(b, 0) for b in seqs_b})
    rows = [(b, h) for b in seqs_b for h in range(2)]
    ref = O.attend_decode(case.q, seqs, 1, rows=rows)
    g = np.stack([got[b, h] for b, h in rows])
    r = np.stack([ref[b, h] for b, h in rows])
    err = float(np.abs(g - r).max() / np.abs(r).max())
    print(f"sampled rows max|d|/|O|inf = {err:.3e}")
    assert err <= TOL
    assert not got[0].any()  # the empty sequence's rows are zero


def test_prefill_at_the_batch_limit():
    gu = _gpu()
    from paper_2502_03589_amd import hack as hk
    from paper_2502_03589_amd import synth
    L = 20
    gu.announce(f"prefill batch={B_MAX} L={L} bits=4 pi=32 G=2 causal")
    case = gu.Case(2025, B_MAX, 1, [L] * B_MAX, 4, 32, group=2).quantize()
    Q = synth.normal_f16(case.seed, "q", (B_MAX, 2, L, 128), sub=7)
    out = hk.hack_attend_prefill(case.layout, case.cache, torch.from_numpy(Q).to(gu.DEV), True)
    torch.cuda.synchronize()
    seqs_b = _sampled(B_MAX, 12, 2)
    rows = [(b, h, i) for b in seqs_b for h in range(2) for i in (0, 7, L - 1)]
    g = np.stack([out[b, h, i].cpu().numpy() for b, h, i in rows])
    del out
    Qs = np.ascontiguousarray(Q[seqs_b])
    seqs = case.oracle_seqs({(b, 0) for b in seqs_b})
    sub = [[seqs[b][0]] for b in seqs_b]
    ref = O.attend_prefill(Qs, sub, 1, causal=True, rows=[(seqs_b.index(b), h, i) for b, h, i in rows])
    r = np.stack([ref[seqs_b.index(b), h, i] for b, h, i in rows])
    err = float(np.abs(g - r).max() / np.abs(r).max())
    print(f"sampled rows max|d|/|O|inf = {err:.3e}")
    assert err <= TOL


def test_prefill_grid_of_two_dimensions():
    """More workgroups (65535 sequences x 65 heads = 4.26 million) than one row of the grid holds.
    Prompts of one token attend it alone, so every output row is that token's V row, exactly;
    the sequences share one page and differ in their open blocks."""
    gu = _gpu()
    from paper_2502_03589_amd import hack as hk
    H, d = 65, 128
    gu.announce(f"prefill batch={B_MAX} L=1 heads={H}/{H} bits=2 pi=32")
    lay = hk.hack_kv_layout_make(d, H, 2, 32, 128)
    table = torch.zeros((B_MAX, 1), dtype=torch.int32, device=gu.DEV)
    cache = hk.KVCache(lay, 1, B_MAX, table, gu.DEV)
    g = torch.Generator(device=gu.DEV)
    g.manual_seed(2026)
    k = torch.randn((1, H, 1, d), generator=g, device=gu.DEV).half()
    one = torch.ones(1, dtype=torch.int32, device=gu.DEV)
    hk.hack_quantize(lay, cache, k, k, one)  # the shared page's K row
    tail = cache.buffers["v_tail"].view(torch.float16)[:B_MAX * H * 32 * d].view(B_MAX, H, 32, d)
    v = torch.randn((B_MAX, H, d), generator=g, device=gu.DEV).half()
    tail[:, :, 0].copy_(v)
    q = torch.randn((B_MAX, H, 1, d), generator=g, device=gu.DEV).half()
    out = hk.hack_attend_prefill(lay, cache, q, True)
    # p = 1 as 128 = 2^7 in three fp16 pieces, times v, times 2^-7 / 1: exact
    assert torch.equal(out[:, :, 0], v.float())

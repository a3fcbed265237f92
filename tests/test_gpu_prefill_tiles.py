"""Prefill attention at the edges of its tiling, against the oracle: rows around the 32-row
waves, 32-token tiles and V blocks, every open-block remainder class, kv groups of 1 to 8
(one, two or four heads to a workgroup, with idle head slots), several sequences, both mask
kinds.  Tolerance as for the other prefill cases: 2e-3 of the largest output (8-bit P codes)."""
import numpy as np
import pytest
import torch

from oracle import hack_oracle as O

pytestmark = pytest.mark.gpu
TOL = 2e-3

CASES = [
    # bits, pi, group, kv_heads, batch, lengths, causal, page
    (2, 32, 1, 1, 1, (1, 31, 32, 33, 64, 129, 161), True, 0),
    (4, 32, 2, 1, 2, (17, 63, 65, 96), True, 64),
    (2, 64, 3, 1, 1, (31, 63, 64, 65, 127, 193), True, 0),
    (4, 64, 5, 1, 1, (33, 95, 128), False, 64),
    (4, 64, 7, 1, 1, (100,), True, 0),
    (2, 64, 8, 2, 1, (66,), True, 0),
    (2, 128, 1, 2, 2, (127, 129), True, 128),
    (4, 128, 6, 1, 1, (33, 160), False, 0),
    # two key groups (four V blocks or more on a grid with free slots), the open block in either
    (2, 32, 4, 1, 2, (128, 129, 159, 161), True, 64),
    (4, 64, 2, 1, 1, (256, 300, 321), False, 0),
    (2, 128, 1, 1, 1, (512, 520, 641), True, 0),
]


@pytest.mark.parametrize("bits,pi,group,H,B,lengths,causal,page", CASES)
def test_prefill_tile_edges(bits, pi, group, H, B, lengths, causal, page):
    import tests.gpu_util as gu
    from paper_2502_03589_amd import hack as hk
    from paper_2502_03589_amd import synth
    for L in lengths:
        gu.announce(f"prefill edges bits={bits} pi={pi} G={group} H={H} B={B} L={L} causal={causal} page={page}")
        case = gu.Case(900 + bits + pi + L, B, H, [L] * B, bits, pi, group=group, paged_page=page).quantize()
        Q = synth.normal_f16(case.seed, "q", (B, case.Hq, L, case.d), sub=7)
        got = hk.hack_attend_prefill(case.layout, case.cache, torch.from_numpy(Q).to(gu.DEV), causal).cpu().numpy()
        assert gu.rel_err(got, O.attend_prefill(Q, case.oracle_seqs(), H, causal=causal)) <= TOL


def test_prefill_wide_key_and_value_ranges():
    """Scale and rank-1 factors far from one: query rows, keys and values scaled by 1/64 to 64,
    constant partitions (zero scales).  Each row is measured against its own largest output.
    A P code that rounds the other way moves a row by up to max(p)/255 of the largest value,
    which is a share of that row's output that no fixed bound covers, but it is rare: nine rows
    in ten have none, and there fp32 is left, whose largest terms (128 s_p s_v sum v' in Eq. 4)
    are up to PI/2 of the value range: 64 * 2^-24 * a few rounding steps < 1e-4.  All rows stay
    within the bound of the whole call."""
    import tests.gpu_util as gu
    from paper_2502_03589_amd import hack as hk
    from paper_2502_03589_amd import synth
    for bits, pi in ((2, 32), (4, 64), (2, 128)):
        gu.announce(f"prefill ranges bits={bits} pi={pi}")
        L, H, G = 150, 1, 4
        case = gu.Case(950 + bits + pi, 1, H, [L], bits, pi, group=G)
        case.k[:, :, 1::7] = (case.k[:, :, 1::7].astype(np.float32) / 64).astype(np.float16)
        case.k[:, :, 2::5, :32] = np.float16(0.75)
        case.v[..., 3::11] = (case.v[..., 3::11].astype(np.float32) * 64).astype(np.float16)
        case.v[..., 4::9] = np.float16(-1.5)
        case.quantize()
        Q = synth.normal_f16(case.seed, "q", (1, case.Hq, L, case.d), sub=7)
        Q[:, 1] = (Q[:, 1].astype(np.float32) / 64).astype(np.float16)
        Q[:, 2, :, :64] = np.float16(0.25)
        got = hk.hack_attend_prefill(case.layout, case.cache, torch.from_numpy(Q).to(gu.DEV), True).cpu().numpy()
        ref = O.attend_prefill(Q, case.oracle_seqs(), H, causal=True)
        rows = np.abs(got - ref).max(-1) / np.abs(ref).max(-1)
        print(f"rows: median {np.median(rows):.2e} 90% {np.quantile(rows, 0.9):.2e} max {rows.max():.2e}")
        assert np.quantile(rows, 0.9) <= 1e-4
        assert gu.rel_err(got, ref) <= TOL


@pytest.mark.parametrize("bits,pi,L,qp", [(2, 32, 33, 8), (4, 64, 66, 4), (2, 128, 129, 8)])
def test_prefill_stochastic_few_rows_and_constant_partitions(bits, pi, L, qp):
    """Stochastic Q codes are drawn on every lane: the last row block holds one or two rows, and
    constant partitions (scale 0, code 0 whatever the threshold) lie among the others."""
    import tests.gpu_util as gu
    from paper_2502_03589_amd import hack as hk
    from paper_2502_03589_amd import synth
    gu.announce(f"prefill stochastic rows bits={bits} pi={pi} L={L} qp={qp}")
    case = gu.Case(980 + bits + pi, 1, 2, [L], bits, pi, group=3, rounding=O.STOCHASTIC, qp_bits=qp).quantize()
    Q = synth.normal_f16(case.seed, "q", (1, case.Hq, L, case.d), sub=7)
    Q[:, 1, ::3, :pi] = np.float16(0.5)
    Q[:, 4, L - 1] = np.float16(-0.25)
    got = hk.hack_attend_prefill(case.layout, case.cache, torch.from_numpy(Q).to(gu.DEV), True).cpu().numpy()
    ref = O.attend_prefill(Q, case.oracle_seqs(), 2, causal=True, qp_bits=qp, stochastic_seed=case.seed)
    assert gu.rel_err(got, ref) <= TOL


SAMPLED = [
    # Four V blocks or more.  bits, pi, q_heads, kv_heads, batch, length, causal, rounding, page, key groups
    (2, 32, 32, 8, 2, 1999, True, 0, 256, 1),     # open block, pages
    (4, 32, 8, 8, 24, 190, True, 1, 0, 1),        # stochastic codes, a head to a workgroup
    (4, 64, 16, 2, 24, 300, True, 1, 64, 1),      # stochastic codes, pages, open block
    (2, 64, 4, 4, 60, 300, False, 0, 0, 1),       # no mask
    (4, 128, 8, 2, 30, 600, False, 0, 0, 1),      # no mask, open block
    (2, 128, 2, 1, 40, 650, True, 0, 128, 1),     # two heads to a workgroup, pages
    (2, 32, 8, 1, 60, 150, True, 0, 0, 1),
    (2, 128, 8, 2, 16, 640, True, 1, 0, 1),       # stochastic codes, whole blocks
    (2, 32, 8, 2, 1, 700, True, 1, 32, 2),        # stochastic codes in two key groups
    (4, 64, 4, 1, 1, 1000, True, 1, 0, 2),
]


@pytest.mark.parametrize("bits,pi,hq,hkv,B,L,causal,rounding,page,groups", SAMPLED)
def test_prefill_sampled_rows_of_larger_grids(bits, pi, hq, hkv, B, L, causal, rounding, page, groups):
    """Chains of several blocks in one key group of waves (a full grid) and in two (a short one);
    that each case takes the number beside it is checked on the CPU with the launch rules."""
    import tests.gpu_util as gu
    from paper_2502_03589_amd import hack as hk
    from paper_2502_03589_amd import synth
    gu.announce(f"prefill sampled bits={bits} pi={pi} heads={hq}/{hkv} B={B} L={L} causal={causal} page={page} "
                f"rounding={rounding}")
    case = gu.Case(1100 + bits + pi + L, B, hkv, [L] * B, bits, pi, group=hq // hkv, paged_page=page,
                   rounding=rounding).quantize()
    Q = synth.normal_f16(case.seed, "q", (B, hq, L, case.d), sub=7)
    got = hk.hack_attend_prefill(case.layout, case.cache, torch.from_numpy(Q).to(gu.DEV), causal).cpu().numpy()
    g = np.random.default_rng(L)
    rows = [(0, 0, 0), (B - 1, hq - 1, L - 1), (0, hq - 1, L // pi * pi - 1), (B - 1, 0, L // 2)]
    rows += [(int(g.integers(B)), int(g.integers(hq)), int(g.integers(L))) for _ in range(28)]
    group = hq // hkv
    ref = O.attend_prefill(Q, case.oracle_seqs({(b, h // group) for b, h, _ in rows}), hkv, causal=causal, rows=rows,
                           stochastic_seed=case.seed if rounding else None)
    g = np.stack([got[r] for r in rows])
    r = np.stack([ref[r] for r in rows])
    assert np.abs(g - r).max() <= TOL * np.abs(r).max()

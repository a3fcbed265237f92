"""Decode over fp16 open blocks whose sizes sit at the edges of the batches their rows are
loaded in, and steps whose new token opens, fills or follows a block, against the oracle
(the decode tolerance: 2e-3 of the largest output)."""
import numpy as np
import pytest
import torch

from oracle import hack_oracle as O

pytestmark = pytest.mark.gpu
TOL = 2e-3

OPEN = {32: [1, 3, 4, 5, 31], 64: [1, 31, 32, 33, 36, 63], 128: [1, 7, 8, 9, 64, 127]}


@pytest.mark.parametrize("bits,pi,group", [(2, 32, 4), (4, 32, 5), (2, 64, 1), (4, 64, 8), (2, 128, 3), (4, 128, 8)])
def test_decode_open_block_sizes(bits, pi, group):
    import tests.gpu_util as gu
    from paper_2502_03589_amd import hack as hk
    lens = OPEN[pi] + [4 * pi + t for t in OPEN[pi]] + [4 * pi, 16 * pi + OPEN[pi][-1]]
    gu.announce(f"open block bits={bits} pi={pi} G={group} lens={lens}")
    case = gu.Case(700 + bits + pi, len(lens), 1, lens, bits, pi, group=group).quantize()
    got = hk.hack_attend_decode(case.layout, case.cache, torch.from_numpy(case.q).to(gu.DEV), case.lens_dev,
                                case.max_len).cpu().numpy()
    assert gu.rel_err(got, O.attend_decode(case.q, case.oracle_seqs(), 1)) <= TOL


@pytest.mark.parametrize("bits,pi", [(2, 32), (4, 32), (4, 64)])
def test_step_at_block_and_span_edges(bits, pi):
    """The appended token (not waited for until the query is quantized) is read back by the
    step's own attention, also where it completes a block or a whole four-block span."""
    import tests.gpu_util as gu
    from paper_2502_03589_amd import hack as hk
    lens = [0, 1, pi - 1, pi, 4 * pi - 1, 4 * pi, 16 * pi - 1, 16 * pi]
    gu.announce(f"step edges bits={bits} pi={pi} lens={lens}")
    case = gu.Case(720 + bits + pi, len(lens), 2, lens, bits, pi, group=4, spare_tokens=1).quantize()
    kn = np.stack([case.k[b, :, n] for b, n in enumerate(lens)])
    vn = np.stack([case.v[b, :, n] for b, n in enumerate(lens)])
    out_lens = torch.zeros_like(case.lens_dev)
    got = hk.hack_decode_step(case.layout, case.cache, torch.from_numpy(kn).to(gu.DEV), torch.from_numpy(vn).to(gu.DEV),
                              torch.from_numpy(case.q).to(gu.DEV), case.lens_dev, out_lens, case.max_len).cpu().numpy()
    case.lens = np.asarray(lens, np.int32) + 1
    assert np.array_equal(out_lens.cpu().numpy(), case.lens)
    assert gu.rel_err(got, O.attend_decode(case.q, case.oracle_seqs(), 2)) <= TOL


def _infinite_case(gu, seed, lens, bits, pi, group):
    """A cache whose every open block ends in a row with infinities in four channels (the
    quantized blocks stay finite), and the oracle's sequences."""
    case = gu.Case(seed, len(lens), 1, lens, bits, pi, group=group)
    for b, n in enumerate(lens):
        case.v[b, :, n - 1, [5, 64]] = np.inf
        case.v[b, :, n - 1, [0, 127]] = -np.inf
    return case.quantize()


def _same_infinities(got, ref):
    """The infinities of ref at their places with their signs; elsewhere the tolerance."""
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)
    assert inf.any() and np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf] > 0, ref[inf] > 0)
    fin = np.isfinite(ref)
    assert np.abs(got[fin] - ref[fin]).max() <= TOL * np.abs(ref[fin]).max()


@pytest.mark.filterwarnings("ignore::RuntimeWarning")  # the oracle's codes of the open block
@pytest.mark.parametrize("bits,pi,group", [(2, 32, 4), (4, 32, 5), (2, 64, 1), (4, 64, 8), (2, 128, 3)])
def test_decode_infinite_value_in_the_open_block(bits, pi, group):
    """An infinite V value of the open block's last row, whatever the row's place in the batch
    it is loaded in, gives infinite outputs in its channels and changes no other."""
    import tests.gpu_util as gu
    from paper_2502_03589_amd import hack as hk
    lens = [4 * pi + t for t in OPEN[pi]] + [4 * pi + 2, pi - 1]
    gu.announce(f"open block infinities bits={bits} pi={pi} G={group} lens={lens}")
    case = _infinite_case(gu, 740 + bits + pi, lens, bits, pi, group)
    got = hk.hack_attend_decode(case.layout, case.cache, torch.from_numpy(case.q).to(gu.DEV), case.lens_dev,
                                case.max_len).cpu().numpy()
    _same_infinities(got, O.attend_decode(case.q, case.oracle_seqs(), 1))


@pytest.mark.filterwarnings("ignore::RuntimeWarning")
@pytest.mark.parametrize("bits,pi,group,L", [(2, 32, 4, 70), (4, 64, 2, 100), (2, 64, 4, 300), (4, 128, 1, 150)])
def test_prefill_infinite_value_in_the_open_block(bits, pi, group, L):
    """As in decode, where the weights are split into pieces of which some are zero: every row
    that attends the token has infinite outputs in its channels, also the first one, whose
    weight for it is about 2^-57; causal rows that end before the block are untouched."""
    import tests.gpu_util as gu
    from paper_2502_03589_amd import hack as hk
    from paper_2502_03589_amd import synth
    gu.announce(f"prefill open block infinities bits={bits} pi={pi} G={group} L={L}")
    case = _infinite_case(gu, 760 + bits + pi + L, [L], bits, pi, group)
    case.k[0, :, L - 1] = np.float16(-3.5)  # against a query of ones: a score of -39.6
    case.quantize()
    Q = synth.normal_f16(case.seed, "q", (1, case.Hq, L, case.d), sub=7)
    Q[:, :, 0] = np.float16(1.0)
    seqs = case.oracle_seqs()
    got = hk.hack_attend_prefill(case.layout, case.cache, torch.from_numpy(Q).to(gu.DEV), False).cpu().numpy()
    _same_infinities(got, O.attend_prefill(Q, seqs, 1, causal=False))
    got = hk.hack_attend_prefill(case.layout, case.cache, torch.from_numpy(Q).to(gu.DEV), True).cpu().numpy()
    last = [(0, h, L - 1) for h in range(case.Hq)]
    ref = O.attend_prefill(Q, seqs, 1, causal=True, rows=last)
    _same_infinities(np.stack([got[r] for r in last]), np.stack([ref[r] for r in last]))
    case.v[0, :, L - 1] = 0  # not attended by the rows before the open block
    early = L // pi * pi // 32 * 32
    ref = O.attend_prefill(Q, case.oracle_seqs(), 1, causal=True)[:, :, :early]
    assert gu.rel_err(got[:, :, :early], ref) <= TOL

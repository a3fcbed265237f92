"""The projection at each of its tile shapes and at their edges: the host picks the shape from
the number of tiles and hidden, so the cases below reach all five (that each reaches the shape
beside it is checked on the CPU with the launch rules).  Where the products are exact
(embeddings k/4, weights j/64, |k|, |j| <= 8: every sum over 4096 channels needs at most 19
bits) the query heads equal the float64 product and every cache byte that of hack_quantize of
its key and value heads (which has its own parity tests)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [
    # bits, pi, batch, q_heads, kv_heads, lengths, page, rounding (hidden 192)
    (2, 32, 1, 32, 8, (1, 31, 32, 33, 65), 0, 0),          # 32-token tiles
    (2, 32, 1, 32, 8, (192, 250), 256, 0),                 # 64-token tiles
    (4, 64, 3, 28, 4, (63, 129), 0, 0),                    # 64-token tiles, several sequences
    (2, 16, 1, 32, 8, (511, 600), 0, 1),                   # 64-token tiles, stochastic codes
    (4, 128, 1, 16, 2, (127, 257), 0, 0),                  # 128-token tiles (one V block each)
    (4, 64, 1, 32, 8, (1000,), 0, 0),                      # 256 tokens x one head
    (2, 32, 1, 32, 8, (1537,), 256, 0),                    # 64-token tiles, more than one round
    (2, 64, 1, 5, 5, (1300,), 0, 0),                       # 64-token tiles, an odd number of heads
]
TILES = [(32, 128), (64, 128), (64, 128), (64, 128), (128, 128), (256, 128), (64, 128), (64, 128)]

# hidden 4096, one length: bits, pi, batch, q_heads, kv_heads, length, page, rounding, tile.  With
# an odd number of heads the last tile of two heads has one (clamped weight rows beside it), and
# with an odd number of query heads one tile holds a query and a key head.
DEEP = [
    (2, 32, 1, 13, 1, 4400, 0, 0, (256, 256)),
    (4, 128, 2, 13, 1, 2300, 0, 0, (256, 256)),   # two sequences
    (2, 16, 1, 13, 1, 4400, 0, 1, (256, 256)),    # stochastic codes, the finest partition
    (4, 64, 1, 32, 8, 1500, 256, 0, (256, 256)),  # pages
    (2, 16, 1, 13, 1, 3000, 0, 1, (256, 128)),
    (4, 128, 1, 11, 1, 4700, 0, 0, (256, 128)),
    (2, 32, 1, 32, 8, 2590, 256, 0, (128, 128)),
    (4, 64, 2, 28, 4, 250, 0, 1, (64, 128)),      # two workgroups a compute unit
    (2, 16, 2, 28, 4, 200, 0, 0, (32, 128)),
]


@pytest.mark.parametrize("bits,pi,B,Hq,H,L,page,rounding,tile", DEEP)
def test_project_tile_shapes_of_a_deep_projection_bit_exact(bits, pi, B, Hq, H, L, page, rounding, tile):
    _check(bits, pi, B, Hq, H, L, page, rounding, 4096)


@pytest.mark.parametrize("bits,pi,B,Hq,H,lengths,page,rounding", CASES)
def test_project_tile_shapes_bit_exact(bits, pi, B, Hq, H, lengths, page, rounding):
    for L in lengths:
        _check(bits, pi, B, Hq, H, L, page, rounding, 192)


def _check(bits, pi, B, Hq, H, L, page, rounding, hidden):
    import tests.gpu_util as gu
    from paper_2502_03589_amd import hack as hk
    gu.announce(f"project tiles bits={bits} pi={pi} B={B} heads={Hq}/{H} L={L} hidden={hidden} page={page} "
                f"rounding={rounding}")
    g = np.random.default_rng(1000 + L)
    e = (g.integers(-8, 9, (B, L, hidden)) / 4).astype(np.float16)
    w = (g.integers(-8, 9, ((Hq + 2 * H) * 128, hidden)) / 64).astype(np.float16)
    e, w = torch.from_numpy(e).to(gu.DEV), torch.from_numpy(w).to(gu.DEV)
    ref = torch.stack([(x.double() @ w.double().T).half() for x in e])
    ref = ref.reshape(B, L, Hq + 2 * H, 128).transpose(1, 2)
    if page:
        blocks = -(-L // page)
        table = torch.from_numpy(g.permutation(B * blocks).astype(np.int32).reshape(B, blocks)).to(gu.DEV)
        pages, pt = B * blocks, page
    else:
        table, pages, pt = None, B, -(-L // pi) * pi
    lay = hk.hack_kv_layout_make(128, H, bits, pi, pt, 8, rounding, 77)
    got, want = (hk.KVCache(lay, pages, B, table, gu.DEV) for _ in range(2))
    q = hk.hack_project_qkv(lay, got, e, w, Hq)
    k, v = ref[:, Hq:Hq + H].contiguous(), ref[:, Hq + H:].contiguous()
    hk.hack_quantize(lay, want, k, v, torch.full((B,), L, dtype=torch.int32, device=gu.DEV))
    assert torch.equal(q.view(torch.int16), ref[:, :Hq].contiguous().view(torch.int16))
    for name in hk.SECTIONS:
        assert torch.equal(got.buffers[name], want.buffers[name]), name

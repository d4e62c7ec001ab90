"""GPU parity of moe_quant_pack against the oracle: codes and {scale, zero}
words must be identical bit for bit (Sec. IV-A quantizer, Sec. V-B packing)."""
import numpy as np
import pytest
import torch

import moe_inputs as mi
from gpu_util import dev

pytestmark = pytest.mark.gpu


def _weights(rng, R, K, kind):
    if kind == "normal":
        return (rng.standard_normal((R, K)) * 0.02).astype(np.float32)
    if kind == "edge":
        w = (rng.standard_normal((R, K)) * 0.02).astype(np.float32)
        w[0] = 0.0                                    # degenerate groups
        w[1] = np.abs(w[1])                           # all positive
        w[2] = -np.abs(w[2])                          # all negative
        w[3] *= 1e-7                                  # subnormal fp16 scales
        w[4, ::7] = 3.0                               # outliers
        w[5] = 0.37                                   # constant
        return w
    raise ValueError(kind)


def _gpu_pack(w, bits, group, rows=None):
    import paper_2503_21135_amd as P
    R, K = w.shape
    n = R if rows is None else len(rows)
    codes = torch.zeros(n * K * bits // 32, dtype=torch.int32, device=dev())
    sz = torch.zeros(n * (K // group), dtype=torch.int32, device=dev())
    st = torch.zeros(1, dtype=torch.int32, device=dev())
    rt = None if rows is None else torch.tensor(rows, dtype=torch.int32, device=dev())
    P.moe_quant_pack(torch.from_numpy(w).to(dev()), bits, group, codes, sz, n=n, rows=rt,
                     ld_codes=K * bits // 32, sz_row_stride=K // group, sz_group_stride=1,
                     status=st)
    torch.cuda.synchronize()
    return (codes.cpu().numpy().view(np.uint32).reshape(n, -1),
            sz.cpu().numpy().view(np.uint32).reshape(n, -1), int(st.item()))


@pytest.mark.parametrize("bits,group", [(2, 64), (4, 64), (8, 64), (2, 128), (3, 128),
                                        (4, 128), (6, 128), (8, 128)])
@pytest.mark.parametrize("kind", ["normal", "edge"])
def test_pack_bitexact(orc, bits, group, kind):
    rng = np.random.default_rng(bits * 100 + group)
    R, K = 40, 1408 if group == 128 else 512
    w = _weights(rng, R, K, kind)
    codes, sz, st = _gpu_pack(w, bits, group)
    assert st == 0
    s, q, s16, z16 = orc.quantize(w, bits, group)
    assert s == 0
    assert np.array_equal(codes, orc.pack(q, bits))
    assert np.array_equal(sz, orc.sz_words(s16, z16))


def test_pack_row_subset_and_overflow(orc):
    rng = np.random.default_rng(9)
    w = (rng.standard_normal((64, 256)) * 0.02).astype(np.float32)
    rows = [63, 0, 17, 17, 5]
    codes, sz, st = _gpu_pack(w, 8, 64, rows)
    s, q, s16, z16 = orc.quantize(w[rows], 8, 64)
    assert st == 0
    assert np.array_equal(codes, orc.pack(q, 8))
    assert np.array_equal(sz, orc.sz_words(s16, z16))
    w[3, 5] = 1e9
    _, _, st = _gpu_pack(w, 2, 64)
    assert st == -6


@pytest.mark.parametrize("name", ["mixtral-decode", "deepseek-decode"])
def test_pack_full_size_sampled_rows(orc, name):
    """Full-size expert matrices: GPU pack of whole matrices, sampled rows
    compared with the oracle."""
    import moe_inputs as mi
    inp = mi.LayerInputs(mi.WORKLOADS[name].layer)
    rng = np.random.default_rng(1)
    E = inp.cfg.n_experts
    for e in (0, E - 1):
        b = int(inp.bits[e])
        for kind in (0, 2):
            w = inp.weight(e, kind)
            codes, sz, st = _gpu_pack(w, b, inp.cfg.group)
            assert st == 0
            rows = np.sort(rng.choice(w.shape[0], 64, replace=False))
            s, q, s16, z16 = orc.quantize(w[rows], b, inp.cfg.group)
            assert np.array_equal(codes[rows], orc.pack(q, b))
            assert np.array_equal(sz[rows], orc.sz_words(s16, z16))


@pytest.mark.parametrize("bits,group", [(2, 64), (4, 64), (8, 64), (3, 128), (6, 128), (8, 128), (16, 64)])
@pytest.mark.parametrize("R,K", [(1, 128), (17, 2048), (33, 2176)])
def test_pack_tile_edges_and_ties(orc, bits, group, R, K):
    """Row and column remainders of the pack tile (16 rows x 2048 columns), a
    matrix whose rows start off 16-byte alignment, and weights whose quotient
    by the scale is exactly a half integer or within a few ulp of one, where
    the code depends on the exact quotient."""
    import paper_2503_21135_amd as P
    rng = np.random.default_rng([bits, group, R, K])
    qmax = (1 << min(bits, 8)) - 1
    half = (rng.integers(0, qmax, (R, K)) + 0.5).astype(np.float32) * np.float32(2.0 ** -7)
    off = rng.integers(-2, 3, (R, K))
    w = np.where(off < 0, np.nextafter(half, np.float32(0)), np.where(off > 0, np.nextafter(half, np.float32(9)), half))
    w[:, ::group] = 0.0                                # every group spans [0, qmax] steps of 2^-7
    w[:, 1::group] = np.float32(qmax * 2.0 ** -7)
    buf = torch.zeros(R * (K + 5) + 3, dtype=torch.float32, device=dev())
    wt = buf[3:].view(R, K + 5)[:, 1:K + 1]
    wt.copy_(torch.from_numpy(w))
    codes = torch.zeros(R * K * bits // 32, dtype=torch.int32, device=dev())
    sz = torch.zeros(R * (K // group), dtype=torch.int32, device=dev())
    P.moe_quant_pack(wt, bits, group, codes, sz, ld_codes=K * bits // 32, sz_row_stride=1, sz_group_stride=R)
    codes = codes.cpu().numpy().view(np.uint32).reshape(R, -1)
    sz = sz.cpu().numpy().view(np.uint32).reshape(K // group, R).T
    if bits == 16:
        bf = mi.bf16_bits(w).astype(np.uint32)
        assert np.array_equal(codes, bf[:, 0::2] | (bf[:, 1::2] << 16)) and np.all(sz == 0x3C00)
        return
    s, q, s16, z16 = orc.quantize(w, bits, group)
    assert s == 0
    assert np.array_equal(codes, orc.pack(q, bits))
    assert np.array_equal(sz, orc.sz_words(s16, z16))


def _periodic_pack_matches(R, K, bits, rows=None):
    """Packs R weight rows of 64 columns repeated along K (and, with `rows`,
    listed over and over) and compares every word with the small matrix's."""
    import paper_2503_21135_amd as P
    group = 64
    small = torch.randn(R, group, device=dev()) * 0.02
    words = group * bits // 32
    c1 = torch.zeros(R, words, dtype=torch.int32, device=dev())
    s1 = torch.zeros(R, dtype=torch.int32, device=dev())
    P.moe_quant_pack(small, bits, group, c1, s1)
    w = small.repeat(1, K // group)
    n = R if rows is None else rows.numel()
    codes = torch.zeros(n, K * bits // 32, dtype=torch.int32, device=dev())
    sz = torch.zeros(n, K // group, dtype=torch.int32, device=dev())
    P.moe_quant_pack(w, bits, group, codes, sz, rows=rows)
    step = 1 << 24    # rows of a comparison
    for i in range(0, n, step):
        r = torch.arange(R, device=dev()) if rows is None else rows[i:i + step].long()
        assert torch.equal(codes[i:i + step].view(len(r), -1, words), c1[r][:, None].expand(-1, K // group, -1))
        assert torch.equal(sz[i:i + step], s1[r][:, None].expand(-1, K // group))


def test_pack_row_wider_than_a_grid_dimension():
    # more column tiles of 2048 than a grid's second dimension holds (65535)
    _periodic_pack_matches(2, 2048 * 65536 + 64, 2)


def test_pack_row_list_longer_than_a_grid():
    # narrow rows, 16 of them per workgroup: more than 2^32 threads
    n = (1 << 28) + 1000
    rows = torch.arange(n, dtype=torch.int32, device=dev()).remainder_(7)
    _periodic_pack_matches(7, 64, 2, rows)

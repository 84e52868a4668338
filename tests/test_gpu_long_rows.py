"""Attention over rows of more key blocks than one tile of the score epilogue holds (16 or 32 per wavefront): dense
attention, score maps and lists on sampled rows of 133 query blocks, for every head_dim and block.
Bars as in test_gpu_short_rows."""
import numpy as np
import pytest

from tests.test_gpu_short_rows import _check_out

pytestmark = pytest.mark.gpu

# ends of the epilogue's tiles (every 16 to 32 blocks, every 64 and 128 of a workgroup) and of the rows' strands
ROWS = [0, 1, 15, 16, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 132]


@pytest.mark.parametrize("d,B", [(128, 128), (128, 64), (64, 128), (64, 64)])
def test_long_rows_dense_and_lists(d, B):
    import torch
    import oracle
    import paper_2505_19578_amd as sp
    from synth import random_qkv, bf16_bits_to_f32
    from tests.gpu_util import to_dev
    nqb = 133
    bits = random_qkv(97, nqb * B, 4, 2, d, 1.5)
    q, k, v = (to_dev(x) for x in bits)
    hq, hk, hv = (bf16_bits_to_f32(x) for x in bits)
    shape = sp.shape_of(q, k, None, B)
    ws = torch.empty(sp.sp_workspace_bytes(shape, 2), dtype=torch.uint8, device="cuda")
    heads, rows = [3, 1], np.asarray(ROWS, dtype=np.int32)
    at = np.concatenate([np.arange(i * B, (i + 1) * B) for i in rows])
    o = torch.zeros_like(q)
    sc = torch.full((1, 2, nqb, nqb), -1.0, dtype=torch.float32, device="cuda")
    sp.sp_dense_attn_with_block_scores(shape, q, k, v, heads, o, sc, ws)
    torch.cuda.synchronize()
    og, sg = o.float().cpu().numpy()[0], sc.cpu().numpy()[0]
    assert np.all(np.triu(sg[0], 1) == 0) and np.all(np.abs(sg.sum(-1) - 1) <= 1e-3)
    for n, h in enumerate(heads):
        ref, s_ref, _ = oracle.dense_rows(hq[:, h], hk[:, h // 2], hv[:, h // 2], B, rows)
        _check_out(og[at, h], ref, hv[:, h // 2], (d, B, h))
        assert np.abs(sg[n][rows] - s_ref).max() <= 1e-3
    rng = np.random.default_rng(d + B)
    idx, cnt = np.full((2, nqb, nqb), -1, np.int32), np.zeros((2, nqb), np.int32)
    for m in range(2):
        for i in range(nqb):
            sel = np.flatnonzero(rng.random(i + 1) < (0.2, 0.9)[m])
            sel = np.union1d(sel, [i]) if i % 3 else sel
            idx[m, i, :len(sel)], cnt[m, i] = sel, len(sel)
    o = torch.zeros_like(q)
    sp.sp_block_sparse_attn(shape, q, k, v, heads, [1, 0], torch.from_numpy(idx).cuda().unsqueeze(0),
                            torch.from_numpy(cnt).cuda().unsqueeze(0), 2, o, ws)
    torch.cuda.synchronize()
    og = o.float().cpu().numpy()[0]
    for m, h in ((1, 3), (0, 1)):
        ref = oracle.masked_rows(hq[:, h], hk[:, h // 2], hv[:, h // 2], B, idx[m][rows], cnt[m][rows], rows)
        _check_out(og[at, h], ref, hv[:, h // 2], (d, B, m, h))


@pytest.mark.parametrize("d,B", [(128, 128), (128, 64), (64, 128), (64, 64)])
def test_lists_longer_than_a_chunk(d, B):
    """The kernel holds 64 entries of a list at a time: lengths around the multiples of 64, the diagonal block as the last
    entry or absent."""
    import torch
    import oracle
    import paper_2505_19578_amd as sp
    from synth import random_qkv, bf16_bits_to_f32
    from tests.gpu_util import to_dev
    nqb, lengths = 261, [62, 63, 64, 65, 66, 70, 71, 127, 128, 129, 130, 191, 192, 193, 255, 256, 257, 258]
    rows = np.asarray([nqb - 1 - x for x in range(len(lengths))], dtype=np.int32)[::-1].copy()
    rows[:7] = [64, 65, 66, 70, 71, 72, 73]  # short lists in short rows
    bits = random_qkv(101, nqb * B, 2, 1, d, 1.5)
    q, k, v = (to_dev(x) for x in bits)
    hq, hk, hv = (bf16_bits_to_f32(x) for x in bits)
    shape = sp.shape_of(q, k, None, B)
    ws = torch.empty(sp.sp_workspace_bytes(shape, 0), dtype=torch.uint8, device="cuda")
    at = np.concatenate([np.arange(i * B, (i + 1) * B) for i in rows])
    rng = np.random.default_rng(d * B)
    idx, cnt = np.full((2, nqb, nqb), -1, np.int32), np.ones((2, nqb), np.int32)
    idx[:, :, 0] = 0
    for i, n in zip(rows, lengths):
        n = min(n, int(i) + 1)
        with_diag = np.union1d(rng.choice(i, size=n - 1, replace=False), [i])
        without = np.sort(rng.choice(i, size=min(n, i), replace=False))
        for m, sel in enumerate((with_diag, without)):
            idx[m, i, :len(sel)], cnt[m, i] = sel, len(sel)
    o = torch.zeros_like(q)
    sp.sp_block_sparse_attn(shape, q, k, v, [0, 1], [0, 1], torch.from_numpy(idx).cuda().unsqueeze(0),
                            torch.from_numpy(cnt).cuda().unsqueeze(0), 2, o, ws)
    torch.cuda.synchronize()
    og = o.float().cpu().numpy()[0]
    for h in (0, 1):
        ref = oracle.masked_rows(hq[:, h], hk[:, 0], hv[:, 0], B, idx[h][rows], cnt[h][rows], rows)
        _check_out(og[at, h], ref, hv[:, 0], (d, B, h))

"""Attention over rows of few key blocks (lists of every length from none, with and without the diagonal) and the
chunked vertical-slash search, at the sizes where their loops leave remainders: rows of less than a step, an odd number
of sub-tiles, a last chunk of one key block, a single chunk per head.
Bars: every output within its rounding bound.  Weights and outputs are rounded to bf16 (relative error 2^-9 each), sums
are fp32: the numerator is off by at most 2^-9 max|V|, the normaliser by 2^-9, i.e. by 2^-9 |O| <= 2^-9 max|V| of the
output, the stored output by 2^-9 |O| (these peaked inputs have outputs above 4, where one bf16 half step is 0.0156
already); mean error 2e-3 and score maps 1e-3 as in the other parity tests; search sums as in test_gpu_vertical_slash."""
import numpy as np
import pytest

from tests.test_gpu_vertical_slash import _check_lists, _search, _sum_check

pytestmark = pytest.mark.gpu

OUT_MEAN = 2e-3


def _check_out(got, want, v, what):
    err = np.abs(got.astype(np.float64) - want)
    bound = 2.0 ** -9 * np.abs(want) + 2.0 ** -8 * np.abs(v).max() + 1e-4  # 1e-4: fp32 sums and the exponential
    assert np.all(err <= bound) and err.mean() <= OUT_MEAN, (what, float((err / bound).max()), float(err.mean()))


# odd and even numbers of query blocks: 7 is one row per strand but the last, 8 one each, 9 and 11 leave strands short
@pytest.mark.parametrize("d,B", [(128, 128), (128, 64), (64, 128), (64, 64)])
@pytest.mark.parametrize("nqb", [7, 8, 9, 11])
def test_short_rows_dense_and_lists(d, B, nqb):
    import torch
    import oracle
    import paper_2505_19578_amd as sp
    from synth import random_qkv, bf16_bits_to_f32
    from tests.gpu_util import to_dev
    N = nqb * B
    bits = random_qkv(83, N, 4, 2, d, 2.0)
    q, k, v = (to_dev(x) for x in bits)
    hq, hk, hv = (bf16_bits_to_f32(x) for x in bits)
    shape = sp.shape_of(q, k, None, B)
    ws = torch.empty(sp.sp_workspace_bytes(shape, 4), dtype=torch.uint8, device="cuda")
    heads = [2, 1]
    o = torch.full_like(q, 7.0)
    sc = torch.full((1, 2, nqb, nqb), -1.0, dtype=torch.float32, device="cuda")
    sp.sp_dense_attn_with_block_scores(shape, q, k, v, heads, o, sc, ws)
    torch.cuda.synchronize()
    og, sg = o.float().cpu().numpy()[0], sc.cpu().numpy()[0]
    assert np.all(og[:, [0, 3]] == 7.0)
    for n, h in enumerate(heads):
        ref, s_ref, _ = oracle.dense_rows(hq[:, h], hk[:, h // 2], hv[:, h // 2], B)
        _check_out(og[:, h], ref, hv[:, h // 2], (d, B, nqb, h))
        assert np.abs(sg[n] - s_ref).max() <= 1e-3
    # list lengths 0 .. i + 1 in turn, with and without the diagonal block
    rng = np.random.default_rng(d + B + nqb)
    idx, cnt = np.full((2, nqb, nqb), -1, np.int32), np.zeros((2, nqb), np.int32)
    for m in range(2):
        for i in range(nqb):
            n = min(i + 1, (i + m) % 6) if i < nqb - 1 else i + 1 - m
            sel = np.sort(rng.choice(i + 1, size=n, replace=False))
            idx[m, i, :n], cnt[m, i] = sel, n
    o = torch.full_like(q, 7.0)
    sp.sp_block_sparse_attn(shape, q, k, v, [3, 0], [0, 1], torch.from_numpy(idx).cuda().unsqueeze(0),
                            torch.from_numpy(cnt).cuda().unsqueeze(0), 2, o, ws)
    torch.cuda.synchronize()
    og = o.float().cpu().numpy()[0]
    for m, h in ((0, 3), (1, 0)):
        ref = oracle.masked_rows(hq[:, h], hk[:, h // 2], hv[:, h // 2], B, idx[m], cnt[m])
        _check_out(og[:, h], ref, hv[:, h // 2], (d, B, nqb, h))


# key blocks: one alone; 64 chunks of one; 33 chunks of two and one of one; (block 128) 34 chunks of two
@pytest.mark.parametrize("d,B,nkb", [(64, 64, 1), (64, 64, 64), (128, 64, 67), (128, 128, 1), (64, 128, 68)])
def test_search_chunks(d, B, nkb):
    import oracle
    import paper_2505_19578_amd as sp
    from synth import random_qkv, bf16_bits_to_f32
    from tests.gpu_util import to_dev
    qb, kb, _ = random_qkv(87, nkb * B, 4, 2, d, 2.5)
    q, k = to_dev(qb), to_dev(kb)
    hq, hk = bf16_bits_to_f32(qb), bf16_bits_to_f32(kb)
    heads = [1, 2]
    _, sums_h, idx, cnt = _search(sp, q, k, B, heads, 0.8, True)
    for n, h in enumerate(heads):
        a_v, a_s = oracle.vertical_slash_sums(hq[:, h], hk[:, h // 2], B)
        _sum_check(sums_h[n, 0], a_v, f"head {h} a_v")
        _sum_check(sums_h[n, 1], a_s, f"head {h} a_s")
    _check_lists(oracle, sums_h, idx.cpu().numpy()[0], cnt.cpu().numpy()[0], B, 0.8, True, f"nkb {nkb}")


# vectors of 16384 entries are selected in one launch, longer ones over several; ties: all keys alike
@pytest.mark.parametrize("B,nkb", [(128, 128), (64, 256), (64, 257)])
@pytest.mark.parametrize("alike", [False, True])
def test_vector_selection_at_the_edge_of_the_single_launch(B, nkb, alike):
    import oracle
    import paper_2505_19578_amd as sp
    from synth import random_qkv
    from tests.gpu_util import to_dev
    qb, kb, _ = random_qkv(89, nkb * B, 2, 1, 64, 2.5)
    if alike:
        kb[1:] = kb[:1]
    _, sums_h, idx, cnt = _search(sp, to_dev(qb), to_dev(kb), B, [0, 1], 0.6, False)
    _check_lists(oracle, sums_h, idx.cpu().numpy()[0], cnt.cpu().numpy()[0], B, 0.6, False, f"nkb {nkb}")

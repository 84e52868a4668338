"""What a head gives does not depend on what else is in the call: its output, score map and search sums are the same
bits whether it is listed alone, beside fifteen others or in a batch of two (a row has one order of tiles and sums)."""
import pytest

pytestmark = pytest.mark.gpu

HQ, HK = 16, 4


def _inputs(seed, N, d, batch=2):
    import torch
    from synth import random_qkv
    from tests.gpu_util import to_dev
    q, k, v = zip(*[[to_dev(x) for x in random_qkv(seed + b, N, HQ, HK, d, 2.0)] for b in range(batch)])
    return torch.cat(q), torch.cat(k), torch.cat(v)


# the launches of the two calls differ 16-fold: 2 x 16 heads of 4096 tokens fill the chip, 2 heads leave it idle
@pytest.mark.parametrize("d,B,nqb", [(128, 128, 32), (64, 128, 32), (128, 64, 64), (64, 64, 64)])
def test_attention_of_a_head_alone_and_among_others(d, B, nqb):
    import torch
    import paper_2505_19578_amd as sp
    q, k, v = _inputs(31, nqb * B, d)
    g = torch.Generator().manual_seed(7)
    keep = torch.rand((2, 2, nqb, nqb), generator=g) < 0.4
    keep |= torch.eye(nqb, dtype=torch.bool)
    keep &= torch.ones(nqb, nqb, dtype=torch.bool).tril()
    key = torch.where(keep, torch.arange(nqb), nqb).sort(dim=-1).values
    idx, cnt = torch.where(key < nqb, key, -1).int().cuda(), keep.sum(-1, dtype=torch.int32).cuda()

    def run(q, k, v, heads, idx, cnt):
        shape, b, n = sp.shape_of(q, k, None, B), q.shape[0], len(heads)
        ws = torch.empty(sp.sp_workspace_bytes(shape, n), dtype=torch.uint8, device="cuda")
        o, ol = torch.zeros_like(q), torch.zeros_like(q)
        sc = torch.full((b, n, nqb, nqb), -1.0, dtype=torch.float32, device="cuda")
        sp.sp_dense_attn_with_block_scores(shape, q, k, v, heads, o, sc, ws)
        sp.sp_block_sparse_attn(shape, q, k, v, heads, [h % 2 for h in heads], idx, cnt, 2, ol, ws)
        torch.cuda.synchronize()
        return o[:, :, heads], sc, ol[:, :, heads]

    everything = run(q, k, v, list(range(HQ)), idx, cnt)
    few = [3, 8]
    for b in range(2):
        alone = run(q[b:b + 1], k[b:b + 1], v[b:b + 1], few, idx[b:b + 1].contiguous(), cnt[b:b + 1].contiguous())
        for what, a, e in zip(("dense output", "score map", "output over lists"), alone, everything):
            e = e[b:b + 1, few] if what == "score map" else e[b:b + 1][:, :, few]
            assert torch.equal(a, e), f"{what}, batch entry {b}: {int((a != e).sum())} of {a.numel()} differ"


@pytest.mark.parametrize("d", [64, 128])
def test_weights_are_rounded_at_the_same_points_for_both_block_sizes(d):
    """Dense attention of one input under blocks of 64 and of 128: the running reference moves once per 64 keys under
    both, so the weights are the same bf16 numbers and O's sums the same bits; only the general steps near the diagonal
    (one block of them) add weights to the second normaliser sum that the fast steps leave out, each below 1/32 of its
    row: outputs close to a rounding step of bf16 may fall on the other side."""
    import torch
    import paper_2505_19578_amd as sp
    q, k, v = _inputs(37, 2048, d, batch=1)
    out = []
    for B in (64, 128):
        shape = sp.shape_of(q, k, None, B)
        nqb = 2048 // B
        ws = torch.empty(sp.sp_workspace_bytes(shape, HQ), dtype=torch.uint8, device="cuda")
        o, sc = torch.zeros_like(q), torch.empty((1, HQ, nqb, nqb), dtype=torch.float32, device="cuda")
        sp.sp_dense_attn_with_block_scores(shape, q, k, v, list(range(HQ)), o, sc, ws)
        out.append(o)
    torch.cuda.synchronize()
    differ = float((out[0] != out[1]).float().mean())
    print(f"[block sizes] d {d}: {differ:.5f} of the outputs differ", flush=True)
    assert differ <= 1e-3


# 65 key blocks and more: the keys are dealt to fewer, longer chunks the more heads a call lists
@pytest.mark.parametrize("d,B,nkb", [(128, 128, 67), (64, 64, 130), (64, 128, 64), (128, 64, 257)])
def test_search_of_a_head_alone_and_among_others(d, B, nkb):
    import torch
    import paper_2505_19578_amd as sp
    q, k, _ = _inputs(41, nkb * B, d)

    def run(q, k, heads):
        shape, b, n = sp.shape_of(q, k, None, B), q.shape[0], len(heads)
        ws = torch.empty(sp.sp_vs_workspace_bytes(shape, n), dtype=torch.uint8, device="cuda")
        sums = torch.full((b, n, 2, nkb * B), -1.0, dtype=torch.float32, device="cuda")
        idx = torch.full((b, n, nkb, nkb), -5, dtype=torch.int32, device="cuda")
        cnt = torch.full((b, n, nkb), -5, dtype=torch.int32, device="cuda")
        sp.sp_search_vertical_slash(shape, q, k, heads, 0.9, True, sums, idx, cnt, ws)
        torch.cuda.synchronize()
        return sums, idx, cnt

    everything = run(q, k, list(range(HQ)))
    for b in range(2):
        for h in (0, 11):
            alone = run(q[b:b + 1], k[b:b + 1], [h])
            for what, a, e in zip(("sums", "lists", "counts"), alone, everything):
                e = e[b:b + 1, h:h + 1]
                assert torch.equal(a, e), f"{what}, head {h}, batch entry {b}: {int((a != e).sum())} of {a.numel()} differ"


@pytest.mark.parametrize("nqb", [65, 66, 67])
@pytest.mark.parametrize("scores", [True, False])
def test_dense_rows_two_to_a_workgroup_and_alone(nqb, scores):
    """d 64, blocks of 64: 2 x 16 heads have their rows walked two to a workgroup (the first workgroup of an odd number has
    one row), a single head one to a workgroup."""
    import torch
    import paper_2505_19578_amd as sp
    q, k, v = _inputs(41, nqb * 64, 64)

    def run(q, k, v, heads):
        shape = sp.shape_of(q, k, None, 64)
        ws = torch.empty(sp.sp_workspace_bytes(shape, len(heads)), dtype=torch.uint8, device="cuda")
        o = torch.zeros_like(q)
        sc = torch.full((q.shape[0], len(heads), nqb, nqb), -1.0, dtype=torch.float32, device="cuda") if scores else None
        sp.sp_dense_attn_with_block_scores(shape, q, k, v, heads, o, sc, ws)
        torch.cuda.synchronize()
        return o[:, :, heads], sc

    o_all, s_all = run(q, k, v, list(range(HQ)))
    for b, h in ((0, 2), (1, 15)):
        o, s = run(q[b:b + 1], k[b:b + 1], v[b:b + 1], [h])
        assert torch.equal(o[0, :, 0], o_all[b, :, h])
        assert s is None or torch.equal(s[0, 0], s_all[b, h])


# The rows of up to 16 batch entries are dispatched in one order (17: one entry after the other); head counts on both sides of
# a multiple of 8; d 64 with blocks of 128: launches with two and with three wavefronts per SIMD (from 1024 rows on, over lists of
# several entries above 1024)
@pytest.mark.parametrize("d,B,nqb,batch,heads", [(128, 128, 9, 3, 5), (64, 64, 17, 16, 3), (64, 64, 17, 17, 3), (128, 64, 7, 2, 16),
                                                 (64, 128, 11, 16, 1), (64, 128, 32, 2, 16), (64, 128, 33, 2, 16), (64, 64, 43, 3, 16)])
def test_a_batch_entry_alone_and_among_others(d, B, nqb, batch, heads):
    import torch
    import paper_2505_19578_amd as sp
    q, k, v = _inputs(47, nqb * B, d, batch)
    g = torch.Generator().manual_seed(11)
    keep = torch.rand((batch, 1, nqb, nqb), generator=g) < 0.5
    keep |= torch.eye(nqb, dtype=torch.bool)
    keep &= torch.ones(nqb, nqb, dtype=torch.bool).tril()
    key = torch.where(keep, torch.arange(nqb), nqb).sort(dim=-1).values
    idx, cnt = torch.where(key < nqb, key, -1).int().cuda(), keep.sum(-1, dtype=torch.int32).cuda()
    listed = [(5 * h + 2) % HQ for h in range(heads)]

    def run(q, k, v, idx, cnt):
        shape = sp.shape_of(q, k, None, B)
        ws = torch.empty(sp.sp_workspace_bytes(shape, heads), dtype=torch.uint8, device="cuda")
        o, ol = torch.full_like(q, 7.0), torch.full_like(q, 7.0)
        sc = torch.full((q.shape[0], heads, nqb, nqb), -1.0, dtype=torch.float32, device="cuda")
        sp.sp_dense_attn_with_block_scores(shape, q, k, v, listed, o, sc, ws)
        sp.sp_block_sparse_attn(shape, q, k, v, listed, [0] * heads, idx, cnt, 1, ol, ws)
        torch.cuda.synchronize()
        return o, sc, ol

    print(f"[batch] d{d} B{B} {nqb} blocks, {batch} x {heads} heads", flush=True)
    everything = run(q, k, v, idx, cnt)
    for b in range(batch):
        alone = run(q[b:b + 1], k[b:b + 1], v[b:b + 1], idx[b:b + 1].contiguous(), cnt[b:b + 1].contiguous())
        for what, a, e in zip(("dense output", "score map", "output over lists"), alone, everything):
            assert torch.equal(a[0], e[b]), f"{what}, batch entry {b}: {int((a[0] != e[b]).sum())} of {a.numel()} differ"


@pytest.mark.parametrize("d,B,nqb,batch", [(128, 128, 8, 4), (64, 64, 21, 4), (128, 64, 9, 16), (64, 128, 5, 17)])
def test_a_batch_entry_of_a_gated_layer_alone_and_among_others(d, B, nqb, batch):
    """Entries whose heads all attend alike (every head shares), entries whose estimates are one-hot (no head passes the sparsity
    test: all but the pivots fall back) and ordinary ones: the device's lists of heads have other lengths for every entry,
    none among them."""
    import torch
    import paper_2505_19578_amd as sp
    q, k, v = _inputs(53, nqb * B, d, batch)
    for b in range(batch):
        if b % 4 in (1, 2):
            q[b] = 0  # uniform attention
        if b % 4 == 2:
            k[b, :B] = 0
            k[b, :B, :, 0] = 8.0
            q[b, :, :, 0] = 8.0  # all on the first block
    clusters, pivots = [h // 4 for h in range(HQ)], [0, 4, 8, 12]

    def run(q, k, v):
        shape, b = sp.shape_of(q, k, None, B), q.shape[0]
        ws = torch.empty(sp.sp_workspace_bytes(shape, 4), dtype=torch.uint8, device="cuda")
        o = torch.full_like(q, 7.0)
        idx = torch.empty((b, 4, nqb, nqb), dtype=torch.int32, device="cuda")
        cnt = torch.empty((b, 4, nqb), dtype=torch.int32, device="cuda")
        a_hat = torch.empty((b, HQ, nqb), dtype=torch.float32, device="cuda")
        dist = torch.empty((b, HQ, 2), dtype=torch.float32, device="cuda")
        role = torch.full((b, HQ), -9, dtype=torch.int32, device="cuda")
        sp.sp_prefill_layer_gated(shape, q, k, v, clusters, pivots, 0.9, 0.3, 0.2, sp.SP_SCORE_BLOCK_MASS, sp.SP_SELECT_PER_ROW,
                                  o, None, idx, cnt, a_hat, dist, role, ws)
        torch.cuda.synchronize()
        return o, idx, cnt, dist, role

    print(f"[batch] gated d{d} B{B} {nqb} blocks, batch {batch}", flush=True)
    everything = run(q, k, v)
    fallback = (everything[4] == -1).sum(1).tolist()
    assert 0 in fallback and max(fallback) >= 12, fallback
    for b in range(batch):
        for what, a, e in zip(("output", "lists", "counts", "distances", "roles"), run(q[b:b + 1], k[b:b + 1], v[b:b + 1]), everything):
            assert torch.equal(a[0], e[b]), f"{what}, batch entry {b}"

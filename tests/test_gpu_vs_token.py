"""GPU parity for attention over the token-level vertical-slash pattern (Alg. 5's mask under Sec. 5.1's
A(Q,K,V,M)): sp_vertical_slash_attn and the token-level fallback of sp_prefill_layer_dict against the CPU oracle.

The kept keys / offsets the call reports must be, bit for bit, the oracle's selection fed the GPU's own sums (the
sums themselves are held to the search test's bar there); outputs: max-abs 2e-2 / mean-abs 2e-3 against the
oracle's token-level attention run with the GPU's kept sets; the reported pair count is exact."""
import numpy as np
import pytest

from tests.test_gpu_parity import OUT_MAX, OUT_MEAN, _LazyHost

pytestmark = pytest.mark.gpu
KT = 64  # keys of a tile


def _bits_to_keep(words, N):
    return np.unpackbits(np.ascontiguousarray(words).view(np.uint8), bitorder="little")[:N].astype(np.uint8)


def _run(sp, q, k, v, B, heads, gamma, forced):
    import torch
    shape = sp.shape_of(q, k, None, B)
    N, n = q.shape[1], len(heads)
    ws = torch.empty(sp.sp_vs_token_workspace_bytes(shape, n), dtype=torch.uint8, device="cuda")
    o = torch.zeros_like(q)
    bits = torch.zeros((1, n, 2, N // 64), dtype=torch.int64, device="cuda")
    pairs = torch.full((1, n), -1, dtype=torch.int64, device="cuda")
    sp.sp_vertical_slash_attn(shape, q, k, v, heads, gamma, forced, o, bits, pairs, ws)
    torch.cuda.synchronize()
    return shape, o, bits.cpu().numpy()[0].view(np.uint64), pairs.cpu().numpy()[0]


def _check_kept_sets(oracle, sp, shape, q, k, heads, gamma, bits):
    """The kept keys and offsets are the oracle's selection over the search's own sums (the same bits run to run)."""
    import torch
    B, N, n = shape.block, shape.seq, len(heads)
    ws = torch.empty(sp.sp_vs_workspace_bytes(shape, n), dtype=torch.uint8, device="cuda")
    sums = torch.empty((1, n, 2, N), dtype=torch.float32, device="cuda")
    idx = torch.empty((1, n, N // B, N // B), dtype=torch.int32, device="cuda")
    cnt = torch.empty((1, n, N // B), dtype=torch.int32, device="cuda")
    sp.sp_search_vertical_slash(shape, q, k, heads, gamma, True, sums, idx, cnt, ws)
    torch.cuda.synchronize()
    sums_h = sums.cpu().numpy()[0]
    for a, h in enumerate(heads):
        for x, what in enumerate(("keys", "offsets")):
            want, _ = oracle.select_cumulative(sums_h[a, x], gamma)
            got = _bits_to_keep(bits[a, x], N)
            assert np.array_equal(got, want), f"head {h}: {int((got != want).sum())} {what} differ"


def _pair_count(keep_v, keep_s, B, forced):
    N = len(keep_v)
    total = 0
    cs = np.concatenate([[0], np.cumsum(keep_s.astype(np.int64))])
    for t in range(N):
        s = np.arange(t + 1)
        allow = keep_v[:t + 1].astype(bool) | keep_s[t - s].astype(bool)
        if forced:
            allow |= (s // B == 0) | (s // B == t // B)
        total += int(allow.sum())
    return total


@pytest.mark.parametrize("d,B,N,forced,gamma", [(128, 128, 1024, True, 0.5), (128, 128, 1024, False, 0.5),
                                                (128, 64, 576, True, 0.5), (64, 128, 768, True, 0.5),
                                                (64, 64, 448, False, 0.5),
                                                # nearly everything kept (every tile a band with a mask), and nearly
                                                # nothing
                                                (128, 128, 1536, True, 0.98), (64, 64, 640, False, 0.98),
                                                (128, 128, 1024, False, 0.02), (128, 64, 576, True, 0.02)])
def test_token_attention_random_inputs(d, B, N, forced, gamma):
    import torch
    import oracle
    import paper_2505_19578_amd as sp
    from synth import random_qkv, bf16_bits_to_f32
    from tests.gpu_util import to_dev, err_stats
    qb, kb, _ = random_qkv(71, N, 4, 2, d, 2.0)
    _, _, vb = random_qkv(72, N, 4, 2, d, 1.0)     # |V| < 8: output rounding alone stays under the absolute bar
    q, k, v = to_dev(qb), to_dev(kb), to_dev(vb)
    hq, hk, hv = (bf16_bits_to_f32(x) for x in (qb, kb, vb))
    heads = [0, 3, 2]
    print(f"[vs token] d{d} B{B} N{N} forced {forced} gamma {gamma}", flush=True)
    shape, o, bits, pairs = _run(sp, q, k, v, B, heads, gamma, forced)
    # the search's own sums on the same inputs (bit-identical run to run): what the kept sets must follow from
    ws = torch.empty(sp.sp_vs_workspace_bytes(shape, len(heads)), dtype=torch.uint8, device="cuda")
    sums = torch.empty((1, len(heads), 2, N), dtype=torch.float32, device="cuda")
    nkb = N // B
    idx = torch.empty((1, len(heads), nkb, nkb), dtype=torch.int32, device="cuda")
    cnt = torch.empty((1, len(heads), nkb), dtype=torch.int32, device="cuda")
    sp.sp_search_vertical_slash(shape, q, k, heads, gamma, forced, sums, idx, cnt, ws)
    torch.cuda.synchronize()
    sums_h = sums.cpu().numpy()[0]
    o_h = o.float().cpu().numpy()[0]
    for n, h in enumerate(heads):
        keep_v, keep_s = _bits_to_keep(bits[n, 0], N), _bits_to_keep(bits[n, 1], N)
        kv_o, _ = oracle.select_cumulative(sums_h[n, 0], gamma)
        ks_o, _ = oracle.select_cumulative(sums_h[n, 1], gamma)
        assert np.array_equal(keep_v, kv_o) and np.array_equal(keep_s, ks_o), f"head {h}: kept sets differ"
        assert 0 < keep_v.sum() < N and 0 < keep_s.sum() < N
        ref = oracle.vs_token_rows(hq[:, h], hk[:, h // 2], hv[:, h // 2], B, keep_v, keep_s, forced)
        emax, emean = err_stats(o_h[:, h], ref)
        assert emax <= OUT_MAX and emean <= OUT_MEAN, f"head {h}: {emax} / {emean}"
        assert int(pairs[n]) == _pair_count(keep_v, keep_s, B, forced), f"head {h}: pair count"
    assert np.all(o_h[:, 1] == 0)          # a head that was not listed is not written


def test_token_attention_structured_2k_and_dictionary_fallback():
    """The structured workload at 2K: the stand-alone call on every head, then one dictionary layer in which every
    head falls back (delta = 0) to the token-level pattern: same bits as the stand-alone call."""
    import torch
    import oracle
    import paper_2505_19578_amd as sp
    from synth import CONFIGS, make_layer
    from tests.gpu_util import to_dev, err_stats
    L = make_layer(CONFIGS["llama8b_32k"], seq=2048)
    cfg = L["cfg"]
    B, Hq, G, N = cfg.block, cfg.n_q_heads, cfg.group, cfg.seq
    q, k, v = (to_dev(L[x]) for x in "qkv")
    host = _LazyHost(L)
    heads = list(range(Hq))
    shape, o, bits, pairs = _run(sp, q, k, v, B, heads, cfg.gamma, True)
    o_h = o.float().cpu().numpy()[0]
    dens = []
    for h in [0, 5, 14, 31]:
        keep_v, keep_s = _bits_to_keep(bits[h, 0], N), _bits_to_keep(bits[h, 1], N)
        ref = oracle.vs_token_rows(host.head("q", h), host.head("k", h // G), host.head("v", h // G), B, keep_v, keep_s, True)
        emax, emean = err_stats(o_h[:, h], ref)
        assert emax <= OUT_MAX and emean <= OUT_MEAN, f"head {h}: {emax} / {emean}"
        dens.append(pairs[h] / (N * (N + 1) / 2))
    print(f"[vs token] llama8b@2k kept-pair fraction of sampled heads: {np.round(dens, 3)}", flush=True)
    nqb = N // B
    C = cfg.n_clusters
    valid = torch.zeros((1, C), dtype=torch.int32, device="cuda")
    a_t = torch.zeros((1, C, nqb), dtype=torch.float32, device="cuda")
    didx = torch.full((1, C, nqb, nqb), -9, dtype=torch.int32, device="cuda")
    dcnt = torch.full((1, C, nqb), -9, dtype=torch.int32, device="cuda")
    pd = sp.pattern_dict_of(valid, a_t, didx, dcnt)
    ws = torch.empty(sp.sp_workspace_bytes(shape, C) + sp.sp_vs_token_workspace_bytes(shape, Hq), dtype=torch.uint8, device="cuda")
    sc = torch.empty((1, C, nqb, nqb), dtype=torch.float32, device="cuda")
    role = torch.full((1, Hq), -7, dtype=torch.int32, device="cuda")
    a_hat = torch.empty((1, Hq, nqb), dtype=torch.float32, device="cuda")
    dist = torch.empty((1, Hq, 2), dtype=torch.float32, device="cuda")
    o2 = torch.zeros_like(q)
    sp.sp_prefill_layer_dict(shape, q, k, v, [int(c) for c in L["head_to_cluster"]], cfg.gamma, 0.0, 0.2, 0, 0, pd, o2,
                             sc, role, a_hat, dist, ws, fallback_mode=sp.SP_FALLBACK_VERTICAL_SLASH_TOKEN)
    torch.cuda.synchronize()
    assert np.all(role.cpu().numpy() == -1)
    assert torch.equal(o2.view(torch.int16), o.view(torch.int16))


def test_token_attention_llama8b_128k_sampled_rows():
    """Full size: two heads, outputs on sampled query-block rows, kept-pair fraction next to the block superset's."""
    import torch
    import oracle
    import paper_2505_19578_amd as sp
    from synth import CONFIGS, make_layer
    from tests.gpu_util import to_dev, err_stats
    from tests.test_gpu_full_size import _sample_rows
    L = make_layer(CONFIGS["llama8b_128k"])
    cfg = L["cfg"]
    B, G, N = cfg.block, cfg.group, cfg.seq
    q, k, v = (to_dev(L[x]) for x in "qkv")
    host = _LazyHost(L)
    heads = [1, 22]
    shape, o, bits, pairs = _run(sp, q, k, v, B, heads, cfg.gamma, True)
    o_h = o.float().cpu().numpy()[0]
    _check_kept_sets(oracle, sp, shape, q, k, heads, cfg.gamma, bits)
    rows = _sample_rows(cfg.nqb, 77, extra=1)
    sel_t = np.concatenate([np.arange(i * B, (i + 1) * B) for i in rows])
    for n, h in enumerate(heads):
        keep_v, keep_s = _bits_to_keep(bits[n, 0], N), _bits_to_keep(bits[n, 1], N)
        ref = oracle.vs_token_rows(host.head("q", h), host.head("k", h // G), host.head("v", h // G), B, keep_v, keep_s,
                                   True, rows=rows)
        emax, emean = err_stats(o_h[sel_t, h], ref)
        assert emax <= OUT_MAX and emean <= OUT_MEAN, f"head {h}: {emax} / {emean}"
        idx_b, cnt_b = oracle.vs_block_lists(keep_v, keep_s, B, True)
        frac_tok = pairs[n] / (N * (N + 1) / 2)
        frac_blk = cnt_b.sum() / (cfg.nqb * (cfg.nqb + 1) / 2)
        print(f"[vs token] cfg3 head {h}: kept keys {int(keep_v.sum())}, kept offsets {int(keep_s.sum())}, "
              f"pairs {frac_tok:.4f} of causal, block superset {frac_blk:.4f} of causal blocks", flush=True)
        assert frac_tok <= frac_blk + 1e-9


# vectors of 16384 entries are selected in one launch, longer ones over several; ties: all keys alike
@pytest.mark.parametrize("B,nkb", [(128, 128), (64, 256), (64, 257), (128, 129)])
@pytest.mark.parametrize("alike", [False, True])
def test_kept_sets_at_the_edge_of_the_single_launch(B, nkb, alike):
    import oracle
    import paper_2505_19578_amd as sp
    from synth import random_qkv
    from tests.gpu_util import to_dev
    qb, kb, vb = random_qkv(93, nkb * B, 2, 1, 64, 2.0)
    if alike:
        kb[1:] = kb[:1]
    q, k, v = to_dev(qb), to_dev(kb), to_dev(vb)
    for gamma in (0.3, 0.9):
        shape, _, bits, _ = _run(sp, q, k, v, B, [0, 1], gamma, True)
        _check_kept_sets(oracle, sp, shape, q, k, [0, 1], gamma, bits)


@pytest.mark.parametrize("token_level", [True, False])
def test_dictionary_fallback_above_16k_tokens(token_level):
    """A dictionary layer of 129 key blocks whose heads take every role: the selection's launches over long vectors
    skip the heads that do not fall back, and those that do give the bits of a stand-alone call on them."""
    import torch
    import paper_2505_19578_amd as sp
    from synth import CONFIGS, make_layer
    from tests.gpu_util import to_dev
    from tests.test_gpu_dict import _Dict
    L = make_layer(CONFIGS["llama8b_128k_regime"], seq=16512)
    cfg = L["cfg"]
    B, Hq, C, nqb = cfg.block, cfg.n_q_heads, cfg.n_clusters, cfg.seq // cfg.block
    q, k, v = (to_dev(L[x]) for x in "qkv")
    shape = sp.shape_of(q, k, None, B)
    D = _Dict(sp, 1, C, nqb)
    ws = torch.empty(sp.sp_workspace_bytes(shape, C) + max(sp.sp_vs_workspace_bytes(shape, Hq),
                                                             sp.sp_vs_token_workspace_bytes(shape, Hq)),
                     dtype=torch.uint8, device="cuda")
    o, sc = torch.zeros_like(q), torch.empty((1, C, nqb, nqb), dtype=torch.float32, device="cuda")
    role = torch.full((1, Hq), -7, dtype=torch.int32, device="cuda")
    a_hat = torch.empty((1, Hq, nqb), dtype=torch.float32, device="cuda")
    dist = torch.empty((1, Hq, 2), dtype=torch.float32, device="cuda")
    vi = torch.full((1, Hq, nqb, nqb), -3, dtype=torch.int32, device="cuda")
    vc = torch.full((1, Hq, nqb), -3, dtype=torch.int32, device="cuda")
    mode = sp.SP_FALLBACK_VERTICAL_SLASH_TOKEN if token_level else sp.SP_FALLBACK_VERTICAL_SLASH
    sp.sp_prefill_layer_dict(shape, q, k, v, [int(x) for x in L["head_to_cluster"]], cfg.gamma, 0.3, 0.2, 0, 0, D.c, o, sc,
                             role, a_hat, dist, ws, fallback_mode=mode, **({} if token_level else dict(vs_idx=vi, vs_cnt=vc)))
    torch.cuda.synchronize()
    role_h = role.cpu().numpy()[0]
    fb = [h for h in range(Hq) if role_h[h] == -1]
    assert fb and (role_h == -2).any() and (role_h >= 0).any()
    print(f"[vs token] {cfg.seq} tokens: {len(fb)} of {Hq} heads fall back", flush=True)
    if token_level:
        _, alone, _, _ = _run(sp, q, k, v, B, fb, cfg.gamma, True)
    else:
        n = len(fb)
        wv = torch.empty(max(sp.sp_vs_workspace_bytes(shape, n), sp.sp_workspace_bytes(shape, 0)), dtype=torch.uint8,
                         device="cuda")
        idx = torch.empty((1, n, nqb, nqb), dtype=torch.int32, device="cuda")
        cnt = torch.empty((1, n, nqb), dtype=torch.int32, device="cuda")
        sp.sp_search_vertical_slash(shape, q, k, fb, cfg.gamma, True, None, idx, cnt, wv)
        alone = torch.zeros_like(q)
        sp.sp_block_sparse_attn(shape, q, k, v, fb, list(range(n)), idx, cnt, n, alone, wv)
        torch.cuda.synchronize()
        assert torch.equal(vi[:, fb], idx) and torch.equal(vc[:, fb], cnt)
    assert torch.equal(o[:, :, fb].view(torch.int16), alone[:, :, fb].view(torch.int16))


def test_token_attention_rows_in_two_launches():
    """A length at which the items of all rows do not fit their room (more than 32 block^2 tokens): rows on both sides of
    the cut, and at the ends, against the oracle with the kept sets that the call reports."""
    import torch
    import oracle
    import paper_2505_19578_amd as sp
    from synth import random_qkv, bf16_bits_to_f32
    from tests.gpu_util import to_dev, err_stats
    d, B, nqb = 64, 64, 3000
    N = nqb * B
    qb, kb, _ = random_qkv(75, N, 1, 1, d, 2.0)
    _, _, vb = random_qkv(76, N, 1, 1, d, 1.0)
    q, k, v = to_dev(qb), to_dev(kb), to_dev(vb)
    print(f"[vs token] d{d} B{B} N{N}", flush=True)
    _, o, bits, _ = _run(sp, q, k, v, B, [0], 0.9, True)
    keep_v, keep_s = _bits_to_keep(bits[0, 0], N), _bits_to_keep(bits[0, 1], N)
    # the first launch takes the last rows, as many as fit: 16 bytes an item, i + 1 items for row i
    room = (4 * N * B) // 16
    cut = next(r for r in range(nqb) if nqb * (nqb + 1) // 2 - r * (r + 1) // 2 <= room)
    assert 1000 < cut < 2000
    rows = np.asarray([0, 1, 500, cut - 3, cut - 2, cut - 1, cut, cut + 1, cut + 2, 2500, nqb - 1], dtype=np.int32)
    at = np.concatenate([np.arange(i * B, (i + 1) * B) for i in rows])
    hq, hk, hv = (bf16_bits_to_f32(x)[:, 0] for x in (qb, kb, vb))
    ref = oracle.vs_token_rows(hq, hk, hv, B, keep_v, keep_s, True, rows)
    emax, emean = err_stats(o.float().cpu().numpy()[0, at, 0], ref)
    assert emax <= OUT_MAX and emean <= OUT_MEAN, (emax, emean)


@pytest.mark.parametrize("d,B", [(128, 128), (128, 64), (64, 128), (64, 64)])
def test_weight_that_rules_a_row_is_not_rounded(d, B):
    """One kept key has about half of every row's weight, the sink block's keys, which a row meets first, have the rest, each
    a factor 30 to 110 below it.  Dimension x has 1 at the one key and -g_x at the others, so outputs near 0 show their
    weights' rounding: of the one key's weight s (1 - s) (1 + g) 2^-9 at most, 5e-4 to 1e-3 rms over the queries, if it is
    rounded; of B independent others sqrt(sum r^2) g 2^-9, 1e-4 to 2e-4 rms with the output's own rounding, if it is exactly 1."""
    import torch
    import paper_2505_19578_amd as sp
    rng = np.random.default_rng([d, B])
    nqb, one = 6, 2 * B + 5
    N = nqb * B
    bf16 = lambda x: torch.from_numpy(np.asarray(x, np.float32)).to(torch.bfloat16)
    f64 = lambda x: x.to(torch.float64).numpy()
    alpha = bf16(rng.uniform(7, 8, N) * np.sqrt(d) / 8)
    beta = bf16(np.where(np.arange(N) < B, rng.uniform(6, 7, N), -8.0))
    x = f64(alpha)[:, None] * f64(beta)[None, :B] / np.sqrt(d)
    beta[one] = bf16((np.log(np.exp(x).sum(1)) / (f64(alpha) / np.sqrt(d))).mean())
    lead = (f64(alpha) * f64(beta)[one] / np.sqrt(d) - x.max(1)) / np.log(2)
    assert 4.0 < lead.min() and lead.max() < 7.5
    g = np.exp(np.linspace(np.log(0.25), np.log(4), d))
    q, k, v = (torch.zeros((1, N, 1, d), dtype=torch.bfloat16) for _ in range(3))
    q[0, :, 0, 0], k[0, :, 0, 0] = alpha, beta
    v[0, :B, 0], v[0, one, 0] = -bf16(g), 1.0
    print(f"[vs token] one heavy key, d{d} B{B}", flush=True)
    _, o, bits, _ = _run(sp, q.cuda(), k.cuda(), v.cuda(), B, [0], 0.9, True)
    keep_v, keep_s = _bits_to_keep(bits[0, 0], N).astype(bool), _bits_to_keep(bits[0, 1], N).astype(bool)
    assert keep_v[one]
    t, s = np.arange(3 * B, N)[:, None], np.arange(N)[None, :]
    allow = (s <= t) & (keep_v[s] | keep_s[np.maximum(t - s, 0)] | (s // B == 0) | (s // B == t // B))
    w = np.where(allow, np.exp(f64(alpha)[t] * f64(beta)[s] / np.sqrt(d)), 0.0)
    ref = (w / w.sum(1, keepdims=True)) @ f64(v[0, :, 0])
    near_0 = np.abs(ref) < 0.05
    assert near_0.sum() > 4 * B
    err = np.sqrt(np.mean((f64(o[0, 3 * B:, 0].cpu()) - ref)[near_0] ** 2))
    print(f"[vs token] rms error of the outputs near 0: {err:.2e}", flush=True)
    assert err <= 3.5e-4


def _row_items(keep_v, keep_s, B, forced):
    """The items of every row, as the kernel's rule makes them: [rows] x (gathered images that lie in no band, bands of which
    every offset is kept, gathered images with a mask, bands with a mask, whether all tiles are walked as bands)."""
    N, spb = len(keep_v), B // KT
    kept = np.cumsum(np.concatenate([[0], keep_s]))
    lo, hi = KT * np.arange(N // KT) - KT + 1, KT * np.arange(N // KT) + B - 1  # the offsets of a tile x below the row's first
    n = kept[np.minimum(hi, N - 1) + 1] - kept[np.maximum(lo, 0)]
    band, full = n > 0, n == B + KT - 1
    keys = np.flatnonzero(keep_v)
    keys = keys[keys >= (B if forced else 0)]
    rows = []
    for i in range(N // B):
        first, below = i * spb, i * spb - (spb if forced and i > 0 else 0)
        nb, nf = int(band[1:below + 1].sum()), int((band & full)[1:below + 1].sum())
        images = np.array_split(keys[keys < i * B], np.arange(KT, max(1, (keys < i * B).sum()), KT))
        left = [int((~band[first - x // KT]).sum()) for x in images]
        gf, gp = sum(x == KT for x in left), sum(0 < x < KT for x in left)
        if nb + gf + gp > below:
            rows.append((0, int((band & full)[1:below + 1].sum()), 0, below - int((band & full)[1:below + 1].sum()), 1))
        else:
            rows.append((gf, nf, gp, nb - nf, 0))
    return np.asarray(rows)


def _weights_by_choice(rng, d, B, N, keys, offsets, share):
    """q, k of which each query of the last block has `share` of its weight on `keys`, alike, the rest on the keys `offsets`
    below it, alike; the other queries' weights are random, on few keys each."""
    h = d // 2
    q, k = rng.normal(size=(N, d)) * 4, rng.normal(size=(N, d))
    k[:, :h] = 0
    code = rng.normal(size=(B, h - 1))
    code /= np.linalg.norm(code, axis=1, keepdims=True)
    for o in offsets:
        k[N - B - o:N - o, 1:h] = 4 * code
    k[keys, 1:h] = 0
    k[keys, 0] = (20 + np.log(share / (1 - share) * max(1, len(offsets)) / len(keys))) / 5 if len(offsets) else 4
    q[N - B:] = 0
    q[N - B:, 1:h] = code * 5 * np.sqrt(d)
    q[N - B:, 0] = 5 * np.sqrt(d)
    return q, k


@pytest.mark.parametrize("d,B", [(128, 128), (128, 64), (64, 128), (64, 64)])
@pytest.mark.parametrize("forced", [True, False])
@pytest.mark.parametrize("kind", ["runs", "all_tiles"])
def test_token_attention_every_kind_of_item(d, B, forced, kind):
    """runs: one run of kept keys and one of kept offsets, which give runs of items without masks of both kinds (the unmasked
    steps) beside ones with masks.  all_tiles: 20 keys of every tile, single offsets 2 to 4 tiles apart and a run of both, so that
    rows have more items than tiles and walk all of their tiles as bands, some without masks."""
    import torch
    import oracle
    import paper_2505_19578_amd as sp
    from tests.gpu_util import err_stats
    rng = np.random.default_rng([d, B])
    if kind == "runs":
        N = 24 * B
        keys, offsets, share, gamma = np.arange(N // 4, N // 4 + N // 3), [], 1.0, 0.9
    else:
        tiles, run, gaps = (24, 6 * B, [2, 3]) if B == 64 else (32, 4 * B, [4])
        N = tiles * KT
        keys = (KT * np.arange(tiles)[:, None] + 3 * np.arange(20) + 3).ravel()
        keys = np.union1d(keys[keys < N - B], np.arange(N - B - run, N - B))
        offsets, x = [], B // KT + 1 + run // KT
        while KT * x + 33 < N - B:
            offsets.append(KT * x + 33)
            x += gaps[(len(offsets) - 1) % len(gaps)]
        share = (len(keys) + 0.0) / (2 * len(keys) - run)  # as much on the single keys as on the single offsets
        gamma = share - 0.05
    bf16 = lambda x: torch.from_numpy(np.asarray(x, np.float32)).to(torch.bfloat16)
    q, k = (bf16(x) for x in _weights_by_choice(rng, d, B, N, keys, offsets, share))
    v = bf16(rng.normal(size=(N, d)))
    print(f"[vs token] {kind} d{d} B{B} N{N} forced {forced}", flush=True)
    q4, k4, v4 = (x[None, :, None].contiguous().cuda() for x in (q, k, v))
    shape, o, bits, pairs = _run(sp, q4, k4, v4, B, [0], gamma, forced)
    _check_kept_sets(oracle, sp, shape, q4, k4, [0], gamma, bits)
    keep_v, keep_s = _bits_to_keep(bits[0, 0], N), _bits_to_keep(bits[0, 1], N)
    items = _row_items(keep_v, keep_s, B, forced)
    print(f"[vs token] rows with each kind of item: {(items > 0).sum(0)} of {N // B}", flush=True)
    if kind == "runs":  # (U > 2: the unmasked steps are taken)
        assert (items[:, :4] > 0).any(0).all() and (items[:, :2].sum(1) > 2).any()
    else:
        assert items[:, 4].sum() > 2 and (items[items[:, 4] > 0, 1] > 0).any()
    f32 = lambda x: x.float().numpy()
    ref = oracle.vs_token_rows(f32(q), f32(k), f32(v), B, keep_v, keep_s, forced)
    emax, emean = err_stats(o.float().cpu().numpy()[0, :, 0], ref)
    assert emax <= OUT_MAX and emean <= OUT_MEAN, (emax, emean)
    assert int(pairs[0]) == _pair_count(keep_v, keep_s, B, forced)


# (a) rows in two launches, more than one head and batch entry: every head's items start at their own place; (b) more than 3
# groups of 8 chunks (384 rows) of heads of 8 KV heads, and more than 6 (768) of heads of 5, which run head by head; (c) fewer of
# them, more heads than XCDs
@pytest.mark.parametrize("B,nqb,batch,Hq,Hkv", [(64, 2050, 2, 4, 2), (128, 385, 1, 16, 8), (64, 770, 1, 10, 5), (64, 390, 1, 10, 5),
                                                (128, 385, 1, 9, 3), (64, 383, 2, 9, 9)])
def test_a_heads_rows_do_not_depend_on_the_other_heads(B, nqb, batch, Hq, Hkv):
    import torch
    import oracle
    import paper_2505_19578_amd as sp
    from synth import random_qkv, bf16_bits_to_f32
    from tests.gpu_util import to_dev, err_stats
    d, N = 64, nqb * B
    parts = [random_qkv(180 + b, N, Hq, Hkv, d, 2.0) for b in range(batch)]
    q, k, v = (torch.cat([to_dev(p[x]) for p in parts]) for x in range(3))
    print(f"[vs token] B{B} N{N} batch {batch} heads {Hq}/{Hkv}", flush=True)
    shape = sp.shape_of(q, k, None, B)
    ws = torch.empty(sp.sp_vs_token_workspace_bytes(shape, Hq), dtype=torch.uint8, device="cuda")
    o = torch.zeros_like(q)
    pairs = torch.full((batch, Hq), -1, dtype=torch.int64, device="cuda")
    sp.sp_vertical_slash_attn(shape, q, k, v, list(range(Hq)), 0.9, True, o, None, pairs, ws)
    torch.cuda.synchronize()
    for b in range(batch):
        for h in range(Hq):
            _, alone, bits, n = _run(sp, q[b:b + 1], k[b:b + 1], v[b:b + 1], B, [h], 0.9, True)
            assert torch.equal(o[b, :, h].view(torch.int16), alone[0, :, h].view(torch.int16)), (b, h)
            assert int(pairs[b, h]) == int(n[0]), (b, h)
    # the last one is held to the oracle on a few rows: the first and last, and the border (rows 77, 78) of (a)'s launches
    rows = np.asarray([0, 1, 40, 77, 78, 79, nqb - 1], dtype=np.int32)
    at = np.concatenate([np.arange(i * B, (i + 1) * B) for i in rows])
    hq, hk, hv = (bf16_bits_to_f32(parts[-1][x])[:, -1] for x in range(3))
    ref = oracle.vs_token_rows(hq, hk, hv, B, _bits_to_keep(bits[0, 0], N), _bits_to_keep(bits[0, 1], N), True, rows)
    emax, emean = err_stats(o[-1, at, Hq - 1].float().cpu().numpy(), ref)
    assert emax <= OUT_MAX and emean <= OUT_MEAN, (emax, emean)

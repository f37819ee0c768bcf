"""Kernel variants at the sizes where their dispatch or tiling changes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _T():
    import paper_2502_12216_amd as T
    return T


def _keys(h, n, kind, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if kind == "ties":  # small integers: many exactly equal distances
        K = torch.zeros(h, n, 128, device="cuda")
        K[..., :4] = torch.randint(-1, 2, (h, n, 4), generator=g, device="cuda").float()
    elif kind == "zeros":  # half of the keys are zero: one cluster of thousands of keys
        K = torch.randn(h, n, 128, generator=g, device="cuda")
        K[torch.rand(h, n, generator=g, device="cuda") < 0.5] = 0.0
    else:
        c = torch.randn(h, max(1, n // 16), 128, generator=g, device="cuda")
        lab = torch.randint(0, c.shape[1], (h, n), generator=g, device="cuda")
        K = torch.stack([c[i][lab[i]] for i in range(h)]) + 0.3 * torch.randn(h, n, 128, generator=g, device="cuda")
    return K.to(torch.bfloat16).contiguous()


@pytest.mark.parametrize("warm", [False, True])
@pytest.mark.parametrize("kind", ["mixture", "ties", "zeros"])
@pytest.mark.parametrize("lens,ncl", [([300], [18]), ([2049, 255, 256], [129, 16, 16]), ([5000, 600], [4, 97]),
                                      ([9000], [1]), ([20011], [1250]), ([33001, 17000], [3, 40])])
def test_kmeans_later_iterations_equal_full_steps(lens, ncl, kind, warm):
    """A later iteration measures only pairs whose centroid changed (from the third
    on, from the second of a warm start, which begins from the centroids of
    other keys, so that most of them move); a call of one iteration measures
    every pair.  Chained through the warm start, t such calls must give bit
    for bit what one call of t iterations gives (member lists in LDS, of more
    than 64 members, and in memory, there also of more than 256 among more
    than 16384 tokens)."""
    T = _T()
    h = 2
    K, V = _keys(h, sum(lens), kind, 1), _keys(h, sum(lens), "mixture", 2)
    rng = np.random.default_rng(3)
    init = torch.as_tensor(np.concatenate([np.stack([rng.choice(n, c, replace=False) for _ in range(h)])
                                           for n, c in zip(lens, ncl)], 1).astype(np.int32), device="cuda")
    batch = T.RaggedBatch(lens, h, h)
    one = T.ClusterBuilder(batch, ncl, max_iters=1)
    start = _cluster_set(V[:, :sum(ncl)].contiguous(), ncl) if warm else None
    prev = start
    for t in range(1, 7):
        step = one(K, V, init, prev=prev)
        many = T.ClusterBuilder(batch, ncl, max_iters=t)
        many.workspace.fill_(0xA5)  # contents on entry are irrelevant
        got = many(K, V, init, prev=start)
        for name, x, y in (("assign", got.assign, step.assign), ("offsets", got.clusters.offsets, step.clusters.offsets),
                           ("perm", got.perm, step.perm),
                           ("centroids", got.clusters.centroids.view(torch.int16), step.clusters.centroids.view(torch.int16)),
                           ("K_sorted", got.K_sorted.view(torch.int16), step.K_sorted.view(torch.int16))):
            assert torch.equal(x, y), f"{name} after {t} iterations"
        prev = step.clusters


def _check_one_step(K, init):
    """The layout is the stable order of the assignment, bit for bit, and every mean is that of the
    cluster's keys, summed in four interleaved chains (a bound of the fp32 sums: members / 4 + 2 additions, each
    2^-24 of the sum of magnitudes, then a factor and a rounding to bf16, 2^-8 with a margin of 2^-20)."""
    T = _T()
    n, C = K.shape[1], init.shape[1]
    r = T.ClusterBuilder(T.RaggedBatch([n], 1, 1), [C], max_iters=1)(K, K, init)
    a = r.assign[0].long()
    assert torch.equal(r.perm[0].long(), torch.sort(a, stable=True).indices)
    cnt = torch.bincount(a, minlength=C)
    assert torch.equal(r.clusters.offsets[0].long()[1:], torch.cumsum(cnt, 0))
    assert torch.equal(r.K_sorted[0], K[0][r.perm[0].long()])
    s = torch.zeros(C, 128, dtype=torch.float64, device="cuda").index_add_(0, a, K[0].double())
    m = torch.zeros(C, 128, dtype=torch.float64, device="cuda").index_add_(0, a, K[0].double().abs())
    full = cnt > 0
    c = cnt[full, None].double()
    mean, err = s[full] / c, m[full] / c * (c / 4 + 3) * 2.0 ** -24
    got = r.clusters.centroids[0][full].double()
    assert torch.all((got - mean).abs() <= err + (mean.abs() + err) * (2.0 ** -8 + 2.0 ** -20))
    assert torch.equal(r.clusters.centroids[0][~full], K[0][init[0].long()][~full])
    return cnt


@pytest.mark.parametrize("C", [1, 2, 3, 64, 65, 100])
def test_kmeans_sizes_at_the_limits_of_the_sums(C):
    """Clusters of given sizes around the limits of a wave (64), of lists in memory (256) and of a slice's keys in
    LDS (4096 together), in every slice; numbers of clusters at and beside powers of two."""
    sizes = np.resize([5000, 64, 257, 1, 65, 256, 63, 1500, 4096, 300, 2, 255, 700], C)
    g = torch.Generator(device="cuda")
    g.manual_seed(C)
    lab = torch.repeat_interleave(torch.arange(C, device="cuda"), torch.as_tensor(sizes, device="cuda"))
    lab = lab[torch.randperm(len(lab), generator=g, device="cuda")]
    centre = torch.randn(C, 128, generator=g, device="cuda")
    K = (centre[lab] + 0.05 * torch.randn(len(lab), 128, generator=g, device="cuda")).to(torch.bfloat16)[None]
    first = torch.as_tensor([int((lab == c).nonzero()[0]) for c in range(C)], dtype=torch.int32, device="cuda")
    assert np.array_equal(_check_one_step(K, first[None]).cpu().numpy(), sizes)


@pytest.mark.parametrize("n,C", [(700, 3), (5001, 300), (20011, 4), (20011, 200), (70000, 2), (270001, 5)])
@pytest.mark.parametrize("kind", ["mixture", "zeros"])
def test_kmeans_one_step_layout_and_means(n, C, kind):
    rng = np.random.default_rng(n)
    init = torch.as_tensor(rng.choice(n, C, replace=False).astype(np.int32)[None], device="cuda")
    _check_one_step(_keys(1, n, kind, n + C), init)


def _cluster_set(cen, ncl):
    off = torch.zeros(cen.shape[0], sum(ncl) + len(ncl), dtype=torch.int32, device="cuda")
    return _T().ClusterSet(cen, off, ncl)


def test_kmeans_equal_scores_of_zero():
    """A key whose own, unmoved centroid scores exactly 0 and a centroid of smaller id that moved and scores 0 too
    goes to the smaller id (two dimensions, the rest zero, every value exact in bf16).  From c0 = (1, -1.5) and
    c1 = (1, 1) the first step assigns (1, 0), (1, 2), (1, -1) to 1, 1, 0; c0 moves to (1, -1), c1 stays; then
    (1, 0) scores 1 - (1 + 1) / 2 = 0 with both."""
    T = _T()

    def rows(x):
        t = torch.zeros(1, len(x), 128, device="cuda")
        t[0, :, :2] = torch.tensor(x, device="cuda")
        return t.to(torch.bfloat16)

    K = rows([[1.0, 0.0], [1.0, 2.0], [1.0, -1.0]])
    prev = _cluster_set(rows([[1.0, -1.5], [1.0, 1.0]]), [2])
    init = torch.zeros(1, 2, dtype=torch.int32, device="cuda")
    got = T.ClusterBuilder(T.RaggedBatch([3], 1, 1), [2], max_iters=10)(K, K, init, prev=prev)
    assert got.assign.tolist() == [[0, 1, 0]]
    assert torch.equal(got.clusters.centroids, rows([[1.0, -0.5], [1.0, 2.0]]))
    assert got.perm.tolist() == [[0, 2, 1]] and got.clusters.offsets.tolist() == [[0, 2, 3]]


def _decode(lens, ncl, hq, hkv, seed, sizes=None, union=1, target=0.9, tail=None, change=None):
    """A sparse decode over random keys with the given cluster sizes (default: random, some empty), `tail` recent
    tokens per sequence behind the clusters; change(q, centroids) edits them in place."""
    T = _T()
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rng = np.random.default_rng(seed)
    total = sum(lens)
    K = torch.randn(hkv, total, 128, generator=g, device="cuda").to(torch.bfloat16)
    V = torch.randn(hkv, total, 128, generator=g, device="cuda").to(torch.bfloat16)
    cen = torch.randn(hkv, sum(ncl), 128, generator=g, device="cuda").to(torch.bfloat16)
    off = []
    tail = tail or [0] * len(lens)
    for n, c in zip([n - t for n, t in zip(lens, tail)], ncl):
        if c == 0:
            off.append(np.zeros((hkv, 1), np.int64))
            continue
        cuts = np.sort(rng.integers(0, n + 1, size=(hkv, c - 1)), axis=1) if sizes is None else \
            np.tile(np.cumsum(sizes)[:-1], (hkv, 1))
        off.append(np.concatenate([np.zeros((hkv, 1), np.int64), cuts, np.full((hkv, 1), n)], 1))
    offs = np.concatenate(off, 1).astype(np.int32)
    batch = T.RaggedBatch(lens, hq, hkv)
    dec = T.SparseDecoder(batch, ncl, T.decode_params(target, use_union=union, max_tail=max(tail)))
    q = (0.3 * torch.randn(len(lens), hq, 128, generator=g, device="cuda")).to(torch.bfloat16)
    if change:
        change(q, cen)
    out, sq, skv = dec(q, K, V, T.ClusterSet(cen, torch.as_tensor(offs, device="cuda"), ncl))
    torch.cuda.synchronize()
    return dict(q=q, K=K, V=V, off=off, out=out, tail=tail, sq=sq.cpu().numpy(), skv=skv.cpu().numpy(),
                view={k: v.cpu().numpy() for k, v in dec.view().items()}, batch=batch)


def _positions(n):
    """Sampled positions (1-based) of a list of n tokens, default parameters."""
    N = min(n, max(1, -(-n // 100)))
    W = max(8, -(-n * 50 // 10000))
    s1 = max((n * 1000 + 5000) // 10000 - W // 2, N + 1)
    s2 = max((n * 6000 + 5000) // 10000 - W // 2, N + 1)
    t1, t2 = min(s1 + W - 1, n), min(s2 + W - 1, n)
    if N == n or s1 > t1 or s2 > t2 or t1 >= s2:
        return np.arange(1, n + 1)
    return np.concatenate([np.arange(1, N + 1), np.arange(s1, t1 + 1), np.arange(s2, t2 + 1)])


def _check_selection(r, lens, ncl, hq, hkv, union=1):
    G = hq // hkv
    v, c0 = r["view"], 0
    for b, (n, C) in enumerate(zip(lens, ncl)):
        if C == 0:
            assert not np.any(r["sq"][b]) and not torch.any(r["out"][b])
            continue
        lengths = np.zeros((hq, C), np.int64)
        for h in range(hq):
            off = r["off"][b][h // G]
            size = np.diff(off)
            order = np.lexsort((np.arange(C), -v["scores"][b, h, :C]))
            assert np.array_equal(v["order"][b, h, :C], order), (b, h)
            pre = np.concatenate([[0], np.cumsum(size[order])])
            assert np.array_equal(v["rank_prefix"][b, h, :C + 1], pre), (b, h)
            nc, tail = n - r["tail"][b], r["tail"][b]
            pos = _positions(nc)
            rank = np.searchsorted(pre, pos, side="left") - 1  # the largest rank with fewer tokens ahead
            rows = off[order[rank]] + pos - 1 - pre[rank]
            rows = np.concatenate([rows, np.arange(nc, n)])  # then the recent tokens
            assert np.array_equal(v["sample_rows"][b, h, :len(rows)], rows), (b, h)
            k = int(r["sq"][b, h]) - tail
            lengths[h, order] = np.minimum(np.maximum(k - pre[:-1], 0), size[order])
        groups = [range(g * G, (g + 1) * G) for g in range(hkv)] if union else [[h] for h in range(hq)]
        for j, heads in enumerate(groups):
            want = lengths[list(heads)].max(0)
            assert np.array_equal(v["union_len"][j, c0:c0 + C], want), (b, j)
            if union:
                assert r["skv"][b, j] == want.sum() + r["tail"][b]
        c0 += C


@pytest.mark.parametrize("C", [1, 1024, 1025, 2049, 4096, 4097, 8192, 8193, 16384, 16385, 20001])
def test_sort_at_slot_edges(C):
    """Slots per thread of the LDS sort (1024, 2048, 4096, 8192 and 16384 clusters), and the pieces beyond."""
    lens, ncl = [max(1, 2 * C + 7), 33], [C, 5]
    _check_selection(_decode(lens, ncl, 4, 1, C), lens, ncl, 4, 1)


def test_sort_two_heads_per_compute_unit():
    """More than 256 heads of up to 8192 clusters: slots by each head's own count."""
    ncl = [4100, 8192, 1, 700, 1500, 3000, 4096, 5000, 1024]
    lens = [2 * c + 11 for c in ncl]
    _check_selection(_decode(lens, ncl, 32, 8, 5), lens, ncl, 32, 8)


@pytest.mark.parametrize("ncl,hq,hkv", [([9001], 4, 1), ([16384], 4, 1), ([4100, 8192, 1, 700, 1500, 3000, 4096, 5000, 1024], 32, 8),
                                        ([33000], 4, 1)])
@pytest.mark.parametrize("distinct", [1, 3, 97, 400])
def test_sort_of_repeated_scores(ncl, hq, hkv, distinct):
    """Few distinct scores: buckets of tens to thousands of clusters, equal ones by id, on the sorts with 16-bit ids
    (8193 to 16384 clusters; more than 256 heads) and in the workspace."""
    def change(q, cen):
        cen[:] = cen[:, torch.arange(cen.shape[1], device="cuda") % distinct]
    lens = [2 * c + 11 for c in ncl]
    _check_selection(_decode(lens, ncl, hq, hkv, 8, change=change), lens, ncl, hq, hkv)


@pytest.mark.parametrize("lens,ncl,hq,hkv", [
    ([70001], [32768], 64, 8),  # four workgroups per head, 8192 clusters each: two pieces
    ([41000] * 4, [20000] * 4, 32, 8),  # two per head, 10000 clusters: two pieces
    ([35003] * 8, [17000] * 8, 32, 8),  # one per head: three pieces
    ([41000, 35000, 39999], [20000, 16500, 18001], 16, 4),  # five per head
    ([50000, 6000], [20000, 3000], 8, 2),  # a short sequence among them
    ([50000, 0, 40000], [20000, 0, 16500], 8, 2)])  # an empty one
def test_sort_pieces(lens, ncl, hq, hkv):
    """16385 to 32768 clusters: a head's buckets shared by several workgroups, each taking its share in pieces of
    at most 6144 clusters."""
    _check_selection(_decode(lens, ncl, hq, hkv, 3), lens, ncl, hq, hkv)


@pytest.mark.parametrize("union", [1, 0])
def test_sort_pieces_with_recent_tokens(union):
    lens, ncl = [50000, 9000], [20000, 500]
    _check_selection(_decode(lens, ncl, 8, 2, 4, tail=[300, 120], union=union), lens, ncl, 8, 2, union)


@pytest.mark.parametrize("kind", ["equal", "bucket", "repeated"])
@pytest.mark.parametrize("hq", [4, 96])
def test_sort_pieces_fall_back(kind, hq):
    """Heads of 20000 clusters that the pieces do not take (the head's first workgroup sorts them in the workspace):
    all scores equal, or more than 6144 in a bucket; 96 heads: two workgroups each."""
    def change(q, cen):
        if kind == "equal":
            q[0, ::2] = 0.0  # beside ordinary heads
        elif kind == "bucket":
            cen[:, 500:7500] = cen[:, 500:501]
        else:
            cen[:] = cen[:, torch.arange(cen.shape[1], device="cuda") % 3]
    lens, ncl = [45000], [20000]
    _check_selection(_decode(lens, ncl, hq, hq // 4, 5, change=change), lens, ncl, hq, hq // 4)


@pytest.mark.parametrize("C,big", [(9, 1 << 19), (8193, 1 << 18), (20001, 70000)])
def test_sort_cluster_sizes_beyond_the_packed_word(C, big):
    sizes = np.ones(C, np.int64)
    sizes[C // 2] = big
    lens, ncl = [int(sizes.sum())], [C]
    _check_selection(_decode(lens, ncl, 2, 1, 9, sizes=sizes), lens, ncl, 2, 1)


def _scored(scores, hq=4):
    """A decode whose cluster scores are the given ones (a centroid is its score's bf16 pair of factors in one
    dimension): scores = (q value, centroid values [C])."""
    T = _T()
    qv, cv = scores
    C = len(cv)
    n = 2 * C
    g = torch.Generator(device="cuda")
    g.manual_seed(C)
    K = torch.randn(1, n, 128, generator=g, device="cuda").to(torch.bfloat16)
    cen = torch.zeros(1, C, 128, dtype=torch.bfloat16, device="cuda")
    cen[0, :, 5] = cv.cuda().to(torch.bfloat16)
    q = torch.zeros(1, hq, 128, dtype=torch.bfloat16, device="cuda")
    q[0, :, 5] = qv
    off = torch.arange(0, n + 1, 2, dtype=torch.int32, device="cuda")[None]
    dec = T.SparseDecoder(T.RaggedBatch([n], hq, 1), [C], T.decode_params(0.9))
    return dec, q, K, T.ClusterSet(cen, off.contiguous(), [C])


def _kinds(kind, C):
    g = torch.Generator().manual_seed(C)
    x = torch.randn(C, generator=g)
    if kind == "ordinary":
        return 1.0, x
    if kind == "tiny":  # squares of the differences underflow
        return 1e-25, x
    if kind == "denormal":
        return 1e-38, x * 0.01
    if kind == "huge":  # squares overflow, differences from the mean too
        return 1.0, torch.where(x > 0, 1.0, -1.0) * 3.2e38 * torch.rand(C, generator=g).clamp_min(0.1) * (x.abs() < 0.002)
    if kind == "infinite":
        return 1.0, torch.full((C,), float("inf"))
    return 1.0, torch.where(x > 0, float("inf"), x)  # some infinite


@pytest.mark.parametrize("C", [200, 3000, 8192, 16384, 20001, 33000])
@pytest.mark.parametrize("kind", ["tiny", "denormal", "huge", "infinite", "some infinite"])
def test_sort_of_extreme_scores(C, kind):
    dec, q, K, cl = _scored(_kinds(kind, C))
    dec(q, K, K, cl)
    v = {k: t.cpu().numpy() for k, t in dec.view().items()}
    for h in range(4):
        order = np.lexsort((np.arange(C), -v["scores"][0, h, :C]))
        assert np.array_equal(v["order"][0, h, :C], order), h


def test_sort_time_of_tiny_or_equal_infinite_scores():
    """8192 clusters whose scores' squares underflow, or which are all infinite: the buckets of the sort must not
    crowd (quadratic work: 18 to 35 times an ordinary call).  A bound of three ordinary calls."""
    def us(kind):
        dec, q, K, cl = _scored(_kinds(kind, 8192))
        best = float("inf")
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            dec(q, K, K, cl)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3)
        return best
    t = {k: us(k) for k in ("ordinary", "tiny", "infinite")}
    print({k: round(x, 1) for k, x in t.items()})
    assert t["tiny"] <= 3 * t["ordinary"] and t["infinite"] <= 3 * t["ordinary"], t


@pytest.mark.parametrize("C", [6143, 6144, 6145, 13000])
@pytest.mark.parametrize("target", [0.3, 0.97])
def test_union_of_eight_heads(C, target):
    """One workgroup up to 6144 clusters, slices beyond."""
    lens, ncl = [3 * C, 40], [C, 6]
    _check_selection(_decode(lens, ncl, 8, 1, C, target=target), lens, ncl, 8, 1)


@pytest.mark.parametrize("C,hq,union", [(49152, 8, 1), (49153, 8, 1), (65536, 4, 1), (65537, 4, 1), (65537, 2, 0)])
def test_union_beyond_the_slices(C, hq, union):
    """Eight slices hold 49152 clusters of 8 heads, 65536 of fewer; beyond, one workgroup per group takes passes
    over memory."""
    lens, ncl = [2 * C, 700], [C, 40]
    _check_selection(_decode(lens, ncl, hq, 1, 6, union=union), lens, ncl, hq, 1, union)


@pytest.mark.parametrize("n", [1, 3, 4, 63, 64, 65, 127, 255, 513, 4099])
@pytest.mark.parametrize("paged", [False, True])
def test_eight_head_attention_tile_remainders(n, paged):
    """Dense decode of 8 heads per KV head (matrix form, tiles of 64 tokens).  Bound: fp32 logits (error at
    most a few ulp of sum |q_i k_i| / sqrt(128), here below 30: 1e-5 relative in a weight)."""
    T = _T()
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    lens = [n, 70]
    K = torch.randn(2, sum(lens), 128, generator=g, device="cuda").to(torch.bfloat16)
    V = torch.randn(2, sum(lens), 128, generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn(2, 16, 128, generator=g, device="cuda").to(torch.bfloat16)
    batch = T.RaggedBatch(lens, 16, 2)
    dec = T.DenseDecoder(batch)
    out = dec.paged(q, T.PagedCache.from_token_order(K, V, batch, 16)) if paged else dec(q, K, V)
    s = 0
    for b, m in enumerate(lens):
        for h in range(16):
            k, v = K[h // 8, s:s + m].double(), V[h // 8, s:s + m].double()
            ref = torch.softmax(k @ q[b, h].double() / 128 ** 0.5, 0) @ v
            assert (out[b, h].double() - ref).abs().max() <= 1e-5 * max(1.0, float(v.abs().max()))
        s += m


@pytest.mark.parametrize("n", [5952, 5953, 8000, 8001, 11072, 11073, 16192, 16193])
@pytest.mark.parametrize("hq", [8, 32])
def test_dense_shares_at_whole_numbers_per_compute_unit(n, hq):
    """Dense decode where the split's units (tokens and 192 for each of 8 KV heads) reach one share of 192, one of
    256, 1.375 (the last to be rounded down to one) and two of 256 per compute unit, of which there are 256.  Bound as
    above."""
    T = _T()
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    K = torch.randn(8, n, 128, generator=g, device="cuda").to(torch.bfloat16)
    V = torch.randn(8, n, 128, generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn(1, hq, 128, generator=g, device="cuda").to(torch.bfloat16)
    out = T.DenseDecoder(T.RaggedBatch([n], hq, 8))(q, K, V)
    for h in range(hq):
        k, v = K[h * 8 // hq].double(), V[h * 8 // hq].double()
        ref = torch.softmax(k @ q[0, h].double() / 128 ** 0.5, 0) @ v
        assert (out[0, h].double() - ref).abs().max() <= 1e-5 * float(v.abs().max())


def test_eight_head_attention_infinite_values():
    """An infinite value reaches the heads that give its token any weight as that infinity, and a weight that is
    exactly zero times it is NaN: as with one multiplication per weight."""
    T = _T()
    n = 200
    K = torch.zeros(1, n, 128, dtype=torch.bfloat16, device="cuda")
    V = torch.ones(1, n, 128, dtype=torch.bfloat16, device="cuda")
    V[0, 17, 3] = float("inf")
    V[0, 150, 5] = float("-inf")
    K[0, 17, 0] = -100.0  # head 1 below: weight 2^-inf
    q = torch.zeros(1, 8, 128, dtype=torch.bfloat16, device="cuda")
    q[0, 1, 0] = 1000.0
    out = T.DenseDecoder(T.RaggedBatch([n], 8, 1))(q, K, V)[0].cpu()
    for h in range(8):
        assert out[h, 5] == -float("inf")
        assert torch.isnan(out[h, 3]) if h == 1 else out[h, 3] == float("inf")
        rest = torch.cat([out[h, :3], out[h, 4:5], out[h, 6:]])
        assert torch.allclose(rest, torch.ones_like(rest), atol=1e-5)

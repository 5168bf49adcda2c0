"""Kernels at the edges of their tiles and ranges, against the oracle."""
import pytest

from tests.test_gpu_attention import test_block_sparse_attention_parity as _attention_parity
from tests.test_gpu_attention import test_compensation_parity as _compensation_parity
from tests.test_gpu_cluster import test_cluster_parity as _cluster_parity

pytestmark = pytest.mark.gpu


# The eigensolver and the Cholesky factor hold d <= 64 and d <= 128 matrices in
# 4 x 4 register blocks: the smallest sizes, and one to each side of a block
# edge and of the switch between the two kernels.
@pytest.mark.parametrize("dt,d,xf", [
    ("f32", 2, "pca"), ("f32", 3, "metric"), ("f32", 5, "adaptive"),
    ("f32", 17, "metric"), ("f32", 63, "metric"), ("bf16", 65, "metric"), ("f32", 96, "pca"),
    ("f32", 127, "metric"), ("f32", 128, "adaptive"),
])
def test_transform_edges(dt, d, xf):
    _cluster_parity(dt, 900, d, 32, xf)


# fp32 attention and compensation: tiles of 16 queries and 16 keys in clusters
# smaller, larger and no multiple of them; head dimensions that leave part of a
# 16-wide tile empty; a remainder cluster; every cluster kept (nothing to
# compensate).
F32_EDGES = [
    # d, cq, ck, n, k
    (4, 1, 1, 37, 5), (20, 2, 2, 61, 9), (100, 16, 4, 203, 11), (64, 32, 8, 130, 7),
    (128, 256, 256, 700, 2), (32, 64, 128, 1000, 8), (36, 128, 32, 555, 17),
]


@pytest.mark.parametrize("d,cq,ck,n,k", F32_EDGES)
def test_f32_attention_edges(d, cq, ck, n, k):
    _attention_parity("f32", d, cq, ck, n, k)
    _compensation_parity("f32", d, cq, ck, n, k, True)


def test_f32_four_byte_alignment():
    """Dense fp32 tensors need no more than their own 4-byte alignment: the
    same bits from inputs and outputs that start one float past a 16-byte
    boundary."""
    import torch
    import paper_2608_26965_amd as ca
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    H, n, d, c, k = 2, 300, 20, 32, 4
    p = ca.Problem(1, H, n, n, d, c, c, torch.float32)

    def rnd(*shape):
        return torch.randn(*shape, device="cuda", generator=g)

    def off(x):  # a copy one float into a buffer
        b = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")
        b[1:] = x.reshape(-1)
        return b[1:].view(x.shape)

    qp, kp, vp = rnd(H, p.nq_pad, d), rnd(H, p.nk_pad, d), rnd(H, p.nkc, d, c)
    kbar, vbar = rnd(H, p.nkc, d), rnd(H, p.nkc, d)
    cnt = torch.full((H, p.nkc), c, dtype=torch.int32, device="cuda")
    cnt[:, -1] = n - (p.nkc - 1) * c
    lists = torch.stack([torch.randperm(p.nkc, device="cuda", generator=g)[:k].sort().values
                         for _ in range(H * p.nqc)]).view(H, p.nqc, k).to(torch.int32)
    perm = torch.arange(n, dtype=torch.int32, device="cuda").repeat(H, 1)
    got = []
    for f in (lambda x: x, off):
        op, lse = ca.block_sparse_attn(p, f(qp), f(kp), f(vp), cnt, lists, k)
        out, _ = ca.compensate(p, f(qp), f(kbar), f(vbar), cnt, lists, k, f(op), f(lse), perm,
                               out=f(torch.zeros(p.shape(n), device="cuda")))
        got.append((op, lse, out))
    for a, b in zip(*got):
        assert torch.equal(a, b)


# The in-workgroup levels of the split: nodes at the tail size and one token to
# each side, nodes of one wavefront's positions, clusters of one token (six
# levels, 32 sub-nodes), clusters larger than a row of 64 positions, and bf16
# coordinates as they are (runs of equal keys at every threshold).
@pytest.mark.parametrize("dt,n,d,c,xf", [
    ("bf16", 2048, 64, 64, "none"), ("bf16", 2049, 64, 32, "none"), ("bf16", 2047, 128, 16, "none"),
    ("f32", 63, 8, 1, "none"), ("f32", 65, 3, 1, "none"), ("bf16", 4097, 128, 128, "metric"),
    ("bf16", 1500, 64, 256, "pca"), ("f32", 700, 100, 2, "none"),
])
def test_split_tail_edges(dt, n, d, c, xf):
    _cluster_parity(dt, n, d, c, xf)


# Inputs that are not finite, or whose products overflow, leave no coordinate of
# the split with a variance: the results are unspecified, but every call ends and
# the orders stay orders, through levels of several workgroups and of one.
@pytest.mark.parametrize("n,d", [(700, 64), (5000, 64), (9000, 128)])
@pytest.mark.parametrize("xf", ["none", "pca", "metric", "adaptive"])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_split_of_non_finite_coordinates(dt, xf, n, d):
    import torch
    import paper_2608_26965_amd as ca
    from tests import gpu_util as G
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    q, k = (torch.randn(1, 3, n, d, device="cuda", generator=g) for _ in range(2))
    q[:, 0] = float("nan")
    q[:, 1, n // 2] = float("inf")
    k[:, 0] *= 1e30
    k[:, 1, :, 0] = float("nan")
    k[:, 2, ::3] = float("-inf")
    q, k = q.to(G.tdtype(dt)), k.to(G.tdtype(dt))
    p = ca.Problem(1, 3, n, n, d, 32, 32, G.tdtype(dt), xf)
    r = ca.cluster(p, q, k, k)
    want = torch.arange(n, dtype=torch.int32, device="cuda")
    for side in ("q", "k"):
        for h in range(3):
            assert torch.equal(r["perm_" + side][h].sort().values, want)
        assert int(r["count_" + side].sum()) == 3 * n


# Levels of several chunks (4,096 tokens each): one token into the next chunk,
# thresholds in runs of equal keys, all keys equal, and keys that one outlier
# crowds into a bin (more of them than the chunk blocks select among by themselves).
@pytest.mark.parametrize("kind", ["normal", "ties", "run", "const", "outlier"])
@pytest.mark.parametrize("n", [4097, 8191, 12289, 30000])
def test_split_chunk_edges(n, kind):
    _split_against_oracle(n, 8, 64, kind)


# Samples without spread: equal rows (some of a signed zero), rows whose squared
# differences underflow in fp32, and one coordinate that differs in one sample row.
@pytest.mark.parametrize("kind", ["const", "zeros", "tiny", "single"])
@pytest.mark.parametrize("n,d,c", [(9000, 100, 64), (9000, 64, 32), (2000, 128, 16)])
def test_split_of_flat_samples(n, d, c, kind):
    _split_against_oracle(n, d, c, kind)


# Nodes of more than 256 chunks (bins laid by the deviation at d = 3, by the
# sample's order at d = 20): histograms summed by groups of chunks, lists too long
# for the chunk blocks, short and long lists of a chunk, and runs of equal keys at
# the threshold that span chunk 256.
@pytest.mark.parametrize("d", [3, 20])
@pytest.mark.parametrize("kind", ["normal", "rest", "drift"])
def test_split_many_chunks(d, kind):
    _split_against_oracle((1 << 20) + 4096 + 5, d, 256, kind)


# Bins by the sample's order where a few sample rows are far off (to one side and
# to both), where keys lie in two clumps, and heavy tails.
@pytest.mark.parametrize("kind", ["normal", "far", "far2", "clumps", "tails"])
@pytest.mark.parametrize("n,d", [(40000, 64), (9000, 128), (300000, 17)])
def test_split_threshold_bins(n, d, kind):
    _split_against_oracle(n, d, 128, kind)


def _split_against_oracle(n, d, c, kind):
    import numpy as np
    import torch
    import paper_2608_26965_amd as ca
    from oracle import ref
    X = np.random.default_rng(n).standard_normal((2, n, d)).astype(np.float32)
    if kind == "ties":
        X = np.round(X)
    elif kind == "run":
        X[np.random.default_rng(1).random(X.shape) < 0.4] = 0.25
    elif kind == "const":
        X[:] = 0.5
    elif kind == "rest":  # the last 40% of the tokens are equal
        X[:, int(0.6 * n):] = 0.25
    elif kind == "drift":  # neighbours are close: most listed keys are in few chunks
        X += np.linspace(-20, 20, n, dtype=np.float32)[:, None]
    elif kind == "far":
        X[:, (5 * n) // (2 * d), 1] = 1e6
    elif kind == "far2":
        X[:, (5 * n) // (2 * d), 1], X[:, (9 * n) // (2 * d), 1] = -1e6, 1e4
    elif kind == "clumps":
        X = X * np.float32(0.01) + (np.random.default_rng(2).random(X.shape) < 0.5)
    elif kind == "tails":
        X = X / np.abs(np.random.default_rng(3).standard_normal(X.shape)).astype(np.float32)
    elif kind == "zeros":
        X = X * 0
    elif kind == "tiny":
        X = X * np.float32(1e-30)
    elif kind == "single":
        X[:] = 0.5
        X[:, ((2 * d - 1) * n) // (2 * d), d // 2] = 0.75
    elif kind == "outlier":
        X = X * 1e-5
        X[:, 5 * n // 16] = 1e6  # row 2 of the sample of 8
    X = X.astype(np.float32)
    p = ca.Problem(1, 1, n, n, d, c, c, torch.float32, "none")
    q, k = (torch.from_numpy(x[None, None]).cuda() for x in X)
    r = ca.cluster(p, q, k, k)
    for x, side in zip(X, ("q", "k")):
        perm, cid, _ = ref.split(x.astype(np.float64), c)
        assert np.array_equal(r["perm_" + side][0].cpu().numpy(), perm)
        assert np.array_equal(r["cid_" + side][0].cpu().numpy(), cid)


# Top-k of rows of 2049-8192 scores: at the edges of the number of groups the
# filter makes (256 to 2048, at least twice k of them), rows that leave part of
# a wavefront's range empty, and the inputs that leave its common path: ties and
# runs of equal scores at the threshold, all scores equal (but for a few
# infinite ones), infinities, fewer than k finite scores, one or two outliers
# that the others crowd under (narrower bins), long runs of the largest scores,
# close scores in a bin by the hundred (radix passes), rows of several kinds.
@pytest.mark.parametrize("nkc,k", [(2049, 64), (2049, 513), (4095, 128), (4096, 129), (4097, 1),
                                   (8192, 128), (8192, 129), (8191, 1023), (8192, 1025)])
@pytest.mark.parametrize("kind", ["normal", "ties", "halves", "const", "const_inf", "inf", "mask",
                                  "few", "outlier", "outliers", "run", "close", "mixed"])
def test_topk_filter_edges(nkc, k, kind):
    import numpy as np
    import torch
    import paper_2608_26965_amd as ca
    from oracle import ref
    rng = np.random.default_rng([nkc, k])
    S = rng.standard_normal((6, nkc)).astype(np.float32)
    if kind == "ties":
        S = np.round(2 * S)
    elif kind == "halves":
        S = np.sign(S)
    elif kind == "const":
        S[:] = 2.5
    elif kind == "const_inf":
        S[:] = 2.5
        S[:, 5::1000], S[:, 7::50] = np.inf, -np.inf
    elif kind == "mask":  # all after a position of each row's own, and a run before it
        S[np.arange(nkc) >= rng.integers(nkc // 2 + 40, nkc, (6, 1))] = -np.inf
        S[:, 64:64 + nkc // 8] = -np.inf
    elif kind == "few":
        S[:, k // 2:] = -np.inf
    elif kind == "outliers":
        S = S * 1e-5
        S[:, nkc // 2], S[:, nkc // 3], S[:, 11] = 1e20, 1, -1e30
    elif kind == "close":  # more than 64 distinct scores in a bin of the listed ones
        S = np.where(rng.random(S.shape) < 0.3, 3 + 1e-6 * S, S).astype(np.float32)
    elif kind == "mixed":
        S[1], S[3, k // 2:], S[4] = 1, -np.inf, np.round(S[4])
    elif kind == "inf":
        S[:, ::7], S[:, 3::1000] = -np.inf, np.inf
    elif kind == "outlier":
        S = S * 1e-5
        S[:, nkc // 2] = 1e20
    elif kind == "run":
        S[:, nkc // 3:nkc // 3 + min(k + 3, nkc // 2)] += 20
    p = ca.Problem(1, 1, 6 * 64, nkc * 64, 64, 64, 64, torch.float32)
    got, _ = ca.select(p, None, None, k, scores_in=torch.from_numpy(S[None]).cuda())
    assert np.array_equal(got.cpu().numpy()[0], ref.topk(S.astype(np.float64), k))


@pytest.mark.parametrize("nkc,k", [(2100, 20), (4500, 300)])
def test_topk_filter_many_rows(nkc, k):
    """More rows than the blocks that look for the filter's leftovers: some rows
    of each kind, most of them without any."""
    import numpy as np
    import torch
    import paper_2608_26965_amd as ca
    from oracle import ref
    rng = np.random.default_rng(nkc)
    S = rng.standard_normal((4301, nkc)).astype(np.float32)
    S[::7] = 1.5
    S[5:3000:11, k // 2:] = -np.inf
    S[4300] = -np.inf
    p = ca.Problem(1, 1, 4301 * 64, nkc * 64, 64, 64, 64, torch.float32)
    got, _ = ca.select(p, None, None, k, scores_in=torch.from_numpy(S[None]).cuda())
    assert np.array_equal(got.cpu().numpy()[0], ref.topk(S.astype(np.float64), k))


# bf16 compensation: from 257 query clusters of 64 on, two share a workgroup;
# heads with an odd number of clusters (the last one alone), a single one, a
# remainder, several stages of centroids, partners with different lists, and a
# tile of 128 centroids selected whole by one partner only.
@pytest.mark.parametrize("d,n,heads", [(64, 130, 86), (64, 40, 257), (128, 300, 52), (128, 64, 257),
                                       (64, 256, 65)])
def test_compensation_cluster_pairs(d, n, heads):
    import math
    import numpy as np
    import torch
    import paper_2608_26965_amd as ca
    from oracle import ref
    from tests import gpu_util as G
    from synth import bf16_round
    rng = np.random.default_rng([d, n])
    c, nk, k = 64, 64 * 389 + 5, 140
    p = ca.Problem(1, heads, n, nk, d, c, c, torch.bfloat16)
    Q = bf16_round(rng.standard_normal((2, n, d)).astype(np.float32))
    kbar, vbar = (rng.standard_normal((2, p.nkc, d)).astype(np.float32) for _ in range(2))
    perm = np.stack([rng.permutation(n) for _ in range(2)]).astype(np.int32)
    lists = G.random_lists(rng, 2, p.nqc, p.nkc, k)
    lists[:, p.nqc - 1] = np.arange(128, 128 + k)
    cq_n, ck_n = G.counts(n, c), G.counts(nk, c)
    o_s = bf16_round(rng.standard_normal((2, n, d)).astype(np.float32)).astype(np.float64)
    l_s = (rng.standard_normal((2, n)) + 9.0).astype(np.float32)  # about the log of the keys kept
    op, lse = np.zeros((2, p.nq_pad, d), np.float32), np.zeros((2, p.nq_pad), np.float32)
    for h in range(2):
        op[h, :n], lse[h, :n] = o_s[h][perm[h]], l_s[h][perm[h]]
    hs = np.arange(heads) % 2
    out, lse_out = ca.compensate(
        p, G.permuted_rows(Q, perm, c, torch.bfloat16)[hs], G.dev(kbar)[hs], G.dev(vbar)[hs],
        G.dev(np.stack([ck_n] * heads), torch.int32), G.dev(lists, torch.int32)[hs].contiguous(), k,
        G.dev(op, torch.bfloat16)[hs], G.dev(lse)[hs], G.dev(perm, torch.int32)[hs].contiguous(),
        want_lse=True)
    out, lse_out = G.host(out)[0], G.host(lse_out)
    for h in range(2):
        o_w, l_w = ref.compensate(Q[h].astype(np.float64), kbar[h], vbar[h], ck_n, perm[h], cq_n,
                                  lists[h], o_s[h], l_s[h].astype(np.float64), 1 / math.sqrt(d))
        assert np.abs(out[h] - o_w).max() <= G.TOL["bf16"]
        assert np.abs(lse_out[h] - l_w).max() <= 1e-4 * np.abs(l_w).max()
    for h in range(2, heads):
        assert np.array_equal(out[h], out[h % 2]) and np.array_equal(lse_out[h], lse_out[h % 2])


@pytest.mark.parametrize("nkc", [32768, 32769])
def test_compensation_many_key_clusters(nkc):
    """As many key clusters as two query clusters' masks hold together, and one
    more: one query cluster a workgroup, whatever their number. Checked for the
    first clusters, one in the middle and the last one."""
    import numpy as np
    import torch
    import paper_2608_26965_amd as ca
    from oracle import ref
    from tests import gpu_util as G
    from synth import bf16_round
    rng = np.random.default_rng(9)
    n, d, c, k = 64 * 256 + 22, 64, 64, 40
    Q = bf16_round(rng.standard_normal((n, d)).astype(np.float32))
    kbar, vbar = (rng.standard_normal((nkc, d)).astype(np.float32) for _ in range(2))
    p = ca.Problem(1, 1, n, nkc * c, d, c, c, torch.bfloat16)
    perm = np.arange(n, dtype=np.int32)
    lists = G.random_lists(rng, 1, p.nqc, nkc, k)
    lists[0, :, -1] = nkc - 1
    o_s = bf16_round(rng.standard_normal((n, d)).astype(np.float32))
    l_s = (rng.standard_normal(n) + 8.0).astype(np.float32)  # about the log of the keys kept
    op, lse = np.zeros((1, p.nq_pad, d), np.float32), np.zeros((1, p.nq_pad), np.float32)
    op[0, :n], lse[0, :n] = o_s, l_s
    out, lse_out = ca.compensate(
        p, G.permuted_rows(Q[None], perm[None], c, torch.bfloat16), G.dev(kbar[None]),
        G.dev(vbar[None]), torch.full((1, nkc), c, dtype=torch.int32, device="cuda"),
        G.dev(lists, torch.int32), k, G.dev(op, torch.bfloat16), G.dev(lse),
        G.dev(perm[None], torch.int32), want_lse=True)
    out, lse_out = G.host(out)[0, 0], G.host(lse_out)[0]
    for a in (0, 1, 130, p.nqc - 1):
        r = slice(a * c, min(n, (a + 1) * c))
        m = r.stop - r.start
        o_w, l_w = ref.compensate(Q[r].astype(np.float64), kbar, vbar, np.full(nkc, c, np.int32),
                                  np.arange(m), np.array([m]), lists[0, a:a + 1],
                                  o_s[r].astype(np.float64), l_s[r].astype(np.float64), 1 / 8)
        assert np.abs(out[r] - o_w).max() <= G.TOL["bf16"]
        assert np.abs(lse_out[r] - l_w).max() <= 1e-4 * np.abs(l_w).max()


def _compensate_rows(dt, d, cq, Q, kbar, vbar, lists, k, heads=1, lse=-1e4):
    """ca.compensate of heads that are all alike, on rows Q [n, d] in cluster
    order (identity permutation), centroids kbar, vbar [nkc, d] of full clusters
    of 64 keys and a sparse part of zeros with weight e^lse: (out [n, d], lse [n])
    of the last head."""
    import numpy as np
    import torch
    import paper_2608_26965_amd as ca
    from tests import gpu_util as G
    n, nkc = Q.shape[0], kbar.shape[0]
    p = ca.Problem(1, heads, n, nkc * 64, d, cq, 64, G.tdtype(dt))
    perm = np.arange(n, dtype=np.int32)[None]

    def all_heads(x):
        return x.expand(heads, *x.shape[1:]).contiguous()

    out, l = ca.compensate(
        p, all_heads(G.permuted_rows(Q[None], perm, cq, G.tdtype(dt))), all_heads(G.dev(kbar[None])),
        all_heads(G.dev(vbar[None])), torch.full((heads, nkc), 64, dtype=torch.int32, device="cuda"),
        all_heads(G.dev(lists[None], torch.int32)), k,
        torch.zeros(heads, p.nq_pad, d, dtype=G.tdtype(dt), device="cuda"),
        torch.full((heads, p.nq_pad), lse, device="cuda"), all_heads(G.dev(perm, torch.int32)),
        scale=1.0, want_lse=True)
    return G.host(out)[0, -1], G.host(l)[-1]


# The bf16 compensation at d = 64 has one softmax reference per tile of 128
# centroids (the largest logit of the tile), and probabilities rounded to bf16
# against it. The logits are a and b > a in the two halves of one tile, so the
# probabilities are bf16(e^(a - b)) and 1; against a as the reference they would
# be 1 and bf16(e^(b - a)), whose rounding moves the log-sum by over 1e-3. The
# tolerance covers logits and log-sums in fp32.
@pytest.mark.parametrize("cq,n,heads", [(64, 64, 1), (64, 64, 300), (64, 128, 150), (128, 128, 1)])
def test_compensation_tile_reference(cq, n, heads):
    import numpy as np
    from synth import bf16_round
    d, nkc = 64, 192
    step = np.float32(1.390625)  # b - a, in bf16
    Q = np.zeros((n, d), np.float32)
    Q[:, 0] = 1
    kbar = np.zeros((nkc, d), np.float32)
    kbar[64:128, 0] = step
    lists = np.tile(np.arange(128, 192), (n // cq, 1))
    _, lse = _compensate_rows("bf16", d, cq, Q, kbar, np.ones((nkc, d), np.float32), lists, 64, heads)
    up, down = (bf16_round(np.full(1, np.exp(s), np.float32))[0] for s in (step, -step))
    assert abs(up / np.exp(np.float64(step)) - 1) > 1e-3
    want = step + np.log(64.0) + np.log(64 * np.float64(down) + 64)
    assert np.abs(lse - want).max() <= 1e-5


def test_compensation_stage_of_one_partner():
    """Two query clusters share a workgroup's centroid tiles: a tile whose
    centroids one of them has all selected takes no part in that one's result,
    even where a value centroid is infinite."""
    import numpy as np
    rng = np.random.default_rng(2)
    for d in (64, 128):
        Q = rng.standard_normal((128, d)).astype(np.float32)
        kbar, vbar = (rng.standard_normal((384, d)).astype(np.float32) for _ in range(2))
        lists = np.stack([np.arange(128), np.arange(200, 328)])
        want, _ = _compensate_rows("bf16", d, 64, Q, kbar, vbar, lists, 128, 150)
        vbar[5] = np.inf
        got, _ = _compensate_rows("bf16", d, 64, Q, kbar, vbar, lists, 128, 150)
        assert np.array_equal(got[:64], want[:64])


@pytest.mark.parametrize("d", [32, 64, 128])
def test_f32_compensation_selected_infinite_value(d):
    """A selected key cluster is left out of the fp32 compensation, also where
    its value centroid is infinite."""
    import numpy as np
    rng = np.random.default_rng(3)
    Q = rng.standard_normal((40, d)).astype(np.float32)
    kbar, vbar = (rng.standard_normal((77, d)).astype(np.float32) for _ in range(2))
    lists = np.sort(rng.choice(77, (2, 9)), axis=1)
    lists[:, 0] = 3
    want, _ = _compensate_rows("f32", d, 32, Q, kbar, vbar, lists, 9)
    vbar[3] = -np.inf
    got, _ = _compensate_rows("f32", d, 32, Q, kbar, vbar, lists, 9)
    assert np.array_equal(got, want)


# fp32: the number of wavefronts of a workgroup follows the tiles of 16 keys (1,
# 2 or 4 with 4 tiles each, then 4 with two parts; 1, 2 or 4 with 2 at d = 128)
# where there are more than 256 workgroups: the last tile count of each, the next
# one, and parts of several steps, against one head alone (64 workgroups, all
# wavefronts): the same bits.
@pytest.mark.parametrize("d,tiles", [(64, t) for t in (1, 4, 5, 8, 9, 16, 17, 33, 70)] +
                         [(128, t) for t in (2, 3, 4, 5)] + [(32, 16), (32, 17), (32, 70)])
def test_f32_wavefronts_of_a_workgroup(d, tiles):
    import torch
    import paper_2608_26965_amd as ca
    g = torch.Generator(device="cuda")
    g.manual_seed(tiles)
    H, n, c, nkc = 5, 1024, 64, 16 * tiles

    def case(heads, ck, k, x):
        p = ca.Problem(1, heads, n, nkc * ck, d, c, ck, torch.float32)
        qp, kp, vp, kbar, vbar = (t[:heads] for t in x)
        cnt = torch.full((heads, nkc), ck, dtype=torch.int32, device="cuda")
        lists = torch.arange(k, dtype=torch.int32, device="cuda").repeat(heads, p.nqc, 1)
        perm = torch.arange(n, dtype=torch.int32, device="cuda").repeat(heads, 1)
        op, lse = ca.block_sparse_attn(p, qp, kp, vp, cnt, lists, k)
        out, _ = ca.compensate(p, qp, kbar, vbar, cnt, lists, k, op, lse, perm)
        return op[0], lse[0], out[0, 0]

    for ck, k in ((16, tiles), (1, tiles)):
        x = [torch.randn(H, *s, device="cuda", generator=g) for s in
             ((n, d), (nkc * ck, d), (nkc, d, ck), (nkc, d), (nkc, d))]
        for a, b in zip(case(1, ck, k, x), case(H, ck, k, x)):
            assert torch.equal(a, b)

"""Top-k_t selection of one row at the edges of its register blocks (4096, 8192
and 16384 slots), with logits that crowd the bound it selects by."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2510_13847_amd import dynahead as D  # noqa: E402

DEV = "cuda"
SIZES = [3, 17, 4096, 4097, 8192, 8193, 16384, 16385]


@pytest.fixture(scope="module")
def layout():
    of = np.repeat(np.arange(len(SIZES), dtype=np.int32), SIZES)
    of = of[np.random.default_rng(1).permutation(len(of))]
    W = torch.zeros((len(of), 8), dtype=torch.bfloat16, device=DEV)
    return D.build_layout(torch.from_numpy(of).to(DEV), W, len(SIZES))


def _logits(kind, n, rng):
    z = rng.standard_normal(n).astype(np.float32)
    if kind == "equal":  # every key reaches the bound
        z[:] = 0.25
    elif kind == "runs":  # large values side by side, then equal ones
        z[n // 3:n // 3 + 40] += 20
        z[n // 2:n // 2 + 300] = 9.0
    elif kind == "lanes":  # only every sixteenth slot is finite
        z[np.arange(n) % 16 != 5] = -np.inf
    elif kind == "special":
        z[::3], z[1::7] = np.nan, -np.inf
        z[n // 2] = np.inf
    elif kind == "lowest":
        z[:] = np.finfo(np.float32).min
    return z


@pytest.mark.parametrize("kind", ["random", "equal", "runs", "lanes", "special", "lowest"])
@pytest.mark.parametrize("k_t", [1, 2, 10, 16])
def test_top_kt(layout, kind, k_t):
    rng = np.random.default_rng(k_t)
    B = len(SIZES)
    sel, off, length, ids = D.shortlist(layout, torch.arange(B, dtype=torch.int32, device=DEV)[:, None])
    vids, cap = ids.cpu().numpy(), layout.cap(1)
    z = np.full((B, cap), np.nan, np.float32)
    for b, n in enumerate(SIZES):
        z[b, :n] = _logits(kind, n, rng)
    out = D.draft_select(layout, torch.from_numpy(z).to(DEV), sel, off, length, mode=D.SEL_TOPK, k_t=k_t)
    got, lp = out["ids"].cpu().numpy(), out["logprobs"].cpu().numpy()
    for b, n in enumerate(SIZES):
        zz = np.where(np.isnan(z[b, :n]), -np.inf, z[b, :n]).astype(np.float64)
        order = np.lexsort((vids[b, :n], -zz))[:k_t]
        assert got[b, :len(order)].tolist() == vids[b, order].tolist()
        assert (got[b, len(order):] == -1).all()
        if np.isfinite(zz.max()):
            ref = zz[order] - zz.max() - np.log(np.exp(zz - zz.max()).sum())
            fin = np.isfinite(ref)
            # fp32: the exponentials' sum over at most 16385 terms in blocks of 16, and one logarithm
            assert np.abs(lp[b, :len(order)][fin] - ref[fin]).max() <= 1e-5 * max(1.0, np.abs(ref[fin]).max())


# one context, one launch: shortlists to both sides of 4096 slots (the blocks
# in which workgroup 0 reads the logits), of 6144 and of 8192 (the key lists
# beyond, for small k_t and for all), and long ones, with random rows and with
# equal ones
@pytest.mark.parametrize("n", [1, 15, 4096, 4097, 6144, 6145, 8192, 8193, 16384, 16385])
@pytest.mark.parametrize("equal", [False, True])
@pytest.mark.parametrize("k_t", [2, 10, 16])
def test_one_launch_top_kt(n, equal, k_t):
    d, V, M = 64, 20000, 3
    g = torch.Generator().manual_seed(n + k_t)
    of = torch.full((V,), 2, dtype=torch.int32)
    mine = torch.randperm(V, generator=g)[:n].sort().values
    of[mine[: (n + 1) // 2]], of[mine[(n + 1) // 2:]] = 0, 1
    W = (torch.randn((V, d), generator=g) / 8).to(torch.bfloat16)
    if equal:
        W[:] = W[0]
    W1 = torch.zeros((M, d), dtype=torch.bfloat16)
    W1[0, 0], W1[1, 0], W1[2, 0] = 2, 1, -1
    h = torch.randn((1, d), generator=g).to(torch.bfloat16)
    h[0, 0] = 1
    L = D.build_layout(of.to(DEV), W.to(DEV), M)
    D.set_option(D.OPT_FUSED_B1, 3)
    try:
        head = D.draft_head(D.Router(W1.to(DEV), act="none"), L, h.to(DEV), h.to(DEV), 2, mode=D.SEL_TOPK, k_t=k_t)
        torch.cuda.synchronize()
    finally:
        D.set_option(D.OPT_FUSED_B1, 0)
    assert head.clusters.cpu().tolist() == [[0, 1]]
    z = head.logits[0, :n].cpu().numpy().astype(np.float64)
    ids = mine.numpy()
    assert np.abs(z - (W[mine].double() @ h[0].double()).numpy()).max() <= 1e-5
    order = np.lexsort((ids, -z))[:k_t]
    assert head.ids[0, :len(order)].cpu().tolist() == ids[order].tolist()
    assert (head.ids[0, len(order):].cpu() == -1).all()
    ref = z[order] - z.max() - np.log(np.exp(z - z.max()).sum())
    assert np.abs(head.logprobs[0, :len(order)].cpu().numpy() - ref).max() <= 1e-5 * max(1.0, np.abs(ref).max())


# one launch, hundreds of slots at the bound of the selection: a run of equal
# logits, the same value in every sixteenth slot (fewer groups than k_t hold
# the largest), and contexts of zeros and NaN (every logit the same)
@pytest.mark.parametrize("n", [300, 4097, 6144, 8192, 16384])
@pytest.mark.parametrize("kind", ["run", "lanes", "lanes+1", "zero", "nan"])
@pytest.mark.parametrize("k_t", [2, 10, 16])
def test_one_launch_crowded_top_kt(n, kind, k_t):
    d, V, M = 64, 20000, 3
    g = torch.Generator().manual_seed(n + k_t)
    of = torch.full((V,), 2, dtype=torch.int32)
    mine = torch.randperm(V, generator=g)[:n].sort().values
    mine = torch.cat([mine[::2], mine[1::2]])  # slot -> vocabulary id: two clusters, interleaved ids
    of[mine[: (n + 1) // 2]], of[mine[(n + 1) // 2:]] = 0, 1
    z = torch.randint(-99, 100, (n,), generator=g).float()
    if kind == "run":
        z[n // 4:n // 4 + 280] = 101
    elif kind.startswith("lanes"):
        z[5::16] = 101
        if kind == "lanes+1":
            z[[7, n - 1]] = 102
    W = torch.zeros((V, d), dtype=torch.bfloat16)
    W[mine, 1] = z.to(torch.bfloat16)
    W1 = torch.zeros((M, d), dtype=torch.bfloat16)
    W1[0, 0], W1[1, 0], W1[2, 0] = 2, 1, -1
    x, h = torch.zeros((1, d), dtype=torch.bfloat16), torch.zeros((1, d), dtype=torch.bfloat16)
    x[0, 0], h[0, 1] = 1, 1
    if kind == "zero":
        h[:] = 0
        z[:] = 0
    elif kind == "nan":
        h[:] = float("nan")
        z[:] = -float("inf")
    L = D.build_layout(of.to(DEV), W.to(DEV), M)
    D.set_option(D.OPT_FUSED_B1, 3)
    try:
        head = D.draft_head(D.Router(W1.to(DEV), act="none"), L, x.to(DEV), h.to(DEV), 2, mode=D.SEL_TOPK, k_t=k_t)
        torch.cuda.synchronize()
    finally:
        D.set_option(D.OPT_FUSED_B1, 0)
    order = np.lexsort((mine.numpy(), -z.numpy()))[:k_t]
    assert head.ids[0].cpu().tolist() == mine.numpy()[order].tolist()
    if kind != "nan":
        zz = z.double().numpy()
        ref = zz[order] - zz.max() - np.log(np.exp(zz - zz.max()).sum())
        assert np.abs(head.logprobs[0].cpu().numpy() - ref).max() <= 1e-5 * max(1.0, np.abs(ref).max())


# rows beyond 16 slots per thread go block after block: to both sides of two
# and three blocks of 8192, with the best slots in one block, spread over all
# of them, or of equal value, and rows that a long row stride makes the wide
# kernel take
@pytest.mark.parametrize("n", [1, 700, 5000, 16385, 24576, 24577, 60000])
@pytest.mark.parametrize("kind", ["random", "rising", "falling", "equal", "runs", "lanes", "special"])
@pytest.mark.parametrize("k_t", [2, 15, 16])
def test_long_row_top_kt(n, kind, k_t):
    rng = np.random.default_rng(n + k_t)
    V, M = 70000, 2
    of = np.ones(V, np.int32)
    of[rng.permutation(V)[:n]] = 0
    L = D.build_layout(torch.from_numpy(of).to(DEV), torch.zeros((V, 8), dtype=torch.bfloat16, device=DEV), M)
    sel, off, length, ids = D.shortlist(L, torch.zeros((1, 1), dtype=torch.int32, device=DEV))
    z = np.full((1, L.cap(1)), np.nan, np.float32)
    z[0, :n] = np.sort(rng.standard_normal(n)) if kind in ("rising", "falling") else _logits(kind, n, rng)
    if kind == "falling":
        z[0, :n] = z[0, :n][::-1]
    out = D.draft_select(L, torch.from_numpy(z).to(DEV), sel, off, length, mode=D.SEL_TOPK, k_t=k_t)
    vids = ids.cpu().numpy()[0, :n]
    zz = np.where(np.isnan(z[0, :n]), -np.inf, z[0, :n]).astype(np.float64)
    order = np.lexsort((vids, -zz))[:k_t]
    got = out["ids"].cpu().numpy()[0]
    assert got[:len(order)].tolist() == vids[order].tolist() and (got[len(order):] == -1).all()
    if np.isfinite(zz.max()):
        ref = zz[order] - zz.max() - np.log(np.exp(zz - zz.max()).sum())
        fin = np.isfinite(ref)
        lp = out["logprobs"].cpu().numpy()[0, :len(order)]
        # fp32: at most 64 terms per thread, a tree over 1024 threads, one logarithm
        assert np.abs(lp[fin] - ref[fin]).max() <= 1e-5 * max(1.0, np.abs(ref[fin]).max())


# the k best clusters at the edges of the workgroup sizes (1024 and 2048
# clusters) and, at the most clusters, of the LDS budget: from k = 1792 on 256
# threads run, and up to k = 1917 only they fit
@pytest.mark.parametrize("M,k", [(1024, 64), (1025, 1025), (2048, 7), (2049, 2049), (8192, 1), (8192, 1791),
                                 (8192, 1792), (8192, 1917)])
def test_top_clusters(M, k):
    g = torch.Generator().manual_seed(M + k)
    W1 = torch.randint(-4, 5, (M, 8), generator=g).to(torch.bfloat16)  # (few distinct scores: many ties)
    x = torch.randint(-4, 5, (3, 8), generator=g).to(torch.bfloat16)
    ids, sc, scores = D.route(D.Router(W1.to(DEV), act="none"), x.to(DEV), k, want_scores=True)
    s = (x.float() @ W1.float().T).numpy()
    assert (scores.cpu().numpy() == s).all()
    for b in range(3):
        order = np.lexsort((np.arange(M), -s[b]))[:k]
        assert ids[b].cpu().tolist() == order.tolist() and sc[b].cpu().tolist() == s[b][order].tolist()

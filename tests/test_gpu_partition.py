"""The partition builder's kernels at the edges of their tiles and chunks: the
counting sort behind the layout, the nearest-centroid product and the update."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2510_13847_amd import dynahead as D  # noqa: E402

DEV = "cuda"


# V around the 64 tokens of a wave step and the 4096 of a chunk, and past 32
# chunks (one batch of the scan); M to both sides of 1024 (one pass of the
# scan) and to the most clusters (fewer counting waves)
@pytest.mark.parametrize("V,M", [(1, 1), (64, 5), (65, 64), (4096, 1024), (4097, 3), (9000, 1025), (9000, 8192),
                                 (140000, 2048)])
@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 8), (torch.float32, 520), (torch.bfloat16, 1032)])
def test_layout(V, M, dtype, d):
    rng = np.random.default_rng(V + M)
    of = np.minimum(rng.geometric(min(1.0, 4.0 / M), V) - 1, M - 1).astype(np.int32)  # crowded and empty clusters
    W = torch.randn((V, d), generator=torch.Generator().manual_seed(V)).to(dtype)
    L = D.build_layout(torch.from_numpy(of).to(DEV), W.to(DEV), M)
    perm = np.argsort(of, kind="stable")
    assert (L.perm.cpu().numpy() == perm).all()
    assert (L.offsets.cpu().numpy() == np.concatenate([[0], np.cumsum(np.bincount(of, minlength=M))])).all()
    assert torch.equal(L.W_perm.cpu(), W[torch.from_numpy(perm)])


def test_layout_of_more_rows_than_one_launch():
    """2^26 rows and more need more waves than a launch can hold, one per row."""
    V, M, d = (1 << 26) + 4999, 3, 8
    g = torch.Generator(device=DEV).manual_seed(1)
    of = torch.randint(0, M, (V,), generator=g, device=DEV, dtype=torch.int32)
    W = torch.randint(-30000, 30000, (V, d), generator=g, device=DEV, dtype=torch.int16).view(torch.bfloat16)
    L = D.build_layout(of, W, M)
    assert L.offsets.cpu().tolist()[1:] == torch.bincount(of, minlength=M).cumsum(0).cpu().tolist()
    perm = torch.argsort(of, stable=True)
    assert torch.equal(L.perm.long(), perm)
    W = W.view(torch.int16)
    for r in range(0, V, 1 << 24):  # (torch's own indexing of all rows at once stops at 2^26)
        assert torch.equal(L.W_perm[r:r + (1 << 24)].view(torch.int16), W[perm[r:r + (1 << 24)]])


@pytest.mark.parametrize("bad", [-1, 7, 1 << 30])
def test_layout_bad_id_is_reported(bad):
    of = np.zeros(5000, np.int32)
    of[4321] = bad
    with pytest.raises(D.DynaError) as e:
        D.build_layout(torch.from_numpy(of).to(DEV), torch.zeros((5000, 8), dtype=torch.bfloat16, device=DEV), 7)
    assert e.value.status == D.ERR_DEVICE_DATA


@pytest.mark.parametrize("bad", [[0], [4095, 4096, 8999], list(range(9000))])
def test_layout_refused_leaves_the_weights(bad):
    """A partition with a bad id is refused before any row is copied: W_perm keeps
    what it held, whatever perm held before; perm lists the good tokens, then -1."""
    V, M, d = 9000, 7, 16
    of = np.random.default_rng(5).integers(0, M, V).astype(np.int32)
    of[bad] = M
    ofd = torch.from_numpy(of).to(DEV)
    W = torch.randn((V, d), device=DEV).to(torch.bfloat16)
    W_perm = torch.full_like(W, 3.0)
    perm = torch.arange(V, dtype=torch.int32, device=DEV)  # every entry a valid row
    offsets = torch.empty(M + 1, dtype=torch.int32, device=DEV)
    cap, n = np.zeros(M + 1, np.int32), D.layout_workspace_bytes(V, M)
    ws = torch.zeros(n, dtype=torch.uint8, device=DEV)
    status = D.lib().dyna_build_layout(ofd.data_ptr(), V, M, W.data_ptr(), D.BF16, d, W_perm.data_ptr(),
                                       perm.data_ptr(), offsets.data_ptr(), cap.ctypes.data_as(ctypes.c_void_p), None,
                                       ws.data_ptr(), n, torch.cuda.current_stream().cuda_stream)
    assert status == D.ERR_DEVICE_DATA
    assert bool((W_perm == 3.0).all())
    good = np.flatnonzero(of < M)
    good = good[np.argsort(of[good], kind="stable")]
    assert perm.cpu().tolist() == good.tolist() + [-1] * (V - good.size)


# both tile sides (128, and 256 from 256 tiles on), rows and centroids on
# either side of them, K of one piece, of ragged stages and of one to three
@pytest.mark.parametrize("V,M,d", [(1, 1, 8), (127, 127, 64), (130, 129, 72), (300, 257, 192), (5000, 512, 1032),
                                   (33000, 513, 40), (65537, 255, 64), (66000, 257, 136)])
def test_nearest_centroid(V, M, d):
    g = torch.Generator().manual_seed(V + M + d)
    W = torch.randn((V, d), generator=g).to(torch.bfloat16)
    mu = torch.randn((M, d), generator=g)
    if V > 100:
        W[17] = 0  # no direction: every product is 0, the lowest id
        mu[M - 1] = mu[M // 2]  # an exact tie: the lower id
    a, s = D.kmeans_assign(W.to(DEV), mu.to(DEV), want_score=True)
    torch.cuda.synchronize()
    a, s = a.cpu().long(), s.cpu().double()
    assert int(a.min()) >= 0 and int(a.max()) < M
    C = mu.to(torch.bfloat16).double()
    S = W.double() @ C.T
    # fp32 sums of exact products, at most d / 4 + 64 roundings deep
    tol = (d / 4 + 64) * 2.0 ** -24 * (W.double().abs() @ C.abs().T).max(dim=1).values
    mine = S.gather(1, a[:, None])[:, 0]
    assert bool((mine >= S.max(dim=1).values - 2 * tol).all())
    assert bool(((s - mine).abs() <= tol).all())
    if V > 100:
        assert int(a[17]) == 0 and not bool((a == M - 1).any())
    # again on the same workspace (its maxima are left cleared)
    ws = D.kmeans_workspace(W.to(DEV), M)
    for _ in range(2):
        b, _ = D.kmeans_assign(W.to(DEV), mu.to(DEV), ws=ws)
        assert torch.equal(b.cpu().long(), a)


@pytest.mark.parametrize("d", [8, 2048, 2056, 4104, 8192])
def test_update(d):
    """Mean directions of clusters of 0 to 9 rows (batches of four and what is
    left of them), with an all-zero row and skipped assignments."""
    g = torch.Generator().manual_seed(d)
    sizes = list(range(10))
    a = torch.tensor(sum(([m] * n for m, n in enumerate(sizes)), []) + [-1, 10], dtype=torch.int32)
    a = a[torch.randperm(len(a), generator=g)]
    W = torch.randn((len(a), d), generator=g).to(torch.bfloat16)
    W[int((a == 5).nonzero()[0])] = 0
    mu0 = torch.nn.functional.normalize(torch.randn((10, d), generator=g), dim=1)
    mu = D.kmeans_update(W.to(DEV), a.to(DEV), mu0.clone().to(DEV)).cpu().double()
    U = torch.nn.functional.normalize(W.double(), dim=1)
    for m, n in enumerate(sizes):
        ref = torch.nn.functional.normalize(U[a == m].sum(dim=0), dim=0) if n else mu0[m].double()
        # a few fp32 roundings per element (the norm, the scale, up to nine sums)
        assert float((mu[m] - ref).abs().max()) <= 32 * 2.0 ** -24 * max(1.0, float(ref.abs().max()))


@pytest.mark.parametrize("d", [512, 520, 2048, 2056, 4096, 4104])
@pytest.mark.parametrize("copies", [1, 40, 70])
def test_update_batches(d, copies):
    """Clusters at the edges of every batch length (4, 8 and 16 rows), few and
    many of them (each side of 256 and 512 clusters takes another batch)."""
    g = torch.Generator().manual_seed(d + copies)
    sizes = torch.tensor([1, 3, 4, 5, 8, 9, 16, 17] * copies)
    M = len(sizes)
    a = torch.arange(M, dtype=torch.int32).repeat_interleave(sizes)
    a = a[torch.randperm(len(a), generator=g)]
    W = torch.randn((len(a), d), generator=g).to(torch.bfloat16)
    mu = D.kmeans_update(W.to(DEV), a.to(DEV), torch.zeros((M, d), device=DEV))
    U = torch.nn.functional.normalize(W.to(DEV).double(), dim=1)
    ref = torch.zeros((M, d), dtype=torch.float64, device=DEV).index_add_(0, a.to(DEV).long(), U)
    ref = torch.nn.functional.normalize(ref, dim=1)
    # a few fp32 roundings per element (the norm, the scale, up to 17 sums)
    assert float((mu.double() - ref).abs().max()) <= 32 * 2.0 ** -24

"""The row-streaming product (dense and union heads of a few contexts) at the
edges of its tiles, k shares and context groups, against float64 products."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2510_13847_amd import dynahead as D  # noqa: E402

DEV = "cuda"


def _inputs(rows, d, B, seed):
    g = torch.Generator().manual_seed(seed)
    W = (torch.randn((rows, d), generator=g) / d ** 0.5).to(torch.bfloat16)
    h = torch.randn((B, d), generator=g).to(torch.bfloat16)
    return W, h


def _check(got, W, h):
    """fp32 sums of exact products: at most (d / 4 + 64) roundings of 2^-24 of
    sum |w h| (every kernel's summation depth stays below that)."""
    z = h.double() @ W.double().T
    bound = (h.shape[1] / 4 + 64) * 2.0 ** -24 * (h.double().abs() @ W.double().abs().T)
    assert bool(((got.double() - z).abs() <= bound).all())


# K: one k step, ragged tails, each stage shape (up to 4, 8, 12, 16 steps per
# wave, and two stages beyond 4096); B: both sides of every context group;
# rows: one, around a tile, and a few hundred tiles
@pytest.mark.parametrize("d", [8, 40, 256, 1032, 2048, 3000, 4096])
@pytest.mark.parametrize("B", [5, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("rows", [1, 16, 17, 4999])
def test_dense_rows(rows, B, d):
    W, h = _inputs(rows, d, B, rows + 31 * B + d)
    head = D.DenseHead(W.to(DEV), rows, B, D.SEL_ARGMAX, 1, keep_logits=True)
    head(h.to(DEV))
    torch.cuda.synchronize()
    _check(head.logits.cpu(), W, h)


@pytest.mark.parametrize("d", [4104, 6000, 8192])
@pytest.mark.parametrize("rows", [15, 5003])
def test_dense_rows_two_stages(rows, d):
    W, h = _inputs(rows, d, 13, rows + d)
    head = D.DenseHead(W.to(DEV), rows, 13, D.SEL_ARGMAX, 1, keep_logits=True)
    head(h.to(DEV))
    torch.cuda.synchronize()
    _check(head.logits.cpu(), W, h)


# (d, B, tile sequences): every instance, k steps per wave of 4, 8, 12 and 16,
# one and two stages, 16 and 32 contexts per workgroup, tiles shared by two
# workgroups; the sequences are as many as the chip holds of that instance
INSTANCES = [(1000, 16, 512), (1000, 32, 512), (1000, 64, 256), (2040, 13, 512), (2040, 29, 256), (2040, 57, 128),
             (3000, 16, 256), (3000, 32, 256), (3000, 40, 128), (4096, 5, 256), (4096, 17, 256), (4096, 64, 128),
             (6000, 16, 256), (8192, 9, 256)]


def _close(got, W, h):
    """_check on the GPU, in pieces of the rows."""
    hd = h.to(DEV).double()
    for r in range(0, W.shape[0], 8192):
        w = W[r:r + 8192].to(DEV).double()
        bound = (h.shape[1] / 4 + 64) * 2.0 ** -24 * (hd.abs() @ w.abs().T)
        assert bool(((got[:, r:r + 8192].double() - hd @ w.T).abs() <= bound).all())


@pytest.mark.parametrize("d,B,seqs", INSTANCES)
def test_dense_many_tiles(d, B, seqs):
    """Three tiles and more for every workgroup, the last round partial and its
    last tile ragged: registers, LDS and partial sums are used again and again."""
    rows = 16 * (3 * seqs + 5) - 3
    W, h = _inputs(rows, d, B, d + B)
    head = D.DenseHead(W.to(DEV), rows, B, D.SEL_ARGMAX, 1, keep_logits=True)
    head(h.to(DEV))
    torch.cuda.synchronize()
    _close(head.logits, W, h)


# both sides of the lines between the row-streaming and the union kernel: by
# row length and contexts, and long tables of unaligned rows
@pytest.mark.parametrize("rows,d,B", [(8320, 64, 34), (8321, 64, 34), (13824, 128, 40), (13825, 128, 40),
                                      (32256, 4096, 40), (32257, 4096, 40), (43008, 2112, 64), (43009, 2112, 64),
                                      (49920, 512, 33), (49921, 512, 33), (73728, 1536, 64), (73729, 1536, 64),
                                      (110208, 896, 50), (110209, 896, 50), (110209, 392, 50),
                                      (98000, 312, 40), (98000, 328, 40)])
def test_dense_lines(rows, d, B):
    W, h = _inputs(rows, d, B, rows)
    head = D.DenseHead(W.to(DEV), rows, B, D.SEL_ARGMAX, 1, keep_logits=True)
    head(h.to(DEV))
    torch.cuda.synchronize()
    _close(head.logits, W, h)


@pytest.mark.parametrize("B,d", [(3, 280), (29, 280), (3, 288), (29, 296), (16, 384), (16, 392), (16, 440), (16, 448)])
def test_union_lines(B, d):
    """Unions of more than 64 rows per column: short aligned rows take the
    union kernel, the others the row-streaming one."""
    M = 32
    V = 64 * d + 2000
    of = torch.arange(V, dtype=torch.int32) % M
    W, h = _inputs(V, d, B, B + d)
    W1 = (torch.randn((M, d), generator=torch.Generator().manual_seed(1)) / d ** 0.5).to(torch.bfloat16)
    L = D.build_layout(of.to(DEV), W.to(DEV), M)
    head = D.draft_head(D.Router(W1.to(DEV), act="none"), L, h.to(DEV), h.to(DEV), M,
                        mode=D.SEL_TOPK | D.SEL_UNION, k_t=1)
    torch.cuda.synchronize()
    ids = torch.arange(V).reshape(-1, 1)[torch.argsort(of, stable=True)].flatten()
    _close(head.logits[:, :V], W[ids], h)
    assert head.ids[:, 0].cpu().tolist() == ids[head.logits[:, :V].argmax(1).cpu()].tolist()


def test_special_values_stay_in_their_row():
    """Infinities and NaN of one row (and of the last row, beside the tile's
    unused rows) reach that row's logits only; a context's columns past K
    never meet them."""
    W, h = _inputs(35, 1032, 7, 3)
    W[4, 0], W[34, 1031], W[20, 7] = float("inf"), float("nan"), float("-inf")
    h[:, 0].abs_().clamp_(min=0.5)
    head = D.DenseHead(W.to(DEV), 35, 7, D.SEL_ARGMAX, 1, keep_logits=True)
    head(h.to(DEV))
    torch.cuda.synchronize()
    z = head.logits.cpu()
    keep = [r for r in range(35) if r not in (4, 20, 34)]
    _check(z[:, keep], W[keep], h)
    assert bool((z[:, 4] == float("inf")).all()) and bool(torch.isnan(z[:, 34]).all())
    assert bool(torch.isinf(z[:, 20]).logical_or(torch.isnan(z[:, 20])).all())


@pytest.mark.parametrize("B,d", [(2, 520), (16, 4096), (17, 1000), (40, 640), (11, 5376), (9, 24), (25, 32), (60, 64)])
def test_union_rows(B, d):
    """Over a union plan (chunks of 1-16 rows at any slot): every logit is its
    row's product and every slot's id its row's."""
    rng = np.random.default_rng(B + d)
    V, M, k = 3000, 37, 3
    sizes = rng.multinomial(V - 2 * M, np.full(M, 1.0 / M)) + 2
    of = np.repeat(np.arange(M, dtype=np.int32), sizes)[rng.permutation(V)]
    W, h = _inputs(V, d, B, 5 * B + d)
    W1 = (torch.randn((M, d), generator=torch.Generator().manual_seed(1)) / d ** 0.5).to(torch.bfloat16)
    L = D.build_layout(torch.from_numpy(of).to(DEV), W.to(DEV), M)
    head = D.draft_head(D.Router(W1.to(DEV), act="none"), L, h.to(DEV), h.to(DEV), k,
                        mode=D.SEL_TOPK | D.SEL_UNION, k_t=4)
    torch.cuda.synchronize()
    chosen = np.unique(head.clusters.cpu().numpy())
    ids = np.concatenate([np.flatnonzero(of == m) for m in chosen])
    z = head.logits.cpu()[:, :ids.size]
    _check(z, W[ids], h)
    top = np.argsort(-z.numpy(), axis=1, kind="stable")[:, :1]
    assert (head.ids.cpu().numpy()[:, :1] == ids[top]).all()


@pytest.mark.parametrize("d,B,seqs", INSTANCES)
def test_union_many_tiles(d, B, seqs):
    """A union of more than three tiles per workgroup (chunks of 1-16 rows):
    every slot's logit and every row's best ids, whose table the kernel wrote."""
    rng = np.random.default_rng(B + d)
    M, k, k_t = 37, 36, 4
    V = 16 * 3 * seqs + 6000
    sizes = rng.multinomial(V - 2 * M, np.full(M, 1.0 / M)) + 2
    of = np.repeat(np.arange(M, dtype=np.int32), sizes)[rng.permutation(V)]
    W, h = _inputs(V, d, B, 7 * B + d)
    W1 = (torch.randn((M, d), generator=torch.Generator().manual_seed(1)) / d ** 0.5).to(torch.bfloat16)
    L = D.build_layout(torch.from_numpy(of).to(DEV), W.to(DEV), M)
    head = D.draft_head(D.Router(W1.to(DEV), act="none"), L, h.to(DEV), h.to(DEV), k,
                        mode=D.SEL_TOPK | D.SEL_UNION, k_t=k_t)
    torch.cuda.synchronize()
    chosen = np.unique(head.clusters.cpu().numpy())
    ids = np.concatenate([np.flatnonzero(of == m) for m in chosen])
    assert sum(-(-int(sizes_m) // 16) for sizes_m in np.bincount(of, minlength=M)[chosen]) > 3 * seqs
    _close(head.logits[:, :ids.size], W[ids], h)
    z = head.logits[:, :ids.size].cpu().numpy()
    for b in range(B):
        best = np.lexsort((ids, -z[b]))[:k_t]
        assert head.ids[b].cpu().tolist() == ids[best].tolist()

"""GPU parity, 0 ULP against the CPU oracle, of the matrix-core kernels that
spread a product's k blocks over a workgroup's waves, of the staged kernels'
short last block, and of the automatic choice between them and the other
kernels.

The contraction's length is taken around the ends of slices (16), blocks (64),
rounds of blocks (4, 8, 16 or 32 blocks) and groups of blocks that share one
instruction; rows and columns around the tiles' edges; operands in all four
layouts, with leading dimensions and origins that are 16-byte aligned and that
are not.
"""
import ctypes

import numpy as np
import pytest

import oracle
from bitcmp import assert_bits_equal
from gpu_util import announce, dev, host, same_bits
from paper_2502_19405_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    from paper_2502_19405_amd import repops
    repops.load()
    return repops


def operand(a, transposed, pad):
    """Device view of a, stored transposed or not, `pad` floats into each row."""
    import torch
    s = np.ascontiguousarray(a.T) if transposed else a
    buf = torch.full((s.shape[0], s.shape[1] + pad), float("nan"), device="cuda:0")
    v = buf[:, pad:] if pad else buf
    v.copy_(dev(s))
    return v.t() if transposed else v


def entries(rp):
    """Launches of the split kernels and of the staged entries with a short last
    block (64-deep blocks of 16-deep slices, one ring turn each)."""
    names = rp.gemm_configs(rp.LAUNCH_GEMM_MFMA)
    out = [("auto", None)]
    for i, n in enumerate(names):
        if "/k" in n or i in (0, 8, 9):
            out.append((n, rp.Launch(rp.LAUNCH_GEMM_MFMA, (i,))))
    assert len(out) > 9
    return out


# (m, n): one row; tiles of 4, 16, 32 and 64 rows with one row or column more
# or less than whole tiles; multiples of 4 for the staged kernels
SHAPES = [(1, 68), (17, 31), (64, 132), (67, 65)]
DEPTHS = [1, 3, 16, 18, 63, 64, 67, 100, 128, 191, 256, 260, 511, 1025, 2051]


@pytest.mark.parametrize("k", DEPTHS)
@pytest.mark.parametrize("pad", [0, 1, 4])
def test_contraction_ends(rp, k, pad):
    for m, n in SHAPES:
        g = inputs.rng(40 * k + m + n)
        A, B = inputs.normal(g, (m, k)), inputs.normal(g, (k, n))
        bias = inputs.uniform(g, (n,), -0.1, 0.1)
        want = oracle.matmul(A, B, bias)
        dbias = dev(bias)
        for ta in (0, 1):
            for tb in (0, 1):
                a, b = operand(A, ta, pad), operand(B, tb, pad)
                for name, launch in entries(rp):
                    announce("contraction end", m, n, k, pad, ta, tb, name)
                    got = rp.matmul(a, b, dbias, launch=launch)
                    assert_bits_equal(host(got), want, f"{m}x{n}x{k} pad {pad} {ta}{tb} {name}")


@pytest.mark.parametrize("k", [64, 70, 333])
def test_batched_causal_and_epilogues(rp, k):
    """The same kernels with two batch strides, both causal masks, the GELU
    output and the GELU backward's input."""
    import torch
    b0, b1, m, n = 2, 3, 70, 66
    g = inputs.rng(8800 + k)
    A, B = inputs.normal(g, (b0, b1, m, k)), inputs.normal(g, (b0, b1, n, k))
    want = oracle.bmm(A, B, alpha=0.125, trans_b=True)
    square = inputs.normal(g, (b0, b1, k, k))
    square[..., np.triu(np.ones((k, k), bool), 1)] = 0.0
    V = inputs.normal(g, (b0, b1, k, n))
    want_v = oracle.bmm(square, V)
    X = inputs.uniform(g, (m, n), -4.0, 4.0)
    a2, b2 = A[0, 0], np.ascontiguousarray(B[0, 0].T)
    prod = oracle.matmul(a2, b2)
    want_g, want_gb = oracle.gelu(prod), oracle.gelu_backward(X, prod)
    lower = np.tril(np.ones((m, n), bool))
    for name, launch in entries(rp):
        announce("batched, causal, epilogues", k, name)
        for mask in (0, rp.CAUSAL_OUTPUT):
            C = torch.full((b0, b1, m, n), float("nan"), device="cuda:0")
            rp.bmm_raw(b0, b1, m, n, k, dev(A), b1 * m * k, m * k, k, 0, dev(B), b1 * n * k, n * k,
                       k, 1, 0.125, C, b1 * m * n, m * n, n, launch=launch, causal=mask)
            keep = lower if mask else np.ones((m, n), bool)
            assert_bits_equal(np.where(keep, host(C), 0), np.where(keep, want, 0), f"{name} {mask}")
        C = torch.full((b0, b1, k, n), float("nan"), device="cuda:0")
        rp.bmm_raw(b0, b1, k, n, k, dev(square), b1 * k * k, k * k, k, 0, dev(V), b1 * k * n, k * n,
                   n, 0, 1.0, C, b1 * k * n, k * n, n, launch=launch, causal=rp.CAUSAL_A)
        assert_bits_equal(host(C), want_v, f"{name} causal A")
        h, gl = rp.matmul_gelu(dev(a2), dev(b2), None, launch=launch)
        assert_bits_equal(host(h), prod, f"{name} H")
        assert_bits_equal(host(gl), want_g, f"{name} GELU")
        gb = rp.matmul_gelu_backward(dev(a2), dev(b2), dev(X), launch=launch)
        assert_bits_equal(host(gb), want_gb, f"{name} GELU backward")


# tokens: few (each product by itself, on the split kernels) to many (one
# grouped launch), with contractions over the tokens that end inside a slice
@pytest.mark.parametrize("tokens", [1, 40, 333, 1001, 2050])
def test_grouped_choice_keeps_the_bits(rp, tokens):
    g = inputs.rng(6600 + tokens)
    X, dY = inputs.normal(g, (tokens, 768)), inputs.normal(g, (tokens, 3072))
    W = inputs.normal(g, (768, 3072))
    dX_, dY_, W_ = dev(X), dev(dY), dev(W)
    announce("grouped choice", tokens)
    a, b = rp.matmul_grouped([(dY_, W_.t(), None, None), (dX_.t(), dY_, None, None)])
    simple = rp.Launch(rp.LAUNCH_GEMM_SIMPLE)
    assert same_bits(a, rp.matmul(dY_, W_.t(), launch=simple))
    assert same_bits(b, rp.matmul(dX_.t(), dY_, launch=simple))
    r, c = inputs.sample_indices(tokens, 256, tokens, 768)
    assert_bits_equal(host(a)[r, c], oracle.matmul_at(dY, W, r, c, trans_b=True), "dX")
    r, c = inputs.sample_indices(tokens + 1, 256, 768, 3072)
    assert_bits_equal(host(b)[r, c], oracle.matmul_at(X, dY, r, c, trans_a=True), "dW")


def in_one_launch(rp, prods):
    """Whether the grouped call's rule runs these products in one launch here."""
    import torch
    descs = (rp.GemmDescT * len(prods))()
    for d, (A, B, *_) in zip(descs, prods):
        d.A, d.m, d.k, d.lda, d.trans_a = rp._mat(A, "A")
        d.B, _, d.n, d.ldb, d.trans_b = rp._mat(B, "B")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return rp.load().repops_internal_grouped_choice(ctypes.byref(rp.Order().c()), len(prods),
                                                    descs, cus) == 1


# Ends of the contraction behind whole blocks: inside the first slice, behind one,
# two and three whole slices, and just short of a block; then one short block alone
@pytest.mark.parametrize("blocks,end", [(9, 4), (9, 20), (9, 36), (9, 52), (9, 60), (0, 36)])
def test_grouped_short_last_blocks_in_every_layout(rp, blocks, end):
    """One grouped launch (asserted) of all four layouts under the default order, rows
    and columns ragged, with a bias and with a GELU input, K ending inside a block;
    transposed A with plain B takes any K, the others multiples of 4."""
    g = inputs.rng(6700 + 64 * blocks + end)
    k = 64 * blocks + end
    shapes = [(1301, 1412, k, 0, 0), (1143, 1337, k, 0, 1), (1204, 1500, k + 1, 1, 0),
              (1108, 1237, k, 1, 1), (2052, 1028, k + 3, 1, 0)]
    prods, hosts = [], []
    for i, (m, n, kk, ta, tb) in enumerate(shapes):
        A, B = inputs.normal(g, (kk, m) if ta else (m, kk)), inputs.normal(g, (n, kk) if tb else (kk, n))
        bias = inputs.uniform(g, (n,), -0.1, 0.1) if i in (0, 2) else None
        X = inputs.uniform(g, (m, n), -4.0, 4.0) if i in (1, 4) else None
        hosts.append((A, B, bias, X))
        prods.append((dev(A).t() if ta else dev(A), dev(B).t() if tb else dev(B),
                      None if bias is None else dev(bias), None,
                      *([] if X is None else [dev(X)])))
    assert in_one_launch(rp, prods)
    announce("grouped short last blocks", blocks, end)
    outs = rp.matmul_grouped(prods)
    simple = rp.Launch(rp.LAUNCH_GEMM_SIMPLE)
    for i, (out, p, (A, B, bias, X)) in enumerate(zip(outs, prods, hosts)):
        m, n, kk, ta, tb = shapes[i]
        if X is None:
            want = rp.matmul(p[0], p[1], p[2], launch=simple)
        else:
            want = rp.matmul_gelu_backward(p[0], p[1], p[4], launch=simple)
        assert same_bits(out, want), shapes[i]
        r, c = inputs.sample_indices(6700 + i, 200, m, n)
        r, c = np.append(r, [0, m - 1, m - 1]), np.append(c, [n - 1, 0, n - 1])
        ref = oracle.matmul_at(A, B, r, c, bias, trans_a=bool(ta), trans_b=bool(tb))
        if X is not None:
            ref = oracle.gelu_backward(np.ascontiguousarray(X[r, c]), ref)
        assert_bits_equal(host(out)[r, c], ref, f"product {i} {shapes[i]}")


@pytest.mark.parametrize("k", [16, 36, 70, 129, 515])
def test_infinities_and_nan_near_the_cut(rp, k):
    """Infinities and NaN in operands at the last k index, in the last whole slice and
    at k 0: what lies past the end, and the values that stand in for it, must not
    meet them (the products' own infinities and NaN must come out)."""
    m, n = 68, 132
    g = inputs.rng(8950 + k)
    for where in sorted({0, k - 1, max(0, k // 16 * 16 - 1)}):
        A, B = inputs.normal(g, (m, k)), inputs.normal(g, (k, n))
        A[3, where], A[5, where], B[where, 7] = np.inf, np.nan, -np.inf
        B[where, 9] = 0.0  # inf * 0
        want = oracle.matmul(A, B)
        assert np.isnan(want[5]).all() and np.isnan(want[3, 9]) and np.isfinite(want[4, 8])
        for ta in (0, 1):
            for tb in (0, 1):
                a, b = operand(A, ta, 0), operand(B, tb, 0)
                for name, launch in entries(rp):
                    announce("infinities", k, where, ta, tb, name)
                    got = host(rp.matmul(a, b, launch=launch))
                    label = f"k {k} at {where} {ta}{tb} {name}"
                    # which NaN a chain gives is not fixed: compare where, not its bits
                    assert np.array_equal(np.isnan(got), np.isnan(want)), label
                    assert_bits_equal(np.where(np.isnan(want), 0, got),
                                      np.where(np.isnan(want), 0, want), label)


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_leading_dimensions_over_2_to_the_22(rp, ta, tb):
    """The split kernels' lane offsets take leading dimensions up to 2^22; past it
    they decline, under AUTO and by name, and the bits stay."""
    m, n, k = 9, 12, 20
    ld = (1 << 22) + 4
    g = inputs.rng(8970)
    A, B = inputs.normal(g, (m, k)), inputs.normal(g, (k, n))
    want = oracle.matmul(A, B)
    import torch

    def wide(a, transposed):
        s = np.ascontiguousarray(a.T) if transposed else a
        buf = torch.full(((s.shape[0] - 1) * ld + s.shape[1],), float("nan"), device="cuda:0")
        v = buf.as_strided(s.shape, (ld, 1))
        v.copy_(dev(s))
        return v.t() if transposed else v

    a, b = wide(A, ta), wide(B, tb)
    for name, launch in entries(rp):
        announce("wide leading dimensions", ta, tb, name)
        assert_bits_equal(host(rp.matmul(a, b, launch=launch)), want, f"{ta}{tb} {name}")


def test_products_of_more_tiles_than_one_launch_holds(rp):
    """2^24 products of one output each: a workgroup per tile would be 2^32 threads
    or more, so the split kernels decline and the others loop over the rest.  All
    batch elements read the same operands, so every output is the one oracle value."""
    import torch
    k, batch = 64, 1 << 24
    g = inputs.rng(8900)
    A, B = inputs.normal(g, (1, k)), inputs.normal(g, (1, k))
    want = oracle.matmul(A, np.ascontiguousarray(B.T))
    split = next(i for i, n in enumerate(rp.gemm_configs(rp.LAUNCH_GEMM_MFMA)) if "/k" in n)
    dA, dB = dev(A), dev(B)
    C = torch.empty(batch, device="cuda:0")
    for name, launch in [("auto", None), ("simple", rp.Launch(rp.LAUNCH_GEMM_SIMPLE)),
                         ("mfma0", rp.Launch(rp.LAUNCH_GEMM_MFMA, (0,))),
                         ("split", rp.Launch(rp.LAUNCH_GEMM_MFMA, (split,)))]:
        announce("more tiles than one launch holds", name)
        C.fill_(float("nan"))
        rp.bmm_raw(batch, 1, 1, 1, k, dA, 0, 0, k, 0, dB, 0, 0, k, 1, 1.0, C, 1, 1, 1,
                   launch=launch)
        assert_bits_equal(host(C[:1]), want.reshape(1), name)
        assert same_bits(C, C[:1].expand(batch)), name

"""Kernel variants that the host chooses by the shape of a call, each at shapes
where its rule takes it."""
import math

import pytest
import torch

from tol import fp32_block_tol

pytestmark = pytest.mark.gpu


def ddst():
    from paper_2510_25991_amd import ddst as mod
    return mod


def plane_schur(M, skew, dtype=torch.float64):
    """The limit of the plane Schur complements of a 2D Laplacian, D = T - D^{-1}
    with T = tridiag(-1, 4, -1), rows and columns scaled apart by up to
    exp(skew) (skew 0: symmetric)."""
    i = torch.arange(1, M + 1, device="cuda", dtype=dtype)
    q = math.sqrt(2 / (M + 1)) * torch.sin(math.pi * i[:, None] * i[None, :] / (M + 1))
    lam = 4 - 2 * torch.cos(math.pi * i / (M + 1))
    D = (q * ((lam + torch.sqrt(lam * lam - 4)) / 2)) @ q
    s = torch.exp(skew * i / M)
    return (D + D.T) / 2 if skew == 0 else s[:, None] * D / s[None, :]


@pytest.mark.parametrize("symmetric", [False, True])
@pytest.mark.parametrize("ld,M,tiles", [(896, 800, 74), (1152, 1025, 45), (1280, 1225, 36),
                                        (1664, 1536, 22), (896, 896, 260)])
def test_outer_elimination_is_as_accurate(ld, M, tiles, symmetric):
    """Many matrices are eliminated in outer blocks, two of them in one level:
    the same sums in another order, so the same error, up to a factor of 2 in
    the Frobenius norm and of 4 in the largest entry."""
    batch = tiles * (2 if symmetric else 1)
    print(f"\n[gpu] outer elimination ld={ld} M={M} batch={batch}", flush=True)
    one = torch.eye(ld, device="cuda", dtype=torch.float32)
    one[:M, :M] = plane_schur(M, 0.0 if symmetric else 1.0).float()
    if symmetric:
        one[:M, :M] = torch.tril(one[:M, :M]) + torch.tril(one[:M, :M], -1).T
    ref = torch.linalg.inv(one.double())
    few = one.repeat(2, 1, 1)
    many = one.repeat(batch, 1, 1)
    ddst().kernel_invert(few, symmetric=symmetric)
    ddst().kernel_invert(many, symmetric=symmetric)
    e1 = few[0].double() - ref
    for b in (0, batch // 2, batch - 1):
        e = many[b].double() - ref
        assert float(e.norm()) <= 2 * float(e1.norm())
        assert float(e.abs().max()) <= 4 * float(e1.abs().max())


@pytest.mark.parametrize("dim,n,slabs,b", [(2, 895, 64, 10.0), (2, 1023, 64, 0.0),
                                           (3, 47, 8, 10.0), (3, 47, 24, 0.0)])
def test_builds_by_outer_blocks(dim, n, slabs, b):
    """FP32 transfer blocks of builds that eliminate in outer blocks against FP64
    ones (one level)."""
    print(f"\n[gpu] outer build {dim}D n={n} slabs={slabs} b={b}", flush=True)
    ops = [ddst().Operator(dim, n, slabs, bvec=(b, 0.0, 0.0), precision=p, keep_factors=False)
           for p in ("fp32", "fp64")]
    worst = scale = 0.0
    for j in (1, 2, slabs // 2, slabs - 1):
        for x, y in zip(ops[0].transfer(j), ops[1].transfer(j)):
            worst = max(worst, float((x.double() - y.double()).abs().max()))
            scale = max(scale, float(y.abs().max()))
    for op in ops:
        op.close()
    assert worst <= fp32_block_tol((n + 1) // slabs, n ** (dim - 1)) * scale


@pytest.mark.parametrize("batch,ld", [(225, 512), (224, 512), (21, 1664), (6, 1664), (60, 1024)])
def test_products_at_the_tiles_rule(batch, ld):
    """FP32 products on both sides of the rule: 128 x 128 tiles, 256 x 256 ones,
    whole and with half tiles at the edges (sums of up to 1664 terms: 2e-5 per
    384 of them, as the other product tests)."""
    print(f"\n[gpu] products {batch} x {ld}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(ld + batch)
    A = torch.randn(batch, ld, ld, generator=g, device="cuda")
    B = torch.randn(batch, ld, ld, generator=g, device="cuda")
    C = torch.empty_like(A)
    ddst().kernel_gemm(A, B, C)
    for b in (0, batch // 2, batch - 1):
        ref = A[b].double() @ B[b].double()
        assert float((C[b].double() - ref).abs().max() / ref.abs().max()) <= 2e-5 * ld / 384


@pytest.mark.parametrize("dim,n,slabs", [(2, 31, 4), (2, 127, 4), (2, 299, 10), (2, 511, 256),
                                         (3, 13, 7), (3, 31, 16)])
def test_transposed_products_of_symmetric_builds(dim, n, slabs):
    """The right blocks of a symmetric operator, products with a transposed right
    operand, by both tile sizes: FP32 against FP64."""
    print(f"\n[gpu] symmetric build {dim}D n={n} slabs={slabs}", flush=True)
    ops = [ddst().Operator(dim, n, slabs, precision=p) for p in ("fp32", "fp64")]
    worst = scale = 0.0
    for j in range(1, slabs):
        x, y = (op.transfer(j)[1] for op in ops)
        worst = max(worst, float((x - y).abs().max()))
        scale = max(scale, float(y.abs().max()))
    for op in ops:
        op.close()
    assert worst <= fp32_block_tol((n + 1) // slabs, n ** (dim - 1)) * scale


@pytest.mark.parametrize("factors", ["bf16", "fp32", "fp64"])
@pytest.mark.parametrize("dim,n,slabs,rank,leaf", [(2, 127, 4, 1, 1), (2, 255, 8, 8, 16),
                                                   (2, 299, 10, 16, 37), (2, 639, 8, 48, 128),
                                                   (3, 23, 6, 64, 128)])
def test_sampled_product_by_node_size(dim, n, slabs, rank, leaf, factors):
    """y = S x through trees whose nodes hold one to four rows per group of lanes
    (clusters of one point to 128): the transposed product is the transpose of
    the plain one, entry by entry (FP64 sums of the same factors: 1e-12)."""
    print(f"\n[gpu] sampled product {dim}D n={n} rank={rank} leaf={leaf} {factors}", flush=True)
    op = ddst().Operator(dim, n, slabs, precision="fp32")
    op.compress_hbs(rank=rank, oversample=10, leaf=leaf, factor_dtype=factors, seed=3)
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn(2, op.n_ds * op.M, generator=g, device="cuda", dtype=torch.float64)
    y = op.apply(x[0], which="hbs").reshape(-1)
    z = op.apply(x[1], which="hbs", transpose=True).reshape(-1)
    assert abs(float(y @ x[1] - z @ x[0])) <= 1e-12 * float(x[0].norm() * x[1].norm())
    # column by column against the whole product, at both ends and between
    cols = [0, 1, op.M // 2, op.M - 1, op.M, op.n_ds * op.M - 1]
    e = torch.zeros_like(x[0])
    for c in cols:
        e.zero_()
        e[c] = 1.0
        col = op.apply(e, which="hbs").reshape(-1)
        assert abs(float(col @ x[1]) - float(z[c])) <= 1e-12 * float(x[1].norm())
    op.close()


@pytest.mark.parametrize("n,slabs", [(1023, 64), (1151, 48), (899, 60), (2047, 16)])
def test_wide_matrix_vector_products(n, slabs):
    """FP32 products of launches with 1024 columns at a time (the last of 1023, 127,
    899 and 1023 columns), against the blocks themselves: FP64 sums, 1e-12."""
    print(f"\n[gpu] wide products n={n} slabs={slabs}", flush=True)
    op = ddst().Operator(2, n, slabs, bvec=(5.0, 1.0, 0.0), precision="fp32", keep_factors=False)
    g = torch.Generator(device="cuda").manual_seed(n)
    J, M = op.n_ds, op.M
    x = torch.randn(J, M, generator=g, device="cuda", dtype=torch.float64)
    out = op.apply(x.reshape(-1)).reshape(J, M)
    for j in (0, 1, J // 2, J - 1):
        a, b = op.transfer(j + 1)
        y = x[j].clone()
        if j > 0:
            y -= (a * x[j - 1]).sum(1)
        if j < J - 1:
            y -= (b * x[j + 1]).sum(1)
        assert float((out[j] - y).abs().max()) <= 1e-12 * float(y.abs().max())
    op.close()


@pytest.mark.parametrize("symmetric", [False, True])
@pytest.mark.parametrize("batch,ld,M", [(256, 128, 100), (257, 128, 100), (300, 256, 200),
                                        (260, 640, 520)])
def test_more_matrices_than_cus(batch, ld, M, symmetric):
    """Inverses in FP32 with the pivots' work-groups one and two on a CU: the same
    arithmetic, so the inverses of one matrix by both are equal."""
    print(f"\n[gpu] inverses {batch} x {ld}", flush=True)
    one = torch.eye(ld, device="cuda", dtype=torch.float32)
    one[:M, :M] = plane_schur(M, 0.0 if symmetric else 1.0).float()
    if symmetric:
        one[:M, :M] = torch.tril(one[:M, :M]) + torch.tril(one[:M, :M], -1).T
    few = one.repeat(2, 1, 1)
    many = one.repeat(batch, 1, 1)
    ddst().kernel_invert(few, symmetric=symmetric)
    ddst().kernel_invert(many, symmetric=symmetric)
    assert torch.equal(many, few[:1].expand_as(many))


@pytest.mark.parametrize("n,slabs", [(383, 192), (511, 256)])
def test_fp32_basis_with_a_partial_chunk(n, slabs):
    """Passes over an FP32 basis of 573 x 128 entries (the last chunk of 256 half
    full) and of whole chunks, classical and lagged steps: as many refinement
    passes as with the FP64 basis, and the same solution."""
    print(f"\n[gpu] FP32 basis n={n} slabs={slabs}", flush=True)
    mod = ddst()
    op = mod.Operator(2, n, slabs, bvec=(4.0, 1.0, 0.0), precision="fp64")
    g = torch.Generator(device="cuda").manual_seed(n)
    f = torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64)
    opts = dict(tol=1e-10, inner_tol=1e-6, max_iter=1500, max_outer=6)
    u64, _, s64 = op.solve(f, opts=mod.SolveOptions(**opts))
    u32, _, s32 = op.solve(f, opts=mod.SolveOptions(basis_fp32=True, **opts))
    op.close()
    assert s64["gmres_iters"] > 128 * s64["outer_iters"]  # lagged steps on both
    assert s32["outer_iters"] == s64["outer_iters"]
    assert float((u32 - u64).abs().max()) <= 1e-9 * float(u64.abs().max())


@pytest.mark.parametrize("factors", ["bf16", "fp32"])
@pytest.mark.parametrize("n,slabs,leaf", [(299, 10, 32), (511, 128, 128), (2303, 8, 128)])
def test_compressed_product_against_its_transpose(n, slabs, leaf, factors):
    """y = S x through the compressed blocks (rows at any alignment, planes that do
    and do not fit LDS) and z = S^T x, which another kernel forms from the same
    factors: x1.(S x2) = x2.(S^T x1) up to the FP32 sums of both, some 300 terms of
    norm 1 each."""
    print(f"\n[gpu] compressed product n={n} leaf={leaf} {factors}", flush=True)
    op = ddst().Operator(2, n, slabs, bvec=(3.0, 1.0, 0.0), precision="fp32", keep_factors=False)
    op.compress(tol=1e-5, leaf=leaf, oversample=10, max_rank=100, factor_dtype=factors)
    g = torch.Generator(device="cuda").manual_seed(n)
    M, J = op.M, op.n_ds
    x1 = torch.randn(J * M, generator=g, device="cuda", dtype=torch.float64)
    z = op.apply(x1, which="hodlr", transpose=True).reshape(-1)
    for c in (0, 1, leaf - 1, leaf, M // 2, M - 1, M, J * M // 2 + 3, J * M - 1):
        e = torch.zeros_like(x1)
        e[c] = 1.0
        col = op.apply(e, which="hodlr").reshape(-1)
        assert abs(float(col @ x1) - float(z[c])) <= 300 * 2.0 ** -24 * float(x1.norm())
    x2 = torch.randn(J * M, generator=g, device="cuda", dtype=torch.float64)
    y = op.apply(x2, which="hodlr").reshape(-1)
    assert abs(float(y @ x1 - z @ x2)) <= 300 * 2.0 ** -24 * float(x1.norm() * x2.norm())
    op.close()


@pytest.mark.parametrize("n,slabs,precision", [(511, 32, "fp32"), (1023, 64, "fp32"),
                                               (899, 60, "fp64"), (1151, 32, "fp64")])
def test_transposed_products_in_both_orders(n, slabs, precision):
    """y = S^T x of small and large launches, against the blocks themselves (FP64
    sums, 1e-12): strips of 256 columns with 127, 255 and none in the last."""
    print(f"\n[gpu] transposed products n={n} slabs={slabs} {precision}", flush=True)
    op = ddst().Operator(2, n, slabs, bvec=(5.0, 1.0, 0.0), precision=precision,
                         keep_factors=False)
    g = torch.Generator(device="cuda").manual_seed(n)
    J, M = op.n_ds, op.M
    x = torch.randn(J, M, generator=g, device="cuda", dtype=torch.float64)
    out = op.apply(x.reshape(-1), transpose=True).reshape(J, M)
    for j in (0, 1, J // 2, J - 1):
        y = x[j].clone()
        if j > 0:
            y -= (op.transfer(j)[1] * x[j - 1][:, None]).sum(0)
        if j < J - 1:
            y -= (op.transfer(j + 2)[0] * x[j + 1][:, None]).sum(0)
        assert float((out[j] - y).abs().max()) <= 1e-12 * float(y.abs().max())
    op.close()

"""The batched dense kernels past one outer block and one tile size.

Bounds: products as in test_gpu_kernels.py (2e-5 for up to 384 terms, growing
with their number); inverses 8e-5 for ld <= 640 there, growing with ld; FP32
transfer blocks against FP64 ones by tol.fp32_block_tol.
"""
import pytest
import torch

from tol import fp32_block_tol

pytestmark = pytest.mark.gpu


def ddst():
    from paper_2510_25991_amd import ddst as mod
    return mod


def relerr(a, b):
    return float((a - b).abs().max() / b.abs().max())


@pytest.mark.parametrize("batch,ld", [(900, 128), (230, 384), (228, 512), (60, 896)])
def test_many_tile_products(batch, ld):
    """FP32 batches large enough for the 256 x 256 tiles, whole and partial."""
    print(f"\n[gpu] products {batch} x {ld}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(ld)
    A = torch.randn(batch, ld, ld, generator=g, device="cuda")
    B = torch.randn(batch, ld, ld, generator=g, device="cuda")
    C = torch.empty_like(A)
    ddst().kernel_gemm(A, B, C, alpha=-1.0)
    for b in (0, batch // 2, batch - 1):
        ref = -(A[b].double() @ B[b].double())
        assert relerr(C[b].double(), ref) <= 2e-5 * max(1.0, ld / 384)


@pytest.mark.parametrize("symmetric", [False, True])
@pytest.mark.parametrize("ld,M", [(1152, 1025), (1152, 1152), (1280, 1225), (1664, 1536)])
def test_outer_block_inverse(ld, M, symmetric):
    """More rows than one outer block takes: a last block of one, two and
    three steps, and one of padding alone."""
    print(f"\n[gpu] kernel invert ld={ld} M={M} symmetric={symmetric}", flush=True)
    g = torch.Generator().manual_seed(M)
    batch = 2
    A = torch.eye(ld, dtype=torch.float64).repeat(batch, 1, 1)
    X = torch.randn(batch, M, M, generator=g, dtype=torch.float64)
    if symmetric:
        X = (X + X.transpose(1, 2)) / 2 ** 0.5
    A[:, :M, :M] = 3.0 * torch.eye(M, dtype=torch.float64) + X / M ** 0.5
    A = A.float()
    Ad = A.cuda()
    ddst().kernel_invert(Ad, symmetric=symmetric)
    ref = torch.linalg.inv(A.double())
    assert relerr(Ad.cpu().double(), ref) <= 8e-5 * ld / 640


@pytest.mark.parametrize("b", [0.0, 10.0])
@pytest.mark.parametrize("n,slabs", [(35, 6), (11, 4), (19, 5), (27, 7)])
def test_transfer_blocks_of_ragged_planes(n, slabs, b):
    """3D planes of 1225 (outer blocks), 121, 361 and 729 rows, padded to tiles;
    symmetric (transposed chains) and not."""
    print(f"\n[gpu] transfer blocks n={n} slabs={slabs} b={b}", flush=True)
    ops = [ddst().Operator(3, n, slabs, bvec=(b, 0.0, 0.0), precision=p)
           for p in ("fp32", "fp64")]
    worst = scale = 0.0
    for j in range(1, slabs):
        for x, y in zip(ops[0].transfer(j), ops[1].transfer(j)):
            worst = max(worst, float((x.double() - y.double()).abs().max()))
            scale = max(scale, float(y.abs().max()))
    for op in ops:
        op.close()
    assert worst <= fp32_block_tol((n + 1) // slabs, n * n) * scale


@pytest.mark.parametrize("n,slabs", [(15, 4), (127, 64), (255, 128), (383, 192), (511, 128), (511, 256)])
def test_krylov_passes_at_each_width(n, slabs):
    """GMRES over bases of 45 entries (less than one chunk) to 130305: one, two
    and four entries per lane, with ragged last chunks.  The estimate of the
    rotations holds for the true residual as long as the basis is orthonormal."""
    print(f"\n[gpu] Krylov passes n={n} slabs={slabs}", flush=True)
    mod = ddst()
    op = mod.Operator(2, n, slabs, bvec=(4.0, 1.0, 0.0), precision="fp64")
    g = torch.Generator(device="cuda").manual_seed(n)
    v = torch.randn(op.n_ds * op.M, generator=g, device="cuda", dtype=torch.float64)
    x, iters, relres = op.gmres(v, tol=1e-10, max_iter=2000)
    r = v - op.apply(x).reshape(-1)
    assert iters < 2000
    assert float(r.norm() / v.norm()) <= 1e-9
    op.close()


@pytest.mark.parametrize("n,slabs,leaf,levels", [(299, 10, 32, 4), (511, 128, 128, 2),
                                                 (2303, 8, 128, 5)])
@pytest.mark.parametrize("factors", ["fp64", "fp32"])
def test_compressed_product(n, slabs, leaf, levels, factors):
    """y = S x through the compressed blocks, rows that begin at any alignment
    and planes that do and do not fit LDS; the bound of the compressed operator
    (4 levels tol), FP32 factors adding their rounding."""
    print(f"\n[gpu] compressed product n={n} leaf={leaf} {factors}", flush=True)
    tol = 1e-8 if factors == "fp64" else 1e-6
    op = ddst().Operator(2, n, slabs, bvec=(3.0, 1.0, 0.0), precision="fp64")
    op.compress(tol=tol, leaf=leaf, oversample=10, max_rank=100, factor_dtype=factors)
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn(op.n_ds * op.M, generator=g, device="cuda", dtype=torch.float64)
    for transpose in (False, True):
        y = op.apply(x, which="hodlr", transpose=transpose).reshape(-1)
        ref = op.apply(x, transpose=transpose).reshape(-1)
        assert float((y - ref).norm() / x.norm()) <= 4 * levels * tol
    op.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("dim,n,slabs", [(2, 5, 3), (2, 127, 8), (2, 331, 4), (2, 899, 10),
                                         (2, 1151, 8), (3, 35, 6)])
def test_block_products(dim, n, slabs, precision):
    """y = S x, its transpose and 5 and 9 vectors at once, against the blocks
    themselves: planes with and without padding, one chunk of columns and
    several.  FP64 sums: 1e-12; with FP32 blocks too, their entries being the
    same on both sides."""
    print(f"\n[gpu] block products {dim}D n={n} {precision}", flush=True)
    op = ddst().Operator(dim, n, slabs, bvec=(5.0, 1.0, 0.0), precision=precision)
    g = torch.Generator(device="cuda").manual_seed(n)
    J, M = op.n_ds, op.M
    x = torch.randn(J, M, generator=g, device="cuda", dtype=torch.float64)
    S = [tuple(b.double() for b in op.transfer(j)) for j in range(1, J + 1)]
    y, yt = x.clone(), x.clone()
    for j in range(J):
        if j > 0:
            y[j] -= (S[j][0] * x[j - 1]).sum(1)
            yt[j] -= (S[j - 1][1] * x[j - 1][:, None]).sum(0)
        if j < J - 1:
            y[j] -= (S[j][1] * x[j + 1]).sum(1)
            yt[j] -= (S[j + 1][0] * x[j + 1][:, None]).sum(0)
    for ref, transpose in ((y, False), (yt, True)):
        out = op.apply(x.reshape(-1), transpose=transpose).reshape(J, M)
        assert relerr(out, ref) <= 1e-12
    for nrhs in (3, 9):
        F = torch.randn((nrhs,) + (n,) * dim, generator=g, device="cuda", dtype=torch.float64)
        opts = ddst().SolveOptions(tol=1e-10, max_iter=400)
        U, _ = op.solve_many(F, opts=opts)
        for v in (0, nrhs - 1):
            u = op.solve(F[v], opts=opts)[0]
            assert relerr(U[v].reshape(-1), u.reshape(-1)) <= 1e-8
    op.close()


@pytest.mark.parametrize("n,slabs,leaf", [(59, 6, 64), (99, 10, 64), (199, 10, 64), (399, 10, 64),
                                          (511, 16, 32), (1023, 16, 32)])
def test_sampled_product(n, slabs, leaf):
    """y = S x through the sampled form with trees of 1 to 32 leaves, whose upper
    levels one work-group takes.  Blocks of this operator decay fast (rank 30
    holds them far below 1e-6); a lost or misplaced node is of order 1."""
    print(f"\n[gpu] sampled product n={n} leaf={leaf}", flush=True)
    op = ddst().Operator(2, n, slabs, bvec=(3.0, 1.0, 0.0), precision="fp64")
    op.compress_hbs(rank=30, oversample=10, leaf=leaf, factor_dtype="fp64")
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn(op.n_ds * op.M, generator=g, device="cuda", dtype=torch.float64)
    for transpose in (False, True):
        y = op.apply(x, which="hbs", transpose=transpose).reshape(-1)
        ref = op.apply(x, transpose=transpose).reshape(-1)
        assert float((y - ref).norm() / ref.norm()) <= 1e-5
    op.close()


@pytest.mark.parametrize("iters", [1, 63, 64, 65, 129, 300])
def test_back_substitution_lengths(iters):
    """x = V y of a run stopped at a given length (blocks of 64 unknowns, whole and
    partial): its true residual is the one the rotations report."""
    print(f"\n[gpu] back substitution {iters}", flush=True)
    op = ddst().Operator(2, 255, 128, bvec=(4.0, 1.0, 0.0), precision="fp64")
    g = torch.Generator(device="cuda").manual_seed(7)
    v = torch.randn(op.n_ds * op.M, generator=g, device="cuda", dtype=torch.float64)
    x, used, relres = op.gmres(v, tol=1e-15, max_iter=iters, allow_notconv=True)
    r = float((v - op.apply(x).reshape(-1)).norm() / v.norm())
    assert used == iters
    assert abs(r - relres) <= 1e-10 * max(1.0, relres) + 1e-6 * relres
    op.close()

"""Batches whose rows lie so far apart that the tile chosen by size cannot address
them with 32-bit offsets: another tile takes them."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("path,n,M,N,K,lda,ldb,ldc", [
    ("f64", 0, 10, 12, 20, 5_000_000, 12, 12),          # few rows of A
    ("f64", 0, 31, 6, 2, 2, 120_000_000, 9_000_000),    # few k, C beyond 2^31 bytes
    ("3xbf16", 3, 42, 13, 3, 3, 161_000_000, 5_700_000),
    ("3xbf16", 6, 51, 5, 15, 8_100_000, 21_300_000, 5),
    ("f32", 0, 100, 8, 40, 40, (1 << 24) + 8, 8),       # 32-row slabs of B
])
def test_batch_of_far_rows(path, n, M, N, K, lda, ldb, ldc):
    """Two problems, the second's operands beside the first's in the same rows;
    small integers, exact in every precision."""
    import torch
    import paper_1902_10345_amd as mm
    dtype = torch.float64 if path == "f64" else torch.float32
    batch = 2

    def operand(rows, cols, ld):
        # (second problem `cols` further along each row where it fits, else after the first)
        step = cols if 2 * cols <= ld else (rows - 1) * ld + cols
        buf = torch.empty((rows - 1) * ld + cols + step, device="cuda", dtype=dtype)
        views = [buf[b * step:].as_strided((rows, cols), (ld, 1)) for b in range(batch)]
        return buf, step, views

    a, sa, va = operand(M, K, lda)
    b, sb, vb = operand(K, N, ldb)
    sc = (M - 1) * ldc + N
    c = torch.empty(batch * sc, device="cuda", dtype=dtype)
    g = torch.Generator().manual_seed(M + N)
    for v in va + vb:
        v.copy_(torch.randint(-9, 10, tuple(v.shape), generator=g).to(dtype))
    if path == "f64":
        mm.gemm_f64_strided_batched(M, N, K, 1.0, a, lda, sa, b, ldb, sb, 0.0, c, ldc, sc, batch)
    else:
        mm.gemm_strided_batched(mm.PATH_F32 if path == "f32" else mm.PATH_3XBF16, M, N, K, 1.0, a,
                                lda, sa, b, ldb, sb, 0.0, c, ldc, sc, batch, max(n, 3))
    for i in range(batch):
        got = c[i * sc:].as_strided((M, N), (ldc, 1)).cpu().double()
        assert torch.equal(got, va[i].cpu().double() @ vb[i].cpu().double()), i

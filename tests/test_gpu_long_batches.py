"""Batches with more output tiles than one launch holds (2^32 lanes): outer
products of one row each against a shared row of B, exact in every precision."""
import pytest

pytestmark = pytest.mark.gpu


def _check(C, a, b, chunk=4096):
    import torch
    for i in range(0, C.shape[0], chunk):
        assert torch.equal(C[i:i + chunk], a[i:i + chunk, None] * b[None, :]), i


@pytest.mark.parametrize("path", ["f32", "3xbf16", "f64"])
def test_batch_of_more_lanes_than_a_launch(path):
    """65 535 problems of 1 x N x 1: 64 lanes per 32 outputs (binary32, split
    precision), 256 per 64 (binary64), more than 2^32 in all."""
    import torch
    import paper_1902_10345_amd as mm
    batch, N = 65535, 20000 if path == "f64" else 33000
    assert batch * (-(-N // 64) * 256 if path == "f64" else -(-N // 32) * 64) >= 1 << 32
    dtype = torch.float64 if path == "f64" else torch.float32
    # small integers: every product is exact, in bf16 planes too
    a = (torch.arange(batch, device="cuda") % 127 - 63).to(dtype)
    b = (torch.arange(N, device="cuda") % 101 - 50).to(dtype)
    C = torch.full((batch, N), 7.0, device="cuda", dtype=dtype)
    if path == "f64":
        mm.gemm_f64_strided_batched(1, N, 1, 1.0, a, 1, 1, b, N, 0, 0.0, C, N, N, batch)
    else:
        mm.gemm_strided_batched(mm.PATH_F32 if path == "f32" else mm.PATH_3XBF16, 1, N, 1, 1.0, a,
                                1, 1, b, N, 0, 0.0, C, N, N, batch, 3)
    _check(C, a, b)


def test_long_single_column_product():
    """2^28 rows of one column: 32 x 32 tiles of eight waves would need 2^32
    lanes."""
    import torch
    import paper_1902_10345_amd as mm
    M = 1 << 28
    a = (torch.arange(M, device="cuda", dtype=torch.int32) % 127 - 63).float()
    b = torch.full((1, 1), 3.0, device="cuda")
    C = torch.zeros(M, device="cuda")
    mm.gemm_f32(M, 1, 1, 1.0, a, 1, b, 1, 0.0, C, 1)
    assert torch.equal(C, 3.0 * a)


def test_fp8_quantisation_of_more_lanes_than_a_launch():
    """2^25 rows and as many columns (and a few) of one element: 2^31 lanes each."""
    import torch
    import paper_1902_10345_amd as mm
    R = (1 << 25) + 40
    a = (torch.arange(R, device="cuda", dtype=torch.int32) % 127 - 63).float()
    b = (torch.arange(R, device="cuda", dtype=torch.int32) % 101 - 50).float()
    nbytes = mm.gemm_fp8_workspace_bytes(R, R, 1)
    ws = torch.full((nbytes,), 0x55, dtype=torch.uint8, device="cuda")
    mm.fp8_quantize(R, R, 1, a, 1, b, R, ws, nbytes)
    L = mm.fp8_workspace_layout(R, R, 1)
    for x, q, s in ((a, "qa", "sa"), (b, "qb", "sb")):
        codes = ws[L[q]:L[q] + R * L["Kp"]].view(R, L["Kp"])
        # one element per row: its code is that of +-448, of 0 where it is zero
        want = torch.where(x == 0, 0x00, torch.where(x < 0, 0xFE, 0x7E)).to(torch.uint8)
        assert torch.equal(codes[:, 0], want), q
        assert not bool(codes[:, 1:].any()), q
        scale = ws[L[s]:L[s] + 4 * R].view(torch.float32)
        assert torch.equal(scale, torch.where(x == 0, torch.ones_like(x),
                                              x.abs() / torch.full_like(x, 448.0))), s

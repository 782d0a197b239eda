"""Operands at any 4-byte (binary64: 8-byte) alignment: bases one to three
elements past a 256-byte boundary, odd row strides and odd K, on every path
that reads rows in 128-bit loads.  Integer inputs, so every result is exact
and is compared bit for bit with the integer product; the elements around the
operands are NaN, so a read that strays past a row shows."""
import numpy as np
import pytest

import seeded_inputs as si

pytestmark = pytest.mark.gpu

# K 1023 and 1027: around the length from which the small-product tiles turn
# their operands through LDS
SHAPES = [(65, 33, 17), (257, 130, 97), (300, 70, 255), (40, 300, 1001), (33, 65, 1023),
          (45, 70, 1027), (70, 45, 1283)]


def _placed(x, off, ld, dtype="float32"):
    """x in a NaN buffer at element offset `off` with row stride ld: (address holder, address)."""
    import torch
    rows, cols = x.shape
    buf = np.full(off + rows * ld + 8, np.nan, dtype=dtype)
    np.lib.stride_tricks.as_strided(buf[off:], (rows, cols), (ld * buf.itemsize, buf.itemsize))[:] = x
    t = torch.from_numpy(buf).cuda()
    return t, t.data_ptr() + off * buf.itemsize


def _problem(M, N, K, seed):
    A, B = si.integers((M, K), seed), si.integers((K, N), seed + 1)
    return A, B, (A.astype(np.int64) @ B.astype(np.int64)).astype(np.float32)


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("off", [1, 2, 3])
def test_every_configuration_and_transpose(M, N, K, off):
    import torch
    import paper_1902_10345_amd as mm
    A, B, want = _problem(M, N, K, M + N + K)
    hA, pA = _placed(A, off, K + off)
    hB, pB = _placed(B, 4 - off, N + 1)
    hAt, pAt = _placed(A.T, off, M + 1)
    hBt, pBt = _placed(B.T, off, K + off)
    C = torch.empty((M, N), device="cuda")
    ran = 0
    for path in (mm.PATH_F32, mm.PATH_3XBF16):
        for cfg in range(mm.gemm_num_configs(path)):
            name = mm.gemm_config_name(path, cfg)
            if K % 2 and name.endswith("kg2"):
                continue  # two equal k ranges need an even K
            C.fill_(float("nan"))
            mm.gemm_run_config(path, cfg, M, N, K, 1.0, pA, K + off, pB, N + 1, 0.0, C, N,
                               n_products=6 if "_p6" in name else 3)
            assert np.array_equal(C.cpu().numpy(), want), name
            ran += 1
        for n in ((3,) if path == mm.PATH_F32 else (3, 6)):
            for ta in (False, True):
                for tb in (False, True):
                    C.fill_(float("nan"))
                    mm.gemm_ex(mm.ROW_MAJOR, mm.TRANS if ta else mm.NO_TRANS,
                               mm.TRANS if tb else mm.NO_TRANS, M, N, K, 1.0,
                               pAt if ta else pA, M + 1 if ta else K + off,
                               pBt if tb else pB, K + off if tb else N + 1, 0.0, C, N, path, n)
                    assert np.array_equal(C.cpu().numpy(), want), (path, n, ta, tb)
    assert ran > 15


@pytest.mark.parametrize("off", [1, 2, 3])
def test_grouped_and_batched(off):
    import torch
    import paper_1902_10345_amd as mm
    keep, probs, wants = [], [], []
    for t, (M, N, K) in enumerate(SHAPES + [(5, 7, 3), (64, 64, 64)]):
        A, B, want = _problem(M, N, K, 50 + t)
        (hA, pA), (hB, pB) = _placed(A, off, K + 1), _placed(B, off, N + 2)
        C = torch.full((M, N), float("nan"), device="cuda")
        keep.append((hA, hB, C))
        probs.append((M, N, K, pA, K + 1, pB, N + 2, C, N, 1.0, 0.0))
        wants.append(want)
    wsb = mm.grouped_gemm_workspace_bytes(len(probs))
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    mm.grouped_gemm(mm.problem_array(probs), len(probs), mm.PATH_3XBF16, None, ws, wsb)
    for (_, _, C), want in zip(keep, wants):
        assert np.array_equal(C.cpu().numpy(), want)
    for (M, N, K) in [(31, 17, 33), (64, 40, 19), (100, 72, 91), (130, 9, 35)]:
        batch, sa = 5, M * (K + 1) + off
        A = si.integers((batch * M, K), K).reshape(batch, M, K)
        B = si.integers((K, N), K + 1)
        buf = np.full(off + batch * sa + 4, np.nan, dtype=np.float32)
        for b in range(batch):
            np.lib.stride_tricks.as_strided(buf[off + b * sa:], (M, K), ((K + 1) * 4, 4))[:] = A[b]
        dA = torch.from_numpy(buf).cuda()
        hB, pB = _placed(B, off, N + 1)
        want = (A.astype(np.int64) @ B.astype(np.int64)).astype(np.float32)
        for path, n in ((mm.PATH_F32, 3), (mm.PATH_3XBF16, 3), (mm.PATH_3XBF16, 6)):
            C = torch.full((batch, M, N), float("nan"), device="cuda")
            mm.gemm_strided_batched(path, M, N, K, 1.0, dA.data_ptr() + 4 * off, K + 1, sa, pB,
                                    N + 1, 0, 0.0, C, N, M * N, batch, n)
            assert np.array_equal(C.cpu().numpy(), want), (M, N, K, path, n)


@pytest.mark.parametrize("M,N,K", SHAPES + [(16, 16, 5), (30, 31, 37), (64, 50, 33)])
def test_binary64(M, N, K):
    import torch
    import paper_1902_10345_amd as mm
    A, B, want = _problem(M, N, K, 9 * M + K)
    (hA, pA), (hB, pB) = _placed(A, 1, K + 1, "float64"), _placed(B, 3, N + 1, "float64")
    for cfg in range(mm.gemm_num_configs(mm.PATH_F64)):
        name = mm.gemm_config_name(mm.PATH_F64, cfg)
        if "small_" in name and max(M, N) > int(name.rsplit("_", 1)[1]):
            continue
        C = torch.full((M, N), float("nan"), dtype=torch.float64, device="cuda")
        mm.gemm_f64_run_config(cfg, M, N, K, 1.0, pA, K + 1, pB, N + 1, 0.0, C, N)
        assert np.array_equal(C.cpu().numpy(), want.astype(np.float64)), name

"""Which kernel a bf16 product goes to, on the host (256 compute units where there is no device)."""
import numpy as np
import pytest

from paper_2311_10418_amd import binding as ds
from helpers import gemm_launches

LARGE = ("256", "192", "128")                        # the kernel that addresses 128 rows of its output through one 32-bit buffer length


def _widths(around):
    return [around + 256 * i for i in (-2, -1, 0, 1, 2)]


@pytest.mark.parametrize("around", [1 << 22, 1 << 23, 1 << 24, 1 << 25])
def test_wide_outputs_stay_on_the_matrix_cores(around):
    """Outputs of which 128 rows are longer than 2^32 bytes go to the smaller tiles, and where the stage wants column sums (a layer of that
    inner width) the kernels that give them still do: no width falls back to the plain kernel, which gives none."""
    for N in _widths(around):
        for M in (1, 130, 700):
            for epi, bytes_ in ((ds.DS_EPI_NONE, 2), (ds.DS_EPI_MULR, 2), (ds.DS_EPI_DGELU, 2), (ds.DS_EPI_ACC32, 4)):
                for colsum in ((False, True) if epi in (ds.DS_EPI_MULR, ds.DS_EPI_DGELU) else (False,)):
                    l = gemm_launches(M, N, 64, epilogue=epi, ws_floats=1 << 24, colsum=colsum)
                    assert l and sum(x["rows"] for x in l) == M
                    if 128 * N * bytes_ >= 1 << 32:
                        assert all(x["tile"] not in LARGE for x in l), (N, M, epi)
                    if colsum:
                        assert all(x["tile"] not in ("192", "64x64") and x["splits"] == 1 for x in l), (N, M, epi)


@pytest.mark.parametrize("around", [1 << 23, 1 << 24, 1 << 25])
def test_wide_weight_gradients(around):
    """The same for weight gradients, up to 2^25 either way (a K tile is addressed through a 32-bit length), where the plain kernel takes over."""
    for wide in _widths(around):
        for M, N in ((256, wide), (wide, 256)):
            l = gemm_launches(M, N, 100, trans_a=True, epilogue=ds.DS_EPI_ACC32)
            assert len(l) == (1 if wide <= 1 << 25 else 0), (M, N)
            if l and 128 * N * 4 >= 1 << 32:
                assert l[0]["tile"] not in LARGE, (M, N)


def test_launches_cover_the_rows_once():
    rng = np.random.default_rng(3)
    for _ in range(3000):
        M, N, K = int(2 ** rng.uniform(0, 17)), 256 * int(rng.integers(1, 65)), 64 * int(2 ** rng.uniform(0, 7))
        colsum = bool(rng.random() < 0.3)
        l = gemm_launches(M, N, K, epilogue=ds.DS_EPI_MULR, ws_floats=int(rng.choice([0, 1 << 20, 1 << 24])), colsum=colsum)
        assert 1 <= len(l) <= 2 and sum(x["rows"] for x in l) == M and all(x["rows"] > 0 for x in l)
        if len(l) == 2:
            assert l[0]["rows"] % 256 == 0
        for x in l:
            tiles = (x["rows"] + 255) // 256 * (N // 256)
            if x["tile"] == "256":
                assert x["splits"] == 1 and 0 <= x["whole"] <= tiles and (x["pieces"] > 1) == (x["whole"] < tiles)
                assert not x["persistent"] or x["whole"] >= 512
            if colsum:
                assert x["tile"] not in ("192", "64x64")


def test_fp32_outputs_of_nt_products_split_into_long_pieces():
    """Contractions of 2 816 are cut in two at most (pieces of 1 024 and more): on 204 large tiles, whole."""
    l = gemm_launches(4318, 3072, 2816, epilogue=ds.DS_EPI_ACC32, ws_floats=1 << 26)
    assert [(x["tile"], x["splits"]) for x in l] == [("256", 1)]


def test_gelu_derivative_keeps_off_the_128_row_tile():
    """Its epilogue takes longer there than the K loop saves, alone of the epilogues."""
    for M, N, K in ((6700, 1024, 128), (3633, 2048, 2816), (9130, 768, 768)):
        assert [x["tile"] for x in gemm_launches(M, N, K, epilogue=ds.DS_EPI_MULR, ws_floats=1 << 24)] == ["128"]
        assert [x["tile"] for x in gemm_launches(M, N, K, epilogue=ds.DS_EPI_DGELU, ws_floats=1 << 24)] == ["128x128/2"]

"""Results of 256 tiles and more, the sizes at which FP8 products take k-steps of two stages and products are stored past the caches:
every entry equal to the same call in panels of fewer tiles (other kernels), and entries at the edges of tiles equal to the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import ozaki_oracle as oz  # noqa: E402
from paper_2508_00441_amd import binding as lib, device  # noqa: E402


# FP8: two, three (odd) and even numbers of k-steps per pair, a last stage of zeros (161 stages; 163: an even number of steps), pairs too
# short for that (2, 3 and 65 stages), ragged edges, measured runs (k = 16384 and, with a stage of zeros, 16400: a few pairs fill the window); products stored past the caches in every format
@pytest.mark.parametrize("fmt,m,n,k,s,pairs", [("fp8", 4096, 4080, 128, 4, "triangle"), ("fp8", 4090, 4100, 384, 3, "full"), ("fp8", 4096, 4096, 4160, 3, "triangle"),
                                               ("fp8", 4095, 4097, 180, 5, "triangle"), ("fp8", 4096, 4100, 250, 4, "triangle"),
                                               ("fp8", 4093, 4096, 10300, 3, "triangle"), ("fp8", 4096, 4090, 10420, 2, "full"), ("fp8", 3841, 4100, 16400, 12, "triangle"),
                                               ("fp8", 3900, 4200, 512, 9, "triangle"), ("fp8", 3900, 4200, 500, 9, "triangle"),
                                               ("fp8", 3841, 4096, 16384, 12, "triangle"), ("fp6", 4096, 3999, 128, 9, "triangle"),
                                               ("int8", 4001, 4096, 320, 9, "triangle"), ("int8", 4001, 4096, 256, 9, "triangle"), ("fp16", 4096, 4096, 1024, 9, "triangle")])
def test_large_results(fmt, m, n, k, s, pairs):
    gen = torch.Generator(device="cuda").manual_seed(m + n + k)
    draw = lambda r, c: torch.randn((r, c), dtype=torch.float64, device="cuda", generator=gen).mul_(torch.randn((r, c), dtype=torch.float64, device="cuda", generator=gen).exp_())
    A, B = draw(k, m), draw(n, k)                            # column-major m x k and k x n
    A[:, 40] *= 2.0 ** 9                                     # rows and columns off their group's ladder of units
    A[:, 300] = torch.round(A[:, 300])
    B[70, :] = torch.round(B[70, :] * 4.0)
    f, ps = lib.SLICE_FORMATS[fmt], lib.PAIR_SETS[pairs]
    lib.ozaki_set_stream(torch.cuda.current_stream().cuda_stream)
    ws = device.Workspace.for_problem(m, n, k, f, s, 0, pair_set=ps)
    half = lib.ozaki_workspace_bytes_ex((m + 1) // 2 // 256 * 256 + 256, n, k, f, s, 0, ps, True)
    got = []
    for cap in (0, half):
        C = torch.full((n, m), float("nan"), dtype=torch.float64, device="cuda")
        lib.ozaki_dgemm_ex(m, n, k, A, m, B, k, C, m, f, s, 0, lib.ACCUM_MODES["emu"], ps, lib.SUM_RUNS, cap)
        assert lib.ozaki_last_device_status() == 0
        got.append(C)
    ws.close()
    assert torch.equal(got[0].view(torch.int64), got[1].view(torch.int64))
    rows = [0, 15, 16, 31, 32, 40, 127, 128, 255, 256, 300, m - 1]
    cols = [0, 15, 16, 31, 32, 70, 127, 128, 255, 256, n // 2, n - 1]
    want = oz.ozaki_dgemm(A[:, rows].T.cpu().numpy(), B[cols, :].T.cpu().numpy(), fmt, s, 0, mode=pairs, accumulate="runs")
    C = got[0][cols, :][:, rows].T.cpu().numpy()
    assert np.array_equal(np.ascontiguousarray(C).view(np.uint64), np.ascontiguousarray(want).view(np.uint64))

"""C = alpha (A B) + beta C formed in the last accumulation: every accumulation mode, floating-point and integer products, results of more
positions than the kernels for few of them take, several blocks of the inner dimension, several passes over the pairs in a small work
memory, padded leading dimensions: bit for bit one rounded multiplication per term and one rounded addition on the plain call's
product (whose bits other tests hold against the oracle), C not read where beta is 0 and nothing written beside it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2508_00441_amd import binding as lib, device, inputs  # noqa: E402

FMT, ACC = lib.SLICE_FORMATS, lib.ACCUM_MODES


@pytest.mark.parametrize("accum", ["hw", "emu", "exact"])
@pytest.mark.parametrize("fmt,m,n,k,k_block,s,small", [
    ("fp8", 777, 801, 300, 0, 9, False),           # 650 positions, ragged
    ("int8", 801, 777, 300, 0, 7, False),
    ("fp8", 640, 900, 260, 0, 8, True),            # several passes over the pairs
    ("int8", 900, 640, 260, 0, 6, True),
    ("fp16", 777, 801, 700, 256, 5, False),        # three blocks
    ("fp6", 770, 830, 500, 192, 7, True),          # three blocks of several passes each
    ("int8", 300, 270, 500, 200, 6, False),        # few positions
    ("fp8", 1200, 1100, 64, 0, 6, False),          # more than 1024 positions
])
def test_scaled_call_is_the_plain_product_scaled(fmt, m, n, k, k_block, s, small, accum):
    A, B = inputs.phi_pair(m, n, k, 1.0, seed=m + n + k)
    Ad, Bd = device.to_device_colmajor(A), device.to_device_colmajor(B)
    blocks = -(-k // (k_block or k))
    args = (FMT[fmt], s, k_block)
    ws = device.Workspace.for_problem(m, n, k, *args)
    P = torch.full((n, m), float("nan"), dtype=torch.float64, device="cuda")
    lib.ozaki_dgemm(m, n, k, Ad, m, Bd, k, P, m, *args, ACC[accum])
    assert lib.ozaki_last_device_status() == 0
    P = P.cpu().numpy()
    ws.close()
    need = lib.ozaki_workspace_bytes_scaled(m, n, k, *args)
    if small:
        need = lib.ozaki_workspace_min_bytes(m, n, k, *args) + 8 * m * n + 4096
    ws = device.Workspace(need)
    ldc = m + 5
    C0 = inputs.phi_matrix(n, m, 2.0, np.random.default_rng(m * n))
    for alpha, beta in ((-1.0, 1.0), (0.3, -1.7), (-2.5, 0.0)):
        start = np.full((n, ldc), np.nan)
        if beta != 0.0:
            start[:, :m] = C0
        Cd = torch.from_numpy(start).cuda()
        lib.ozaki_profile_enable(True)
        lib.ozaki_dgemm_scaled(m, n, k, alpha, Ad, m, Bd, k, beta, Cd, ldc, *args, ACC[accum])
        assert lib.ozaki_last_device_status() == 0
        launches = lib.ozaki_profile_read()[1]
        lib.ozaki_profile_enable(False)
        assert launches[2] > blocks if small else launches[2] == blocks, launches
        got = Cd.cpu().numpy()
        assert np.all(np.isnan(got[:, m:]))
        want = alpha * P if beta == 0.0 else alpha * P + beta * C0
        assert np.array_equal(np.ascontiguousarray(got[:, :m]).view(np.uint64), want.view(np.uint64)), (alpha, beta)
    ws.close()


@pytest.mark.parametrize("accum", ["hw", "emu"])
def test_scaled_call_without_inner_dimension(accum):
    """C = beta C, and its time among the accumulation's."""
    m, n, ldc = 70, 33, 73
    C0 = inputs.phi_matrix(n, m, 2.0, np.random.default_rng(7))
    start = np.full((n, ldc), np.nan)
    start[:, :m] = C0
    Cd, X = torch.from_numpy(start).cuda(), torch.zeros(8, dtype=torch.float64, device="cuda")
    args = (FMT["fp8"], 4, 0)
    ws = device.Workspace(lib.ozaki_workspace_bytes_scaled(m, n, 0, *args) + 4096)
    lib.ozaki_profile_enable(True)
    lib.ozaki_dgemm_scaled(m, n, 0, 2.0, X, m, X, 1, -1.7, Cd, ldc, *args, ACC[accum])
    assert lib.ozaki_last_device_status() == 0
    assert lib.ozaki_profile_read()[1] == [0, 0, 1]
    lib.ozaki_profile_enable(False)
    got = Cd.cpu().numpy()
    assert np.all(np.isnan(got[:, m:]))
    assert np.array_equal(got[:, :m], 2.0 * 0.0 + -1.7 * C0)
    ws.close()

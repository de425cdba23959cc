"""Lines on right-angle transforms (conv1d_ra.hip): the single-pass kernels (512 to 8192 complex points, 8 and 16 per
lane) and the three-pass ones (4 to 512 columns' points), at their edges: one point above and below a transform, the
three modes, calls below and above the points-per-lane rule, forward, backward and the operator, and a small
workspace; against the oracle, within the plans' tolerances (relative L2: fp32 1e-5, bf16 2e-2)."""
import numpy as np
import pytest

import oracle
from paper_2607_19378_amd import workloads as W
from gpu_util import TOL, from_device, log, oracle_ref, per_line_worst, rel_l2, run_gpu, to_device

pytestmark = pytest.mark.gpu


def _ref(inp):
    w = inp.workload
    if w.pad_mode != "circular":
        return oracle_ref(inp)
    x1, x2, v, k, D = inp.as_f64()  # the oracle's circular FFT takes powers of two: numpy's serves here
    u, L = x1 * v, w.grid[0]
    return x2 * (np.fft.irfft(np.fft.rfft(u) * np.fft.rfft(k), n=L) + D[None, :, None] * u)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,mode", [(512, "linear"), (257, "centered"), (1023, "linear"), (1024, "centered"),
                                    (2047, "centered"), (3001, "circular"), (4096, "linear"), (4097, "linear"),
                                    (8191, "circular"), (8192, "centered"), (8193, "linear"), (16384, "centered"),
                                    (40000, "circular"), (65537, "linear"), (300001, "centered"), (1 << 20, "linear")])
def test_forward(L, mode, dtype):
    from paper_2607_19378_amd import hyenand as H
    log(f"ra1d forward {L} {mode} {dtype}")
    inp = W.random_case(1, 2, (L,), mode, dtype, seed=L % 1000)
    y = run_gpu(inp)
    assert per_line_worst(y, _ref(inp), 2) <= TOL[dtype]
    small = run_gpu(inp, workspace_bytes=H.workspace_min(inp.workload.shape, mode, dtype))
    assert np.array_equal(y, small)


@pytest.mark.parametrize("L", [2048, 4000])
def test_many_lines(L):
    """More than 512 lines take 16 points per lane, fewer 8."""
    inp = W.random_case(3, 171, (L,), "linear", "f32", seed=3)
    assert per_line_worst(run_gpu(inp), oracle_ref(inp), 513) <= TOL["f32"]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,mode", [(257, "linear"), (512, "centered"), (1000, "centered"), (2048, "linear"),
                                    (3000, "centered"), (8192, "linear"), (5001, "centered"), (8193, "centered"),
                                    (16384, "linear"), (20001, "linear")])
def test_backward(L, mode, dtype):
    import torch
    from paper_2607_19378_amd import hyenand as H
    log(f"ra1d backward {L} {mode} {dtype}")
    inp = W.random_case(2, 1, (L,), mode, dtype, seed=L % 997)
    gy = W.quantise(np.random.default_rng(9).standard_normal(inp.workload.shape), dtype)
    dev = [to_device(a, dtype) for a in (inp.x1, inp.x2, inp.v, inp.k, inp.D, gy)]
    got = H.backward(*dev, pad_mode=mode)
    torch.cuda.synchronize()
    ref = oracle.backward_direct(*inp.as_f64(), W.storage_to_f64(gy, dtype), mode)
    for name, g, r in zip(("gx1", "gx2", "gv", "gk", "gD"), got, ref):
        assert rel_l2(from_device(g), r) <= TOL[dtype], name


@pytest.mark.parametrize("L,mode", [(3000, "linear"), (8192, "centered"), (32768, "linear")])
def test_operator(L, mode):
    import torch
    from paper_2607_19378_amd import hyenand as H
    rng = np.random.default_rng(5)
    shape = (2, 3, L)
    q, kin, vin = (rng.standard_normal(shape).astype(np.float32) for _ in range(3))
    k = (rng.standard_normal(oracle.kernel_shape(shape, mode)) / np.sqrt(L)).astype(np.float32)
    D, wi, wo = (rng.standard_normal(3).astype(np.float32) for _ in range(3))
    y = H.operator(*[torch.from_numpy(a).cuda() for a in (q, kin, vin, k, D, wi, wo)], pad_mode=mode)
    torch.cuda.synchronize()
    ref = oracle.operator(*[a.astype(np.float64) for a in (q, kin, vin, k, D, wi, wo)], pad_mode=mode)
    assert rel_l2(from_device(y), ref) <= TOL["f32"]

"""Single-pass 2D kernels on right-angle row transforms (conv2d_ra.hip): every transform grid they are built for
(one and two rounds of rows per signal), both modes, fp32 and bf16, forward and backward, an odd number of images,
against the fp64 oracle, within the plans' tolerances (relative L2: fp32 1e-5, bf16 2e-2); lines of very different
scales keep their own accuracy."""
import numpy as np
import pytest

import oracle
from paper_2607_19378_amd import workloads as W
from gpu_util import TOL, from_device, log, per_line_worst, rel_l2, run_gpu, to_device

pytestmark = pytest.mark.gpu

GRIDS = [(16, 16), (16, 32), (32, 16), (32, 32), (32, 64), (64, 32), (64, 64)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("mode", ["linear", "centered"])
@pytest.mark.parametrize("grid", GRIDS)
def test_forward_and_backward(grid, mode, dtype):
    import torch
    from paper_2607_19378_amd import hyenand as H
    inp = W.random_case(1, 3, grid, mode, dtype, seed=700 + sum(grid))
    log(f"ra2d {grid} {mode} {dtype}")
    assert H.plan_name(inp.workload.shape, mode, dtype) == "fused2d"
    y = run_gpu(inp)
    f = inp.as_f64()
    assert per_line_worst(y, oracle.conv_fft(*f, mode), 3) <= TOL[dtype]
    gy = W.quantise(np.random.default_rng(5).standard_normal(inp.workload.shape), dtype)
    dev = [to_device(a, dtype) for a in (inp.x1, inp.x2, inp.v, inp.k, inp.D, gy)]
    got = H.backward(*dev, pad_mode=mode)
    torch.cuda.synchronize()
    bwd = oracle.backward_direct if mode == "centered" else oracle.backward_fft
    for name, g, r in zip(("gx1", "gx2", "gv", "gk", "gD"), got, bwd(*f, W.storage_to_f64(gy, dtype), mode)):
        assert tuple(g.shape) == tuple(r.shape)
        assert rel_l2(from_device(g), r) <= TOL[dtype], name


RAGGED = [(9, 9), (14, 14), (9, 17), (16, 31), (17, 9), (32, 17), (28, 28), (31, 33), (57, 40), (33, 64), (64, 33), (63, 63)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("mode", ["linear", "centered", "circular"])
@pytest.mark.parametrize("grid", RAGGED)
def test_other_extents(grid, mode, dtype):
    """The smallest and largest extents of each transform grid, one and both axes off a power of two."""
    import torch
    from paper_2607_19378_amd import hyenand as H
    inp = W.random_case(1, 3, grid, mode, dtype, seed=800 + sum(grid))
    log(f"ra2d {grid} {mode} {dtype}")
    f = inp.as_f64()
    x1, x2, v, k, D = f
    u = x1 * v
    if mode == "circular":  # the oracle's circular FFT takes powers of two: numpy's serves here
        ref = x2 * (np.fft.irfftn(np.fft.rfftn(u, axes=(2, 3)) * np.fft.rfftn(k, axes=(-2, -1)), s=grid, axes=(2, 3))
                    + D[None, :, None, None] * u)
    else:
        ref = oracle.conv_fft(*f, mode)
    assert per_line_worst(run_gpu(inp), ref, 3) <= TOL[dtype]
    if mode == "circular":
        return
    gy = W.quantise(np.random.default_rng(5).standard_normal(inp.workload.shape), dtype)
    dev = [to_device(a, dtype) for a in (inp.x1, inp.x2, inp.v, inp.k, inp.D, gy)]
    got = H.backward(*dev, pad_mode=mode)
    torch.cuda.synchronize()
    for name, g, r in zip(("gx1", "gx2", "gv", "gk", "gD"), got,
                          oracle.backward_direct(*f, W.storage_to_f64(gy, dtype), mode)):
        assert tuple(g.shape) == tuple(r.shape)
        assert rel_l2(from_device(g), r) <= TOL[dtype], name


@pytest.mark.parametrize("mode", ["linear", "centered"])
def test_lines_of_different_scales(mode):
    """u and k of a line are transformed apart, and lines never share a transform: scales 1e6 apart between lines
    and 1e4 between u and k change no line's relative error."""
    inp = W.random_case(1, 4, (32, 32), mode, "f32", seed=77)
    scale = np.array([1e-3, 1e3, 1.0, 1e2], dtype=np.float32).reshape(1, 4, 1, 1)
    inp.x1 *= scale
    inp.k *= np.float32(1e-4)
    inp.D *= np.float32(1e-4)
    assert per_line_worst(run_gpu(inp), oracle.conv_fft(*inp.as_f64(), mode), 4) <= TOL["f32"]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("u,k", [(1e37, 1e-30), (1e30, 1e-36)])
@pytest.mark.parametrize("grid,mode,forward", [((14, 14), "linear", True), ((14, 14), "centered", True),
                                               ((17, 28), "centered", True), ((22, 22), "linear", True),
                                               ((28, 28), "centered", False)])
def test_magnitudes_near_the_range(grid, mode, forward, u, k, dtype):
    """Images of the mixed plan (28 x 28: its backward) scale u, h and k by powers of two: sums of u that leave fp32's
    range, and kernels that the normalisation of the inverse would make subnormal, change no line's relative error."""
    import torch
    from paper_2607_19378_amd import hyenand as H
    rng = np.random.default_rng(31 + sum(grid))
    shape = (1, 3) + grid
    x1 = np.abs(rng.standard_normal(shape)) * u  # one sign: the DC bin is the sum of all
    x2, v, gy = rng.standard_normal(shape), np.ones(shape), 1e-3 * rng.standard_normal(shape)
    kern = rng.standard_normal(oracle.kernel_shape(shape, mode)) * k
    D = rng.standard_normal(3) * k
    arrays = [W.quantise(a, dtype) for a in (x1, x2, v, kern, D, gy)]
    dev = [to_device(a, dtype) for a in arrays]
    log(f"ra2d range {grid} {mode} {dtype} {u:g} {k:g}")
    assert (H.plan_name(shape, mode, dtype) == "mixed2d") == forward
    y = H.fftconv(*dev[:5], pad_mode=mode)
    got = H.backward(*dev, pad_mode=mode)
    torch.cuda.synchronize()
    f = [W.storage_to_f64(a, dtype) for a in arrays]
    assert not forward or per_line_worst(from_device(y), oracle.conv_fft(*f[:5], mode), 3) <= TOL[dtype]
    for name, g, r in zip(("gx1", "gx2", "gv", "gk"), got, oracle.backward_direct(*f, mode)):
        assert per_line_worst(from_device(g), r, 3) <= TOL[dtype], name

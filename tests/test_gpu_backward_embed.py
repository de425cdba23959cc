"""Backward of the centred mode and of grid extents that are not powers of
two, every pad mode, off the mixed-radix kernels (HYENAND_PLAN=nomixed;
tests/test_gpu_backward_mixed.py covers those): the circular backward on the
transform grid of the embedded tensors (circular mode, and centred lines of up
to 256 points) with each circular plan underneath, and the right-angle kernels
(the rest), against the oracle's direct-sum backward, every gradient, fp32 and
bf16, 1D/2D/3D."""
import os

import numpy as np
import pytest

import oracle
from paper_2607_19378_amd import workloads as W

from gpu_util import TOL, from_device, log, rel_l2, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prev = os.environ.get("HYENAND_PLAN")
    os.environ["HYENAND_PLAN"] = "nomixed"
    yield
    if prev is None:
        del os.environ["HYENAND_PLAN"]
    else:
        os.environ["HYENAND_PLAN"] = prev


def _check(shape, mode, dtype, seed):
    import torch
    from paper_2607_19378_amd import hyenand as H
    rng = np.random.default_rng(seed)
    kshape = oracle.kernel_shape(shape, mode)
    npts = int(np.prod(kshape[2:]))
    x1, x2, v, gy = (W.quantise(rng.standard_normal(shape), dtype) for _ in range(4))
    k = W.quantise(rng.standard_normal(kshape) / np.sqrt(npts), dtype)
    D = W.quantise(rng.standard_normal(shape[1]), dtype)
    dev = [to_device(a, dtype) for a in (x1, x2, v, k, D, gy)]
    outs = H.backward(*dev, pad_mode=mode)
    torch.cuda.synchronize()
    f = [W.storage_to_f64(a, dtype) for a in (x1, x2, v, k, D, gy)]
    refs = oracle.backward_direct(*f, pad_mode=mode)
    names = ("gx1", "gx2", "gv", "gk", "gD")
    errs = {n: rel_l2(from_device(o), r) for n, o, r in zip(names, outs, refs)}
    log(f"[bwd-embed] {shape} {mode} {dtype}: " + " ".join(f"{n}={e:.2e}" for n, e in errs.items()))
    for n, o in zip(names, outs):
        assert tuple(o.shape) == tuple(refs[names.index(n)].shape)
    assert max(errs.values()) <= TOL[dtype], errs


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(2, 3, 1), (2, 3, 2), (2, 3, 64), (1, 3, 1000), (2, 2, 16, 16), (1, 2, 32, 32),
                                   (1, 2, 7, 30), (1, 2, 4, 8, 8), (1, 2, 5, 6, 7)])
def test_centered(shape, dtype):
    _check(shape, "centered", dtype, 11 + sum(shape))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(2, 3, 3), (2, 3, 100), (1, 2, 3000), (2, 2, 14, 14), (1, 2, 50, 60),
                                   (1, 2, 5, 6, 7)])
def test_other_extents(shape, dtype):
    _check(shape, "linear", dtype, 21 + sum(shape))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(2, 3, 3), (2, 3, 12), (1, 2, 1000), (2, 2, 14, 14), (1, 2, 7, 30),
                                   (1, 2, 5, 6, 7)])
def test_circular_other_extents(shape, dtype):
    """Circular mode on extents that are not powers of two: the periodic
    kernel embedded on the centred grid; gk gathers both displacements."""
    _check(shape, "circular", dtype, 41 + sum(shape))


def test_centered_long_line():
    """2^14 points centred: the three-pass right-angle lines."""
    _check((1, 2, 1 << 14), "centered", "f32", 31)


def test_circular_long_line_four_step():
    """12000 points: a 2^15-point circular four-step backward underneath the embedded copies."""
    from paper_2607_19378_amd import hyenand as H
    assert H.plan_name((1, 2, 1 << 15), "circular", "f32") == "fourstep1d"
    assert H.backward_workspace_min((1, 2, 12000), "circular", "f32") > 9 * 2 * (1 << 15) * 4
    _check((1, 2, 12000), "circular", "f32", 33)


def test_circular_image_multipass():
    """60 x 50: the 128 x 128 circular grid runs the multi-pass backward underneath the embedded copies."""
    from paper_2607_19378_amd import hyenand as H
    assert H.backward_workspace_min((1, 2, 128, 128), "circular", "f32") > 256
    assert H.backward_workspace_min((1, 2, 60, 50), "circular", "f32") > 9 * 2 * 128 * 128 * 4
    _check((1, 2, 60, 50), "circular", "f32", 32)
    _check((1, 2, 64, 64), "centered", "f32", 32)  # in one pass on right angles

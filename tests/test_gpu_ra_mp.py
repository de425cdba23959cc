"""Multi-pass kernels on right-angle rows (conv_ra_mp.hip, conv_ra_slab.hip): non-circular 2D and 3D grids of any
extents, forward and backward, at the edges of their transforms: one point below and above a power of two on each
axis, rows from 16 to 512 complex points (two and three passes), planes in the slab passes (one and two foldings)
and outside them, periodic kernels, and a small workspace; against the oracle, within the plans' tolerances (relative
L2: fp32 1e-5, bf16 2e-2)."""
import numpy as np
import pytest

import oracle
from paper_2607_19378_amd import workloads as W
from gpu_util import TOL, from_device, log, oracle_ref, rel_l2, run_gpu, to_device

pytestmark = pytest.mark.gpu

GRIDS = [((200, 150), "centered"), ((65, 257), "centered"), ((129, 128), "linear"), ((16, 512), "centered"),
         ((300, 9), "linear"), ((70, 90), "circular"), ((17, 33, 49), "centered"), ((48, 48, 48), "centered"),
         ((9, 65, 127), "centered"), ((5, 128, 128), "linear"), ((20, 24, 28), "linear"), ((3, 129, 130), "centered"),
         ((11, 40, 100), "circular")]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("grid,mode", GRIDS)
def test_forward(grid, mode, dtype):
    from paper_2607_19378_amd import hyenand as H
    log(f"ra_mp forward {grid} {mode} {dtype}")
    inp = W.random_case(1, 2, grid, mode, dtype, seed=40 + sum(grid))
    w = inp.workload
    y = run_gpu(inp)
    x1, x2, v, k, D = inp.as_f64()
    if mode == "circular":  # the oracle's circular FFT takes powers of two: numpy's serves here
        ax = tuple(range(2, 2 + len(grid)))
        u = x1 * v
        ref = x2 * (np.fft.irfftn(np.fft.rfftn(u, axes=ax) * np.fft.rfftn(k, axes=ax), s=grid, axes=ax)
                    + D.reshape((1, 2) + (1,) * len(grid)) * u)
    else:
        ref = oracle_ref(inp)
    assert rel_l2(y, ref) <= TOL[dtype]
    small = run_gpu(inp, workspace_bytes=H.workspace_min(w.shape, mode, dtype))
    assert np.array_equal(y, small)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("grid,mode", [((65, 33), "linear"), ((72, 40), "centered"), ((7, 70, 18), "centered"),
                                       ((6, 17, 33), "linear"), ((3, 20, 65), "centered"), ((4, 65, 65), "linear")])
def test_backward(grid, mode, dtype):
    import torch
    from paper_2607_19378_amd import hyenand as H
    log(f"ra_mp backward {grid} {mode} {dtype}")
    inp = W.random_case(2, 2, grid, mode, dtype, seed=60 + sum(grid))
    gy = W.quantise(np.random.default_rng(9).standard_normal(inp.workload.shape), dtype)
    dev = [to_device(a, dtype) for a in (inp.x1, inp.x2, inp.v, inp.k, inp.D, gy)]
    got = H.backward(*dev, pad_mode=mode)
    torch.cuda.synchronize()
    ref = oracle.backward_direct(*inp.as_f64(), W.storage_to_f64(gy, dtype), mode)
    for name, g, r in zip(("gx1", "gx2", "gv", "gk", "gD"), got, ref):
        assert rel_l2(from_device(g), r) <= TOL[dtype], name


@pytest.mark.parametrize("grid,mode", [((4, 128, 128), "linear"), ((3, 40, 100), "centered"), ((5, 48, 48), "centered"),
                                       ((4, 33, 20), "linear"), ((4, 20, 60), "circular")])
def test_slab_and_axis_passes_agree(monkeypatch, grid, mode):
    """HYENAND_SLAB=0 takes the rows and axis-1 passes in place of the slab ones (two foldings, one, 32-point rows):
    other bits, the same values, forward and backward."""
    import torch
    from paper_2607_19378_amd import hyenand as H
    inp = W.random_case(1, 2, grid, mode, "f32", seed=70 + sum(grid))
    gy = np.random.default_rng(9).standard_normal(inp.workload.shape).astype(np.float32)
    dev = [to_device(a, "f32") for a in (inp.x1, inp.x2, inp.v, inp.k, inp.D, gy)]
    out = {}
    for slab in ("1", "0"):
        monkeypatch.setenv("HYENAND_SLAB", slab)
        log(f"ra_mp slab {slab} {grid} {mode}")
        res = [H.fftconv(*dev[:5], pad_mode=mode)]
        if mode != "circular":  # embedded
            res += H.backward(*dev, pad_mode=mode)[:4]
        torch.cuda.synchronize()
        out[slab] = [from_device(t) for t in res]
    for a, b in zip(out["1"], out["0"]):
        assert not np.array_equal(a, b) and rel_l2(a, b) <= 1e-6


# relative L2 error (1e-7) of y and gk with the packed real transforms, which the right-angle rows replaced, on the
# inputs of test_rounding
PACKED = {((64, 64), "linear"): (1.767, 2.535), ((64, 64), "centered"): (2.159, 2.521),
          ((57, 40), "centered"): (1.749, 2.092), ((200, 150), "centered"): (2.110, 2.607),
          ((100, 300), "linear"): (1.907, 2.590), ((48, 48, 48), "centered"): (2.299, 2.726),
          ((4, 128, 128), "linear"): (1.805, 2.845)}


@pytest.mark.parametrize("grid,mode", list(PACKED))
def test_rounding(grid, mode):
    """fp32 images and volumes are as close to 64 bits as with the packed real transforms (to 1 %).  With the
    constants of the rows' inverse rounded once and no more they are 1 to 4 % further off."""
    import torch
    from paper_2607_19378_amd import hyenand as H
    rng = np.random.default_rng(sum(grid))
    C, nd = (64 if len(grid) == 2 else 16), len(grid)
    shape, axes = (1, C) + grid, tuple(range(-len(grid), 0))
    x1, x2, v, gy = (rng.standard_normal(shape).astype(np.float32) for _ in range(4))
    k = (rng.standard_normal(oracle.kernel_shape(shape, mode)) / np.sqrt(np.prod(grid))).astype(np.float32)
    D = rng.standard_normal(C).astype(np.float32)
    dev = [torch.from_numpy(a).cuda() for a in (x1, x2, v, k, D, gy)]
    y = from_device(H.fftconv(*dev[:5], pad_mode=mode))
    gk = from_device(H.backward(*dev, pad_mode=mode)[3])
    x1, x2, v, k, D, gy = (a.astype(np.float64) for a in (x1, x2, v, k, D, gy))
    P, u = tuple(2 * n for n in grid), x1 * v
    if mode == "centered":  # displacement d at index d mod P
        k = np.roll(np.pad(k, [(0, 0), (0, 0)] + [(0, 1)] * nd), [1 - n for n in grid], axes)
    U, crop = np.fft.rfftn(u, P, axes), (Ellipsis,) + tuple(slice(n) for n in grid)
    z = np.fft.irfftn(U * np.fft.rfftn(k, P, axes), P, axes)[crop] + D.reshape((1, C) + (1,) * nd) * u
    ref = np.fft.irfftn(np.fft.rfftn(gy * x2, P, axes) * U.conj(), P, axes)
    if mode == "centered":
        ref = np.roll(ref, [n - 1 for n in grid], axes)
    ref = ref[(Ellipsis,) + tuple(slice(n) for n in gk.shape[2:])]
    errs = rel_l2(y, x2 * z), rel_l2(gk, ref)
    log(f"ra rounding {grid} {mode} {errs[0]:.3e} {errs[1]:.3e}")
    for e, packed in zip(errs, PACKED[(grid, mode)]):
        assert e <= 1.01 * packed * 1e-7

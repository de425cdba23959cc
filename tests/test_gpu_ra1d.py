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


@pytest.mark.parametrize("u,k", [(1e37, 1e-30), (1e30, 1e-36)])
@pytest.mark.parametrize("L,mode,B", [(300, "circular", 1), (3000, "circular", 1), (3000, "circular", 300),
                                      (1000, "linear", 1), (700, "centered", 1), (300, "linear", 1)])
def test_magnitudes_near_the_range(L, mode, B, u, k):
    """Lines of the mixed plan (circular forward, non-circular backward) scale u, h and k by powers of two: sums of u
    that leave fp32's range, and kernels that the normalisation of the inverse would make subnormal, change no line's
    relative error (few and many lines: 8 and 16 points per lane)."""
    import torch
    from paper_2607_19378_amd import hyenand as H
    rng = np.random.default_rng(L)
    shape = (B, 2, L)
    x1 = np.abs(rng.standard_normal(shape)) * u  # one sign: the DC bin is the sum of all
    x2, v, gy = rng.standard_normal(shape), np.ones(shape), 1e-4 * rng.standard_normal(shape)
    kern = rng.standard_normal(oracle.kernel_shape(shape, mode)) * k
    D = rng.standard_normal(2) * k
    arrays = [W.quantise(a, "f32") for a in (x1, x2, v, kern, D, gy)]
    dev = [to_device(a, "f32") for a in arrays]
    log(f"ra1d range {L} {mode} {B} {u:g} {k:g}")
    f = [a.astype(np.float64) for a in arrays]
    if mode == "circular":  # the oracle's circular FFT takes powers of two: numpy's serves here
        assert H.plan_name(shape, mode, "f32") == "mixed1d"
        y = from_device(H.fftconv(*dev[:5], pad_mode=mode))
        ux = f[0] * f[2]
        ref = f[1] * (np.fft.irfft(np.fft.rfft(ux) * np.fft.rfft(f[3]), n=L) + f[4][None, :, None] * ux)
        assert per_line_worst(y, ref, 2 * B) <= TOL["f32"]
        return
    got = H.backward(*dev, pad_mode=mode)
    torch.cuda.synchronize()
    for name, g, r in zip(("gx1", "gx2", "gv", "gk"), got, oracle.backward_direct(*f, mode)):
        assert per_line_worst(from_device(g), r, 2 * B) <= TOL["f32"], name


def _conv64(u, k, mode):
    """k conv u of lines in 64 bits, and H conj(U) for a given h (numpy's FFT, zero-padded)."""
    L = u.shape[-1]
    K, U = np.fft.fft(k, 2 * L), np.fft.fft(u, 2 * L)
    if mode == "centered":
        K *= np.exp(2j * np.pi * np.arange(2 * L) * (L - 1) / (2 * L))
    return U, K


# relative L2 error (1e-7) of the packed real transforms, which these kernels replaced, on the inputs of test_rounding:
# forward, and the worst of gx1, gx2 and gv (0: more than 7 % further off than these kernels)
PACKED = {(512, "linear"): (1.70, 1.75), (512, "centered"): (1.87, 1.91), (1024, "linear"): (1.80, 1.82),
          (2048, "linear"): (1.90, 1.92), (2048, "centered"): (1.99, 2.04), (3000, "linear"): (1.81, 1.93),
          (8192, "linear"): (2.06, 0), (16384, "linear"): (2.84, 2.87), (65536, "centered"): (4.34, 4.34),
          (1 << 20, "linear"): (3.97, 4.01), (1 << 20, "centered"): (4.18, 4.21)}


@pytest.mark.parametrize("L,mode", list(PACKED))
def test_rounding(L, mode):
    """fp32 lines are as close to 64 bits as with the packed real transforms, to 3 % (8192 points forward: to 7 %; half
    the points of the padded transform's first pass are zeros, which round nothing).  The weights exp(-2 pi i n / (4 N))
    as a product of two or three rounded factors miss it by 4 to 13 %, the three-pass lines' twiddles as one chain of 16
    products by 4 to 18 %."""
    import torch
    from paper_2607_19378_amd import hyenand as H
    rng = np.random.default_rng(L)
    C = 8 if L > 1 << 16 else 64
    shape = (1, C, L)
    x1, x2, v, gy = (rng.standard_normal(shape).astype(np.float32) for _ in range(4))
    k = (rng.standard_normal(oracle.kernel_shape(shape, mode)) / np.sqrt(L)).astype(np.float32)
    D = rng.standard_normal(C).astype(np.float32)
    dev = [torch.from_numpy(a).cuda() for a in (x1, x2, v, k, D, gy)]
    y = from_device(H.fftconv(*dev[:5], pad_mode=mode))
    g = [from_device(t) for t in H.backward(*dev, pad_mode=mode)]
    x1, x2, v, k, D, gy = (a.astype(np.float64) for a in (x1, x2, v, k, D, gy))
    u, h, d = x1 * v, gy * x2, D[None, :, None]
    U, K = _conv64(u, k, mode)
    z = np.fft.ifft(U * K).real[..., :L] + d * u
    gu = np.fft.ifft(np.fft.fft(h, 2 * L) * K.conj()).real[..., :L] + d * h
    forward, backward = PACKED[(L, mode)]
    errs = [rel_l2(y, x2 * z), rel_l2(g[0], gu * v), rel_l2(g[1], gy * z), rel_l2(g[2], gu * x1)]
    log(f"ra1d rounding {L} {mode} " + " ".join(f"{e:.3e}" for e in errs))
    slack = 1.07 if L == 8192 else 1.03
    assert errs[0] <= slack * forward * 1e-7
    assert not backward or max(errs[1:]) <= slack * backward * 1e-7

"""Parity of the multi-pass plans (2D/3D lines per axis, 1D four-step) with
the fp64 oracle, from small ragged cases to the largest transforms each plan
takes (the full-size workloads are compared element by element in
test_gpu_full_workloads.py)."""
import numpy as np
import pytest

from paper_2607_19378_amd import workloads as W

from gpu_util import TOL, log, oracle_ref, rel_l2, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_19378_amd import hyenand as H
    H.lib()


def check_full(inp, tag, **kw):
    w = inp.workload
    log(f"[multipass] {tag}: shape={w.shape} mode={w.pad_mode} dtype={w.dtype}")
    y = run_gpu(inp, **kw)
    ref = oracle_ref(inp)
    err = rel_l2(y, ref)
    log(f"[multipass] {tag}: rel_l2={err:.3e}")
    assert np.all(np.isfinite(y)) and err <= TOL[w.dtype], f"{tag}: {err:.3e}"
    return y


def plan(inp):
    from paper_2607_19378_amd import hyenand as H
    w = inp.workload
    return H.plan_name(w.shape, w.pad_mode, w.dtype)


MP2D = [(2, 2), (4, 8), (16, 4), (32, 32), (8, 64), (64, 16)]


@pytest.mark.parametrize("grid", MP2D)
@pytest.mark.parametrize("mode", ["linear", "circular"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_multipass2d_forced(monkeypatch, grid, mode, dtype):
    monkeypatch.setenv("HYENAND_PLAN", "multipass")
    inp = W.random_case(3, 3, grid, mode, dtype, seed=300 + grid[0] + 7 * grid[1])
    assert plan(inp) == "multipass2d"
    check_full(inp, f"mp2d {grid}")


@pytest.mark.parametrize("grid,mode", [((256, 256), "linear"), ((512, 256), "circular"), ((1024, 64), "circular"),
                                       ((128, 512), "linear")])
def test_multipass2d_natural(grid, mode):
    inp = W.random_case(1, 3, grid, mode, "f32", seed=17)
    assert plan(inp) == "multipass2d"
    check_full(inp, f"mp2d {grid}")


MP3D = [(2, 2, 2), (4, 4, 4), (2, 8, 4), (8, 4, 16), (16, 16, 16), (32, 8, 64), (4, 64, 8)]


@pytest.mark.parametrize("grid", MP3D)
@pytest.mark.parametrize("mode", ["linear", "circular"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_multipass3d(grid, mode, dtype):
    inp = W.random_case(2, 3, grid, mode, dtype, seed=400 + sum(grid))
    assert plan(inp) == "multipass3d"
    check_full(inp, f"mp3d {grid}")


@pytest.mark.parametrize("L,mode", [(16384, "linear"), (32768, "circular"), (65536, "linear"),
                                    (1 << 17, "circular")])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_fourstep(L, mode, dtype):
    inp = W.random_case(1, 3, (L,), mode, dtype, seed=500 + L % 97)
    assert plan(inp) == "fourstep1d"
    check_full(inp, f"fourstep L={L}")


def test_chunked_workspace_matches_full():
    """A workspace of one line per chunk gives bitwise the same result as the
    recommended one (chunking only changes the launch order)."""
    from paper_2607_19378_amd import hyenand as H
    for grid, mode in (((8, 16, 8), "linear"), ((256, 128), "circular"), ((32768,), "linear")):
        inp = W.random_case(2, 3, grid, mode, "f32", seed=21)
        w = inp.workload
        wmin = H.workspace_min(w.shape, w.pad_mode, w.dtype)
        wrec = H.workspace_size(w.shape, w.pad_mode, w.dtype)
        assert 0 < wmin <= wrec
        log(f"[chunk] {grid}: min={wmin} rec={wrec}")
        y1 = run_gpu(inp, workspace_bytes=wmin)
        y2 = run_gpu(inp, workspace_bytes=wmin * 2 + 8)
        y3 = run_gpu(inp)
        assert np.array_equal(y1, y3) and np.array_equal(y2, y3)
        assert rel_l2(y3, oracle_ref(inp)) <= TOL["f32"]


@pytest.mark.parametrize("grid,mode,dtype", [((256, 128), "circular", "f32"), ((8, 8, 16), "linear", "bf16"),
                                             ((16384,), "linear", "f32"), ((100, 70), "centered", "f32")])
def test_side_streams_match_caller_stream(monkeypatch, grid, mode, dtype):
    """Chunks rotating over two or three side streams (7 lines, 3 lines of
    workspace: chunks of one line each) give bitwise the result of every
    chunk on the caller's stream.  The caller's stream is a non-default one
    whose next kernel reads y at once, so a missing join would show."""
    import torch
    from paper_2607_19378_amd import hyenand as H
    from gpu_util import to_device
    inp = W.random_case(1, 7, grid, mode, dtype, seed=33)
    w = inp.workload
    wmin = H.workspace_min(w.shape, w.pad_mode, w.dtype)
    assert wmin > 0, "a single-pass plan, without chunks"
    dev = [to_device(a, w.dtype) for a in (inp.x1, inp.x2, inp.v, inp.k, inp.D)]
    ws = torch.empty(3 * wmin, dtype=torch.uint8, device="cuda")
    outs = []
    for streams in ("1", "2", "3"):
        monkeypatch.setenv("HYENAND_CHUNK_STREAMS", streams)
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            y = torch.full_like(dev[0], float("nan"))
            H.fftconv_into(y, *dev, pad_mode=w.pad_mode, workspace=ws, stream=s)
            y2 = y.float() * 2.0  # consumer on the caller's stream
        s.synchronize()
        outs.append((y.float().cpu().numpy(), y2.cpu().numpy()))
    log(f"[side streams] {grid} {mode} {dtype}")
    a, a2 = outs[0]
    for b, b2 in outs[1:]:
        assert np.array_equal(a, b) and np.array_equal(a2, b2) and np.array_equal(b2, 2.0 * b)
    assert rel_l2(a, oracle_ref(inp)) <= TOL[dtype]


@pytest.mark.parametrize("grid,mode,name", [((256, 128), "circular", "multipass2d"), ((128, 256), "linear", "multipass2d"),
                                            ((32768,), "linear", "fourstep1d")])
def test_graph_capture_with_side_streams(monkeypatch, grid, mode, name):
    """A multi-pass call captured into a graph (chunks on two side streams)
    replays to the eager result, three times, with eager calls in between.
    (By themselves calls this small stay on the caller's stream.)"""
    import torch
    from paper_2607_19378_amd import hyenand as H
    from gpu_util import to_device
    monkeypatch.setenv("HYENAND_CHUNK_STREAMS", "2")
    inp = W.random_case(1, 5, grid, mode, "f32", seed=44)
    w = inp.workload
    assert plan(inp) == name
    wmin = H.workspace_min(w.shape, w.pad_mode, w.dtype)
    dev = [to_device(a, w.dtype) for a in (inp.x1, inp.x2, inp.v, inp.k, inp.D)]
    ws = torch.empty(2 * wmin, dtype=torch.uint8, device="cuda")
    y = torch.empty_like(dev[0])
    H.fftconv_into(y, *dev, pad_mode=w.pad_mode, workspace=ws)
    torch.cuda.synchronize()
    ref = y.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        H.fftconv_into(y, *dev, pad_mode=w.pad_mode, workspace=ws)
    other = torch.empty_like(y)
    for i in range(3):
        y.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        log(f"[graph] replay {i}")
        assert torch.equal(y, ref)
        H.fftconv_into(other, *dev, pad_mode=w.pad_mode, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(other, ref)


def test_workspace_too_small_rejected():
    import torch
    from paper_2607_19378_amd import hyenand as H
    inp = W.random_case(1, 2, (8, 8, 8), "linear", "f32", seed=1)
    w = inp.workload
    wmin = H.workspace_min(w.shape, w.pad_mode, w.dtype)
    with pytest.raises(H.HyenandError) as e:
        run_gpu(inp, workspace_bytes=wmin - 8)
    assert e.value.status == H.ERR_WORKSPACE_TOO_SMALL
    torch.cuda.synchronize()


@pytest.mark.parametrize("grid,mode,dtype", [((1 << 21,), "linear", "bf16"), ((1 << 22,), "circular", "f32"),
                                             ((512, 512), "linear", "f32"), ((1024, 1024), "circular", "bf16"),
                                             ((1024, 8), "circular", "f32"), ((512, 4, 8), "linear", "f32"),
                                             ((4, 1024, 16), "circular", "bf16"), ((8, 4, 512), "linear", "f32")])
def test_maximum_extents(grid, mode, dtype):
    """The largest transforms the plans take: 2^22 points in 1D (N1 = 1024
    columns of the four-step split), 1024 on any axis of a 2D or 3D grid;
    every output element against the oracle."""
    inp = W.random_case(1, 2, grid, mode, dtype, seed=600 + len(grid) + grid[0] % 13)
    assert plan(inp) in ("fourstep1d", "multipass2d", "multipass3d")
    check_full(inp, f"max {grid} {mode}")


def test_other_stream_outside_its_context(monkeypatch):
    """fftconv(stream=s) called while another stream is current (its chunks on
    two side streams of the library): the binding
    allocates y and the workspace on the current stream and hands them to s.
    Allocations made on the current stream right after the call (before s
    finishes) must not take their memory: y matches a call on the current
    stream bitwise, and the filler tensors keep their values."""
    import torch
    from paper_2607_19378_amd import hyenand as H
    from gpu_util import to_device
    monkeypatch.setenv("HYENAND_CHUNK_STREAMS", "2")
    inp = W.random_case(2, 6, (256, 128), "circular", "f32", seed=45)
    w = inp.workload
    assert plan(inp) == "multipass2d"
    dev = [to_device(a, w.dtype) for a in (inp.x1, inp.x2, inp.v, inp.k, inp.D)]
    ref = H.fftconv(*dev, pad_mode=w.pad_mode)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    for rep in range(3):
        y = H.fftconv(*dev, pad_mode=w.pad_mode, stream=s)
        fill = [torch.full((H.workspace_size(w.shape, w.pad_mode, w.dtype) // 4 + 1024,), float(rep + j),
                           device="cuda") for j in range(3)]
        torch.cuda.current_stream().wait_stream(s)
        torch.cuda.synchronize()
        log(f"[other stream] rep {rep}")
        assert torch.equal(y, ref)
        for j, f in enumerate(fill):
            assert bool((f == float(rep + j)).all())


def test_host_threads_each_with_own_side_streams(monkeypatch):
    """Four host threads call multi-pass plans at once, each on a stream of
    its own and with two side streams (ctypes releases the GIL inside the library, so the calls overlap
    on the host); every result matches the single-thread one bitwise."""
    import threading
    import torch
    from paper_2607_19378_amd import hyenand as H
    from gpu_util import to_device
    monkeypatch.setenv("HYENAND_CHUNK_STREAMS", "2")  # calls this small would stay on their stream
    cases = []
    for j, (grid, mode) in enumerate((((256, 128), "circular"), ((32768,), "linear"), ((8, 16, 8), "linear"),
                                      ((128, 256), "linear"))):
        inp = W.random_case(1, 5, grid, mode, "f32", seed=70 + j)
        w = inp.workload
        dev = [to_device(a, w.dtype) for a in (inp.x1, inp.x2, inp.v, inp.k, inp.D)]
        ref = H.fftconv(*dev, pad_mode=w.pad_mode)
        cases.append((w, dev, ref))
    torch.cuda.synchronize()
    errors = []

    def worker(j):
        try:
            w, dev, ref = cases[j]
            s = torch.cuda.Stream()
            ws = torch.empty(H.workspace_size(w.shape, w.pad_mode, w.dtype), dtype=torch.uint8, device="cuda")
            ys = [torch.empty_like(dev[0]) for _ in range(4)]
            torch.cuda.synchronize()
            for y in ys:
                H.fftconv_into(y, *dev, pad_mode=w.pad_mode, workspace=ws, stream=s)
            s.synchronize()
            for y in ys:
                if not torch.equal(y, ref):
                    errors.append(f"case {j}: mismatch")
        except Exception as e:  # reported below
            errors.append(f"case {j}: {e!r}")

    threads = [threading.Thread(target=worker, args=(j,)) for j in range(len(cases))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=60)
    log(f"[threads] {len(cases)} threads done, errors={errors}")
    assert not any(t.is_alive() for t in threads)
    assert not errors, errors


SLAB = [((4, 32, 32), "linear"), ((2, 64, 64), "linear"), ((4, 128, 128), "linear"), ((2, 64, 64), "circular"),
        ((4, 128, 128), "circular"), ((8, 128, 128), "linear")]


@pytest.mark.parametrize("grid,mode", SLAB)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_slab3d(grid, mode, dtype):
    """The three-pass 3D plan (planes transformed on chip along both inner
    axes, the multi-pass core along axis 0) against the oracle, every
    element."""
    inp = W.random_case(2, 3, grid, mode, dtype, seed=800 + sum(grid))
    assert plan(inp) == "slab3d"
    check_full(inp, f"slab3d {grid}")


@pytest.mark.parametrize("grid,mode", [((4, 128, 128), "linear"), ((2, 128, 128), "circular")])
def test_slab3d_and_five_pass_agree_with_oracle(monkeypatch, grid, mode):
    """The same shapes on the five-pass plan (slab plan switched off) also
    match the oracle, and the two plans agree to rounding."""
    inp = W.random_case(1, 3, grid, mode, "f32", seed=850 + grid[0])
    y_slab = check_full(inp, f"slab {grid}")
    monkeypatch.setenv("HYENAND_SLAB", "0")
    assert plan(inp) == "multipass3d"
    y_five = check_full(inp, f"five-pass {grid}")
    assert rel_l2(y_slab, y_five) <= 1e-6


def test_slab3d_chunking_and_shared_k():
    """Chunked workspaces give bitwise the recommended one's result; one
    kernel per channel (k as [C, ...]) through the slab plan."""
    import torch
    from paper_2607_19378_amd import hyenand as H
    from gpu_util import to_device
    inp = W.random_case(2, 3, (4, 128, 128), "linear", "bf16", seed=861)
    w = inp.workload
    assert plan(inp) == "slab3d"
    wmin = H.workspace_min(w.shape, w.pad_mode, w.dtype)
    y1 = run_gpu(inp, workspace_bytes=wmin)
    y2 = run_gpu(inp)
    assert np.array_equal(y1, y2)
    assert rel_l2(y2, oracle_ref(inp)) <= TOL["bf16"]
    # shared k: every sample uses k[0]'s channels
    ksh = inp.k[0]
    dev = [to_device(a, w.dtype) for a in (inp.x1, inp.x2, inp.v, ksh, inp.D)]
    y = H.fftconv(*dev, pad_mode=w.pad_mode, shared_k=True)
    torch.cuda.synchronize()
    import oracle
    x1, x2, v, k, D = inp.as_f64()
    kb = np.broadcast_to(k[:1], k.shape).copy()
    ref = oracle.conv_fft(x1, x2, v, kb, D, w.pad_mode)
    from gpu_util import from_device
    err = rel_l2(from_device(y), ref)
    log(f"[slab shared k] rel_l2={err:.3e}")
    assert err <= TOL["bf16"]

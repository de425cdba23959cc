"""The multi-pass kernels on right-angle rows must fit in the workspace that the plans' queries report, for every
shape that reaches them: the power-of-two non-circular grids have no other kernels."""
import itertools

from paper_2607_19378_amd import hyenand as H


def _ra_bytes(grid, mode, backward):
    """Spectra of a line: planes x P1 x N complex fp32 (conv_ra_mp.hip)."""
    p = [2 * n for n in grid]
    n = max(16, p[-1] // 2)
    p1 = p[1] if len(grid) == 3 else 1
    if len(grid) == 3 and p[-1] >= 32 and 32 <= p1 <= 256 and max(32, n) <= 128:
        n = max(32, n)
    kp = grid[0] if mode == "linear" else 2 * grid[0] - 1
    return ((2 if backward else 1) * grid[0] + kp) * p1 * n * 8


def _sums(grid, lines):
    """The gD sums of h u: up to 64 parts of 8192 points a line, in a 256-byte block."""
    data = 1
    for n in grid:
        data *= n
    return (lines * min(64, -(-data // 8192)) * 4 + 255) // 256 * 256


def test_power_of_two_grids_fit(monkeypatch):
    """With one line and with many: the gD sums, which come before the spectra, grow with the lines.  Backward shapes
    whose least workspace is one float per line run in a single pass and are left out."""
    monkeypatch.setenv("HYENAND_PLAN", "multipass")
    sizes = [2, 4, 8, 16, 32, 64, 128, 256, 512]
    grids = [g for nd in (2, 3) for g in itertools.product(sizes, repeat=nd)]
    multipass = 0
    for grid, mode, lines in itertools.product(grids, ("linear", "centered"), (1, 4095)):
        shape = (1, lines) + grid
        try:
            name = H.plan_name(shape, mode, "f32")
        except H.HyenandError as e:  # 4095 lines of the largest grids
            assert e.status == H.ERR_UNSUPPORTED and lines > 1
            continue
        assert name[:6] in ("multip", "slab3d"), (grid, mode)
        assert _ra_bytes(grid, mode, False) <= H.workspace_min(shape, mode, "f32"), (grid, mode)
        try:
            least = H.backward_workspace_min(shape, mode, "f32")
        except H.HyenandError as e:  # the centered mode's copies of 2^31 elements
            assert e.status == H.ERR_UNSUPPORTED and lines > 1
            continue
        if least > (lines * 4 + 255) // 256 * 256:
            multipass += 1
            assert _sums(grid, lines) + _ra_bytes(grid, mode, True) <= least, (grid, mode, lines)
    assert multipass > 1000


def test_other_extents_fit():
    """Ragged grids beyond the single-pass kernels, down to the narrowest rows, where the right-angle rows keep 16
    values; and no shape of that plan is left without passes: a row of N values is no longer than the circular
    problem's half row, and 3 L0 - 1 planes are at most its 2 P0."""
    sizes = [3, 5, 7, 9, 17, 31, 33, 63, 65, 129, 200, 511]
    seen = 0
    for nd in (2, 3):
        for grid, mode, lines in itertools.product(itertools.product(sizes, repeat=nd), ("linear", "centered", "circular"),
                                                   (1, 21)):
            try:
                name = H.plan_name((1, lines) + grid, mode, "bf16")
            except H.HyenandError as e:  # more than 2^31 points on the transform grid
                assert e.status == H.ERR_UNSUPPORTED and lines * (4 * max(grid)) ** nd > 1 << 31
                continue
            if not name.startswith("embedded"):
                continue
            seen += 1
            p = [1 << (2 * n - 2).bit_length() for n in grid]
            n, p1 = max(16, p[-1] // 2), p[1] if nd == 3 else 1
            if nd == 3 and p[-1] >= 32 and 32 <= p1 <= 256 and max(32, n) <= 128:
                n = max(32, n)
            planes = 2 * grid[0] if mode == "linear" else 3 * grid[0] - 1
            assert planes * p1 * n * 8 <= H.workspace_min((1, lines) + grid, mode, "bf16"), (grid, mode)
    assert seen > 1000


def test_lines_fit():
    """Three-pass lines: two (backward three) spectra of N = P / 2 points, and the sums of h u."""
    for L, mode, lines in itertools.product((16384, 20000, 65537, 300001, 1 << 20, 1 << 21), ("linear", "centered"),
                                            (1, 300)):
        n = 1 << (2 * L - 2).bit_length() - 1
        shape = (1, lines, L)
        assert 2 * n * 8 <= H.workspace_min(shape, mode, "f32"), (L, mode)
        assert _sums((L,), lines) + 3 * n * 8 <= H.backward_workspace_min(shape, mode, "f32"), (L, mode)


def test_scaled_lines_have_kernels():
    """The right-angle kernels that take the mixed plan's calls scale u, k and h by powers of two; the kernels built
    without that (images beyond 32 x 32 points, non-circular lines, lines beyond 4096) must
    not be reached by the plan."""
    for n0, n1 in itertools.product(range(17, 65), repeat=2):
        if max(n0, n1) > 32 and not (n0 & (n0 - 1) == 0 and n1 & (n1 - 1) == 0):
            for mode in ("linear", "centered"):
                assert H.plan_name((2, 3, n0, n1), mode, "f32") == "fused2d_any", (n0, n1, mode)
    for L in list(range(257, 4097, 7)) + [4099, 5000, 8191]:
        assert L & (L - 1) == 0 or H.plan_name((2, 3, L), "linear", "f32") == "fused1d_any", L
        assert L <= 4096 or H.plan_name((2, 3, L), "circular", "f32") == "fused1d_any", L


def test_backward_asks_for_what_it_uses():
    """Centered and ragged backward calls on right angles hold the gD sums, and in several passes their spectra: no
    copies on the transform grid (4 x 64 volumes of 48^3 asked for 19.5 GB of them)."""
    for shape, mode in (((4, 64, 48, 48, 48), "centered"), ((4, 64, 200, 150), "centered"), ((2, 64, 500, 500), "linear"),
                        ((1, 64, 300001), "linear"), ((8, 64, 128, 128), "centered"), ((1, 64, 1 << 20), "centered")):
        lines, grid = shape[0] * shape[1], shape[2:]
        if len(grid) == 1:
            per = 3 * (1 << (2 * grid[0] - 2).bit_length() - 1) * 8
        else:
            p = [1 << (2 * n - 2).bit_length() for n in grid]
            planes = 2 * grid[0] + (grid[0] if mode == "linear" else 2 * grid[0] - 1)
            per = planes * (p[1] if len(grid) == 3 else 1) * (p[-1] // 2) * 8
        least, size = (f(shape, mode, "bf16") for f in (H.backward_workspace_min, H.backward_workspace_size))
        assert least == _sums(grid, lines) + per, (shape, mode)
        assert least <= size <= _sums(grid, lines) + max(640 << 20, 2 * per), (shape, mode)
    for shape, mode in (((8, 64, 5000), "linear"), ((8, 64, 57, 40), "centered"), ((8, 64, 8192), "centered")):
        assert H.backward_workspace_min(shape, mode, "f32") == H.backward_workspace_size(shape, mode, "f32") == 8 * 64 * 4

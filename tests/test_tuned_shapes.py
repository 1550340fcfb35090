"""What a launch makes of a shape that the autotuner stored and of one that was
pinned, read from the runtime calls of the library (no kernel runs)."""
from tests._fake_hip import run

COMMON = """
def shape(s, *n):
    g, v, z = ctypes.c_int(), ctypes.c_int(), ctypes.c_int()
    assert L.hydro_get_launch_shape(ctypes.byref(s), *n, ctypes.byref(g), ctypes.byref(v), ctypes.byref(z)) == 0
    return g.value, v.value, z.value
def launched():  # (kernel, workgroups) of the launches since the last call
    return [(w.split()[1], n) for w, a, n in calls() if w.startswith("launch")]
def groups(s, n):  # a solve of n ghosted groups
    assert L.hydro_solve_groups(P(1 << 40), P(1 << 41), None, n, D(1e-3), D(1.0), D(s.gamma), s.scheme, s.reconstruction,
                                s.riemann, s.limiter, s.flags, None) == 0
def box(s, n):
    assert L.hydro_step_box(P(1 << 40), P(1 << 41), None, n, n, n, P(1 << 42), D(1.0), D(1.0), D(s.gamma), s.scheme,
                            s.reconstruction, s.riemann, s.limiter, s.flags, None) == 0
CHAR, F64 = 2, 1
"""


def test_tuning_keeps_small_launches_split(tmp_path):
    """Every interval takes the same time here, so the tuner keeps its first
    candidate, the variant that has no split kernels in FP32.  It times whole
    groups at one group count: launches that the untuned shape splits stay
    split, at its hint and elsewhere; others take the tuned shape."""
    run(tmp_path, COMMON + """
for scheme in (0, 1, 2):
    for flags, waves in ((CHAR, 4), (CHAR | F64, 2)):
        s = Spec(scheme, 1, 1, 1, flags, 1.4)
        untuned = {n: shape(s, n, n, n) for n in (32, 64)}
        assert untuned[32] == (128, waves, 1) and untuned[64][0] > 64
        for hint in (8, 64, 4096):
            assert L.hydro_autotune(ctypes.byref(s), hint, None) == min(hint, 256)
            for n in (32, 64):
                assert shape(s, n, n, n) == untuned[n], (scheme, flags, hint, n)
            calls()
            groups(s, 8), box(s, 32)
            assert [g for k, g in launched() if "predict" not in k] == [128, 128]
        assert shape(s, 256, 256, 256)[:2] == (256, 2)
""")


def test_saved_shape_keeps_small_launches_split(tmp_path):
    cache = tmp_path / "tune"
    cache.write_text("gfx950/f32/s2/r1/rs1/c1 512 2 1 512\n")
    run(tmp_path, COMMON + f"""
os.environ["HYDRO_TUNE_CACHE"] = {str(cache)!r}
ctypes.CDLL(None).setenv(b"HYDRO_TUNE_CACHE", {str(cache)!r}.encode(), 1)
s = Spec(2, 1, 1, 1, CHAR, 1.4)
assert shape(s, 32, 32, 32) == (128, 4, 1)
assert shape(s, 256, 256, 256) == (512, 2, 1)
""")


def test_pinned_grid_is_used(tmp_path):
    """A pinned grid is the number of workgroups, clamped to the groups; only
    without one are groups split."""
    run(tmp_path, COMMON + """
for scheme in (0, 1, 2):
    for flags, waves in ((CHAR, 4), (CHAR | F64, 2)):
        s = Spec(scheme, 1, 1, 1, flags, 1.4)
        for grid in (5, 8, 9, 128, 4096):
            assert L.hydro_set_launch_shape(ctypes.byref(s), grid, waves, 0) == 0
            want = min(grid, 8)
            assert shape(s, 32, 32, 32) == (want, waves, 1), (scheme, flags, grid)
            calls()
            groups(s, 8), box(s, 32)
            assert {g for k, g in launched()} == {want}, (scheme, flags, grid)
        assert L.hydro_set_launch_shape(ctypes.byref(s), 0, waves, 0) == 0
        assert shape(s, 32, 32, 32) == (128, waves, 1)
""")

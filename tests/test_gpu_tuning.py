"""The instruments that a user tunes and measures with: the kernel-class timing and the tile
autotuner, where a launch is preceded or replaced by another kernel."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2505_24504_amd import jfmg, workloads as W  # noqa: E402

from gpu_common import DEV  # noqa: E402


def setup_module(module):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    jfmg.load_library()


@pytest.mark.parametrize("prec", [32, 64])
def test_stage_timing_behind_summed_partials(prec):
    """1024 x 1024 cells in 256-cell tiles: 4096 partial sums of ||x||^2, which a kernel of a
    few us adds up before each stage.  The class times the stage and not that kernel: its mean
    launch is at least half of what the autotuner measures for the same shape, whose launches
    have 1024 partials and no such kernel before them (a sum alone is below a tenth of it)."""
    d = W.small(nx=256, nz=256, k=3, mg_levels=1, mg_key="mg008802V", rk_stages=1, mg_precision=prec,
                x1=256 * 40.0, z1=256 * 40.0)
    p = jfmg.Problem(d, device=DEV)
    U = p.initial_state(dict(shape=0, amp=1.0, xc=5000.0, zc=5000.0, xr=2000.0, zr=2000.0))
    p.linearize(U, 0.3)
    _, times = p.autotune(reps=10)
    p.set_tiles(["64x4_512"])
    b = torch.randn(p.fv_size(0), device=DEV, generator=torch.Generator(device=DEV).manual_seed(3), dtype=p.fv_dtype)
    p.mg_fv(b)
    p.profile_enable(["fv_stage"])
    p.mg_fv(b)
    r = p.profile_read()["fv_stage"]
    mean = 1e3 * r["ms"] / r["launches"]
    print(f"fp{prec}: stage {mean:.1f} us, autotuner {times[0]['64x4_512']:.1f} us", flush=True)
    assert r["launches"] == 15
    assert mean >= 0.5 * times[0]["64x4_512"]


# (config, the levels that go in one launch in 8x4 tiles)
def _tuned_cases():
    d, _, _ = W.bubble_small()
    out = []
    for prec in (32, 64):
        out.append((dict(d, mg_precision=prec), [1, 2]))                       # 16x16, 8x8
        out.append((dict(d, mg_precision=prec, nx=12, nz=8, rk_stages=1), [1, 2]))   # 12x8, 6x4
        out.append((dict(d, mg_precision=prec, nx=16, nz=8, mg_levels=4), [1, 2, 3]))   # 16x8, 8x4, 4x2
    return out


@pytest.mark.parametrize("case", _tuned_cases())
def test_tuned_problem_keeps_the_one_launch_levels(case):
    """The coarse levels that go in one launch in the default shapes do so after tuning: that
    launch saves half of the time of the levels' own, so that no other shape is the fastest."""
    d, levels = case
    p = jfmg.Problem(d, device=DEV)
    assert [l for l, t in enumerate(p.get_tiles()) if t == "8x4"][-len(levels):] == levels
    U = p.initial_state(dict(shape=0, amp=0.5, xc=500.0, zc=350.0, xr=250.0, zr=250.0))
    p.linearize(U, 0.5)
    mv = p.implicit_step(U.clone())["fv_matvecs"]
    for _ in range(3):
        shapes, times = p.autotune(reps=20)
        print([(l, {s: round(t, 2) for s, t in times[l].items()}) for l in levels], flush=True)
        assert [shapes[l] for l in levels] == ["8x4"] * len(levels)
    assert p.implicit_step(U.clone())["fv_matvecs"] == mv


@pytest.mark.parametrize("physics", [0, 1])
def test_jvp_bytes_are_the_librarys(physics):
    """bench.py's bytes of a JVP call are the library's of its kernel and a pass over y."""
    import bench
    d = W.small(nx=7, nz=5, k=3, physics=physics, mu=75.0 if physics else 0.0, mg_levels=1)
    p = jfmg.Problem(d, device=DEV)
    U = p.initial_state(dict(shape=0, amp=1.0, xc=500.0, zc=400.0, xr=200.0, zr=200.0))
    p.linearize(U, 0.3)
    p.profile_enable(["dg_jvp"])
    p.jvp(U)
    r = p.profile_read()["dg_jvp"]
    assert r["launches"] == 1
    assert bench.jvp_bytes(7, 5, 3, physics == 1) == r["bytes"] + 8 * p.ndof

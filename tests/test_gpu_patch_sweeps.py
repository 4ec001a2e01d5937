"""Patch sweeps on 8^3 tiles with the prolongation included, one or two sweeps a launch,
against a launch per sweep and a separate prolongation (GRMG_PATCH_SWEEP=0).

The point updates and their order are the same, so the fields agree to rounding (1e-12 of
the largest value, the bar of the whole solve) after the same number of cycles.
"""
import pytest

from paper_1905_08890_amd import grmg, synth
from test_gpu_patches import PRM, _load

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# sides that 8 divides and does not, one to three levels above the single-workgroup cycle,
# one patch inside another
SIDES = (18, 20, 22, 28, 34, 40, 56, 72)


@pytest.mark.parametrize("two", ["0", "40", "100000"])
@pytest.mark.parametrize("nu", [2, 4])
def test_tiled_sweeps_match_a_launch_per_sweep(two, nu, monkeypatch):
    """No level, some and every level with both sweeps in a launch; other sweep counts."""
    boxes = [64]
    patches = [(n, 1 / 160, 0, ((3 + 2 * j) / 64, 9 / 64, (5 + j) / 64)) for j, n in enumerate(SIDES)]
    patches.append((24, 1 / 400, len(boxes) + 7, (24 / 64, 18 / 64, 20 / 64)))
    print(f"[gpu] patch sweeps two<={two} nu={nu}", flush=True)
    monkeypatch.setenv("GRMG_PATCH_SWEEP", "0")
    A = grmg.Batch(boxes, **PRM, patches=patches)
    monkeypatch.delenv("GRMG_PATCH_SWEEP")
    monkeypatch.setenv("GRMG_PATCH_TWO", two)
    B = grmg.Batch(boxes, **PRM, patches=patches)
    src = [synth._matter_sources(64, 700, 0.3)], [synth._matter_sources(n, 710 + j, 0.3)
                                                  for j, (n, _, _, _) in enumerate(patches)]
    reps = []
    for X in (A, B):
        _load(X, boxes, *src)
        reps.append(X.solve(rtol=0.0, max_cycles=3, nu1=nu, nu2=nu))
        torch.cuda.synchronize()
    assert reps[0]["cycles"] == reps[1]["cycles"]
    for j in range(len(patches)):
        for f in range(10):
            a, b = A.get_field(1 + j, f).cpu(), B.get_field(1 + j, f).cpu()
            assert float((a - b).abs().max()) <= 1e-12 * float(a.abs().max()), (j, f)

"""Graphs that lbw_step replays (launch field graph), against a stand-in for the
HIP runtime: one per state the calls meet, captured once, and none destroyed by a
step, whose replays may still be running."""
import pytest

from fakehip import run


@pytest.mark.parametrize("form", ["", "has_s=True, kappa_s=1e-3", "fluid_mode=lbw.FLUID_FROZEN",
                                  "fluid_mode=lbw.FLUID_FROZEN, has_s=True, kappa_s=1e-3"])
@pytest.mark.parametrize("size", ["nx=64, ny=128", "nx=2048, ny=2048"])
def test_one_graph_per_state(tmp_path, form, size):
    """Calls of two steps run the stages and, on the small grid, longer calls the
    one-launch transport; odd calls also change the streaming parity."""
    states = (1 if "FROZEN" in form and "has_s" not in form else 2) * (2 if "64" in size else 1)
    run(tmp_path, f"""
h = handle(lbw.RunConfig({size}, {form}), graph=1)
for n in (2, 10, 2, 3, 1, 2, 5, 4, 1, 2, 10, 3, 2, 10, 2, 10):
    lbw.check(lib.lbw_step(h, n))
lines = log()
made = [l.split()[1] for l in lines if l.startswith("instantiate")]
assert len(made) == {states}, made
assert not [l for l in lines if l.startswith("destroy")], lines
assert {{l.split()[1] for l in lines if l.startswith("replay")}} == set(made)
lbw.check(lib.lbw_set_launch(h, ctypes.byref(lbw.CLaunch(graph=1))))
assert sorted(l.split()[1] for l in log() if l.startswith("destroy")) == sorted(made)
""")

"""Pinned slots of the reductions, against a stand-in for the HIP runtime.

A kernel writes its partials straight into a slot of host memory, so a slot may
serve another call only after a wait has shown that the kernel of the last one
has ended.  A launch can be reported as failed though the kernel runs: the
status also holds an older error that another library left on the thread."""
from fakehip import run

BODY = r"""
h = handle(lbw.RunConfig(nx=64, ny=128))
out = ctypes.c_double(0.0)
def reduce():
    rc = lib.lbw_reduce(h, lbw.MASS_C, ctypes.byref(out))
    lines = log()
    slot = [l.split()[-1] for l in lines if l.startswith("launch") and "k_partial" in l]
    return rc, slot[0], [l for l in lines if l.startswith("wait")]
rc, first, waits = reduce()
assert rc == 0 and waits == ["wait 0"], (rc, waits)
rc, again, waits = reduce()
assert rc == 0 and again == first            # given back after its wait
fake.fake_last_error(101)                    # left by another library on this thread
"""


def test_slot_is_waited_for_after_a_reported_launch_error(tmp_path):
    run(tmp_path, BODY + r"""
rc, slot, waits = reduce()
assert rc == lbw.ERR_HIP
rc, later, _ = reduce()
assert rc == 0
assert waits == ["wait 0"] or later != slot, (slot, later, waits)
""")


def test_slot_is_not_used_again_when_that_wait_fails(tmp_path):
    run(tmp_path, BODY + r"""
fake.fake_sync_error(719)
rc, slot, waits = reduce()
assert rc == lbw.ERR_HIP
fake.fake_sync_error(0)
rc, later, _ = reduce()
assert rc == 0 and later != slot, (slot, later, waits)
""")

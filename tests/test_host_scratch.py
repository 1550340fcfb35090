"""Scratch memory that a kernel needs zeroed is zero before the kernel starts."""
from tests._fake_hip import run

SCRIPT = """
U, out = P(1 << 20), P(1 << 30)
for k in range(70):  # the pool's 64 slots and memory of the streams' own
    assert L.hydro_cfl_dt(U, 1, D(1.0), D(1.4), D(0.5), 0, out, P(4096 + 64 * k)) == 0
cleared, launches = False, 0
for what, a, n in calls():
    if what == "memset":
        cleared = True   # enqueued on the null stream, asynchronous to the host
    elif what == "devsync" or (what == "sync" and a == 0):
        cleared = False
    elif what.startswith("launch"):
        assert not cleared, (what, launches)
        launches += 1
assert launches == 70, launches
"""


def test_cleared_scratch_is_waited_for(tmp_path):
    """The first reduction on a stream starts after the clearing of its counters,
    which is on the null stream (other streams need not wait for that one)."""
    run(tmp_path, SCRIPT)

"""Planning with little memory: what a plan that cannot be completed leaves behind.  Each plan is made in a process whose
address space may grow by so many megabytes and no further.  No GPU."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.skipif("asan" in os.environ.get("LD_PRELOAD", ""), reason="a sanitizer reserves address space of its own")
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OK, ENOMEM, ESTATE = 0, -2, -5

CHILD = """
import json, resource, sys
import csb_inputs
from paper_2005_05758_amd import CsbMatrix, load_library

A = csb_inputs.small_matrix(7, 4096, 4096, 32, 32, rate=12.0).A
L = load_library()
hard = resource.getrlimit(resource.RLIMIT_AS)[1]
def limit(room):
    size = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
    resource.setrlimit(resource.RLIMIT_AS, (size + (room << 20), hard))
out = []
for first_mode in (None, 1):                    # the matrix's first plan, and one after a plan of another mode
    for room in range(0, 80, 4):
        M = CsbMatrix(A, 32, 32)
        if first_mode is not None:
            M.plan(mode=first_mode)
        limit(room)
        planned = L.csb_plan(M._h, 0, None)
        resource.setrlimit(resource.RLIMIT_AS, (hard, hard))
        out.append((first_mode, room, planned, L.csb_plan_validate(M._h), L.csb_device_bytes(M._h)))
        M.close()
M = CsbMatrix(A, 32, 32)
M.plan()
print(json.dumps(out), flush=True)
limit(16)
print(L.csb_plan_validate(M._h))                # (it keeps the dense matrix twice: 128 MB)
"""


@pytest.fixture(scope="module")
def child():
    # (freed memory goes back to the system, so that every plan starts from the same size)
    env = dict(os.environ, PYTHONPATH=ROOT, MALLOC_MMAP_THRESHOLD_="65536", MALLOC_TRIM_THRESHOLD_="0", MALLOC_TOP_PAD_="0")
    res = subprocess.run([sys.executable, "-c", CHILD], env=env, stdout=subprocess.PIPE, text=True, timeout=300)
    return res.returncode, res.stdout.splitlines()


@pytest.fixture(scope="module")
def plans(child):
    return json.loads(child[1][0])


def test_what_is_left_is_a_whole_plan_or_none(plans):
    assert {p[2] for p in plans} == {OK, ENOMEM}      # both are met
    for first_mode, room, planned, valid, size in plans:
        assert valid in (OK, ESTATE), (first_mode, room, planned)


# 34 MB is what the tile sections and the row-owned section of this matrix take to plan.  No room is set aside for the section
# of the batched products, which is there for speed alone: where it does not fit, the plan is made without it.
def test_plan_without_the_batched_section(plans):
    by_room = {room: (planned, size) for first_mode, room, planned, valid, size in plans if first_mode is None}
    assert all(planned == OK for room, (planned, size) in by_room.items() if room >= 36)
    assert by_room[36][1] < by_room[76][1]


def test_validation_without_memory_is_an_error_code(child):
    status, lines = child
    assert status == 0 and int(lines[1]) == ENOMEM

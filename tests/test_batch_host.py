"""The host side of amg_solve_batch without a GPU (tests/host/batch_calls.hip: the program's own HIP runtime calls)."""
import os

import pytest

from paper_1209_5421_amd import amg
from tests import host_program


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    lib = os.path.dirname(amg.LIB_PATH)
    return host_program.build("batch_calls.hip", tmp_path_factory.mktemp("host"),
                              [f"-L{lib}", "-lquadamg", f"-Wl,-rpath,{lib}", "-lpthread", "-ldl", "-rdynamic"])


def result(exe, *args):
    out = host_program.run(exe, *args).split()
    return dict(zip(out[::2], map(int, out[1::2])))


@pytest.mark.parametrize("mode", ["drain", "drain-noalloc"])
def test_a_failed_launch_leaves_nothing_queued(exe, mode):
    r = result(exe, mode)
    assert r["launches"] > 20 and r["bad"] == 0 and r["queued"] == 0


def test_the_callers_allocator_is_called_on_the_callers_thread(exe):
    """It may depend on the thread (torch's current stream does), and amg_solve_batch called it on that thread before it
    ran two routes side by side."""
    assert result(exe, "allocator") == {"status": 0, "blocks": 1, "foreign": 0}


def test_a_call_that_gets_no_thread_runs_its_routes_in_turn(exe):
    assert result(exe, "no-threads") == {"status": 0, "ok": 4}


@pytest.mark.parametrize("mode", ["no-memory", "no-memory-noalloc"])
def test_no_exception_leaves_a_call(exe, mode):
    """Each host allocation of a call fails in turn: the call answers AMG_ERR_NOMEM or does without, leaves nothing
    queued, and the next call is whole."""
    r = result(exe, mode)
    assert r["bad"] == 0 and r["queued"] == 0


@pytest.mark.parametrize("mode", ["refused-engine", "refused-top"])
def test_a_list_with_a_kernel_that_cannot_be_shared_is_refused(exe, mode):
    """(Planning's rules keep such systems out.) Launched beside the recording, the kernel would run at once."""
    assert result(exe, mode) == {"planning": 0, "in_step": 0, "status": 0, "launches": 1}


def test_a_call_without_allocation_takes_no_host_memory_either(exe):
    """Not in its first call: what it launches is recorded when the systems are planned."""
    assert result(exe, "heap-noalloc") == {"status": 0, "allocations": 0}

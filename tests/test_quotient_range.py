"""The range of the quotient by a stored reciprocal, on the CPU (tests/host/quotient.hip)."""
from tests import host_program


def test_quotient_is_correctly_rounded_down_to_the_smallest_normal_diagonal(tmp_path):
    out = host_program.run(host_program.build("quotient.hip", tmp_path)).split()
    got = dict(zip(out[::2], map(int, out[1::2])))
    assert got == {"wrong32": 0, "wrong64": 0, "below32": 1, "below64": 1}

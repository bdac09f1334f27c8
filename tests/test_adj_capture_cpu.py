"""Host: an adjoint run whose graphs cannot be instantiated falls back to launches
and reads the same tape.

In the device of tests/host no captured graph instantiates.  The adjoint steps then
have to read the tape entries of the states T - 1, T - 2, ..., 0, whatever number
of launches a segment takes.
"""
import pytest

from tests import host


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    return host.build(tmp_path_factory.mktemp("host"))


@pytest.mark.parametrize("every", [3, 4, 5, 6, 10, 15, 25])
def test_backward_reads_the_tape_of_every_state(program, every):
    T = 3 * every + 1
    tried, *levels = [float(v) for v in host.run(program, "adjoint", 32, T, every)[0].split()]
    assert tried == 1  # one attempt, launches from then on
    assert levels == list(range(T - 1, -1, -1))

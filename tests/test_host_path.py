"""The host side of a solve (no GPU needed)."""
import subprocess

from paper_1506_08435_amd import build


def test_waiting_for_the_device_allocates_nothing():
    """The wait of each CG iteration takes its predicate as it is: a type-erased
    one (std::function) goes to the host heap when it captures more than two
    words, on the latency path, and a refusal there would leave the C ABI as an
    exception."""
    names = subprocess.run(["nm", "-C", build.LIB], check=True, capture_output=True, text=True).stdout
    assert " T nn_solve_nonneg" in names
    assert not [n for n in names.splitlines() if "std::function" in n or "std::_Function" in n]

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


def test_iterations_enqueued_ahead(tmp_path):
    """cg_chunk: 0 and the default are the library's choice, any other number is
    taken as it is."""
    src = tmp_path / "ahead.cpp"
    src.write_text('#include "ahead.hpp"\n#include <cstdio>\n#include <cstdlib>\n'
                   "int main(int n, char **v) { for (int i = 1; i < n; i++) std::printf(\"%d \", nnqp::cg_ahead(std::atoi(v[i]))); }\n")
    exe = str(tmp_path / "ahead")
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, "-o", exe, str(src)], check=True)
    asked = [0, 1, 2, 3, 15, 16, 17, 64, 5000]
    out = subprocess.run([exe, *map(str, asked)], check=True, capture_output=True, text=True).stdout
    assert list(map(int, out.split())) == [2, 1, 2, 3, 15, 2, 17, 64, 5000]

"""The walk that shrinks S-box circuits (gen/sbox_walk.c): it prints correct circuits no larger than the
one it starts from, and refuses a wrong one.
"""
import subprocess

import pytest

from paper_1305_4376_amd.gen import gen_sbox


@pytest.fixture(scope="module")
def tool(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("walk") / "sbox_walk")
    subprocess.check_call(["gcc", "-O2", "-Wall", "-Werror", "-o", exe, gen_sbox.WALK_SRC])
    return exe


def _run(tool, steps, tab, circuit):
    return subprocess.run([tool, "5", str(steps), "1"] + [str(v) for v in tab], input=circuit.dump(),
                          capture_output=True, text=True, timeout=120)


def _long_circuit(tab):
    """The first output as a tree of multiplexers: many more gates than needed."""
    gates, mux = [], 0b11001010  # bit 4a + 2b + c: c where a = 0, b where a = 1

    def build(points, depth):
        if depth == 5:  # both values of the last input: a gate of it alone
            gates.append((6 + len(gates), 5, 5, 5, points[0] | points[1] << 7))
            return gates[-1][0]
        half = len(points) // 2
        lo, hi = build(points[:half], depth + 1), build(points[half:], depth + 1)
        gates.append((6 + len(gates), depth, hi, lo, mux))
        return gates[-1][0]

    root = build([v >> 3 for v in tab], 0)
    return gen_sbox.Circuit(gates, [root] * 4)


@pytest.mark.parametrize("box", [0, 3, 7])
def test_walk_keeps_the_stored_circuits_correct(tool, box):
    tab, start = gen_sbox.sbox_tables()[box], gen_sbox.load_store()[box]
    res = _run(tool, 5000, tab, start)
    assert res.returncode == 0, res.stderr
    circuit = gen_sbox.last_circuit(res.stdout)
    circuit.polarities(tab)  # raises if an output is wrong
    assert len(circuit.gates) <= len(start.gates)


def test_walk_shrinks_a_long_circuit(tool):
    tab = [15 * (v >> 3) for v in gen_sbox.sbox_tables()[4]]  # all four outputs alike
    start = _long_circuit(tab)
    start.polarities(tab)
    res = _run(tool, 20000, tab, start)
    assert res.returncode == 0, res.stderr
    circuit = gen_sbox.last_circuit(res.stdout)
    circuit.polarities(tab)
    assert len(circuit.gates) < len(start.gates) // 2


def test_walk_refuses_a_wrong_start(tool):
    res = _run(tool, 10, gen_sbox.sbox_tables()[4], gen_sbox.load_store()[3])
    assert res.returncode != 0 and "not correct" in res.stderr

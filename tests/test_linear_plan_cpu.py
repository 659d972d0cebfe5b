"""Host logic of the linear schedules (CNOTs as a change of basis): tests/
linear_replay.cpp builds plans of random circuits (entangler-poor to dense, and
the whole gate library), replays every instruction, LDS exchange and tile
address in double precision and compares the measured <Z>, the probabilities
and the adjoint's walk back with the circuit's gates applied one by one.  The
replay also checks that exchanges are permutations without bank conflicts and
that a tile's local address columns are distinct single bits."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_11985_amd", "csrc")


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("replay") / "linear_replay")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-I", os.path.join(ROOT, "include"),
                           "-I", CSRC, os.path.join(ROOT, "tests", "linear_replay.cpp"),
                           os.path.join(CSRC, "planner.cpp"), "-o", exe])
    return exe


# (n, circuits, gates, tile_qubits, reg_bits): resident with 8 and 16 amplitudes
# per thread, streaming with one to several global qubits and every tile size,
# 32 amplitudes per thread, circuits with no gate at all, and long ones
@pytest.mark.parametrize("n,count,gates,tile,rb", [
    (9, 16, 60, 0, 0), (10, 8, 120, 0, 0), (11, 8, 3, 0, 0), (12, 8, 90, 0, 0), (12, 4, 60, 0, 3),
    (13, 4, 80, 0, 0), (14, 8, 80, 12, 0), (14, 4, 80, 13, 0), (14, 4, 60, 14, 0),
    (15, 4, 100, 12, 0), (15, 4, 100, 12, 5), (16, 4, 150, 12, 0), (17, 4, 60, 13, 0),
    (18, 2, 60, 12, 0), (16, 4, 0, 12, 0), (9, 2, 9000, 0, 0)])
def test_replay(replay, n, count, gates, tile, rb):
    out = subprocess.run([replay, str(n), "0", str(count), str(gates), str(tile), str(rb)],
                         capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.endswith("ok\n"), out.stdout[-500:] + out.stderr


def test_replay_more_greedy_passes(replay):
    """A circuit whose greedy linear passes outnumber those with the CNOTs as
    gates: the replay refuses more passes, so the fewer have to be taken."""
    out = subprocess.run([replay, "16", "1009", "1", "150", "12", "0"], capture_output=True,
                         text=True)
    assert out.returncode == 0 and out.stdout.endswith("ok\n"), out.stdout[-500:] + out.stderr


# (prefix, n, circuits, gates, tile_qubits): entanglers before the first rotation
# (linear_replay.cpp, Prefix), of which the passes that run no rotation go, though
# a plan's first pass has to start in logical order.  1-3 without a layer of
# rotations in front, 4-6 with one, which the training step's plan leaves out.
@pytest.mark.parametrize("prefix", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("n,count,gates,tile", [
    (12, 2, 12, 0), (14, 4, 1, 12), (15, 4, 12, 12), (15, 4, 1, 13), (16, 4, 1, 12),
    (16, 4, 12, 13), (18, 2, 1, 12), (20, 1, 1, 12), (14, 2, 60, 12)])
def test_replay_entanglers_first(replay, prefix, n, count, gates, tile):
    out = subprocess.run([replay, str(n), "0", str(count), str(gates), str(tile), "0",
                          str(prefix)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.endswith("ok\n"), out.stdout[-500:] + out.stderr

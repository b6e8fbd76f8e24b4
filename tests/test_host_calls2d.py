"""What the 2D entry points launch, read on the CPU: the host code of a V-cycle and of a Newton step
with the launches recorded (tests/host/calls2d.cpp, against the built library's planning functions)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2505_10857_amd")


@pytest.fixture(scope="module")
def calls(tmp_path_factory):
    lib = os.path.join(PKG, "libnmg.so")
    if not os.path.exists(lib):
        pytest.skip("libnmg.so not built (run __graft_entry__.build())")
    exe = str(tmp_path_factory.mktemp("host") / "calls2d")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                           os.path.join(ROOT, "tests", "host", "calls2d.cpp"), lib, "-Wl,-rpath," + PKG,
                           "-Wl,-rpath-link,/opt/rocm/lib", "-o", exe])

    def run(queries):
        """One list of launches (tuples, the kind first) and the status of the call, per query."""
        text = "\n".join(" ".join(map(str, q)) for q in queries) + "\n"
        out = subprocess.run([exe], input=text, text=True, capture_output=True, check=True).stdout
        results, now = [], []
        for line in out.splitlines():
            kind, *v = line.split()
            if kind == "end":
                results.append((now, int(v[0])))
                now = []
            else:
                now.append((kind, *map(int, v)))
        assert len(results) == len(queries)
        return results

    return run


def _grids():
    """Grids cx 2^k x cy 2^k of at most 40 coarsest cells, thin and square ones, odd sizes."""
    for cx, cy in ((8, 4), (5, 3), (3, 2), (7, 5), (10, 4), (20, 1), (1, 13), (40, 1), (2, 2), (6, 6), (1, 1)):
        for k in range(1, 11):
            if (cx << k) * (cy << k) <= 1 << 20:
                yield cx << k, cy << k, k + 1


@pytest.mark.parametrize("jac", [9, 21])
@pytest.mark.parametrize("prec", [0, 1])
def test_every_phase_of_several_workgroups_exchanges(calls, prec, jac):
    """A workgroup of a cooperative phase reads dU of its neighbours' cells at the start and writes
    its own in place at the end; an exchange in between is what orders the two.  So every such phase
    needs one, for all smoothing counts, and its numbers have to lie apart from the next phase's."""
    nus = [(0, 0), (0, 1), (1, 0), (1, 1), (2, 1), (1, 2), (0, 3), (3, 0), (2, 3), (4, 4), (20, 20)]
    queries = [(entry, nx, ny, lv, jac, prec, a, b, 3, 0, 0, 256)
               for nx, ny, lv in _grids() for a, b in nus for entry in ("setup", "step")]
    seen = 0
    for q, (launches, status) in zip(queries, calls(queries)):
        assert status == 0, q
        free = 0                                  # exchanges numbered so far
        for kind, *v in launches:
            if kind not in ("resident", "streamed"):
                continue
            nx, ny, nb, C, tx, ty, gx, gy, m, nu, prolong, restr, tiled, tag, reserved = v
            runs = nu * 4 * (C - 1) + 1 if nu > 0 else 0
            done = 0 if runs == 0 else (-(-runs // m) if restr else (runs - 1) // m)
            assert tag >= free and reserved >= done, (q, kind, v)
            free = tag + done
            assert gx * gy == 1 or done >= 1, f"{q}: {kind} {v} has no exchange"
            seen += 1
    assert seen > 1000


# grids whose finest level is streamed: exact and ragged tiles, FP64 and FP32
STREAMED = [(1024, 512, 8, 0), (1024, 512, 8, 1), (768, 384, 8, 0), (64, 2112, 7, 0), (128, 4224, 8, 1)]


@pytest.mark.parametrize("nx,ny,levels,prec", STREAMED)
def test_the_operator_lies_where_the_set_up_left_it(calls, nx, ny, levels, prec):
    """A set-up call and a call that reuses its operator agree on the order of the rows, whatever
    differs between them: the workspace's size, a capture, the device's compute units.  And each way
    of a call runs as it is meant to: streamed where that is possible, else a launch a pass."""
    ways = {(0, 0, 256): True, (1, 0, 256): False, (0, 1, 256): False, (0, 0, 64): False}
    for entry in ("setup", "vcycle"):
        for way, streams in ways.items():
            (launches, status), = calls([(entry, nx, ny, levels, 9, prec, 2, 2, 3, *way)])
            assert status == 0
            assert any(kind == "streamed" for kind, *_ in launches) == streams
            assert any(kind == "pass" and v[:2] == [nx, ny] for kind, *v in launches) == (not streams)
            rows = [v[2] for kind, *v in launches if kind == "rows"]
            assert len(rows) == (2 if entry == "setup" else 1) and set(rows) == {1}, (entry, way)


def test_rows_in_tiles_have_a_slot_each(calls):
    sizes = [(nx, ny, tw, th) for nx in (1, 2, 16, 31, 64, 90) for ny in (1, 3, 34, 47, 70)
             for tw in (16, 17, 18, 32) for th in (4, 5, 6, 34)]
    queries = [("order", *q) for q in sizes]
    for q, (_, bad) in zip(sizes, calls(queries)):
        assert bad == 0, (q, bad)

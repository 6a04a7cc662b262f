"""The rows of the damage passes, checked on the CPU entry by entry against the meshes they
were built from: every neighbour of every owned and ring node once, with the elements at the
pair, column ids inside the rings that a pass of each degree keeps, and element lists by ring.
Meshes: grids with and without random diagonals, one cell, a strip, fans (a node with more
neighbours than a row's base entries, and with so many that only one ring fits), an edge with
three triangles."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_row_plan_matches_its_meshes(tmp_path):
    from paper_2606_23458_amd import build as b
    if not os.path.exists(b.LIB):
        b.build()
    exe = str(tmp_path / "row_plan")
    cmd = [b.hipcc(), "-std=c++17", "-O1", "-I", os.path.join(b.ROOT, "include"),
           os.path.join(HERE, "row_plan_driver.cpp"), "-o", exe, "-L", b.PKG, "-lpfrac", f"-Wl,-rpath,{b.PKG}"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout[-2000:] + run.stderr[-500:]
    assert run.stdout.count(" ok") == 8

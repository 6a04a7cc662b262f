"""Every LDS read of the damage passes, checked on the CPU against the bytes their launch asks
for: each degree a caller may ask for, both widths, lanes past a tile's rows, batches whose
instances run different degrees, and a mesh that only the row plan's second cut fits."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_damage_passes_read_inside_their_lds(tmp_path):
    from paper_2606_23458_amd import build as b
    if not os.path.exists(b.LIB):
        b.build()
    exe = str(tmp_path / "row_reads")
    cmd = [b.hipcc(), "-std=c++17", "-O2", "-I", os.path.join(b.ROOT, "include"),
           os.path.join(HERE, "row_reads_driver.cpp"), "-o", exe, "-L", b.PKG, "-lpfrac", f"-Wl,-rpath,{b.PKG}"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout[-2000:] + run.stderr[-500:]
    assert run.stdout.count(" ok") == 21

"""The sums that stand in for the first stages of a transform on small inputs, on the host."""
import os
import shutil
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_sums_of_small_samples(tmp_path):
    """tests/arith_sum_check.cpp on moduli of every size a policy takes, 2^b - c with the smallest and largest c."""
    cxx = shutil.which("g++") or shutil.which("clang++")
    exe = str(tmp_path / "check")
    subprocess.check_call([cxx, "-O2", "-std=c++17", "-w", "-o", exe, os.path.join(ROOT, "tests", "arith_sum_check.cpp")])
    moduli = [12289, 65537, (1 << 29) + 11, (1 << 30) - 35, (1 << 36) - 5, (1 << 43) + 3, (1 << 44) - 17]
    moduli += [(1 << b) - c for b in (45, 50, 54, 55, 56, 60) for c in (1, 262143, 36044799, (1 << 31) - 1)]
    out = subprocess.run([exe] + [str(q) for q in moduli], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout
    counts = [int(v) for v in out.stdout.split()]
    assert counts[:4] == [2, 2, 2, 2] and min(counts[:7]) == 1 and sum(c == 2 for c in counts[7:]) >= 10, out.stdout

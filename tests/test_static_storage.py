"""The static device array behind jatam_classify_static: the tally's counter sets,
not the queues of a pipeline that the call does not run.  (The array's host
stand-in has its size.)"""
import subprocess

from paper_2205_15311_amd import jatam


def test_static_array_is_small():
    out = subprocess.run(["nm", "-S", jatam.LIB_PATH], capture_output=True, text=True,
                         check=True).stdout
    sizes = [int(line.split()[1], 16) for line in out.splitlines()
             if len(line.split()) == 4 and line.split()[2] in "bBdD"]
    assert sizes and max(sizes) <= 64 * 1024, max(sizes)

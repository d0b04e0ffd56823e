"""What the kernels promise the compiler about their pointers, read off the compiler's own view of the
source (no optimisation passes, no GPU)."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rows_that_a_step_edits_are_not_noalias(tmp_path):
    """The best-move kernel edits the starts and ends it reads in a descent: its instantiations for that (SEARCH, the fourth
    argument, without KEPT, the fifth) must not declare them free of other writers."""
    out = tmp_path / "nb.ll"
    subprocess.run(["hipcc", "--offload-arch=gfx950", "--offload-device-only", "-O1", "-std=c++17", "-S", "-emit-llvm", "-Xclang", "-disable-llvm-passes",
                    "-I", os.path.join(ROOT, "include"), "-o", str(out), os.path.join(ROOT, "paper_2304_14463_amd", "csrc", "moc_neighbours.hip")],
                   check=True, capture_output=True)
    seen = {True: 0, False: 0}
    for line in out.read_text().splitlines():
        kernel = re.match(r"define amdgpu_kernel .*best_neighbours_kernelILi\d+ELb[01]ELi\d+ELb([01])ELb([01])EE[^(]*\((.*)\) #", line)
        if not kernel:
            continue
        search, kept = kernel.group(1) == "1", kernel.group(2) == "1"
        assert search != kept
        starts, ends = kernel.group(3).split(", ptr addrspace(1) ")[1:3]   # the first two plain pointers
        assert starts.startswith("noalias") == ends.startswith("noalias") == kept, line[:200]
        seen[kept] += 1
    assert seen[True] > 0 and seen[False] > 0

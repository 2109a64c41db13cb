"""The halt word within one launch.  The p update's block 0 sets ctl->halt while
other blocks of the same launch may only be starting, so a block there must
take one reading of it for all its waves: through the copy of the control
block that one thread per word brings to LDS, after a barrier.  Every other
kernel that reads the word leaves it alone.  A property of the source (the
window of the race is too narrow to meet in a run).  No GPU."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2206_14780_amd", "csrc")


def _kernels():
    """Name and body of every kernel of the solver, comments taken out."""
    text = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, "solver.hip")).read())
    out = {}
    for m in re.finditer(r"__global__[^;{]*?\b(k_\w+)\s*\(", text):
        i = text.index("{", m.end())
        depth, j = 1, i + 1
        while depth:
            depth += {"{": 1, "}": -1}.get(text[j], 0)
            j += 1
        out[m.group(1)] = text[i:j]
    return out


def test_no_kernel_reads_the_halt_word_that_it_sets():
    ks = _kernels()
    assert len(ks) > 8 and "k_pupd" in ks
    sets = {k for k, b in ks.items() if re.search(r"ctl->halt\s*=[^=]", b)}
    reads = {k for k, b in ks.items() if re.search(r"ctl->halt\b(?!\s*=[^=])", b)}
    assert sets == {"k_pupd"}
    assert not sets & reads


def test_the_p_update_asks_its_copy_after_a_barrier():
    body = _kernels()["k_pupd"]
    stop = re.search(r"stop\s*=\s*\[&\]\s*(?:\(\)\s*)?\{(.*?)\}", body, re.S).group(1)
    assert re.search(r"__syncthreads\(\);.*get\(\)->halt", stop, re.S)
    assert body.index("copy.load(ctl)") < body.index("stop")

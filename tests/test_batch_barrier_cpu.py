"""The batched kernel's grid-wide barrier, from the listing of its compiled
code: one wave of a workgroup issues the write-back that makes the workgroup's
stores visible to the others, so every wave has to have waited for its own
stores before the workgroup barrier in front of that write-back."""
import re
import subprocess

from paper_2502_05279_amd import build

LABEL = re.compile(r"^\.LBB\w+:")
STORE = re.compile(r"^(flat|global|buffer|scratch)_(store|atomic)")


def listing(tmp_path):
    out = tmp_path / "batch.s"
    cmd = [a for a in build.command(str(out)) if a != "-shared" and not a.endswith(".hip")]
    subprocess.run(cmd + ["-S", "--cuda-device-only", build.CSRC + "/bmg_batch.hip"], check=True,
                   stderr=subprocess.DEVNULL)
    text = [re.sub(r"\s*;.*", "", s).strip() for s in out.read_text().splitlines()]
    return [s for s in text if s and (LABEL.match(s) or not s.startswith("."))]


def arrivals(code):
    """Indices of the workgroup barriers that a write-back follows."""
    for k, s in enumerate(code):
        if s.startswith("buffer_wbl2"):
            j = k - 1
            while not code[j].startswith(("s_barrier", "buffer_wbl2", "global_atomic", "flat_atomic")):
                j -= 1
            if code[j].startswith("s_barrier"):
                yield j


def test_every_wave_waits_for_its_stores_before_the_grid_barrier(tmp_path):
    code = listing(tmp_path)
    found = list(arrivals(code))
    assert len(found) >= 6          # one per use of the barrier
    for j in found:
        k = j - 1
        while not (code[k].startswith("s_waitcnt") and "vmcnt(0)" in code[k]):
            assert not LABEL.match(code[k]) and not STORE.match(code[k]), code[k:j + 1]
            k -= 1

"""How the one-launch quantiser (csrc/lordba_ptq_run.h) ends, read off its source: faults here would be races between workgroups, which
no run shows reliably and none should be made to show on a GPU."""
import os
import re

from paper_2605_24058_amd import binding


def _kernel():
    """The kernel's text without comments, as lines."""
    with open(os.path.join(binding._CSRC, "lordba_ptq_run.h")) as f:
        text = re.sub(r"/\*.*?\*/|//[^\n]*", "", f.read(), flags=re.S)
    return [line.strip() for line in text[text.index("lordba_ptq_run_kernel(PtqRunArgs)"):].splitlines() if line.strip()]


def test_one_thread_reads_the_end_flag_for_its_workgroup():
    # The flag is set inside the launch (by the workgroup that sees the run end), so waves that read it for themselves could part.
    lines = _kernel()
    reads = [i for i, line in enumerate(lines) if "kDone" in line and not re.search(r"ctrl\[kDone\] = ", line)]
    assert len(reads) == 1 and re.match(r"if \(published\(arg->a\.ctrl \+ kDone\) != 0\.0\) sh_numbers = ", lines[reads[0]]), reads
    guard = max(i for i in range(reads[0]) if lines[i].startswith("if (threadIdx.x == 0) {"))
    assert not any("}" in line for line in lines[guard:reads[0]])   # (still inside the block of one thread)
    used = [i for i, line in enumerate(lines) if re.search(r"readfirstlane\(sh_numbers\)", line)]
    assert len(used) == 1 and "__syncthreads();" in lines[reads[0]:used[0]]


def test_stop_bits_are_written_before_their_workgroup_counts_as_gone():
    # The last workgroup to leave zeroes the counters; a stop bit that landed after that would end the next piece of the run.
    lines = _kernel()
    bits = [i for i, line in enumerate(lines) if "__hip_atomic_fetch_or(" in line]
    gone = [i for i, line in enumerate(lines) if "__hip_atomic_fetch_add(arg->g.sync + kSyncStride" in line]
    assert len(bits) == 1 and len(gone) == 1 and bits[0] < gone[0]
    waits = [i for i in range(bits[0], gone[0]) if "s_waitcnt vmcnt(0)" in lines[i]]
    leaves = [i for i in range(bits[0], gone[0]) if lines[i].startswith("break;")]
    assert waits and leaves and waits[0] < leaves[0]
    assert re.match(r"if \(done && ", lines[bits[0]])   # (at the end of a piece nobody waits: no bits at all)

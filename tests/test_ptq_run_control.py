"""How the one-launch quantiser (csrc/lordba_ptq_run.h) ends, read off its source: faults here would be races between workgroups, which
no run shows reliably and none should be made to show on a GPU."""
import os
import random
import re

import pytest

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


# What a block of each kind of step waits for by arrivals (step, sweeps back) before it looks at the shares (step, sweeps back) that it takes
# by their mark, the parity of the sweep; step 0 takes the shares of step 2 first, those of step 3 behind another wait.
_STEPS = {0: [([(1, 1)], (2, 1)), ([(2, 1)], (3, 1))], 1: [([(3, 1)], (0, 0))], 2: [([(0, 0)], (1, 0))], 3: [([(1, 0)], (2, 0))]}


def _stale_reads(steps, seed, workgroups, blocks, sweeps=6):
    """Runs the steps' blocks on `workgroups` in a random order of events; returns the reads that took shares of another sweep for theirs."""
    rng = random.Random(seed)
    order = [(t, p, b) for t in range(sweeps) for p in range(4) for b in range(blocks)]
    shares = {(p, b): -1 for p in range(4) for b in range(blocks)}   # the sweep whose shares lie there (complete at sweep -1)
    arrived = {(p, -1): blocks for p in range(4)}
    taken, stale, left = 0, 0, len(order)

    def block(t, p, b):   # a generator: True where the block goes on, False where it waits
        nonlocal stale
        for waits, (source, back) in steps[p]:
            for step, behind in waits:
                while arrived.get((step, t - behind), 0) < blocks and t - behind >= 0:
                    yield False
            if t - back < 1:   # the first sweep goes by the arrivals
                while arrived.get((source, t - back), 0) < blocks and t - back >= 0:
                    yield False
            for other in range(blocks):
                while shares[source, other] & 1 != (t - back) & 1:
                    yield False
                stale += shares[source, other] != t - back
                yield True
        yield "ask"
        shares[p, b] = t
        yield True
        arrived[p, t] = arrived.get((p, t), 0) + 1

    held = [[] for _ in range(workgroups)]
    while left:
        w = rng.choice([k for k in range(workgroups) for _ in range(1 + 8 * (k % 3 == 0))])   # (some are much slower than others)
        if not held[w] and taken < len(order):
            held[w].append(block(*order[taken]))
            taken += 1
        if held[w]:
            try:
                if next(held[w][0]) == "ask" and taken < len(order):
                    held[w].append(block(*order[taken]))
                    taken += 1
            except StopIteration:
                held[w].pop(0)
                left -= 1
    return stale


@pytest.mark.parametrize("workgroups,blocks", [(1, 2), (3, 1), (5, 2), (9, 2), (40, 3)])
def test_shares_taken_by_their_mark_are_those_of_the_sweep(workgroups, blocks):
    assert sum(_stale_reads(_STEPS, seed, workgroups, blocks) for seed in range(40)) == 0


def test_the_model_finds_a_step_that_looks_two_sweeps_ahead():
    planted = dict(_STEPS)
    planted[0] = [([], (2, 1)), ([(2, 1)], (3, 1))]
    assert sum(_stale_reads(planted, seed, 9, 1) for seed in range(40)) > 0


def test_the_kernel_waits_as_the_model_does():
    lines = "\n".join(_kernel())
    tikhonov = lines[lines.index("const bool update = p == 0"):]
    first, second = tikhonov.index("if (wait_for(1, t - 1)) break;"), tikhonov.index("gather(arg->g.partS[0]")
    third, fourth = tikhonov.index("if (wait_for(p + 2, t - 1)) break;"), tikhonov.index("double total = gather(")
    assert first < second < third < fourth
    scale = tikhonov[tikhonov.index("if (p == 2 ? wait_for(0, t) : wait_for(1, t)) break;"):]
    assert scale.index("wait_for(0, t)") < scale.index("gather(")

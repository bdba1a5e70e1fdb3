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


# The whole control flow of a run of `sweeps` sweeps (from the start of a launch at sweep 0, the warm start done): the keeper, which publishes beta and
# the penalty of every sweep, the number that is asked for ahead, the stop bits and who leaves on them.  `end`: the sweep after which the run
# is over (None: the last one, no bits).
def _run(seed, workgroups, blocks, sweeps, end, kept_stops=True, waits_for_beta=True):
    """Returns how many reads took something of another sweep, and whether every workgroup left with every sweep up to the end done."""
    rng = random.Random(seed)
    order = [(t, 0, -1) if b < 0 else (t, p, b) for t in range(sweeps) for p in range(4) for b in range(-1 if p == 0 else 0, blocks)]
    order.append((sweeps, 0, -1))   # behind the last sweep: its beta and penalty
    per = [blocks + 1, blocks, blocks, blocks]
    shares = {(p, b, v): -1 for p in range(4) for b in range(blocks) for v in range(2)}   # two values of each, which may come one by one
    slot, arrivals, stop, kept, kept_stop = [-1, -1], [0] * 4, [False] * 4, 0, False
    wrong, done_sweeps, taken = 0, 0, 0

    class Over(Exception):
        pass

    def wait(p, t):   # arrivals of step p through sweep t
        while not stop[p] and arrivals[p] < per[p] * (t + 1):
            yield False
        if stop[p]:
            raise Over

    def gather(p, t, want_kept=0):   # by the mark; the shares of the workgroups come as they come
        nonlocal wrong
        for b in range(blocks):
            for v in range(2):
                while shares[p, b, v] & 1 != t & 1 or (waits_for_beta and kept < want_kept):
                    if kept_stop:
                        raise Over
                    yield False
                wrong += shares[p, b, v] != t

    def block(t, p, b):
        nonlocal wrong, kept, kept_stop, done_sweeps
        update, marked = p == 0 and t > 0, t > (1 if p == 0 else 0)
        if update:
            yield from wait(1, t - 1)
            if marked:
                yield from gather(2, t - 1)
            yield from wait(2, t - 1)
            yield from (gather(3, t - 1) if marked else wait(3, t - 1))
        elif p == 1:
            yield from wait(3, t - 1)
            yield from (gather(0, t, t + 1) if marked else wait(0, t))
        elif p >= 2:
            yield from wait(p - 2, t)
            wrong += slot[t & 1] != t
            yield from (gather(p - 1, t) if marked else wait(p - 1, t))
        yield "ask"
        over = update and end == t - 1
        if b < 0:
            slot[t & 1] = t
            yield True
            if over or t == sweeps:
                done_sweeps = t
                if over:
                    for k in rng.sample(range(5), 5):
                        if k < 4:
                            stop[k] = True
                        else:
                            kept_stop = kept_stops
                        yield True
                raise Over
            arrivals[0] += 1
            yield True
            kept += 1
            return
        if over:
            raise Over
        if p == 1:
            wrong += slot[t & 1] != t
        for v in rng.sample(range(2), 2):
            shares[p, b, v] = t
            yield True
        arrivals[p] += 1

    held, idle = [[] for _ in range(workgroups)], 0
    gone = [False] * workgroups
    while not all(gone) and idle < 400 * workgroups:
        w = rng.choice([k for k in range(workgroups) if not gone[k] for _ in range(1 + 8 * (k % 3 == 0))])
        idle += 1
        if not held[w]:
            if taken >= len(order):
                gone[w], idle = True, 0
                continue
            held[w].append(block(*order[taken]))
            taken += 1
        try:
            said = next(held[w][0])
            if said == "ask":
                if taken < len(order):
                    held[w].append(block(*order[taken]))
                taken += 1
            idle = 0 if said else idle
        except StopIteration:
            held[w].pop(0)
            idle = 0
        except Over:
            gone[w], idle = True, 0
    return wrong, all(gone) and done_sweeps == (sweeps if end is None else end + 1)


@pytest.mark.parametrize("workgroups,blocks", [(1, 2), (2, 1), (5, 2), (9, 2), (14, 3)])
@pytest.mark.parametrize("sweeps,end", [(1, None), (5, None), (1, 0), (6, 0), (6, 1), (6, 4), (6, 5)])
def test_a_run_ends_and_every_workgroup_leaves(workgroups, blocks, sweeps, end):
    for seed in range(12):
        assert _run(seed, workgroups, blocks, sweeps, end) == (0, True), seed


def test_the_model_of_a_run_finds_planted_faults():
    # Without the stop bit of the keeper's word somebody waits for shares that nobody makes; without the wait for it somebody takes beta of another sweep
    assert not all(_run(seed, 9, 2, 6, 2, kept_stops=False)[1] for seed in range(25))
    assert any(_run(seed, 9, 2, 6, None, waits_for_beta=False)[0] for seed in range(25))


def test_the_kernel_ends_a_run_as_the_model_does():
    text = "\n".join(_kernel())
    # the keeper sets all five words, and counts itself in its own word behind its arrival
    assert re.search(r"if \(done && tid < 5\) __hip_atomic_fetch_or\(tid < 4 \? arrivals\(tid\) : kept, kStop,", text)
    arrive = text[text.index("auto arrive = "):text.index("auto gather = ")]
    assert arrive.index("fetch_add(arrivals(p)") < arrive.index("fetch_add(kept")
    # U2's step waits for as many sweeps' beta as there are with its own; the others take theirs behind an arrival that the keeper is part of
    assert re.search(r"blk, p == 0 \? 0u : static_cast<uint32_t>\(t - arg->g\.t_begin \+ 1\)\);", text)
    # whoever sees the stop bit leaves, for the whole workgroup behind a barrier
    assert len(re.findall(r"readfirstlane\(sh_over\) != 0u\) break;", text)) == 3 and text.count("sh_over = 1u;") == 1

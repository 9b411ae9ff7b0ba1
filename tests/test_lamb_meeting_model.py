"""A plain Python model of how the workgroups of a single-launch LAMB step wait for each other (no GPU).

`lamb_one_launch_kernel` publishes every workgroup's sums, waits for everybody's and then writes w.  A wave may give up, and
then the waves that are still there share the shard's chunks.  Here every wave is a small state machine whose steps are
the kernel's shared accesses, and EVERY interleaving is walked through, with every look free to be the one after which a wave gives
up or glances at the outcome word, and with any number of workgroups resident at a time.  What has to hold:

  * from every state that can be reached the launch can still end (no deadlock; a wave that only looks does not move);
  * nobody writes w before every workgroup has published;
  * when the launch has ended, the w of every chunk was written by its own waves or taken from the counter and computed again,
    and the chunks on the counter were all done by the wave that drew them.

The second half runs two launches over the same words, as calls that overlap on one plan would, with counted looks: whatever
they read, every wave leaves."""
import random

import pytest

OPEN, ABANDONED, CLOSED = 0, 1, 2


class Launch:
    """n workgroups of `waves` waves, at most `resident` of them on the device, groups of `group` chunks (0: no groups).
    A state is (arrived, chunks published, groups published, outcome, next ticket, own parts written, chunks done again, waves);
    a wave is None before its workgroup starts, then (pc, last, sure, chunk in hand)."""

    def __init__(self, n, waves, resident, group, stays):
        self.n, self.waves, self.resident, self.group, self.stays = n, waves, resident, group, stays
        self.groups = -(-n // group) if group else 0

    def start(self):
        first = tuple(("arrive", False, False, -1) if w // self.waves < self.resident else None for w in range(self.n * self.waves))
        return (0, 0, 0, OPEN, 0, 0, 0, first)

    def gave_up_or_glanced(self, wave, state, b):
        """What a wave may do after a look in vain, besides looking again."""
        pc, last, sure, _ = wave
        if not last and not sure:
            yield ("giveup_" + pc, last, sure, -1)
        if not sure and state[3] == ABANDONED:
            yield ("help", last, sure, -1) if last else ("exit", last, sure, -1)
            if not last and self.stays[b]:
                yield ("help", last, sure, -1)

    def steps(self, state):
        arrived, pub, gpub, outcome, ticket, own, again, waves = state
        everybody = (1 << self.n) - 1
        for i, wave in enumerate(waves):
            if wave is None or wave[0] == "exit":
                continue
            b, k = divmod(i, self.waves)
            pc, last, sure, c = wave
            mates = [waves[b * self.waves + m] for m in range(self.waves)]
            leader = self.group and b % self.group == 0 and k == self.waves - 1
            to = lambda pc_, **kw: self.move(state, i, (pc_, kw.pop("last", last), kw.pop("sure", sure), kw.pop("c", -1)), **kw)
            if pc == "arrive":
                yield to("barrier", last=arrived + 1 == self.n * self.waves, arrived=arrived + 1)
            elif pc == "barrier":
                if all(m[0] != "arrive" for m in mates):
                    yield to("publish" if k == 0 else "lead" if leader else "wait")
            elif pc == "publish":
                yield to("lead" if leader else "wait", pub=pub | 1 << b)
            elif pc in ("lead", "wait"):
                if pc == "lead":
                    g = b // self.group
                    need = sum(1 << x for x in range(g * self.group, min((g + 1) * self.group, self.n)))
                    found, then = pub & need == need, "gpub"
                else:
                    found = gpub == (1 << self.groups) - 1 if self.group else pub == everybody
                    then = "write"
                if found:
                    yield to(then)
                else:
                    for w in self.gave_up_or_glanced(wave, state, b):
                        yield self.move(state, i, w)
            elif pc.startswith("giveup_"):
                yield to(pc[7:], sure=True) if outcome == CLOSED else to("exit", outcome=ABANDONED)
            elif pc == "gpub":
                yield to("wait", gpub=gpub | 1 << b // self.group)
            elif pc == "write":
                assert pub == everybody, "w written before everybody has published"
                if last:                                                   # the exchange, before its own part is written
                    yield to("own", c=ticket if outcome == ABANDONED else -1, outcome=CLOSED)
                else:
                    yield to("own")
            elif pc == "own":
                yield to("after", own=own | 1 << i, c=c)
            elif pc == "after":
                if last:
                    yield to("exit") if c < 0 else to("help", outcome=ABANDONED, ticket=c)
                else:
                    yield to("exit")                                       # did not wait long and saw nobody leave
                    if outcome == ABANDONED:
                        yield to("help")
            elif pc == "help":
                if pub == everybody:
                    yield to("draw")
                elif not last:
                    yield to("exit")
            elif pc == "draw":
                assert pub == everybody
                if outcome != ABANDONED:                                   # the last arrival's exchange: it puts the old word back
                    assert not last
                    yield to("exit")
                else:
                    yield to("redo", c=ticket, ticket=ticket + 1) if ticket < self.n else to("exit", ticket=ticket + 1)
            elif pc == "redo":
                yield to("draw", again=again | 1 << c)

    def move(self, state, i, wave, **kw):
        names = ("arrived", "pub", "gpub", "outcome", "ticket", "own", "again")
        shared = tuple(kw.get(name, old) for name, old in zip(names, state))
        waves = list(state[7])
        waves[i] = wave
        if wave[0] == "exit":                                              # a workgroup that has left makes room for the next
            W, gone = self.waves, lambda b: all(w is not None and w[0] == "exit" for w in waves[b * self.waves:(b + 1) * self.waves])
            here = sum(waves[b * W] is not None and not gone(b) for b in range(self.n))
            for b in range(self.n):
                if waves[b * W] is None and here < self.resident:
                    waves[b * W:(b + 1) * W] = [("arrive", False, False, -1)] * W
                    here += 1
        return shared + (tuple(waves),)

    def ended(self, state):
        return all(w is not None and w[0] == "exit" for w in state[7])

    def check_end(self, state):
        own, again = state[5], state[6]
        for b in range(self.n):
            mine = ((1 << self.waves) - 1) << b * self.waves
            assert own & mine == mine or again >> b & 1, "chunk %d has no w: %r" % (b, state)

    def walk(self):
        """Every reachable state; returns how many there are and how many ends had waves that left."""
        start = self.start()
        seen, before, todo, ends = {start}, {}, [start], []
        while todo:
            state = todo.pop()
            if self.ended(state):
                self.check_end(state)
                ends.append(state)
                continue
            for nxt in self.steps(state):
                before.setdefault(nxt, []).append(state)
                if nxt not in seen:
                    seen.add(nxt)
                    todo.append(nxt)
        can_end, todo = set(ends), list(ends)
        while todo:
            for s in before.get(todo.pop(), ()):
                if s not in can_end:
                    can_end.add(s)
                    todo.append(s)
        assert can_end == seen, "stuck: %r" % next(iter(seen - can_end))
        return len(seen), sum(s[3] == ABANDONED for s in ends)


@pytest.mark.parametrize("n,waves,group", [(1, 2, 0), (2, 2, 0), (3, 1, 0), (2, 2, 1), (3, 1, 1), (3, 1, 2), (4, 1, 3)])
def test_every_interleaving_ends_with_every_w_written(n, waves, group):
    for resident in range(1, n + 1):
        for stays in {(False,) * n, (True,) * n, tuple(b % 2 == 1 for b in range(n))}:
            if n * waves == 4 and resident == 3:
                continue                                                   # the largest walks: 1, 2 and all are enough
            states, left = Launch(n, waves, resident, group, stays).walk()
            assert states > 1
            assert left > 0 or n == 1                                      # the model does reach the rare road


def test_a_model_without_the_handing_over_is_found_out():
    """The walk would notice: leave out what the last arrival does for those that have left."""
    class Broken(Launch):
        def steps(self, state):
            for nxt in super().steps(state):
                yield nxt[:7] + (tuple(w if w is None or w[0] != "help" else ("exit",) + w[1:] for w in nxt[7]),)
    with pytest.raises(AssertionError):
        Broken(2, 1, 1, 0, (False, False)).walk()


# ---- two launches over the same words ------------------------------------------------------------------------------------

LIMIT, PATIENCE, BOUND = 2, 4, 60


def wave(x, tag, b, n, out):
    """The kernel's waits with their counters.  `x` is shared: arrivals, each chunk's tag, and (tag, state, ticket)."""
    x["arrived"] += 1
    last = x["arrived"] % n == 0
    yield
    x["chunk"][b] = tag
    yield
    polls, sure, most = 0, False, LIMIT * (PATIENCE if b & 1 else 1)

    def mine(state):
        return x["outcome"][:2] == (tag, state)
    help_ = False
    while any(t != tag for t in x["chunk"]):
        polls += 1
        yield
        if polls > BOUND:
            return out.append((tag, b, last))
        if not last and not sure and polls > most:
            if not mine(CLOSED):
                x["outcome"] = (tag, ABANDONED, 0)
                return out.append((tag, b, False))
            sure = True
        if mine(ABANDONED) and not sure:
            if not last and polls <= LIMIT:
                return out.append((tag, b, False))
            help_ = True
            break
    yield
    if not help_:
        if last:
            was = x["outcome"]
            x["outcome"] = (tag, CLOSED, 0)
            yield
            if was[:2] != (tag, ABANDONED):
                return out.append((tag, b, False))
            x["outcome"] = was
        elif polls <= LIMIT or not mine(ABANDONED):
            return out.append((tag, b, False))
    while any(t != tag for t in x["chunk"]):
        polls += 1
        yield
        if polls > (BOUND if last else most):
            return out.append((tag, b, last))
    while True:
        yield
        t, state, ticket = x["outcome"]
        x["outcome"] = (t, state, ticket + 1)
        if (t, state) != (tag, ABANDONED):
            return out.append((tag, b, last))
        if ticket >= n:
            return out.append((tag, b, False))
        for _ in range(2):                                                 # the chunk
            yield


@pytest.mark.parametrize("n", [1, 2, 3, 5, 8])
def test_overlapping_calls_end(n):
    lost = 0
    for seed in range(300):
        rng = random.Random(seed)
        x = {"arrived": 0, "chunk": [0] * n, "outcome": (0, OPEN, 0)}
        out = []
        alive = [wave(x, tag, b, n, out) for tag in (1, 2) for b in range(n)]
        for _ in range(2 * n * (3 * BOUND + 3 * n + 10)):
            if not alive:
                break
            # now and then one wave runs alone for a while
            i = rng.randrange(len(alive)) if seed % 2 else rng.randrange(min(2, len(alive)))
            try:
                next(alive[i])
            except StopIteration:
                alive.pop(i)
        assert not alive and len(out) == 2 * n
        lost += any(gone for _, _, gone in out)
    assert lost > 0 or n == 1                                              # some last arrival had to end its wait

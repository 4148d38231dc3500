"""A host model of the counter of a cluster of sampled acceptance's pieces, over random schedules in which waits may
give up, with the field layout read from the kernels' header.

Each piece clears its exchange slots, counts itself in, waits until every piece has (or gives up), reads the other
pieces' slots, and counts itself out; the last to leave resets the counter.  The model checks that a piece whose wait
did not give up reads only slots that their owners have cleared, and that the counter ends at zero, reset once and
after every piece has left."""
import os
import re

import numpy as np
import pytest

HEADER = os.path.join(os.path.dirname(__file__), "..", "paper_2606_00535_amd", "csrc", "kernels.h")


def layout():
    text = open(HEADER).read()
    m = re.search(r"constexpr uint32_t kClusterLeft = 1u << (\d+);", text)
    assert m, "the counter's fields were not found"
    return 1 << int(m.group(1)), int(re.search(r"constexpr int kSampledMaxPieces = (\d+);", text).group(1))


LEFT, MAX_PIECES = layout()


def run_schedule(chunks, rng, give_up):
    counter, cleared, resets = 0, [False] * chunks, 0
    state = ["new"] * chunks
    while any(s != "done" for s in state):
        k = int(rng.choice([i for i in range(chunks) if state[i] != "done"]))
        if state[k] == "new":
            cleared[k] = True
            counter += 1
            state[k] = "waiting"
        elif state[k] == "waiting":
            if counter & (LEFT - 1) == chunks:
                assert all(cleared), "a slot read before its owner cleared it"
                state[k] = "leaving"
            elif rng.random() < give_up:
                state[k] = "leaving"
        else:
            last = counter // LEFT == chunks - 1
            counter += LEFT
            state[k] = "done"
            if last:
                assert all(s == "done" for s in state), "reset while a piece was still in"
                counter, resets = 0, resets + 1
    assert counter == 0 and resets == 1


@pytest.mark.parametrize("chunks", [2, 3, 8, 64])
@pytest.mark.parametrize("give_up", [0.0, 0.3, 1.0])
def test_slots_are_read_only_once_cleared(chunks, give_up):
    assert chunks <= MAX_PIECES < LEFT
    rng = np.random.default_rng(chunks)
    for _ in range(200):
        run_schedule(chunks, rng, give_up)

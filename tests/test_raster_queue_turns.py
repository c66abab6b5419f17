"""CPU check of how the raster counts the back-facing triangles that a chunk queues (k_raster_bins, second phase).

Per chunk a wavefront adds its own count to a word in LDS, meets a barrier, and reads the word; short chunks go on to
the next one without a second barrier.  Every order in which two wavefronts can take these steps is gone through: all
must read the same counts, for a wavefront that read another one would meet a barrier alone.  One or two words are not
enough, and the model says so; the kernel has as many as the model needs."""
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHUNKS = 6


def _steps(wave, words):
    """Steps of one wavefront: ("add", word, n), ("bar",), ("read", word), ("clear", word); wavefront 0 clears."""
    out = []
    for c in range(CHUNKS):
        turn = c % words
        out += [("add", turn, 1 + wave + 2 * c), ("bar",), ("read", turn)]
        if wave == 0:
            out.append(("clear", (turn - 1) % words))
    return out


def _uniform(words):
    """True if no order of the two wavefronts' steps lets one read another count than was queued by the chunk."""
    prog = [_steps(w, words) for w in (0, 1)]
    want = [sum(1 + w + 2 * c for w in (0, 1)) for c in range(CHUNKS)]
    seen, todo = set(), [((0, 0), (0, 0), (0,) * words)]   # next step and reads of each, the words
    while todo:
        state = todo.pop()
        if state in seen:
            continue
        seen.add(state)
        at, reads, mem = state
        for w in (0, 1):
            if at[w] == len(prog[w]):
                continue
            step = prog[w][at[w]]
            nxt, rd, m = list(at), list(reads), list(mem)
            if step[0] == "bar":
                other = prog[1 - w][at[1 - w]] if at[1 - w] < len(prog[1 - w]) else None
                if other != ("bar",):
                    continue      # waits
                nxt[1 - w] += 1
            elif step[0] == "add":
                m[step[1]] += step[2]
            elif step[0] == "clear":
                m[step[1]] = 0
            else:
                if m[step[1]] != want[rd[w]]:
                    return False
                rd[w] += 1
            nxt[w] += 1
            todo.append((tuple(nxt), tuple(rd), tuple(m)))
    return True


@pytest.mark.parametrize("words,enough", [(1, False), (2, False), (3, True)])
def test_words_that_chunks_take_in_turn(words, enough):
    assert _uniform(words) == enough


def test_the_kernel_has_as_many():
    with open(os.path.join(ROOT, "paper_2409_02482_amd", "csrc", "vs_raster.h")) as f:
        src = f.read()
    words = re.search(r"__shared__ uint32_t qadd\[(\d+)\]", src)
    assert words and int(words.group(1)) == 3
    chunk = src[src.index("atomicAdd(&qadd[turn]"):]
    order = [chunk.index(s) for s in ("atomicAdd(&qadd[turn]", "__syncthreads()", "q += qadd[turn]",
                                      "qadd[turn == 0 ? 2 : turn - 1] = 0")]
    assert order == sorted(order)

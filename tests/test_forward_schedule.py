"""The bfloat16 forward tile kernel's requests into the LDS, played on the CPU.

Its wavefronts request rows, row numbers, list entries and query rows straight into the LDS, several steps ahead, and wait for them by count.
A request of one wavefront is ordered against what another one does only by its own wait and the barrier behind it.  This
file mirrors the kernel's steps (attn_fwd.hip: `step`, the loop over the tiles and what comes before it) as a list of requests, waits, barriers and
reads, and checks every word: what is read was requested for this purpose and has landed, and nothing else is on its way to it."""
import os
import random
import re
import subprocess

import pytest

from paper_2506_23858_amd import build

SOURCE = open(os.path.join(build.HERE, "csrc", "attn_fwd.hip")).read()
ROW_RINGS = int(re.search(r"\bROW_RINGS = (\d+)", SOURCE)[1])


class Op:
    def __init__(self, wave, data, epoch):
        self.wave, self.data, self.issued, self.landed, self.seen = wave, data, epoch, False, None


class Lds:
    """Requests per word; an epoch is what lies between two barriers."""
    def __init__(self, n_waves):
        self.epoch, self.flight, self.words, self.reads, self.faults = 0, [[] for _ in range(n_waves)], {}, {}, []

    def request(self, wave, *parts):
        """One load or store of a wavefront; parts: (word, data) it writes."""
        ops = []
        for word, data in parts:
            op = Op(wave, data, self.epoch)
            for o in self.words.get(word, []):
                if o.data != data and o.wave != wave and (o.seen is None or o.seen > self.epoch):
                    self.faults.append(f"{word}: {data} requested while {o.data} may be on its way")
            for data_read, until in self.reads.get(word, []):
                if data_read != data and until > self.epoch:
                    self.faults.append(f"{word}: {data} requested while {data_read} is read")
            self.words[word] = [o for o in self.words.get(word, []) if o.data == data or o.seen is None or o.seen > self.epoch] + [op]
            self.reads[word] = [r for r in self.reads.get(word, []) if r[1] > self.epoch]
            ops.append(op)
        self.flight[wave].append(ops)

    def wait(self, wave, n):
        gone = self.flight[wave][:len(self.flight[wave]) - n] if n else self.flight[wave]
        self.flight[wave] = self.flight[wave][len(gone):]
        for op in sum(gone, []):
            op.landed, op.seen = True, self.epoch + 1

    def read(self, wave, word, data, across_barrier=False):
        """across_barrier: the value may still be on its way when the wavefront passes the next barrier."""
        ops = [o for o in self.words.get(word, []) if o.data == data]
        if not any((o.wave == wave and o.landed) or (o.seen is not None and o.seen <= self.epoch) for o in ops):
            self.faults.append(f"{word}: {data} read before it has landed")
        if self.words.get(word, [None])[-1] not in ops:
            self.faults.append(f"{word}: {data} read after other data were requested")
        self.reads.setdefault(word, []).append((data, self.epoch + (2 if across_barrier else 1)))


def play(lengths, n_waves, D, in_place, rings):
    """Faults found while a workgroup walks tiles of blocks of these lengths."""
    lds, waves = Lds(n_waves), range(n_waves)
    rpi, L = 1024 // (2 * D), lambda t: lengths[min(t, len(lengths) - 1)]
    tile = lambda t: min(t, len(lengths) - 1)
    groups = lambda t: max(-(-L(t) // 32), 4)
    n_step = 3 if in_place else 2
    n_first = (1 if in_place else 0) + D * 2 * 32 // 1024 + 1 + 2 + 32 // rpi

    def number(t, x):                                   # row numbers of group x: past the block's end all are the last key's
        return ("row", tile(t), min(x, -(-L(t) // 32)))

    def row_numbers(w, t, x):
        lds.request(w, (("tok", t % rings, x & 15), number(t, x)), (("tok", t % rings, (x & 15) + 1), number(t, x + 1)))

    def first_row_numbers(w, t):
        row_numbers(w, t, 2 * (w & 3))

    def rows(w, tensor, slot, t, x):
        lds.request(w, ((tensor, slot & 3, w), (tensor, t, x)))

    def take_number(w, t, x):
        lds.read(w, ("tok", t % rings, x & 15), number(t, x), across_barrier=True)
        return (t, x)

    def barrier():
        lds.epoch += 1

    def group_at(t, x):                                 # group x of tile t, counted on into the tiles behind it
        while x >= groups(t):
            t, x = t + 1, x - groups(t)
        return t, x

    def read_rows(tensor, slot, t, x, across):
        for w in waves:
            for part in waves:
                lds.read(w, (tensor, slot & 3, part), (tensor, t, x), across)

    krow, vrow = {}, {}
    for w in waves:
        lds.request(w, (("entries", 0, w), 0))
        lds.request(w, (("entries", 1, w), 1))
        if in_place:
            first_row_numbers(w, 0)
            first_row_numbers(w, 1)
            lds.wait(w, 0)
    if in_place:
        barrier()
    for w in waves:
        for x in range(4):
            if in_place:
                lds.read(w, ("tok", 0, x), number(0, x))
            rows(w, "K", x, 0, x)
            if x < 2:
                rows(w, "V", x, 0, x)
        lds.wait(w, 6)
        lds.read(w, ("entries", 0, w), 0)
        for _ in range(32 // rpi):
            lds.request(w, (("queries", w), 0))
        lds.wait(w, 0)
    barrier()
    for w in waves:
        lds.read(w, ("queries", w), 0)
        if in_place:
            krow[w], vrow[w] = take_number(w, *group_at(0, 4)), take_number(w, 0, 2)
    read_rows("K", 0, 0, 0, False)
    n = 0                                               # step of the stream
    for t in range(len(lengths)):
        ge = groups(t)
        for g in range(ge):
            for w in waves:
                lds.wait(w, n_step + (n_first if g in (1, 2) and g < ge - 2 or g == 1 else 0))
            barrier()
            if g or t:
                read_rows("V", n - 1, *((t, g - 1) if g else (t - 1, groups(t - 1) - 1)), False)
            read_rows("K", n + 1, *group_at(t, g + 1), False)
            for w in waves:
                if g == ge - 2:
                    lds.read(w, ("queries", w), t + 1)
                if in_place:
                    assert (krow[w], vrow[w]) == (group_at(t, g + 4), group_at(t, g + 2))
                rows(w, "K", n + 4, *group_at(t, g + 4))
                rows(w, "V", n + 2, *group_at(t, g + 2))
                if in_place:
                    krow[w], vrow[w] = take_number(w, *group_at(t, g + 5)), take_number(w, *group_at(t, g + 3))
                    row_numbers(w, t, g + 8)
            read_rows("K", n + 2, *group_at(t, g + 2), True)
            read_rows("V", n, t, g, True)
            n += 1
            if g == 0:
                for w in waves:
                    if in_place:
                        first_row_numbers(w, t + 2)
                    if t:
                        for _ in range(D * 2 * 32 // 1024 + 1):         # partial rows and LSE leave
                            lds.request(w)
                    lds.request(w, (("descriptor", w), t + 3))
                    lds.request(w, (("entries", t & 1, w), t + 2))
                    lds.read(w, ("entries", (t + 1) & 1, w), t + 1)
                    for _ in range(32 // rpi):
                        lds.request(w, (("queries", w), t + 1))
                    if t == 0:
                        lds.wait(w, 0)
        for w in waves:
            lds.read(w, ("descriptor", w), t + 3)
    return lds.faults


def walks():
    """Tiles of 1 to 40 groups: runs of one length, short beside long, any order."""
    rng = random.Random(3)
    for n in list(range(1, 22)) + [28, 33, 40]:
        yield [32 * n - 7 * (n % 3)] * 4
        yield [32 * n, 20, 32 * n - 1, 100, 96, 32 * n]
    for _ in range(12):
        yield [rng.choice([rng.randint(1, 128), rng.randint(1, 1280)]) for _ in range(7)]


@pytest.mark.parametrize("D,n_waves", [(64, 4), (128, 8)])
@pytest.mark.parametrize("in_place", [False, True])
def test_requests_of_the_forward_kernel_are_ordered(D, n_waves, in_place):
    for lengths in walks():
        faults = play(lengths, n_waves, D, in_place, ROW_RINGS)
        assert not faults, (lengths, len(faults), faults[:5])


def test_the_check_sees_a_ring_that_is_taken_too_early():
    """A ring per tile in sight, none for the tile just ended: the last surplus numbers of 13 groups lie where groups 4 and 5 go, those of 8 groups
    beside the first eight."""
    assert any("on its way" in f for f in play([390] * 4, 4, 64, True, 3))
    assert not play([256] * 4, 4, 64, True, 3)


def test_a_request_that_advances_an_offset_loads_from_the_old_one(tmp_path):
    """dma16_advance adds before it loads, so the offset loaded from needs a register of its own, also where it is the one that is advanced."""
    (tmp_path / "k.hip").write_text('''#include "attn_common.h"
__global__ void k(const char* base, uint32_t* off, uint32_t advance, uint32_t lds) {
    uint32_t o = off[threadIdx.x];
    dma16_advance(base, o, o, advance, lds, 0);
    off[threadIdx.x] = o;
}''')
    subprocess.run([build.HIPCC] + [f for f in build.FLAGS if f != "-shared"] + ["--cuda-device-only", "-S", "k.hip", "-o", "k.s"], check=True, cwd=tmp_path,
                   capture_output=True)
    asm = (tmp_path / "k.s").read_text()
    advanced, = re.findall(r"\bs_add_u32 m0, .*\n\s*v_add_u32(?:_e32)? (v\d+),", asm)
    loaded, = re.findall(r"\bglobal_load_lds_dwordx4 (v\d+),", asm)
    assert advanced != loaded

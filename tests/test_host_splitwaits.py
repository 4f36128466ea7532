"""The bf16 row stream waits for its direct loads by count in both kernels that
instantiate it (host-only: reads the compiled gfx950 assembly, as for the other
rings)."""
import re

import pytest

from test_host_waitcounts import _asm, _events

# Design (stream_rows, one body per tile count NT with a ring of D stages): a
# stage is k = 8 + NT / 2 direct loads per wave (8 row groups, NT / 2 map
# fragments), D stages are issued before the loop and one per pass after the
# stage's compute, and the wait before stage s's barrier leaves the loads of up
# to D - 1 later stages outstanding, so the hand waits are multiples of k up to
# D - 1 of them.
RING = {2: 4, 4: 3, 6: 3, 8: 2}  # NT: D


def _function(lines, symbol):
    start = next(i for i, l in enumerate(lines) if l.startswith(symbol) and ":" in l)
    end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
    return [l.strip() for l in lines[start:end]]


def _vmcnt(body):
    return {int(m.group(1)) for t in body for m in [re.match(r"s_waitcnt vmcnt\((\d+)\)$", t)] if m}


def _no_drain_before_reads(body):
    # The fragment reads are inline assembly: between a stage's barrier and its
    # reads there must be no vmcnt wait, which would drain the ring each stage.
    # From each run of fragment reads (6 to 12 in one asm block) back to its
    # barrier or the block before it:
    reads = [i for i, t in enumerate(body) if t.startswith("ds_read_b128")]
    assert reads
    for i in reads:
        j = i - 1
        while j >= 0 and body[j] != "s_barrier" and not body[j].startswith("ds_read_b128"):
            assert not body[j].startswith("s_waitcnt vmcnt"), (i, body[j])
            j -= 1


def test_split_stream_waits():
    body = _function(_asm("split.hip"), "_ZN6dattri19split_stream_kernelILi2E")
    want = {k * (8 + nt // 2) for nt, d in RING.items() for k in range(1, d)}
    counts = _vmcnt(body)
    assert counts >= want and counts <= want | {0}, (counts, want)
    # every issue of a stage holds the row loads twice (with and without the
    # non-temporal hint, one of the two taken) and the map loads once
    n_d = sum(e == "D" for e in _events(body))
    assert n_d == sum((d + 1) * (2 * 8 + nt // 2) for nt, d in RING.items()), n_d
    _no_drain_before_reads(body)


@pytest.fixture(scope="module")
def few_asm():
    return _asm("score_few.hip")


@pytest.mark.parametrize("nt", [2, 4])
@pytest.mark.parametrize("norm", [0, 1])
def test_score_stream_waits(few_asm, nt, norm):
    # one body per kernel, always non-temporal; with norms the squares are taken
    # between the fragment reads and the MFMA
    body = _function(few_asm, f"_ZN6dattri19score_stream_kernelILi{nt}ELb{norm}E")
    k, d = 8 + nt // 2, RING[nt]
    ev = [e for e in _events(body) if isinstance(e, str)]
    d_pos = [i for i, e in enumerate(ev) if e == "D"]
    assert len(d_pos) == (d + 1) * k, (len(d_pos), k, d)
    assert all(e == "D" for e in ev[:d_pos[-1] + 1]), "".join(ev)  # nothing else is counted by vmcnt
    want = {i * k for i in range(1, d)}
    counts = _vmcnt(body)
    assert counts >= want and counts <= want | {0}, (counts, want)
    _no_drain_before_reads(body)

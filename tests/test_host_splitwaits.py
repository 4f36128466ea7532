"""The bf16 split form's row stream waits for its direct loads by count
(host-only: reads the compiled gfx950 assembly, as for the other rings)."""
import re

from test_host_waitcounts import _asm, _body


def test_split_stream_waits():
    # Design (stream_rows, one body per tile count NT = 2, 4, 6, 8 with rings of
    # D = 4, 3, 3, 2 stages): a stage is 8 + NT / 2 direct loads per wave, and
    # the wait before stage s's barrier leaves the loads of up to D - 1 later
    # stages outstanding, so the hand waits are multiples of 8 + NT / 2 up to
    # D - 1 of them.  The fragment reads are inline assembly: between a stage's
    # barrier and its reads there must be no vmcnt wait, which would drain the
    # ring each stage.
    lines = _asm("split.hip")
    start = next(i for i, l in enumerate(lines) if l.startswith("_ZN6dattri19split_stream_kernelILi2E") and ":" in l)
    end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
    body = [l.strip() for l in lines[start:end]]
    counts = {int(m.group(1)) for t in body for m in [re.match(r"s_waitcnt vmcnt\((\d+)\)$", t)] if m}
    want = {0}
    for nt, d in ((2, 4), (4, 3), (6, 3), (8, 2)):
        want |= {k * (8 + nt // 2) for k in range(1, d)}
    assert counts >= want - {0} and counts <= want, (counts, want)
    # from each run of fragment reads (12 to 48 in one asm block) back to its barrier or the block before it
    reads = [i for i, t in enumerate(body) if t.startswith("ds_read_b128")]
    assert reads
    for i in reads:
        j = i - 1
        while j >= 0 and body[j] != "s_barrier" and not body[j].startswith("ds_read_b128"):
            assert not body[j].startswith("s_waitcnt vmcnt"), (i, body[j])
            j -= 1

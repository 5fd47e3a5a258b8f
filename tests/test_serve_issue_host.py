"""When the batched server issues a batch: beside the batches in flight while they leave part of the
GPU idle and a backlog has formed, behind one that fills it once no request is still to arrive,
else not yet (no GPU)."""
import itertools

from paper_2510_05814_amd.serve import BEHIND, NOW, WAIT, issue


def test_issue_rule():
    for inflight, full, waiting, last, backlog in itertools.product(
            range(4), (False, True), range(1, 6), (False, True), (1, 2, 4)):
        blocks = 0 if not inflight else (4096 if full else 4095)
        got = issue(inflight, blocks, waiting, last, 4096, backlog)
        if not inflight:
            assert got == NOW
        elif not full:   # a lone request, or less than the backlog, waits -- also at the end
            assert got == (NOW if waiting >= backlog else WAIT), (waiting, last, backlog)
        else:
            assert got == (BEHIND if last and inflight == 1 else WAIT)

"""CPU model of the LDS writes of a 128-row MFMA tile (csrc/count.hip, mfma_tile with WM = 2)
against the d'Alembertian's column sums.

Between two barriers the waves of a workgroup are not ordered.  A DMA request may write its
LDS bytes at any time from its issue to the wait of its own wave that covers it; the waits do
not order it against other waves, only the next barrier does.  Requests past the last stage
count too: they write zeros.  The model issues the requests, waits and barriers of a tile in
program order and checks that no request of one wave can land on the bytes of the column sums
in the barrier phase in which another wave stores them.  Where the sums live is read from the
source.
"""
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

BM, WAVES, RING = 128, 4, 2
STAGE = BM * 64                    # bytes of a panel's stage (512 bits per row)
PER_PANEL = BM * 4 // 256          # 16-byte requests per thread and panel
LOADS = 2 * PER_PANEL


def sums_in_ring():
    """Byte offset of the column sums in the DMA ring, or None if they lie outside it."""
    text = open(os.path.join(ROOT, "paper_1805_04463_amd", "csrc", "count.hip")).read()
    where = re.findall(r"double\* const cols = ([^;]+);", text)
    assert len(where) == 1, where
    if "ring" in where[0]:
        return 0
    assert where[0] == "phis + BM + 8", where
    # a row's phi each, the eight words of the coefficients, and a sum per column
    assert "double phis[EPI == 1 ? BM + 8 + (BM == 128 ? BM : 0) : 1];" in text
    return None


def request_bytes(stage, wave, q):
    """Ring bytes [lo, hi) of request q of a stage by one wave: both panels, four waves."""
    lo = (stage % RING) * 2 * STAGE + (q // PER_PANEL) * STAGE + (q % PER_PANEL) * 4096 + wave * 1024
    return lo, lo + 1024


def landing_phases(nst, half):
    """(stage, request, first phase, last phase) of every request that a wave issues, and the
    phase in which the column sums are stored."""
    phase, open_, done = 0, [], []

    def wait(left):
        while len(open_) > left:
            st, q, first = open_.pop(0)
            done.append((st, q, first, phase))

    def issue(st):
        open_.extend((st, q, phase) for q in range(LOADS))

    for st in range(RING):
        issue(st)
    wait((RING - 1) * LOADS)
    phase += 1
    for s in range(nst):
        last = s == nst - 1
        if not last:
            wait((RING - 2) * LOADS)
        phase += 1                      # the barrier at the stage's middle
        if not (last and half):
            issue(s + RING)
    wait(0)
    return done, phase


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("nst", range(1, 9))
def test_column_sums_meet_no_request(nst, half):
    start = sums_in_ring()
    if start is None:
        return
    requests, store = landing_phases(nst, half)
    for st, q, first, last in requests:
        for wave in range(WAVES):
            lo, hi = request_bytes(st, wave, q)
            for other in (2, 3):        # the wave row that stores its sums, 64 columns each
                at = start + (other - 2) * 512
                hit = lo < at + 512 and at < hi
                assert not (hit and wave != other and first <= store <= last), (
                    f"wave {wave}'s request {q} of stage {st} (of {nst}) can land on wave "
                    f"{other}'s column sums")

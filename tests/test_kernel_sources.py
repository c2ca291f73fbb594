"""What the kernels' texts must keep that no run can show: orderings whose loss would corrupt results only now and then."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_05186_amd", "csrc")


def test_no_counted_wait_stands_behind_the_epilogue_s_requests():
    """gemm_bf16.hip, direct_tile: a wait for all but the newest n memory operations tells tile loads from other loads by their
    number, which holds only where every load is written in assembly.  The loads that the epilogue requests are the
    compiler's, to merge and to move: ahead of them nothing may be in flight, and behind them no wait may count."""
    text = open(os.path.join(CSRC, "gemm_bf16.hip")).read()
    body = text[text.index("void direct_tile("):]
    body = body[:body.index("\n}\n")]
    requests = [m.start() for m in re.finditer(r"old_value\(reinterpret_cast|reinterpret_cast<const bf16x4_t\*>\(R \+", body)]
    assert len(requests) == 2
    waits = [(m.start(), int(m.group(1))) for m in re.finditer(r"(?:OPTSTAGE_TILE_SYNC\(|vmcnt\()(\d+)\)", body)]
    ahead = [n for at, n in waits if at < min(requests)]
    behind = [n for at, n in waits if at > min(requests)]
    assert ahead[-1] == 0 and not any(behind), (ahead, behind)
    # and no tile load is written between that wait and the end
    last_wait = max(at for at, _ in waits if at < min(requests))
    assert not re.search(r"trip\([^)]*, true, (?:true|false)\)|issue_one\(", body[last_wait:])

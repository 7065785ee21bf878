"""The staircase and the counters of the fronts count as clean only once the merge that cleans them up has been seen to end:
a call whose launches were made and never ran (or whose wait failed) has them filled anew, since a list that begins at
whatever the counters hold would lie outside its array."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_clean_only_behind_the_wait():
    text = open(os.path.join(ROOT, "paper_2604_03446_amd", "csrc", "mmee.hip")).read()
    text = re.sub(r"//[^\n]*", "", text)
    assert re.findall(r"front_clean\s*=\s*(\w+)", text) == ["false", "false", "true"]     # the member, before the launches, behind the wait
    launches = text[text.index("int enqueue_front("):]
    launches = launches[:launches.index("\n}")]
    assert launches.index("S.front_clean = false") < launches.index("k_front_points") and "S.front_clean = true" not in launches
    assert re.search(r"rc = wait_signalled\(1, ksec\);\s*if \(rc\) return rc;\s*S\.front_clean = true;", text)

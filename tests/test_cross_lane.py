"""Cross-lane reads in the kernel sources.  A lane that reads another one gets its
value only if that one executes the read too, so no shuffle may stand behind a
short-circuit operator or in an arm of a conditional expression, where some lanes
skip it."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_12083_amd", "csrc")
READ = re.compile(r"__shfl\w*\s*\(|__builtin_amdgcn_(ds_bpermute|mov_dpp|update_dpp)\s*\(")


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "mrs_device*.h"))),
                         ids=os.path.basename)
def test_every_lane_executes_its_shuffles(path):
    text = re.sub(r"/\*.*?\*/|//[^\n]*", "", open(path).read(), flags=re.S)
    for statement in re.split(r"[;{}]", text):
        for m in READ.finditer(statement):
            assert not re.search(r"&&|\|\||\?", statement[:m.start()]), " ".join(statement.split())

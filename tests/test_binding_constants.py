"""Facts that the binding and the library both hold (host only)."""
from __future__ import annotations

import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_sets_up_to_which_no_basis_is_kept():
    import paper_2409_19156_amd as zp

    with open(os.path.join(ROOT, "paper_2409_19156_amd", "csrc", "series.hpp")) as f:
        assert re.findall(r"kFusedDotSets = (\d+);", f.read()) == [str(zp._FUSED_SETS)]

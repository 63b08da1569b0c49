"""The cut of the backward's key pass into row chunks and query-head parts: a
host build of the library's own rule (bwd_chunks), checked over 31 sequence
lengths x 4 batch sizes x 28 head layouts x 3 head dims, plain and under
AddressSanitizer and UndefinedBehaviorSanitizer (host code only)."""
import os

import pytest

from test_host_logic import HIPCC, SAN_ENV, SAN_HIPCC, _build_run


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("sanitize", [False, True])
def test_bwd_plan(tmp_path, sanitize):
    out = _build_run(tmp_path, "bwd_plan_check.cpp", "bwd_plan_check",
                     SAN_HIPCC if sanitize else ["-O2"], env=SAN_ENV if sanitize else None)
    assert out.startswith("bwd plan ok")
    assert int(out.split()[-1]) == 31 * 4 * 28 * 3

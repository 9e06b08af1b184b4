"""Loads through a buffer descriptor: what lies beyond a head's valid rows is kept out by the descriptor's range check, which is promised
for the lane's own offset and not for a scalar offset beside it.  So every such load has its whole offset in the lane."""
import os
import re

import numpy as np
import pytest

from paper_2106_09236_amd import build
from tests.test_parity_gpu import check_against_oracle
from tests.test_parts_of_k import _workload
from tests.test_plan import plan

SCALAR_OFFSET = {"load": 2, "store": 3, "load_lds": 4}     # which argument it is


def _calls(text):
    for m in re.finditer(r"__builtin_amdgcn_raw_(?:ptr_)?buffer_(load_lds|load|store)\w*\(", text):
        args, depth, start = [], 0, m.end()
        for at in range(m.end(), len(text)):
            c = text[at]
            if c in ",)" and depth == 0:
                args.append(text[start:at].strip())
                start = at + 1
            depth += (c in "([{") - (c in ")]}")
            if depth < 0:
                break
        yield m.group(1), args


def test_no_scalar_offsets():
    seen = 0
    for name in sorted(os.listdir(build.CSRC)):
        if name.endswith((".h", ".hip")):
            with open(os.path.join(build.CSRC, name)) as f:
                for kind, args in _calls(f.read()):
                    assert args[SCALAR_OFFSET[kind]] == "0", (name, kind, args)
                    seen += 1
    assert seen >= 10


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,L", [("f32", 600), ("f32", 1500), ("bf16", 1100), ("bf16", 2500)])
def test_nothing_is_read_behind_short_items(dtype, L):
    # the gather out of L2: its query rows, indices and V rows come in pieces of 1 KB, all of them beyond the shortest items
    w = _workload(dtype, 11, 2, L, 20, True)
    p = plan(11, 2, L, 20, dtype)
    assert (p["measure"], p["measure_parts"]) == ("stream", "0")
    w.lengths[9], w.lengths[10] = 2, 17
    w.sample_idx[9] %= 2
    w.sample_idx[10] %= 17
    for b in range(11):
        for x in (w.Q, w.K, w.V):
            x[b, :, int(w.lengths[b]):] = np.nan if x.dtype != np.uint16 else 0x7FC0
    check_against_oracle(w, label=f"short items {dtype} L{L}")

"""The committed counters of the predictor are taken as current only while its sources are unchanged: every
file its kernels are compiled from counts, the ones with the launches included."""
import os
import re

import bench

CSRC = os.path.join(bench.HERE, "paper_1803_09563_amd", "csrc")


def test_profile_tag_covers_every_predictor_source():
    want = {f for f in os.listdir(CSRC) if f.startswith("k_predictor")}
    for f in list(want):
        with open(os.path.join(CSRC, f)) as fh:
            want |= set(re.findall(r'#include "(\w+\.h)"', fh.read()))
    assert {"k_predictor_fp64.hip", "k_predictor_mixed.hip", "predictor_async.h"} <= want
    assert want <= {os.path.basename(f) for f in bench.PRED_SOURCES}
    assert all(os.path.isfile(f) for f in bench.PRED_SOURCES)

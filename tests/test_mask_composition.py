"""What dK/dV leaves out of a mask must not be asked for by it: for a canvas it works out which pixels match and nothing else, so that
a composition of a canvas with another predicate has to be refused by the compiler.  (Front end only, no code is made.)"""
import os
import shutil
import subprocess

import pytest

from paper_2412_05496_amd import build

SOURCE = """
#include "flex_common.h"
using namespace flexattn;
__global__ void kernel(const flexattn_mod_params p, const uint32_t* tags, uint32_t* out) {
    const PartialMask<TESTED_MASK> mask(p, 0, 64);
    out[0] = mask.match_queries(tags, mask.key_corners(0), 0).plain;
}
"""


@pytest.mark.skipif(shutil.which(build.HIPCC) is None, reason="no hipcc")
@pytest.mark.parametrize("mask,accepted", [
    ("FLEXATTN_M_NEIGHBORHOOD", True), ("FLEXATTN_M_NEIGHBORHOOD | FLEXATTN_M_CAUSAL", False),
    ("FLEXATTN_M_NEIGHBORHOOD | (FLEXATTN_M_PREFIX << 8)", False)])
def test_canvas_with_another_predicate(mask, accepted, tmp_path):
    src = os.path.join(tmp_path, "mask.hip")
    with open(src, "w") as f:
        f.write(SOURCE)
    r = subprocess.run([build.HIPCC, *build.FLAGS, f"-DTESTED_MASK=({mask})", "--cuda-device-only", "-fsyntax-only", src], capture_output=True, text=True, timeout=300)
    assert (r.returncode == 0) == accepted, r.stderr
    assert accepted or "a canvas with another predicate" in r.stderr


@pytest.mark.parametrize("mask", [0x60, 0x6020, 0x40, 0x61])
def test_the_internal_canvas_flag_is_not_accepted(mask):
    """Bit 6 selects, inside the library, the kernels that compare pixels token by token: no mask of a caller has it."""
    import paper_2412_05496_amd as fa
    assert not fa.flexattn_is_supported(mask, 0, 64) and fa.flexattn_is_supported(fa.MASK_NEIGHBORHOOD, 0, 64)


BOUNDED_SOURCE = """
#include "fwd_kernel.h"
using namespace flexattn;
template __global__ void flexattn::fwd_kernel<64, 4, (FLEXATTN_MASK_NEIGHBORHOOD | kCanvasCells), TESTED_SCORE, TESTED_BOUNDED, false>(const FwdArgs);
"""


@pytest.mark.skipif(shutil.which(build.HIPCC) is None, reason="no hipcc")
@pytest.mark.parametrize("score,bounded", [("FLEXATTN_SCORE_IDENTITY", "false"), ("FLEXATTN_SCORE_SOFTCAP", "true")])
def test_cells_with_a_bounded_score(score, bounded, tmp_path):
    """The weights of a bounded score_mod are made where no maximum is tracked, which is where the masks of cells are worked out: refused, not weighed by
    masks that nobody has set."""
    src = os.path.join(tmp_path, "bounded.hip")
    with open(src, "w") as f:
        f.write(BOUNDED_SOURCE)
    r = subprocess.run([build.HIPCC, *build.FLAGS, f"-DTESTED_SCORE={score}", f"-DTESTED_BOUNDED={bounded}", "--cuda-device-only", "-fsyntax-only", src], capture_output=True, text=True,
                       timeout=300)
    assert (r.returncode == 0) == (bounded == "false"), r.stderr
    assert bounded == "false" or "cells: the running maximum's branch" in r.stderr

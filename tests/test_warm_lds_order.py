"""Order of the warm-start kernels' LDS writes before their first sample: the whole patch buffer is
cleared by all 256 threads, then threads 0 to 191 stage the patch's rows into it.  A word cleared by
one wavefront and staged by another needs a block barrier between the two, or a wavefront that is
late in its clearing wipes values already staged."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2603_00145_amd", "csrc")
WAVE, THREADS = 64, 256


def _inference_rows():
    """word -> staging thread, as patch_row and stage_patch_row lay the two copies out."""
    row, z, c = 6, 60, 600
    copy = 3 * c + 4
    out = {}
    for t in range(192):
        r = (t >> 6) * c + ((t >> 3 & 7) + 1) * z + ((t & 7) + 1) * row
        out.update({r + i: t for i in range(5)})
        out.update({r + copy + i: t for i in range(4)})
    return out, 2 * copy


def _training_rows():
    """element -> staging thread, as stage_patch lays a row out (five words of two)."""
    out = {}
    for t in range(192):
        r = ((t >> 6) * 100 + ((t >> 3 & 7) + 1) * 10 + (t & 7) + 1) * 12
        out.update({r + i: t for i in range(10)})
    return out, 3600


# kernel -> source, {LDS unit: staging thread} and the units, cleared one a thread in turn
KERNELS = {"k_ws_conv12": ("warm_fwd.hip", _inference_rows),
           "k_ws_train12": ("warm_train.hip", _training_rows),
           "k_ws_back12": ("warm_train.hip", _training_rows)}


def _before_first_sample(src, kernel):
    """The kernel's text from its clearing of s.in to its first staging."""
    with open(os.path.join(CSRC, src)) as f:
        text = f.read()
    body = re.sub(r"//[^\n]*", "", text[text.index(f" {kernel}("):])
    clear = body.index("s.in[i] = 0")
    return body[clear:body.index("stage_patch", clear)]


@pytest.mark.parametrize("kernel", KERNELS)
def test_clearing_and_staging_are_ordered(kernel):
    src, layout = KERNELS[kernel]
    staged, units = layout()
    assert max(staged) < units
    shared = sum(u % THREADS // WAVE != t // WAVE for u, t in staged.items())
    assert shared > 0      # wavefronts do write each other's words
    assert "__syncthreads();" in _before_first_sample(src, kernel)

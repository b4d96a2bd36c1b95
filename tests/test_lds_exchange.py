"""LDS exchanges between the lanes of one wavefront, by the source: in the row-marching kernel every
read of a slot that another lane wrote comes after a wave_fence() that follows the write. Lanes have
no barrier there, so without the fence nothing but the compiler's caution orders the two."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1912_07645_amd", "csrc")


def _kernel():
    text = open(os.path.join(CSRC, "fv_stage_y.h")).read()
    text = re.sub(r"//[^\n]*", "", text)
    start = text.index("stage_kernel_y(const StageArgs args)")
    return text[start:text.index("void launch_stage_y", start)]


def _fence_between(body, write, read):
    """Every (write, next read) pair has a fence in it; the loop is followed once around."""
    events = sorted([(m.start(), "w") for m in re.finditer(write, body)] +
                    [(m.start(), "r") for m in re.finditer(read, body)] +
                    [(m.start(), "f") for m in re.finditer(r"wave_fence\(\)", body)])
    dirty, ok = False, True
    for _, e in events:
        if e == "w":
            dirty = True
        elif e == "f":
            dirty = False
        else:
            ok = ok and not dirty
    return ok


def test_row_march_fences_what_lanes_exchange():
    k = _kernel()
    loop = k.index("for (int32_t k = y0; k < y1; ++k)")
    # the row ends, written by one lane per row before the march, read by the first lanes in it
    end_write = r"s\[q \* QS \+ T::END[^\]]*\] ="
    end_read = r"= s\[q \* QS \+ T::END"
    assert len(re.findall(end_write, k[:loop])) == 3 and re.search(end_read, k[loop:])
    assert _fence_between(k, end_write, end_read)
    # the row, read through StripCells by its neighbours, and the x fluxes
    assert _fence_between(k[loop:], r"s\[q \* QS \+ (?:G \+ lane|to)\] =", r"StripCells<")
    assert _fence_between(k[loop:], r"s\[q \* QS \+ T::FX \+ lane\] =", r"s\[q \* QS \+ T::FX \+ pos")

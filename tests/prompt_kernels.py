"""Which kernel a dense call of more than 32 rows takes, asked of the launch rule."""
import ctypes

from paper_2507_07145_amd import binding as b


def prompt_kernel(w, M):
    """"block", "256-row" or "64-row", for a descriptor."""
    assert M > 32
    if b.load().ccq_prompt_plan(ctypes.byref(w), M, (ctypes.c_int32 * 8)()) > 0:
        return "block"
    return "256-row" if b.load().ccq_prompt_block_cols(ctypes.byref(w), M) > 0 else "64-row"

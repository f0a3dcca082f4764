"""Properties of the kernels' source that no output shows (CPU only): what a
race or a lost round trip looks like in the code, not in a result."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2504_11651_amd", "csrc")


def source(name):
    """The file without comments."""
    with open(os.path.join(CSRC, name)) as f:
        return re.sub(r"//[^\n]*", "", f.read())


def body(text, head):
    """The function whose definition starts with `head`, braces included."""
    at = text.index(head)
    at = text.index("{", text.index(")", at))
    depth = 0
    for i in range(at, len(text)):
        depth += {"{": 1, "}": -1}.get(text[i], 0)
        if depth == 0:
            return text[at:i + 1]
    raise AssertionError(f"{head}: no end")


def test_tables_come_from_lds_after_the_barrier():
    """A wave's copy of the long-code tables is read from LDS, not once more
    from memory, and only after the barrier that follows their staging."""
    core = source("df11_decode_core.h")
    assert "a.tables" not in body(core, "Tables staged_tables(")
    assert "a.tables" in body(core, "void stage_table_blob(")
    seen = 0
    for name in ("df11_decode.hip", "df11_gemv.hip"):
        calls = re.findall(r"\b(stage_table_blob|__syncthreads|staged_tables)\(", source(name))
        staged = barrier = False
        for call in calls:
            if call == "stage_table_blob":
                staged, barrier = True, False
            elif call == "__syncthreads":
                barrier = staged
            else:
                assert barrier, f"{name}: tables read before the barrier"
                staged = barrier = False
                seen += 1
    assert seen == 6  # four decode kernels, the fused kernel's two paths


def test_lanes_hand_lds_over_in_the_products():
    """Weights (and up to 16 tokens activations) are written to LDS by some lanes
    of a wave and read by others: the writes come before the reads, and the reads
    before the next writes, by more than the compiler's view of one lane."""
    text = source("df11_gemm.hip")
    for kernel in ("gemm_rows_kernel(", "gemm_slab_kernel("):
        code = body(text, kernel)
        code = re.sub(r"auto \w+ = \[&\].*?\n    \};", "", code, flags=re.S)  # the lambdas
        calls = re.findall(r"\b(put_x|put_w|products|wave_lds_sync|__syncthreads|for \(;;\)|"
                           r"for \(; k1)", code)
        # the loop's body twice, so that its back edge is seen too
        at = next(i for i, c in enumerate(calls) if c.startswith("for"))
        end = calls.index("products", at) + 1
        while end < len(calls) and calls[end] == "__syncthreads":
            end += 1
        order = calls[:at] + 2 * calls[at + 1:end] + calls[end:]
        assert order.count("products") == 3 and order.count("put_w") == 3, (kernel, order)
        last = None
        for call in order:
            if call in ("wave_lds_sync", "__syncthreads"):
                last = None
                continue
            now = "read" if call == "products" else "write"
            assert last in (None, now), f"{kernel} {last} then {call} without a hand-over: {order}"
            last = now

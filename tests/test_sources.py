"""What the compiler does not check about the kernels' inline assembly."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_19124_amd", "csrc")


def _sources():
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(path) as f:
            yield os.path.basename(path), re.sub(r"//[^\n]*", "", f.read())


def test_assembly_that_reads_matrix_results_stands_behind_a_wait():
    """The compiler keeps the distance between a matrix instruction and the reader of its result for its own
    instructions only.  So assembly stays in one file, and there every accumulator passes through the statement that
    waits before the first one of the epilogue is read by assembly."""
    for name, text in _sources():
        emitted = {m.split()[0] for t in re.findall(r'asm(?: volatile)?\(\s*"([^"]*)"', text) for m in t.split("\\n\\t")
                   if m.strip()}
        assert emitted <= ({"v_max_f64", "v_min_f64", "v_max_f32", "s_nop"} if name == "kernels_head_gemm.hip" else set())
        if emitted:
            reads = [m.start() for m in re.finditer(r"logit_key\(acc", text)]
            waits = [m.start() for m in re.finditer(r"matrix_results_settled<MB>\(acc\)", text)]
            products = [m.start() for m in re.finditer(r"__builtin_amdgcn_mfma_f32_32x32", text)]
            assert len(reads) == 1 and len(waits) == 1 and max(products) < waits[0] < reads[0]
            # two s_nop of 16 and 8 states: 16 passes of the instruction and 4 more are needed
            assert text.count('"s_nop 15\\n\\ts_nop 7"') == 4


def test_loads_that_rely_on_a_buffers_end_are_checked_whole():
    """A buffer's range check leaves the scalar offset out: a load that may lie past the end carries all of its position in the
    offset of the lanes.  (Copies into LDS go by scalar offsets, and none of them relies on the check.)"""
    calls = [(name, m) for name, text in _sources() for m in re.findall(r"raw_buffer_load_b128\(([^;]*)\);", text)]
    assert calls
    for name, args in calls:
        assert re.fullmatch(r"\w+, \w+, 0, 2", args), (name, args)


def test_what_lies_in_restricted_buffers_is_reached_through_them_only():
    """Copies into LDS go through restricted pointers, so that a read waits for those into its own buffer alone.  While they are in
    scope nothing may reach that memory by another name; the merges that use it again stand behind."""
    found = 0
    for name, text in _sources():
        for head, body in re.findall(r"\n(__device__[^\n{]*\((?:[^{}]*?)__restrict[^{}]*\) \{)(.*?)\n\}\n", text, re.S):
            if "lds_byte* __restrict" in head:
                found += 1
                assert "smem" not in head + body, name
    assert found == 2

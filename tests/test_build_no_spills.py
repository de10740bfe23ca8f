"""Build-time checks of the draft kernels' machine code (hipcc only, no GPU).

No instantiation may spill vector registers: the in-flight tile windows live in registers, and
a spilled window turns the weight stream into scratch-memory traffic (measured once: 36.8 us
instead of 29.6 us per call on the phi shape with 12 spilled registers).

The streaming kernel copies scale / zero entries into LDS with loads issued from inline assembly
that set the M0 register themselves; the compiler is not told, so nothing else in those kernels
may depend on M0."""
import functools
import os
import re
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@functools.lru_cache(maxsize=None)
def _assembly(name):
    from paper_2511_14102_amd import build as B
    src = os.path.join(B.CSRC, name)
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, name + ".s")
        cmd = [B.HIPCC] + B.FLAGS + ["--cuda-device-only", "-S", src, "-o", out]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return open(out).read()


def _kernel_blocks(text, kernel):
    """Metadata blocks (one per kernel, after '.name:') of the instantiations of `kernel`."""
    return [blk for blk in text.split(".name:")[1:] if kernel in blk.split("\n", 1)[0]]


def test_draft_kernel_instantiations_do_not_spill():
    for src, kernel, count in (("draft_int4.hip", "draft_stream_kernel", 36),     # 2 windows x 3 token capacities x 3 group sizes x 2 formats
                               ("draft_int4.hip", "draft_stream_sums_kernel", 18),    # 3 token capacities x 3 group sizes x 2 formats
                               ("draft_slice.hip", "draft_fused_kernel", 12),     # with and without shared experts x 3 group sizes x 2 formats
                               ("draft_slice.hip", "draft_pair_kernel", 12),      # the same, two items per workgroup
                               ("draft_prefill.hip", "prefill_tile_kernel", 12)): # (gate/up, down) x 3 group sizes x 2 formats
        blocks = _kernel_blocks(_assembly(src), kernel)
        assert len(blocks) == count, (src, len(blocks))
        for blk in blocks:
            m = re.search(r"\.vgpr_spill_count:\s+(\d+)", blk)
            assert m is not None
            assert int(m.group(1)) == 0, blk.split("\n", 1)[0].strip()


def test_streaming_kernel_uses_m0_only_for_its_loads_to_lds():
    body = _assembly("draft_int4.hip")
    uses = [l.strip() for l in body.splitlines() if re.search(r"\bm0\b", l) and not l.strip().startswith(";")]
    assert uses, "the loads to LDS are gone?"
    for l in uses:
        assert l.startswith("s_mov_b32 m0,"), l
    assert "global_load_lds_dwordx4" in body


@pytest.mark.parametrize("src", ["draft_int4.hip", "draft_prefill.hip"])
def test_loads_to_lds_do_not_follow_the_write_of_m0_directly(src):
    """A load to LDS needs a wait state between the scalar write of M0 and itself."""
    code = [l.strip() for l in _assembly(src).splitlines()]
    code = [l for l in code if re.match(r"[a-z]\w*( |$)", l)]            # instructions: no comments, labels, directives
    loads = [(a, b) for a, b in zip(code, code[1:]) if re.match(r"(global_load_lds_|buffer_load_\w+ .*\blds\b)", b)]
    assert loads, "the loads to LDS are gone?"
    for before, load in loads:
        assert not re.search(r"\bm0\b", before), (before, load)


def test_kernel_of_pairs_with_long_rows_does_not_spill():
    blocks = _kernel_blocks(_assembly("draft_slice.hip"), "draft_pair_planes_kernel")
    assert len(blocks) == 12                           # with and without shared experts x 3 group sizes x 2 formats
    for blk in blocks:
        assert int(re.search(r"\.vgpr_spill_count:\s+(\d+)", blk).group(1)) == 0, blk.split("\n", 1)[0].strip()

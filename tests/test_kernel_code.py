"""What the compiler made of a loop whose speed hangs on it, read from the assembly of our own sources (hipcc compiles for
gfx950 without a GPU)."""
import os
import re
import subprocess

import pytest

from paper_2605_05802_amd.build import CSRC, FLAGS, HIPCC


@pytest.fixture(scope="module")
def attention_asm(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "attention.s"
    r = subprocess.run([HIPCC] + FLAGS + ["--cuda-device-only", "-S", os.path.join(CSRC, "attention.hip"), "-o", str(out)],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr
    return out.read_text()


@pytest.mark.parametrize("kernel", ["attn_kernelILi64ELi1E", "attn_kernelILi64ELi2E", "attn_kernelILi128ELi1E",
                                    "attn_kernelILi128ELi2E"])
def test_block_loop_keeps_its_fragments_in_flight(attention_asm, kernel):
    """The blocks of the attention kernel that hold matrix instructions load the next block's K and V fragments; a wait for
    every outstanding vector load among them serialises the block chain."""
    body = re.search(r"^_ZN\S*" + kernel + r"\S*:[^\n]*\n(.*?)^\.Lfunc_end", attention_asm, re.S | re.M).group(1)
    loops = [b for b in re.split(r"^\.LBB\S*:.*$", body, flags=re.M) if "v_mfma" in b]
    assert loops
    for block in loops:
        assert "global_load" in block and "vmcnt(0)" not in block


@pytest.mark.parametrize("kernel", ["attn_prefill_shared_kernelILi64ELi1E", "attn_prefill_shared_kernelILi64ELi2E",
                                    "attn_prefill_shared_kernelILi128ELi1E", "attn_prefill_shared_kernelILi128ELi2E",
                                    "attn_decode_kernelILi64E", "attn_decode_kernelILi128E"])
def test_shared_blocks_are_read_before_they_are_overwritten(attention_asm, kernel):
    """Behind the barrier of the block loop the copies overwrite the buffer of the block before: the wait in front of it covers
    the wavefront's LDS reads as well as its copies."""
    body = re.search(r"^_ZN\S*" + kernel + r"\S*:[^\n]*\n(.*?)^\.Lfunc_end", attention_asm, re.S | re.M).group(1)
    heads = body.split("s_barrier")[:-1]
    assert heads
    for head in heads:
        last = re.findall(r"s_waitcnt[^\n]*", head)[-1]
        assert "lgkmcnt(0)" in last and "vmcnt" in last

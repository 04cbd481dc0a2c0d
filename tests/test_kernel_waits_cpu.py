"""Waits in the assembly of kernels that count their direct-to-LDS copies by hand, from a device-only compilation without a GPU."""
import os
import re
import subprocess

import pytest

from paper_2602_06036_amd import build

SOURCE = r"""
#include "attn_mfma.h"
template __global__ void attn_prefill_kernel<128>(const bf16_t* __restrict__, const bf16_t* __restrict__, SeqGeom, AttnArgs, const int4* __restrict__, int);
"""


def _loop_blocks(asm, kernel):
    """The basic blocks of the kernel's first loop, as lists of lines."""
    body = re.search(r"^_Z\d+%s\w*:.*?^\.Lfunc_end" % kernel, asm, re.S | re.M).group(0)
    blocks = re.split(r"^(?=\.LBB\d+_\d+:|; %bb\.\d+:)", body, flags=re.M)
    head = next(i for i, b in enumerate(blocks) if "Loop Header: Depth=1" in b and "s_barrier" in b)
    label = re.match(r"\.L(BB\d+_\d+):", blocks[head]).group(1)
    return [b.splitlines() for i, b in enumerate(blocks) if i == head or "Header=%s " % label in b]


@pytest.mark.skipif(not os.path.exists(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")), reason="needs hipcc")
def test_prefill_attention_waits_for_its_ring_and_not_for_every_copy(tmp_path):
    """A stage waits until its own copies have landed, eight younger ones in flight.  The compiler does not see the copies, so whatever global load it waits
    for by itself drains them all: only the block that loads page ids, once in sixteen stages, may hold such a wait."""
    (tmp_path / "k.hip").write_text(SOURCE)
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    csrc = os.path.dirname(build.SRC)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--offload-device-only", "-S", "-I", csrc, str(tmp_path / "k.hip"), "-o", str(tmp_path / "k.s")],
                   check=True, capture_output=True)
    blocks = _loop_blocks((tmp_path / "k.s").read_text(), "attn_prefill_kernel")
    waits = [(int(m.group(1)), any("global_load_dword " in x for x in b)) for b in blocks for l in b for m in [re.search(r"s_waitcnt.*vmcnt\((\d+)\)", l)] if m]
    assert sum("global_load_lds_dwordx4" in l for b in blocks for l in b) == 4
    assert (8, False) in waits
    assert [w for w in waits if not w[1]] == [(8, False)], waits

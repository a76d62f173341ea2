"""The attention kernels that pass probabilities from a wave's lanes to its other
lanes through LDS state that order: between the stores and the loads the
compiled kernel holds a wave barrier, over which the compiler moves no LDS
access.  (The order that a build happens to emit without it is no promise.)"""
import os
import re
import subprocess

import pytest

from paper_2607_20357_amd import build

# source, kernel, hand-offs in one pass over a key or query tile
KERNELS = [("fp32_path.hip", "attn_f32_kernel", 1), ("train.hip", "train_attn_fwd_kernel", 1),
           ("train.hip", "train_attn_dq_kernel", 1), ("train.hip", "train_attn_dkv_kernel", 3)]


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    """The gfx950 listing of each source, built as the library builds it."""
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = {}
    for src in sorted({k[0] for k in KERNELS}):
        asm = str(tmp_path_factory.mktemp("asm") / (src + ".s"))
        flags = [f for f in build.COMMON if f != "-fPIC"]
        subprocess.run([build.HIPCC] + flags + ["--cuda-device-only", "-S", "-x", "hip",
                                                os.path.join(build.CSRC, src), "-o", asm],
                       check=True, capture_output=True)
        with open(asm) as f:
            out[src] = f.read()
    return out


@pytest.mark.parametrize("src,kernel,handoffs", KERNELS)
def test_wave_handoff_is_ordered(listings, src, kernel, handoffs):
    bodies = re.findall(rf"^(_Z\w*{kernel}\w*):.*?^\.Lfunc_end", listings[src], re.S | re.M)
    assert len(bodies) == 3                      # head dimensions 32, 64 and 128
    for name in bodies:
        body = re.search(rf"^{name}:.*?^\.Lfunc_end", listings[src], re.S | re.M).group(0)
        assert body.count("; wave barrier") == handoffs, name

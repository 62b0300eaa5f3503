"""The instruction rule of section 3.2 (no fused multiply-add, no packed
float32 arithmetic where values are encoded or decoded) for every kernel that
does so, each counted by name, so that a new or renamed one cannot fall out
of the check."""
import collections
import os
import re

import pytest

from test_abi import ROOT, kernel_bodies

FUSED = re.compile(r"^\s*(v_(?:fma|fmac|mad|mac)\w*_f(?:16|32|64)\w*|v_mad_legacy\w*|"
                   r"v_fma_legacy\w*|v_pk_fma_f32|v_pk_mul_f32|v_pk_add_f32)\b", flags=re.M)


@pytest.fixture(scope="module")
def bodies(tmp_path_factory):
    from paper_2407_15037_amd import build
    out = {}
    for name in ("lcq.hip", "lcq_compress.hip"):
        path = str(tmp_path_factory.mktemp("asm") / (name + ".s"))
        build.asm(path, src=os.path.join(ROOT, "paper_2407_15037_amd", "csrc", name))
        out[name] = kernel_bodies(open(path).read())
    return out


def test_small_field_kernels(bodies):
    """One kernel per dtype, quantizer and chunks per wavefront."""
    found = {}
    for name, body in bodies["lcq.hip"].items():
        m = re.search(r"k_quant_smallI([fd])Li([012])ELi([12])E", name)
        if m:
            found[m.groups()] = body
    assert len(found) == 2 * 3 * 2, sorted(found)
    for key, body in found.items():
        assert not FUSED.findall(body), key


def test_compress_kernels(bodies):
    kernels = {k: v for k, v in bodies["lcq_compress.hip"].items()
               if re.search(r"\d+k_(?:cmp|decompress)", k)}
    count = collections.Counter(re.search(r"\d+(k_\w+?)I[fd]", k).group(1) for k in kernels)
    assert count == {"k_cmp_stage": 6, "k_cmp_write": 12, "k_cmp_scan": 6, "k_decompress": 2}, count
    for name, body in kernels.items():
        assert not FUSED.findall(body), name

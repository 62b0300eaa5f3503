"""Which kernels a call launches, and how, without a GPU: the launches are
recorded by a stand-in for the HIP runtime's launch calls (launch_shim.c).
The section 6 ablations are timed against the guaranteed operations, so each
must be launched as its counterpart is: the same kernels, grids, workgroups
and LDS, at every size."""
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

CHILD = r"""
import ctypes, json, re, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
shim.shim_name.restype = ctypes.c_char_p
shim.shim_lds.restype = ctypes.c_uint64
sys.path.insert(0, sys.argv[2])
import paper_2407_15037_amd as lcq
L = lcq.lib()
fake, big = ctypes.c_void_p(1 << 20), 1 << 60

def launches(call):
    shim.shim_reset()
    assert call() == lcq.OK
    out = []
    for i in range(shim.shim_launches()):
        name = shim.shim_name(i).decode()
        kernel = re.search(r"\d+(k_\w+?)(?:I([fd])|E|P)", name)
        out.append([kernel.group(1), name, shim.shim_grid(i), shim.shim_block(i),
                    shim.shim_lds(i)])
    return out

res = []
for t in (0, 1):
    for base, kind in ((lcq.ABS, lcq.ABL_ABS_UNCHECKED), (lcq.REL, lcq.ABL_REL_LIBM)):
        for n in json.loads(sys.argv[3]):
            q = [launches(lambda: L.lcq_quantize(base, t, 1e-3, fake, n, fake, big, fake, fake, big,
                                                 None)),
                 launches(lambda: L.lcq_quantize_ablation(kind, t, 1e-3, fake, n, fake, big, fake,
                                                          fake, big, None))]
            d = [launches(lambda: L.lcq_dequantize(t, fake, big, fake, n, fake, big, None)),
                 launches(lambda: L.lcq_dequantize_ablation(kind, t, fake, big, fake, n, fake, big,
                                                            None))]
            res.append([t, base, n, q, d])
print(json.dumps(res))
"""

SIZES = [0, 1, 1024, 16 * 1024, 16 * 1024 + 1, 18 * 1024 + 1, 24 * 1024 + 1, 32 * 1024,
         32 * 1024 + 1, 1 << 20, 4096 * 4 * 1024 + 1, 4096 * 8 * 1024 + 1]


@pytest.fixture(scope="module")
def recorded(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("shim") / "launch_shim.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-Wall", "-o", so,
                    os.path.join(HERE, "launch_shim.c"), "-ldl"], check=True)
    r = subprocess.run([sys.executable, "-c", CHILD, so, ROOT, json.dumps(SIZES)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout)


def test_ablations_are_launched_as_their_counterparts(recorded):
    for t, base, n, quant, deq in recorded:
        shape = [[(k, g, b, lds) for k, _, g, b, lds in side] for side in quant]
        assert shape[0] and shape[0] == shape[1], (t, base, n, shape)
        shape = [[(g, b, lds) for _, _, g, b, lds in side] for side in deq]
        assert shape[0] and shape[0] == shape[1], (t, base, n, shape)
        assert deq[0][0][0] == "k_dequantize_chunks" and deq[1][0][0] == "k_dequantize_ablation"

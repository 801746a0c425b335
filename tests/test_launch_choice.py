"""Which variant of a kernel a call launches, where results do not show it: libmimose on the stand-in for the HIP
runtime of test_launch_errors, which launches nothing and here keeps the names."""
import subprocess
import sys
import textwrap

import pytest

from test_launch_errors import ROOT, runtime  # noqa: F401

PRELUDE = """
    import ctypes, sys
    runtime = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
    runtime.shim_kernel.restype = ctypes.c_char_p
    import paper_2209_02478_amd as mi
    import numpy as np
    def launched(call):
        first = runtime.shim_launches()
        call()
        return [runtime.shim_kernel(i).decode() for i in range(first, runtime.shim_launches())]
"""


def run(runtime, code, *args):  # noqa: F811
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(PRELUDE) + textwrap.dedent(code), runtime, *map(str, args)], cwd=ROOT,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("T,ahead", [(16, (1, 16)), (4096, (1, 16)), (4097, (4, 4)), (8192, (4, 4)), (8193, (2, 4)),
                                     (57344, (2, 4)), (57345, (2, 4)), (131072, (2, 4))])
def test_layernorm_bwd_alone(runtime, T, ahead):  # noqa: F811
    """Rows ahead and waves of a block of a call that nothing runs beside."""
    run(runtime, """
    T, ahead, waves = map(int, sys.argv[2:])
    for dtype, wide, H, nc in ((1, 0, 1024, 2), (1, 1, 1024, 2), (1, 0, 512, 1), (0, 0, 512, 2), (0, 0, 768, 3), (0, 0, 1024, 4)):
        at = 1 << 20                                    # (an aligned address that nothing reads)
        names = launched(lambda: mi.mimose_op_layernorm_bwd(dtype, at, wide, at, wide, at, 2 * at, None, at, at, at, T, H, 1e-5))
        assert "ln_bwd_vec_kernel" in names[0] and "Li%dELi%dELi%dEE" % (nc, ahead, waves) in names[0], (dtype, wide, H, names)
    """, T, *ahead)


@pytest.mark.parametrize("rows,ahead", [(57344, 2), (57408, 4)])
def test_layernorm_bwd_beside_weight_gradients(runtime, rows, ahead):  # noqa: F811
    run(runtime, """
    import synthdata
    rows, ahead = map(int, sys.argv[2:])
    shape = synthdata.ModelShape(1, 64, 1, 64, 300, 64, "bf16")
    memory = np.zeros((640 << 20) + 256, np.uint8)
    ctx = mi.mimose_init(mi.make_cfg(synthdata.shape_dict(shape)), 0, (memory.ctypes.data + 255) // 256 * 256, 640 << 20)
    mi.mimose_force_plan(ctx, 0)
    batch = synthdata.make_batch(shape, rows // 64, 64, 3)
    names = [n for n in launched(lambda: mi.mimose_train_step(ctx, *batch, wait=False)) if "ln_bwd_vec" in n]
    assert names and all("Li1ELi%dELi4EE" % ahead in n for n in names), names
    """, rows, ahead)

"""pf_residual_noalloc's reasons for a mesh it does not take (CPU: refused before any launch)."""
import ctypes
import os

import pytest

from paper_2006_16764_amd import binding

pytestmark = pytest.mark.skipif(not os.path.exists(binding.LIB_PATH), reason="library not built")


@pytest.mark.parametrize("n", [(1025, 1024), (4096, 300), (256, 256, 256)], ids=lambda n: "x".join(map(str, n)))
def test_reason(n):
    lib = binding.load()
    p = binding.make_params(len(n), n, [0.4 * k for k in n], 0.2, 0.05, 1.6, 2.0)
    fake = [ctypes.c_void_p(0x10000 + 0x1000 * k) for k in range(3)]
    assert lib.pf_residual_noalloc(ctypes.byref(p), *fake, None) == binding.PF_ERR_INVALID_ARG
    msg = lib.pf_last_error().decode()
    if len(n) == 2:
        # 2-D calls use no scratch: the limit is a number of elements
        assert "bytes" not in msg and str(n[0] * n[1]) in msg and "2^20" in msg, msg
    else:
        assert "bytes of scratch" in msg and "2727" in msg and "2-D" not in msg, msg

"""Replicas and buffers read into device memory (one packing kernel) against
the same read into host memory (copies): every piece width (D and the block
widths multiples of four, of two, odd), a destination that is not 16-byte
aligned, rows that the learners share and rows that they do not."""

import numpy as np
import pytest

import cases

pytestmark = pytest.mark.gpu

# name -> (case, update mode, edit that leaves the learners with rows of their own)
CASES = {
    "four": (cases.case("mlp", 4, 2, 2, 2, B=8, IN=128, H=64, C=4, N=50, momentum=0.9, lr=0.05, seed=301), "eager", False),
    "two_shared": (cases.case("mlp", 18, 2, 2, 2, B=8, IN=102, H=70, C=6, N=50, lr=0.05, seed=302), "delayed", False),
    "odd_shared": (cases.case("mlp", 3, 1, 2, 2, B=8, IN=33, H=31, C=5, N=50, lr=0.05, seed=303), "delayed", True),
    "softmax": (cases.case("softmax", 4, 2, 2, 2, B=8, IN=3072, C=10, N=50, lr=0.05, seed=304), "auto", True),
    "averaging_long_row": (cases.case("averaging", 5, 1, 2, 2, IN=20001, lr=0.1, momentum=0.9, seed=305), "auto", False),
    "averaging_one": (cases.case("averaging", 2, 2, 1, 1, IN=1, lr=0.1, momentum=0.9, seed=306), "auto", False),
}


@pytest.mark.parametrize("offset", [0, 1, 2])
@pytest.mark.parametrize("name", sorted(CASES))
def test_device_reads_equal_host_reads(name, offset, gpu_lib):
    import ctypes
    import torch
    from paper_1903_05133_amd import HierAvg, native
    c, mode, edit = CASES[name]
    print(f"[gpu case] {name} offset {offset}", flush=True)
    with HierAvg(config=cases.native_config(c, mode)) as h:
        h.round()
        if edit:  # learners' rows differ
            w = h.params()
            h.set_params(w + np.arange(c["P"], dtype=np.float32)[:, None])
        n = c["P"] * h.D
        buf = torch.full((n + 8,), 7.0, dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()  # the handle reads on a stream of its own
        h.params_into(buf.data_ptr() + 4 * offset, n)
        got = buf.cpu().numpy()
        assert np.array_equal(got[offset:offset + n].reshape(c["P"], -1), h.params())
        assert np.all(got[:offset] == 7.0) and np.all(got[offset + n:] == 7.0)
        if c["momentum"] > 0:
            native.check(native.lib().hieravg_momentum(h._h, ctypes.c_void_p(buf.data_ptr() + 4 * offset), n))
            assert np.array_equal(buf.cpu().numpy()[offset:offset + n].reshape(c["P"], -1), h.momentum())

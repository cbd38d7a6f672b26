"""hieravg_time_kernel: every class of a workload can be timed on its own, a
class that the workload does not launch is refused, and what the launches
leave behind is the state of extra applications of the kernel."""

import numpy as np
import pytest

import cases

pytestmark = pytest.mark.gpu


def _handle(c, mode="auto"):
    from paper_1903_05133_amd import HierAvg
    print(f"[gpu case] time_kernel {mode} {c}", flush=True)
    return HierAvg(config=cases.native_config(c, mode))


WIDE = cases.case("mlp", 4, 2, 2, 2, B=48, IN=1100, H=500, C=7, N=300, sigma=0.5, lr=0.01, seed=501)


@pytest.mark.parametrize("c,refused", [
    # more than 32 samples, more than 32 classes: no k_head_step
    (WIDE, ("head_step", "head_step_end")),
    (dict(WIDE, B=20, C=40), ("head_step", "head_step_end", "head_fused")),
    (dict(WIDE, B=20), ("z1_delayed", "b1_step")),
], ids=["wide", "many_classes", "narrow"])
def test_classes_of_other_heads_are_refused(c, refused, gpu_lib):
    with _handle(c) as h:
        h.profile(True)
        h.round()
        ran = set(h.profile_read()) - {"draw_indices"}
        h.profile(False)
        for name in refused:
            with pytest.raises(Exception):
                h.time_kernel(name, 1)
        for name in sorted(ran):
            assert h.time_kernel(name, 2) > 0.0


def test_head_step_after_an_eager_round(gpu_lib):
    """A replayed delayed round after an eager one: the head reads the block
    forward's partials in their own split count."""
    with _handle(dict(WIDE, B=20)) as h:
        h.round()
        w = h.params()
        w[1, 0] += 1.0
        h.set_params(w)  # rows that differ: the next round is eager
        h.round()
        h.round()
        assert h.time_kernel("head_step", 3) > 0.0
        assert h.finite()


@pytest.mark.parametrize("c", [WIDE, dict(WIDE, B=20), dict(WIDE, B=20, C=40), dict(WIDE, B=20, momentum=0.9)],
                         ids=["wide", "narrow", "many_classes", "momentum"])
def test_rounds_after_timing_every_class(c, gpu_lib):
    """The launches scale the products by the operands as they are: timing
    every class of a delayed round leaves finite parameters, and so does the
    round after it."""
    with _handle(c) as h:
        h.profile(True)
        h.round()
        ran = set(h.profile_read()) - {"draw_indices"}
        h.profile(False)
        for name in sorted(ran):
            h.time_kernel(name, 2)
            assert h.finite(), name
        h.round()
        assert h.finite()


def test_block_end_of_errors_that_grew(gpu_lib):
    """A unit that no sample activates in the first block and every sample does
    in the second: its first block's errors are zero, those that a block-end
    launch finds are the second's.  Also buffers that grow far beyond the
    round's by repeated launches."""
    c = dict(WIDE, K1=1, B=20, momentum=0.9)
    with _handle(c) as h:
        u, IN, H = 3, c["IN"], c["H"]
        w, v = h.params(), h.momentum()
        w[:, u * IN:(u + 1) * IN] = 0.0  # z = b1 = 0 at step 0 (not active), b1 > 0 at step 1
        v[:, H * IN + u] = -1.0
        h.set_params(w)
        h.set_momentum(v)
        h.round()
        for name in ("scale_errors", "buffer_update_gemm", "block_update_gemm"):
            h.time_kernel(name, 1)
            assert h.finite() and np.isfinite(h.momentum()).all(), name
        h.time_kernel("buffer_update_gemm", 30)
        h.round()
        assert h.finite() and np.isfinite(h.momentum()).all()


@pytest.mark.parametrize("P,S", [(4, 2), (4, 4), (1, 1)])
def test_step_classes_of_averaging_rounds(P, S, gpu_lib):
    """Rounds that take all their steps in one launch: the classes of single
    steps and of the buffers' means can still be timed, before a round and
    after one, and a step is one step."""
    c = cases.case("averaging", P, S, 2, 2, IN=300, lr=0.5, momentum=0.9, avg_momentum=True, seed=502)
    with _handle(c) as h:
        for _ in range(2):
            names = ["momentum", "momentum_group_mean", "momentum_global_mean", "momentum_buffer_group_mean",
                     "momentum_buffer_global_mean"]
            for name in names:
                assert h.time_kernel(name, 2) > 0.0
            assert h.finite()
            h.round()
    with _handle(c) as h:
        w = h.params()
        h.time_kernel("momentum", 1)  # one heavy-ball step of the given gradients from v = 0: w - lr v
        assert np.allclose(h.params(), w - np.float32(0.5) * h.momentum(), rtol=0, atol=1e-7)

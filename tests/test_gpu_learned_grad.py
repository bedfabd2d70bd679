"""Weight gradients over slices of the samples: one sample, one full slice, a
short second slice, slices of 64 samples with a short last one."""
import numpy as np
import pytest

from test_gpu_learned import _params, setup  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("distinct,M", [(1, 32), (8, 32), (12, 36), (12, 528)])
def test_gradient_of_repeated_samples(lib, setup, distinct, M):
    """The loss is a mean over the samples, so repeating a set of samples M /
    distinct times leaves the gradient as it is, up to FP32 sums over M samples
    (M eps = 6e-5 at most)."""
    w, op, thetas, insts, xs, X, Phi, sig = setup
    print(f"[case] gradient of {distinct} samples repeated to {M}", flush=True)
    _, flat = _params(3)
    got = []
    for reps in (1, M // distinct):
        s = lib.Solver()
        s.set_reference_factored(op.A, op.alpha, op.shift, w.Z)
        s.set_pod_modes(Phi)
        s.learned_set_params(flat)
        sel = list(range(distinct)) * reps
        s.learned_prepare(np.stack([insts[m].mask for m in sel]), np.stack([insts[m].b for m in sel]), xs[sel],
                          thetas[sel].astype(np.float32))
        got.append(s.learned_loss_grad())
    (l0, g0), (l1, g1) = got
    np.testing.assert_allclose(l1, np.tile(l0, M // distinct), rtol=1e-12)
    for a, b in ((0, 512), (512, 640), (640, 17024), (17024, 17152), (17152, 82688), (82688, g0.size)):
        assert np.linalg.norm(g1[a:b].astype(float) - g0[a:b]) <= 1e-4 * np.linalg.norm(g0[a:b].astype(float)), (a, b)


@pytest.mark.parametrize("at", range(6))
def test_parameters_after_an_allocation_failed(lib, setup, at):
    """Setting the parameters again after one of their buffers had no room finds all
    of them: the gradient is that of a context with room."""
    w, op, thetas, insts, xs, X, Phi, sig = setup
    print(f"[case] network parameters after allocation {at} failed", flush=True)
    _, flat = _params(3)
    got = []
    for fails in (False, True):
        s = lib.Solver()
        s.set_reference_factored(op.A, op.alpha, op.shift, w.Z)
        s.set_pod_modes(Phi)
        if fails:
            s.fault(3, at)
            with pytest.raises(lib.Adef2Error) as e:
                s.learned_set_params(flat)
            assert e.value.code == lib.E_NOMEM
        s.learned_set_params(flat)
        s.learned_prepare(np.stack([insts[m].mask for m in range(4)]), np.stack([insts[m].b for m in range(4)]),
                          xs[:4], thetas[:4].astype(np.float32))
        got.append(s.learned_loss_grad())
    np.testing.assert_array_equal(got[0][1], got[1][1])

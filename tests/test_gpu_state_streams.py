"""State images of many pieces while steps are still in flight, on a stream of the caller's and on
the per-thread stream (which names another stream in every host thread): they are taken after the
steps enqueued before them, and what is set is what the next step runs on.  And images and moments
of several host threads' solvers at the same time, through the pinned blocks that they share."""
import ctypes
import threading

import numpy as np
import pytest

from paper_1810_08137_amd import ugks
from paper_1810_08137_amd import workloads as WL

pytestmark = pytest.mark.gpu

# 43 x 31 cells, 64 x 61 velocities: 41.6 MB of f, 20 pieces
CASE = dict(WL.CHANNEL_DEFAULTS, lx=2.0, ly=1.0, umax=5.0, vmax=5.0, kn=0.1, seed=9, nx=43, ny=31,
            nu=64, nv=61)
PER_THREAD = 2  # hipStreamPerThread


def _create(stream):
    case = dict(CASE)
    kn = case.pop("kn")
    mesh, vgrid, bc, opts = ugks.make_structs(**case)
    opts.stream = ctypes.c_void_p(stream)
    return ugks.ugks_create(mesh, vgrid, kn, bc, opts)


@pytest.mark.parametrize("kind", ["own", "per thread"])
def test_images_follow_the_steps_in_flight(kind):
    import torch

    own = torch.cuda.Stream()
    a = _create(own.cuda_stream if kind == "own" else PER_THREAD)
    b = _create(None)
    f0, W0 = ugks.ugks_get_state(b)
    ugks.ugks_step(a, 60)  # several ms, still running when the images are asked for
    fa, Wa = ugks.ugks_get_state(a)
    ugks.ugks_step(b, 60)
    ugks.ugks_moments(b)
    fb, Wb = ugks.ugks_get_state(b)
    assert not np.array_equal(fb, f0)
    assert np.array_equal(fa, fb) and np.array_equal(Wa, Wb)
    ugks.ugks_step(a, 60)
    ugks.ugks_set_state(a, f0, W0)
    ugks.ugks_step(a, 60)
    fa, Wa = ugks.ugks_get_state(a)
    assert np.array_equal(fa, fb) and np.array_equal(Wa, Wb)
    ugks.ugks_destroy(a)
    ugks.ugks_destroy(b)


def test_host_threads_share_the_pinned_blocks():
    import torch

    wrong, device = [], torch.cuda.current_device()
    h = _create(None)
    f0, W0 = ugks.ugks_get_state(h)
    ugks.ugks_step(h, 2)
    f2, W2 = ugks.ugks_get_state(h)
    m2 = ugks.ugks_moments(h)
    ugks.ugks_destroy(h)

    def work(t):
        try:
            torch.cuda.set_device(device)
            stream = torch.cuda.Stream()
            for _ in range(2):
                h = _create(stream.cuda_stream)
                for _ in range(2):
                    ugks.ugks_set_state(h, f0 * (t + 1.0), W0 * (t + 1.0))
                    f, W = ugks.ugks_get_state(h)
                    if not (np.array_equal(f, f0 * (t + 1.0)) and np.array_equal(W, W0 * (t + 1.0))):
                        wrong.append((t, "set"))
                ugks.ugks_set_state(h, f0, W0)
                ugks.ugks_step(h, 2)
                if not np.array_equal(ugks.ugks_moments(h), m2):
                    wrong.append((t, "moments"))
                f, W = ugks.ugks_get_state(h)
                if not (np.array_equal(f, f2) and np.array_equal(W, W2)):
                    wrong.append((t, "step"))
                ugks.ugks_destroy(h)
        except Exception as e:
            wrong.append((t, repr(e)))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong

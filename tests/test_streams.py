"""The seeded synthetic streams the other tests share."""
import numpy as np

from synth import make_stream


def test_every_call_returns_its_own_stream():
    """A test that changes its stream must not change the next test's input."""
    a = make_stream("tiny", n_frames=2)
    want, poses, params = a.depth.copy(), a.T_wc.copy(), dict(a.params)
    a.depth = np.zeros_like(a.depth)
    a.T_wc = a.T_wc[::-1]
    a.params["n_excess"] += 1
    b = make_stream("tiny", n_frames=2)
    assert np.array_equal(b.depth, want) and np.array_equal(b.T_wc, poses) and b.params == params
    c = make_stream("tiny", n_frames=2, cache=False)
    assert np.array_equal(c.depth, want) and np.array_equal(c.T_wc, poses) and c.params == params

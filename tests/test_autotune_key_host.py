"""The tuner's cache key: a choice timed on one kernel or shape is not taken for
another; no GPU needed."""
from dataclasses import replace

from paper_2404_03399_amd import autotune
from paper_2404_03399_amd import workloads as W


def test_key_tells_kernels_and_shapes_apart():
    w = W.c2_advection_large("adg_at", n_elem=1 << 14)
    batch = lambda ne: [replace(w, n_elem=ne, pe_size=16)] * 64
    sets = [[w], [replace(w, speed=-1.0)], [replace(w, pe_size=64)], [replace(w, pe_size=8)], [replace(w, scheme="dg")],
            [replace(w, n_elem=25 * 655, pe_size=25)], [replace(w, degree=2)], batch(1008), batch(1024),
            [w, replace(w, n_elem=25 * 655, pe_size=25)]]
    keys = [autotune._key(s, "gpu") for s in sets]
    assert len(set(keys)) == len(keys)
    assert autotune._key([replace(w, seed=7, dt=2 * w.dt)], "gpu") == keys[0]  # neither changes a kernel
    assert autotune._key([w], "another") != keys[0]

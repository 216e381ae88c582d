"""Cached launch shapes belong to the kernels they were timed on (no device needed): the keys tell apart
problems that run different kernels, and differ from those of earlier kernels."""
import hashlib
import json

import numpy as np

from paper_1908_01682_amd import autotune as A
from paper_1908_01682_amd import inputs as I
from tests.test_autotune_cache import _FakeSim


def _sha(**kw):
    return hashlib.sha1(json.dumps(kw, sort_keys=True).encode()).hexdigest()[:16]


def _variants():
    wave = I.dusty_wave(n_side=4000, cells_per_axis=2000)
    out = [wave]
    for kw in (dict(eos=I.ADIABATIC), dict(av_alpha=1.0), dict(av_beta=2.0), dict(h=0.5 * wave.params.h)):
        q = wave.copy()
        q.params = q.params.replace(**kw)
        out.append(q)
    return out


def test_plain_keys_tell_the_kernels_apart():
    # alpha and beta select one and the same force loop: four kinds of kernel
    assert len({A.plain_signature("gfx950", _FakeSim(p)) for p in _variants()}) == 4


def test_keys_of_earlier_kernels_are_not_found():
    wave = _variants()[0]
    old = _sha(dev="gfx950", dim=1, prec=0, ng=4000, nd=4000, cells=[2000], scheme=0, kind="plain")
    assert A.plain_signature("gfx950", _FakeSim(wave)) != old
    ns = np.array([8000])
    hist = np.histogram(np.log2(ns), bins=8, range=(0, 32))[0]
    old = _sha(dev="gfx950", dim=1, prec=0, n=1, hist=hist.tolist(), nmax=8000)
    assert A.signature("gfx950", [wave], 0) != old

"""The packed form of parameter dicts: byte for byte that of FovParams objects, for plain dicts and for what
only make_params converts, and the same refusals."""
import collections

import numpy as np
import pytest

from paper_2012_08655_amd import _native as N
from paper_2012_08655_amd import api

BASE = dict(fix_x=3.25, fix_y=-1.0, e0=32.0, slope=0.03, cap=12.0, block=16, origin_x=-5, origin_y=-9)
SHORT = {k: BASE[k] for k in ("fix_x", "fix_y", "e0", "slope", "cap")}
FORMS = [BASE, SHORT, dict(BASE, block=16.9), dict(BASE, fix_x=np.float32(3), origin_x=np.int64(-3), e0=True, cap=7),
         dict(BASE, cap="7.5"), dict(BASE, origin_y=2**33 + 5), dict(BASE, slope=float("nan"), cap=float("inf")),
         collections.defaultdict(lambda: 7, SHORT), dict(BASE, sigma_map=None, other=1)]


@pytest.mark.parametrize("n", [1, 2, len(FORMS)])
def test_bytes(n):
    for start in range(len(FORMS) - n + 1):
        plist = FORMS[start:start + n]
        arr, npar, keep = api._params_array(plist, n)
        assert (npar, keep) == (n, []) and len(arr) == n
        assert [bytes(a) for a in arr] == [bytes(N.make_params(p)) for p in plist]
        assert bytes(api._frame_params([[p] for p in plist], [])) == bytes(arr)


@pytest.mark.parametrize("n", [63, 64, 65, 128, 150])
@pytest.mark.parametrize("forms", [FORMS[:2], FORMS])  # packed; one frame of them through make_params
def test_many(n, forms):
    plist = [dict(forms[i % len(forms)], e0=float(i)) for i in range(n)]
    assert bytes(api._params_array(plist, n)[0]) == b"".join(bytes(N.make_params(p)) for p in plist)


@pytest.mark.parametrize("bad", [{}, dict(BASE, block="x"), dict(BASE, fix_x=None), dict(BASE, origin_x=float("nan"))])
def test_refusals(bad):
    with pytest.raises(Exception) as want:
        N.make_params(bad)
    for call in (lambda: api._params_array(bad, 1), lambda: api._frame_params([BASE, bad], [])):
        with pytest.raises(want.type):
            call()


def test_counts():
    for call in (lambda: api._params_array([BASE, BASE], 3), lambda: api._frame_params([[BASE, BASE]], [])):
        with pytest.raises(ValueError):
            call()
    with pytest.raises(TypeError):
        api._params_array(dict(BASE, sigma_map=np.zeros(4, np.float32)), 1)

"""A batch call hands the library as many parameter entries as frames, whatever the list given."""
import pytest

from paper_2012_08655_amd import _native as N
from paper_2012_08655_amd import api

P = dict(fix_x=1.0, fix_y=2.0, e0=3.0, slope=0.1, cap=4.0)


class Library:
    def foveate_autotune_batch(self, ins, outs, params, n, *rest):
        assert len(ins) == len(outs) == len(params) == n
        self.params = [bytes(p) for p in params]
        return N.FOV_OK


@pytest.mark.parametrize("given", [0, 1, 2, 3])
def test_entries(monkeypatch, given):
    lib = Library()
    monkeypatch.setattr(api, "tensor_desc", lambda t, layout: N.FovTensor())
    monkeypatch.setattr(api, "_stream_handle", lambda stream=None: 0)
    monkeypatch.setattr(N, "lib", lambda: lib)
    api.autotune_batch([None] * 3, [P] * given, [None] * 3)
    assert lib.params == [bytes(N.make_params(P))] * given + [bytes(N.FovParams())] * (3 - given)


def test_too_many(monkeypatch):
    monkeypatch.setattr(api, "tensor_desc", lambda t, layout: N.FovTensor())
    with pytest.raises(IndexError):
        api.autotune_batch([None] * 2, [P] * 3, [None] * 2)

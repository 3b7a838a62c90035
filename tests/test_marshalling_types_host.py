"""Cameras and groups of other types than the binding's own, subclasses among
them, reach the calls as their own to_c(), dim and stride() say; and an error
that is not a value's passes through instead of turning into the slow way."""
import ctypes

import pytest
import torch

import paper_2601_16736_amd as gs

VIEW = [1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0]


class FarCamera(gs.Camera):
    def to_c(self):
        c = super().to_c()
        c.z_far = 7.0
        return c


class OnlyToC:
    def __init__(self, x):
        self.x = x

    def to_c(self):
        return self.x.to_c()


class FlatGroup(gs.Group):
    """[n] tensors whose rows hold several elements."""

    @property
    def dim(self):
        return 4


class ScaledGroup(gs.Group):
    def to_c(self):
        g = super().to_c()
        g.lr *= 2.0
        return g


def _group(kind=gs.Group, shape=(8, 4)):
    return kind(*(torch.zeros(shape) for _ in range(4)), 1e-3)


def test_cameras_of_other_types():
    own = gs.Camera(VIEW, 500.0, 500.0, 320.0, 240.0, 640, 480, 0.1, 100.0)
    far = FarCamera(VIEW, 500.0, 500.0, 320.0, 240.0, 640, 480, 0.1, 100.0)
    got = gs._cameras_c([own, far, OnlyToC(own), OnlyToC(far)])
    assert [c.z_far for c in got] == [100.0, 7.0, 100.0, 7.0]
    assert bytes(got[0]) == bytes(got[2]) == bytes(own._by_field())
    assert len(gs._cameras_c([])) == 1 and ctypes.sizeof(gs._cameras_c([])) == ctypes.sizeof(gs.gs_camera)


def test_groups_of_other_types():
    own, scaled, flat = _group(), _group(ScaledGroup), _group(FlatGroup, (32,))
    got = gs._groups_c([own, scaled, OnlyToC(own), flat])
    assert [g.lr for g in got] == [1e-3, 2e-3, 1e-3, 1e-3]
    assert [g.dim for g in got] == [4, 4, 4, 4]
    assert bytes(got[2]) == bytes(own._by_field()) == bytes(got[0])
    assert flat.to_c().dim == 4


@pytest.mark.parametrize("make,item", [(gs._cameras_c, gs.Camera(VIEW, 5.0, 5.0, 3.0, 2.0, 6, 4)),
                                       (gs._groups_c, _group())])
def test_other_errors_pass_through(make, item, monkeypatch):
    class Broken:
        def pack(self, *_):
            raise NameError("packing")

    monkeypatch.setattr(gs, "_CAMERA" if make is gs._cameras_c else "_GROUP", Broken())
    with pytest.raises(NameError):
        make([item])

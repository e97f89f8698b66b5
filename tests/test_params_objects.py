"""Parameter objects as a handle takes them: LLGParams, a class of it that fills the
structure itself, and any other object with a to_c()."""
from dataclasses import dataclass

import pytest

from paper_1207_2192_amd._lib import LLGParamsC
from paper_1207_2192_amd.api import Disk, LLGParams


@dataclass
class Doubled(LLGParams):
    def to_c(self):
        p = super().to_c()
        p.alpha *= 2.0
        return p


class Plain:
    def to_c(self):
        return LLGParams(alpha=0.3, hext=(1.0, 2.0, 3.0), renorm=True).to_c()


class Instance(LLGParams):
    """A class that adds a field and keeps the rest."""
    label = "x"


def handle(n):
    disk = object.__new__(Disk)
    disk._h, disk.n = None, n
    return disk


@pytest.mark.parametrize("given", [LLGParams(alpha=0.1, temp=0.2), Doubled(alpha=0.1, freq=3.0), Plain(),
                                   Instance(alpha=0.4)])
def test_every_object_arrives_as_its_to_c(given):
    want = bytes(given.to_c())
    assert [bytes(c) for c in handle(3)._params([given] * 3)] == [want] * 3
    if isinstance(given, LLGParams):
        assert [bytes(c) for c in handle(2)._params(given)] == [want] * 2
    mixed = handle(2)._params([given, LLGParams(c=1.0)])
    assert bytes(mixed[0]) == want and mixed[1].c == 1.0 and isinstance(mixed[0], LLGParamsC)


def test_other_objects_are_refused():
    with pytest.raises(AttributeError):
        handle(1)._params([object()])
    with pytest.raises(ValueError):
        handle(2)._params([LLGParams()])

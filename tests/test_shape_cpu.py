"""tman.Shape is an ordinary value: using it leaves nothing behind in it, and classes made from it are copied whole."""
import copy
import dataclasses
import pickle

import paper_2511_11248_amd as tman


@dataclasses.dataclass(frozen=True)
class Named(tman.Shape):
    name: str = ""


def test_use_leaves_no_trace():
    used, fresh = tman.Shape(64, 256, 4, 64), tman.Shape(64, 256, 4, 64)
    assert tman.tman_packed_bytes(used) > 0
    assert vars(used) == vars(fresh) and tman.Shape(**vars(used)) == fresh
    assert used == fresh and hash(used) == hash(fresh) and repr(used) == repr(fresh)
    assert pickle.dumps(used) == pickle.dumps(fresh)
    for other in (copy.copy(used), copy.deepcopy(used), pickle.loads(pickle.dumps(used)), dataclasses.replace(used)):
        assert other == fresh and tman.tman_packed_bytes(other) == tman.tman_packed_bytes(fresh)
    assert tman.tman_packed_bytes(dataclasses.replace(used, K=512)) > tman.tman_packed_bytes(used)


def test_derived_classes():
    s = Named(64, 256, 4, 64, name="gate")
    assert tman.tman_packed_bytes(s) == tman.tman_packed_bytes(tman.Shape(64, 256, 4, 64))
    for other in (copy.copy(s), copy.deepcopy(s), pickle.loads(pickle.dumps(s))):
        assert type(other) is Named and other == s and other.name == "gate"


def test_anything_with_a_c_form():
    class Rows:
        __slots__ = ("rows",)

        def c(self):
            return tman.Shape(self.rows, 256, 4, 64).c()

    s = Rows()
    for s.rows in (64, 128):
        assert tman.tman_packed_bytes(s) == tman.tman_packed_bytes(tman.Shape(s.rows, 256, 4, 64))

"""A tuning result of another build of the library is measured again; this build's, and one set by hand, are returned."""
import pytest

from paper_2207_06908_amd import autotune as T


class Measured(Exception):
    pass


def _measure(_n):
    raise Measured


GRID = {"variant": 1, "tile_y": 0, "tile_z": 0, "ms_per_step": 1.0}
BATCH = {"tile_x": 60, "tile_y": 8, "tile_z": 32, "persistent": True, "ms_per_step": 1.0}


@pytest.mark.parametrize("tune,value", [(T.tune_grid, GRID), (T.tune_batch, BATCH)])
def test_a_choice_of_another_build_is_measured_again(tune, value, tmp_path):
    p = str(tmp_path / "tune.json")
    T.store("old", dict(value, candidates=26), p)                              # written before builds were named
    T.store("other", dict(value, candidates=26, library="0" * 16), p)
    T.store("same", dict(value, candidates=26, library=T.library_stamp()), p)
    T.store("hand", value, p)
    for key in ("old", "other", "absent"):
        with pytest.raises(Measured):
            tune(_measure, key, path=p)
    for key in ("same", "hand"):
        assert tune(_measure, key, path=p)["ms_per_step"] == 1.0
        with pytest.raises(Measured):
            tune(_measure, key, path=p, force=True)

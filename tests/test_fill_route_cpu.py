"""CPU checks of the rules that choose a fill's kernel (mrg_fill_route,
mrg_leapfrog_route): computed on the host alone, for a device of 256 compute
units.  The GPU tests check what the kernels write on each side of a rule."""
import pytest

from paper_1412_8266_amd import _abi

LANES, WAVE, BLOCKS, PARTS, HALVES, STEPS, DEAL = range(7)
U32, F32, F64 = 0, 1, 2
ROWS, ILV = 0, 1


def rows(count, n, dtype=U32, off=0, streams=None):
    return _abi.mrg_fill_route(streams or count, count, n, dtype, ROWS, off)


def steps(count, n, dtype=U32, off=0, streams=None):
    return _abi.mrg_fill_route(streams or count, count, n, dtype, ILV, off)


@pytest.fixture
def keys():
    old = {}

    def set_(**kw):
        for k, v in kw.items():
            old.setdefault(k, _abi.mrg_config_get(k))
            _abi.mrg_config_set(k, v)
    yield set_
    for k, v in old.items():
        _abi.mrg_config_set(k, v)


@pytest.mark.parametrize("key,value", [("coop_lanes", 32), ("coop_wgs_per_cu", 4), ("coop_order", 1)])
def test_a_key_that_is_set_is_honoured(keys, key, value):
    assert rows(64, 1 << 20).kernel == BLOCKS
    keys(**{key: value})
    r = rows(64, 1 << 20)
    assert r.kernel == WAVE
    assert r.lanes == (32 if key == "coop_lanes" else 64)


def test_strategies_other_than_automatic_cut_nothing(keys):
    for s in (1, 2):
        keys(strategy=s)
        assert rows(64, 1 << 20).kernel == (LANES if s == 1 else WAVE)
        assert steps(64, 4096).kernel == STEPS
        assert steps(1, 4096).kernel == STEPS


def test_refused():
    for args in ((4, 0, 1), (4, 5, 1), (4, 1, 0)):
        with pytest.raises(_abi.MRGError):
            _abi.mrg_fill_route(*args, U32, ROWS)
    with pytest.raises(_abi.MRGError):
        _abi.mrg_leapfrog_route(1, 0, 4, U32, ROWS)

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


def test_streams_move_in_the_fill_unless_arrivals_queue():
    """At most 256 arrivals a ticket; on a line that 32 tickets share, 256 by
    waves and 2048 (4096 from 512 streams on) by lanes; none without tickets."""
    # own lines (4096 streams and fewer), packed tickets, no tickets
    for streams, n, want in ((4096, 16384, 1), (4096, 65536, 0), (4097, 2048, 1), (4097, 16384, 0),
                             (1 << 20, 2048, 1), ((1 << 20) + 1, 2048, 0)):
        r = steps(64, n, streams=streams)
        assert r.kernel == PARTS and r.moves == want, (streams, n, r.parts)
    assert steps(1024, 8192, streams=5000).moves == 1      # 128 segments
    assert steps(300, 8192, streams=5000).moves == 0
    for streams, want in ((4096, 1), (4097, 0)):
        r = rows(40, 1 << 16, streams=streams)
        assert r.kernel == BLOCKS and 8 < r.parts <= 256 and r.moves == want
    assert rows(1, 1 << 16, streams=1 << 20).moves == 1
    assert rows(1, 1 << 16, streams=(1 << 20) + 1).moves == 0


# (streams, steps, dtype, offset, cut): both sides of each line of the rule that
# cuts interleaved streams into segments
STEP_RULE = [
    (64, 127, U32, 0, False), (64, 128, U32, 0, True), (32768, 4096, U32, 20, True),
    (32800, 4096, U32, 20, False), (32800, 191, U32, 0, False), (32800, 192, U32, 0, True),
    (40960, 1000, U32, 0, True), (40992, 1000, U32, 0, False), (40959, 1000, U32, 0, False),
    (57344, 999, F32, 0, False), (57344, 1000, F32, 0, True), (65536, 4096, F32, 0, True),
    (65536, 4096, F32, 20, False), (65535, 4096, F32, 0, False), (65537, 4096, U32, 0, False),
    (18432, 4096, F64, 24, True), (18433, 4096, F64, 24, False), (18448, 4096, F64, 0, True),
    (28672, 4096, F64, 0, True), (28688, 4096, F64, 0, False), (32768, 999, F64, 0, True),
    (32768, 1000, F64, 0, False), (32768, 512, F64, 8, True), (32768, 513, F64, 8, False),
    (32784, 512, F64, 0, False), (38912, 800, U32, 4, True), (38912, 801, F32, 4, False),
    (38913, 800, U32, 0, False), (43008, 600, F32, 20, True), (43008, 601, U32, 20, False),
    (43009, 600, U32, 0, False), (43008, 192, U32, 4, True), (43008, 191, U32, 4, False)]


@pytest.mark.parametrize("count,n,dtype,off,cut", STEP_RULE)
def test_interleaved_streams_are_cut_where_it_pays(count, n, dtype, off, cut):
    r = steps(count, n, dtype, off)
    assert r.kernel == (PARTS if cut else STEPS)
    if cut:
        assert r.part_values % 16 == 0 and (r.parts - 1) * r.part_values < n <= r.parts * r.part_values


# (MiB of one stream in order, dtype, block bytes, chunk bytes): both sides of
# the block sizes' lines
ORDER_RULE = [(1, U32, 8, 8), (11, U32, 8, 8), (12, U32, 16, 16), (47, F32, 16, 16), (48, U32, 32, 16),
              (191, F32, 32, 16), (192, U32, 64, 64), (193, U32, 48, 16), (256, U32, 64, 64),
              (257, F32, 48, 16), (319, F32, 64, 64), (319, F64, 32, 16), (320, F64, 64, 64),
              (320, U32, 64, 64), (2047, U32, 64, 64), (2048, F64, 128, 64)]


@pytest.mark.parametrize("mib,dtype,block,chunk", ORDER_RULE)
def test_blocks_of_a_stream_in_order(mib, dtype, block, chunk):
    es = 8 if dtype == F64 else 4
    n = (mib << 20) // es
    for r in (_abi.mrg_leapfrog_route(1, n // 4, 4, dtype, ILV), rows(1, n, dtype), steps(1, n, dtype),
              rows(64, n // 64, dtype)):
        assert r.kernel == BLOCKS
        assert (r.part_values * es, r.chunk_values * es) == (block << 10, chunk << 10)
        assert (r.parts - 1) * r.part_values <= n


# (players, cards, waves, waves to a workgroup, players a lane, moved in the
# kernel): both sides of 4 and of 15 waves per CU at 64 players a lane, and of
# 4096 cards
DEAL_RULE = [(2, 5, 1, 1, 1, 1), (1000, 1000, 512, 2, 32, 1), (65536, 52, 2048, 8, 32, 1),
             (65537, 52, 1025, 5, 64, 1), (245696, 52, 3839, 15, 64, 1), (245697, 52, 3840, 15, 64, 1),
             (4096, 4096, 4096, 16, 64, 1), (4096, 4097, 4096, 1, 64, 0),
             (60, 64 * 3839, 3839, 15, 60, 1), (60, 64 * 3840, 3840, 1, 60, 0),
             (65536, 8000, 4096, 1, 497, 0), (65536, 65536, 4096, 1, 4096, 0)]


@pytest.mark.parametrize("players,cards,waves,per,lane,moves", DEAL_RULE)
def test_deals_by_player(players, cards, waves, per, lane, moves):
    r = _abi.mrg_leapfrog_route(1, players, cards, U32, ROWS)
    assert r.kernel == DEAL
    assert r.waves_per_group == per and r.moves == moves and r.part_values == lane
    assert r.waves == waves == min(r.parts, 4096) and r.parts * lane * r.lanes >= players * cards
    assert (r.waves + per - 1) // per <= 256 or not moves


# (streams, row bytes, dtype, offset, several lanes): both sides of the shortest
# row that several lanes draw
LANE_RULE = [(1, 380, U32, 0, False), (1, 384, U32, 4, True), (1, 384, U32, 0, False), (1, 512, U32, 0, True),
             (2048, 504, F64, 8, True), (2048, 384, F64, 0, False), (2048, 512, F64, 0, True),
             (8192, 508, U32, 4, False), (8192, 512, U32, 4, True), (8192, 512, F32, 0, False),
             (8192, 640, F32, 0, True), (8192, 640, F64, 0, False), (8192, 768, F64, 0, True),
             (16384, 1020, F32, 0, False), (16384, 1028, F32, 0, True), (16384, 1408, U32, 0, False),
             (16384, 1536, U32, 0, True), (16384, 2816, F64, 0, False), (16384, 2944, F64, 0, True),
             (20000, 1660, U32, 0, False), (20000, 1672, U32, 0, True), (28672, 3328, F32, 0, False),
             (28672, 3456, F32, 0, True), (32768, 2728, U32, 0, False), (32768, 2732, U32, 0, True),
             (32768, 5504, F32, 0, False), (32768, 5632, F32, 0, True), (32768, 8064, F64, 0, False),
             (32768, 8192, F64, 0, True), (32769, 8188, U32, 0, False), (32769, 8192, U32, 0, True)]


@pytest.mark.parametrize("count,row,dtype,off,several", LANE_RULE)
def test_shortest_row_of_several_lanes(count, row, dtype, off, several):
    r = rows(count, row // (8 if dtype == F64 else 4), dtype, off)
    assert (r.kernel == WAVE) == several


@pytest.mark.parametrize("dtype,es", [(U32, 4), (F32, 4), (F64, 8)])
def test_rows_of_whole_4_kib_take_two_lanes(dtype, es):
    """On lines, in the lane writer: 4 KiB at any number of streams it takes,
    12 KiB from a wave of lanes per SIMD on."""
    n = 4096 // es
    for count in (40000, 65536, 262144):
        assert rows(count, n, dtype).kernel == HALVES
        assert rows(count, n, dtype, 4).kernel != HALVES
        assert rows(count, n + 1, dtype).kernel != HALVES
        assert rows(count, n + 128 // es, dtype).kernel != HALVES
        assert rows(count, 2 * n, dtype).kernel == WAVE
    assert rows(65535, 3 * n, dtype).kernel == WAVE
    assert rows(65536, 3 * n, dtype).kernel == HALVES

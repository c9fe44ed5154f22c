"""GPU: the automatic choice of fill kernels at its edges, against the oracle.

Every shape sits at a line of a dispatch rule (number of streams against the
chip, row bytes, rows on or off 128-byte lines) with remainders on both sides
of it.  Outputs and states are integers or exact conversions of them:
tolerance 0.  Guard words around every output stay untouched, and a second
fill continues the first.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

GUARD = 32


@pytest.fixture(scope="module")
def mg():
    import torch
    import paper_1412_8266_amd as m
    assert torch.cuda.is_available()
    return m


def check(mg, first, count, n, dtype, layout, off, reps=2):
    import torch
    print("dispatch", first, count, n, dtype, layout, off, flush=True)
    base = oracle.seed_from_master(20120719)
    ss = mg.StreamSet(first + count + 1, seed=[int(x) for x in base])
    st = oracle.streams(base, first, count)
    buf = torch.zeros(count * n + off + 2 * GUARD, dtype=mg.torch_dtype(dtype), device="cuda")
    lo, hi = GUARD + off, GUARD + off + count * n
    for rep in range(reps):
        buf.zero_()
        ss.fill_ptr(n, dtype, layout, buf[lo:hi].data_ptr(), first=first, count=count)
        h = buf.cpu().numpy()
        want, st = oracle.fill(st, n, dtype, layout)
        assert np.array_equal(h[lo:hi].view(np.uint8), want.reshape(-1).view(np.uint8)), rep
        assert not h[:lo].view(np.uint8).any() and not h[hi:].view(np.uint8).any(), rep
    assert np.array_equal(ss.get_states(first, count), st)
    assert np.array_equal(ss.get_states(0, first), oracle.streams(base, 0, first))
    ss.close()


# rows: lanes per stream by the number of streams (64 / 32 / 16 / 8, one) and
# the shortest row given to several lanes (384 bytes; a byte per 16 streams)
ROWS = [(1, 95, 0, 0), (1, 96, 0, 0), (5, 97, 1, 3), (2048, 100, 0, 0), (2049, 100, 0, 1),
        (4096, 190, 2, 0), (4097, 127, 0, 0), (8200, 129, 1, 0), (16384, 256, 0, 0),
        (16384, 255, 0, 1), (20000, 330, 0, 0), (32768, 257, 2, 0), (32769, 600, 0, 0),
        (65535, 600, 1, 0), (65536, 2050, 0, 0)]

# and by the rows' type and place on lines
ROWS += [(8192, 96, 2, 0), (8192, 80, 2, 0), (16384, 352, 0, 0), (16384, 384, 0, 0), (16384, 272, 2, 0),
         (32768, 760, 0, 0), (32768, 1024, 1, 0), (32768, 992, 1, 0), (32768, 768, 2, 0), (32768, 761, 0, 3)]

# two lanes per stream (rows of 4 KiB on lines): whole and partial last waves
ROWS += [(65536, 1024, 0, 0), (65553, 1024, 1, 0), (65569, 512, 2, 0), (65600, 1024, 0, 32)]
# and rows of 12 KiB, from 65536 on
ROWS += [(65536, 3072, 0, 0), (65553, 1536, 2, 0)]


@pytest.mark.parametrize("count,n,dtype,off", ROWS)
def test_rows(mg, count, n, dtype, off):
    check(mg, 3, count, n, dtype, 0, off, reps=1 if count * n > 1 << 25 else 2)


# rows in blocks of a wave each (few streams, rows of 16 or 64 KiB and more):
# one and several blocks, remainders in the last block and in one of their
# own, every chunk size, states moved by the last block or by a launch after
BLOCKS = [(1, 4096, 0, 0), (1, 4097, 0, 31), (3, 8193, 1, 1), (2, 6144, 2, 0), (2, 2049, 2, 15),
          (1, 1 << 20, 0, 5), (1, (1 << 22) + 3, 0, 0), (1, 1 << 21, 2, 1), (1, 5 << 20, 0, 0), (40, 100001, 1, 2),
          (256, 4100, 0, 7), (257, 4100, 0, 7), (512, 16400, 0, 9), (513, 16400, 0, 0)]


# both sides of the sizes where blocks and their chunks grow: 12, 48, 192 and
# 320 MiB in all
BLOCKS += [(1, (3 << 20) - 1, 0, 0), (1, 3 << 20, 0, 3), (5, (3 << 19) // 5 + 1, 2, 1), (1, (12 << 20) - 9, 1, 1),
           (1, 12 << 20, 0, 0), (200, 70001, 0, 1), (40, 170001, 2, 1), (1, (48 << 20) - 100, 0, 3),
           (1, (48 << 20) + 999, 1, 0), (1, (40 << 20) - 99, 2, 5), (1, (40 << 20) + 99, 2, 0),
           (500, 170001, 0, 7)]


@pytest.mark.parametrize("engine", [1, 0], ids=["f64", "int"])
@pytest.mark.parametrize("count,n,dtype,off", BLOCKS)
def test_rows_in_blocks(mg, count, n, dtype, off, engine):
    old = mg.mrg_config_get("engine")
    mg.mrg_config_set("engine", engine)
    try:
        check(mg, 2, count, n, dtype, 0, off)
    finally:
        mg.mrg_config_set("engine", old)


# interleaved in segments: lanes of one wave in two segments and in one, a
# last segment of one step, tickets on lines of their own and packed
STEPS = [(2, 40000, 0, 1), (70, 20000, 2, 0), (1, 64, 0, 0), (1, 70001, 1, 3), (3, 1000, 2, 1), (63, 127, 0, 0), (64, 129, 1, 0),
         (100, 4097, 0, 5), (4095, 300, 2, 0), (4096, 193, 0, 0), (5000, 1000, 1, 1),
         (32768, 129, 2, 0), (32769, 129, 2, 0), (65536, 145, 0, 0), (65537, 145, 0, 0)]


# both sides of the lines where many streams stop being cut
STEPS += [(38912, 799, 0, 1), (43007, 577, 1, 5), (32800, 192, 0, 0), (32800, 192, 0, 5), (57344, 1000, 1, 0), (65536, 1001, 0, 0),
          (18432, 700, 2, 1), (28672, 1000, 2, 0), (28688, 1000, 2, 0), (32768, 520, 2, 0)]


@pytest.mark.parametrize("engine", [1, 0], ids=["f64", "int"])
@pytest.mark.parametrize("count,n,dtype,off", STEPS)
def test_steps_in_segments(mg, count, n, dtype, off, engine):
    old = mg.mrg_config_get("engine")
    mg.mrg_config_set("engine", engine)
    try:
        check(mg, 1, count, n, dtype, 1, off)
    finally:
        mg.mrg_config_set("engine", old)


# deals by player on both sides of 4 and of 15 waves per CU at 64 players a
# lane: the stream moved in the kernel, by a launch after it
@pytest.mark.parametrize("engine", [1, 0], ids=["f64", "int"])
@pytest.mark.parametrize("players,cards,dtype", [(65472, 52, 0), (65473, 52, 2), (245696, 52, 1), (245697, 52, 0),
                                                 (3001, 1001, 1), (75, 64 * 1919, 0), (75, 64 * 1920 + 1, 2)])
def test_deals(mg, players, cards, dtype, engine):
    old = mg.mrg_config_get("engine")
    mg.mrg_config_set("engine", engine)
    try:
        with mg.StreamSet(3, master_seed=8) as ss:
            st = ss.get_states()
            for _ in range(2):
                got = ss.fill_leapfrog(1, players, cards, dtype).cpu().numpy()
                want, st[1:2] = oracle.fill(st[1:2], players * cards, dtype)
                want = np.ascontiguousarray(want.reshape(cards, players).T)
                assert np.array_equal(got.view(np.uint8), want.view(np.uint8))
                assert np.array_equal(ss.get_states(), st)
    finally:
        mg.mrg_config_set("engine", old)


def test_captured_fill_advances_each_replay(mg):
    """A captured fill whose states move inside the fill kernel: every replay,
    with eager work between, continues the streams."""
    import torch
    base = oracle.seed_from_master(5)
    ss = mg.StreamSet(8, seed=[int(x) for x in base])
    st = oracle.streams(base, 0, 8)
    out = torch.empty(8 * 20001, dtype=torch.uint32, device="cuda")
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ss.fill(20001, mg.U32, out=out)  # eager first
        side.synchronize()
        want, st = oracle.fill(st, 20001, oracle.U32)
        assert np.array_equal(out.cpu().numpy(), want.reshape(-1))
        with torch.cuda.graph(g, stream=side):
            ss.fill(20001, mg.U32, out=out)
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        want, st = oracle.fill(st, 20001, oracle.U32)
        assert np.array_equal(out.cpu().numpy(), want.reshape(-1))
        torch.ones(1000, device="cuda").sum().item()
    assert np.array_equal(ss.get_states(), st)
    ss.close()


def test_sets_hold_what_their_fills_need(mg):
    """24 bytes a stream, tickets beside them in sets of up to 2^20 streams of
    the generators that cut streams into parts."""
    import torch
    n = 1 << 26
    for generator in ("mrg32k3a", "philox", "tinymt"):
        with mg.StreamSet(n, master_seed=1, generator=generator, per_param=n) as ss:  # tables, records
            ss.fill(4, mg.U32, count=1)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        with mg.StreamSet(n, master_seed=1, generator=generator, per_param=n):
            used = before - torch.cuda.mem_get_info()[0]
        assert used < 25 * n, (generator, used / n)


# a range of a set with a ticket per stream and of one without: rows in blocks,
# segments, a deal, Philox runs and segments; both move their streams
@pytest.mark.parametrize("streams", [1 << 20, (1 << 20) + 1])
@pytest.mark.parametrize("generator,count,n,layout", [
    ("mrg32k3a", 3, 20001, 0), ("mrg32k3a", 1, 2000, 0), ("mrg32k3a", 2, 4100, 0), ("mrg32k3a", 100, 1000, 1), ("mrg32k3a", 1, 9, 2),
    ("mrg32k3a", 33, 8193, 1), ("philox", 3, 70001, 0), ("philox", 40, 4001, 1),
    ("philox", 40, 20001, 1)])
def test_ranges_of_sets_with_and_without_tickets(mg, streams, generator, count, n, layout):
    with mg.StreamSet(streams, master_seed=3, generator=generator) as ss:
        first = streams - count - 1
        st = ss.get_states(first, count)
        fill = oracle.fill if generator == "mrg32k3a" else oracle.philox_fill
        for _ in range(2):
            if layout == 2:  # n cards to each of 500 players
                got = ss.fill_leapfrog(first, 500, n, mg.U32).cpu().numpy()
                want, st = oracle.fill(st, 500 * n, oracle.U32)
                want = want.reshape(n, 500).T
            else:
                got = ss.fill(n, mg.U32, layout, first=first, count=count).cpu().numpy()
                want, st = fill(st, n, oracle.U32, layout)
            assert np.array_equal(got, want)
            assert np.array_equal(ss.get_states(first, count), st)


class Words:
    """Device words at an address, for torch."""

    def __init__(self, ptr, n):
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": "<i4", "data": (ptr, False),
                                         "version": 2}


# fills whose parts count their arrivals: rows in blocks, interleaved segments,
# Philox runs; sets with a line per ticket and with packed tickets
@pytest.mark.parametrize("generator,streams,first,count,n,layout", [
    ("mrg32k3a", 8, 2, 5, 20001, 0), ("mrg32k3a", 70, 3, 64, 4097, 1), ("mrg32k3a", 5000, 3, 64, 4097, 1),
    ("philox", 8, 2, 5, 70001, 0)])
def test_set_states_makes_spoiled_streams_whole(mg, generator, streams, first, count, n, layout):
    """Fills of one stream that were not ordered can leave its arrivals counted
    in part; set_states restores the stream, not its state words alone."""
    import torch
    with mg.StreamSet(streams, master_seed=9, generator=generator) as ss:
        st = ss.get_states()
        pitch = 32 if streams <= 4096 else 1
        tickets = torch.as_tensor(Words(ss.states_ptr + 24 * streams, streams * pitch), device="cuda")
        assert not tickets.cpu().numpy()[::pitch].any()
        tickets[first * pitch:(first + count) * pitch:pitch] = 1
        torch.cuda.synchronize()
        ss.set_states(st[first:first + count], first=first)
        fill = oracle.fill if generator == "mrg32k3a" else oracle.philox_fill
        for _ in range(2):
            got = ss.fill(n, mg.U32, layout, first=first, count=count).cpu().numpy()
            want, st[first:first + count] = fill(st[first:first + count], n, oracle.U32, layout)
            assert np.array_equal(got, want)
            assert np.array_equal(ss.get_states(), st)
        assert not tickets.cpu().numpy()[::pitch].any()


# Philox: rows in LDS blocks (one block per row, rows that a workgroup cannot
# hold whole, the longest), runs of a row (one, several, more than the tickets
# take), segments of a stream; (streams, n, dtype, layout, offset, position)
PHILOX = [(65537, 2048, 0, 0, 0, 4), (65538, 1024, 2, 0, 0, 1), (300, 1, 0, 0, 1, 3), (5000, 2, 1, 0, 0, 1), (1300, 255, 2, 0, 1, 2), (9000, 61, 0, 0, 3, 0),
          (2, 511, 0, 0, 5, 1), (2, 512, 0, 0, 5, 1), (70, 2001, 1, 0, 2, 0), (3, 1 << 17, 0, 0, 0, 0),
          (2, 70001, 2, 0, 1, 3), (1, 1 << 21, 1, 0, 7, 2), (5000, 1100, 0, 0, 0, 0),
          (70000, 4, 0, 0, 0, 4), (3000, 1020, 0, 0, 0, 8), (3000, 508, 2, 0, 0, 2), (20000, 1030, 1, 0, 0, 1),
          (1, 5001, 0, 1, 0, 1), (33, 4100, 2, 1, 0, 3), (5000, 700, 1, 1, 1, 0), (64, 20000, 0, 1, 0, 1)]


# many rows of one run in the chunked order and not, of two runs of binary64
PHILOX += [(65539, 2049, 0, 0, 0, 1), (65541, 4096, 0, 0, 0, 0), (33333, 4096, 1, 0, 1, 3),
           (65539, 1025, 2, 0, 0, 2), (33333, 2048, 2, 0, 0, 0), (33333, 4096, 2, 0, 0, 1),
           (16411, 4097, 0, 0, 3, 2)]


# several pieces of rows to a workgroup, from 512 MiB (binary64 a GiB) on: whole
# and partial last pieces, 256 rows, on and off 16 bytes and blocks, and below
PHILOX += [(300007, 4, 0, 0, 0, 0), (100003, 128, 1, 0, 0, 2), (70001, 508, 2, 0, 0, 0),
           (700001, 192, 0, 0, 0, 0), (700001, 192, 1, 0, 0, 3), (130001, 1031, 0, 0, 1, 1),
           (400001, 171, 2, 0, 0, 0), (400001, 340, 2, 0, 0, 0), (400001, 340, 2, 0, 0, 1), (400001, 337, 2, 0, 1, 0)]


@pytest.mark.parametrize("count,n,dtype,layout,off,pos", PHILOX)
def test_philox(mg, count, n, dtype, layout, off, pos):
    import torch
    print("philox", count, n, dtype, layout, off, pos, flush=True)
    with mg.StreamSet(count + 2, master_seed=17, generator="philox") as ss:
        ss.jump_uniform(pos)
        ss.jump_uniform(2**64 - 6, first=1, count=1)  # one row across the wrap
        st = ss.get_states()
        buf = torch.zeros(count * n + off + 2 * GUARD, dtype=mg.torch_dtype(dtype), device="cuda")
        lo, hi = GUARD + off, GUARD + off + count * n
        for rep in range(3):
            buf.zero_()
            if rep == 2:  # another key in one row
                st[count // 2 + 1, 4:] = 12345, 678
                ss.set_states(st)
            ss.fill_ptr(n, dtype, layout, buf[lo:hi].data_ptr(), first=1, count=count)
            h = buf.cpu().numpy()
            want, st[1:-1] = oracle.philox_fill(st[1:-1], n, dtype, layout)
            assert np.array_equal(h[lo:hi].view(np.uint8), want.reshape(-1).view(np.uint8)), rep
            assert not h[:lo].view(np.uint8).any() and not h[hi:].view(np.uint8).any(), rep
            assert np.array_equal(ss.get_states(), st)

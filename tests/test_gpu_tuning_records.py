"""Tuning records that lie idle (GPU): the autotuner reports them as such, a
record read and set again has the graph decode as it did, and a decode with an
idle record is the decode without one, also where a flag forces the path."""
import ctypes

import pytest

from paper_2507_10424_amd import workloads as wl

pytestmark = pytest.mark.gpu

CHECK, ONCHIP = 0, 2  # kernel ids of ldpc_timing_read; the LDS-resident decoder is timed as on-chip


def setup(B):
    import torch
    from paper_2507_10424_amd import ldpc
    H = wl.regular_ldpc(2016, 252, 4, 32, seed=2)  # rows of 32: LDS-resident without a record, else streamed
    Hd = torch.from_numpy(H).to("cuda:0")
    rate = 1.0 - 252 / 2016
    llr = torch.from_numpy(wl.bpsk_awgn_llr(None, 4.4, rate, seed=5, n=2016, batch=B)).to("cuda:0")
    return torch, ldpc, Hd, llr


def launches(torch, ldpc, fn):
    """Outputs of fn() and its check and on-chip launches."""
    lib = ldpc.load_library()
    assert lib.ldpc_timing_enable(1) == 0
    out = fn()
    torch.cuda.synchronize()
    counts = []
    for kid in (CHECK, ONCHIP):
        ms, n = ctypes.c_double(), ctypes.c_int64()
        assert lib.ldpc_timing_read(kid, ctypes.byref(ms), ctypes.byref(n)) == 0
        counts.append(n.value)
    assert lib.ldpc_timing_enable(0) == 0
    return out, counts


def test_idle_record_survives_get_and_set():
    torch, ldpc, Hd, llr = setup(200)
    g, other = ldpc.build_graph(Hd), ldpc.build_graph(Hd)
    best = ldpc.autotune(g, 200, 10, 4.4)
    assert best["path"] == 2 and best["ms"] > 0 and best["idle"] == 1, best
    got = ldpc.get_tuning(g)
    assert {k: v for k, v in got.items() if k != "ms"} == {k: v for k, v in best.items() if k != "ms"}
    ref, counts = launches(torch, ldpc, lambda: ldpc.minsum_decode(g, llr, 10))
    assert counts == [0, 1]
    record = {k: v for k, v in got.items() if k != "ms"}
    for idle, want in ((1, [0, 1]), (0, [10, 0])):  # the LDS-resident decoder; the record's own launches
        for graph in (g, other):
            ldpc.set_tuning(graph, **{**record, "stream_chunk": 0, "idle": idle})
            assert ldpc.get_tuning(graph)["idle"] == idle
            out, counts = launches(torch, ldpc, lambda: ldpc.minsum_decode(graph, llr, 10))
            assert counts == want, (idle, counts)
            assert all(torch.equal(a, b) for a, b in zip(ref, out))
    with pytest.raises(ldpc.LdpcError) as e:
        ldpc.set_tuning(g, **{**record, "idle": 2})
    assert e.value.status == -1
    ldpc.set_tuning(g, None)
    assert ldpc.get_tuning(g)["path"] == 0 and ldpc.get_tuning(g)["idle"] == 0


def test_forced_streaming_leaves_an_idle_record_out():
    torch, ldpc, Hd, llr = setup(130)  # three tiles
    g = ldpc.build_graph(Hd)
    flags = ldpc.LDPC_FORCE_STREAM | ldpc.LDPC_NO_EARLY_EXIT
    run = lambda: ldpc.minsum_decode(g, llr, 4, flags=flags)  # noqa: E731
    ref, none = launches(torch, ldpc, run)
    assert none == [4, 0]  # all tiles in one chunk
    for idle, want in ((1, [4, 0]), (0, [12, 0])):  # one tile to a chunk only where the record is in force
        ldpc.set_tuning(g, 2, stream_chunk=1, idle=idle)
        out, counts = launches(torch, ldpc, run)
        assert counts == want, (idle, counts)
        assert all(torch.equal(a, b) for a, b in zip(ref, out))

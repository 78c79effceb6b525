"""Batches around the sizes where the on-chip path changes its launch: one-slot
kernels for few frames, first frames dealt to the workgroups, further ones from
the counters.  Every frame against the streaming path, some against the oracle."""
import numpy as np
import pytest

from paper_2507_10424_amd import workloads as wl
from parity import assert_parity, note, oracle_decode

pytestmark = pytest.mark.gpu


def _codes():
    fam = wl.qc_multi_code_family(seed=7)
    out = {f"qc{k}": (c["H"], c["rate"]) for k, c in enumerate(fam)}
    out["regular96"] = (wl.regular_ldpc(96, 48, 3, 6, seed=1), 0.5)
    out["regular1024"] = (wl.regular_ldpc(1024, 512, 3, 6, seed=2), 0.5)
    # masked columns (no layout), and layouts padded without a degree profile
    out["masked_columns"] = (wl.regular_ldpc(600, 300, 4, 8, seed=3), 0.5)
    out["columns_8"] = (wl.regular_ldpc(240, 180, 6, 8, seed=3), 0.3)
    for k, (dv, dc) in enumerate([(2, 6), (4, 9), (5, 12), (3, 16)]):
        out[f"padded_{dv}_{dc}"] = (wl.regular_ldpc(dc * 36, dv * 36, dv, dc, seed=5 + k), 1 - dv / dc)
    return out


CODES = _codes()


@pytest.mark.parametrize("name", sorted(CODES))
def test_small_batches(name):
    import torch
    from paper_2507_10424_amd import ldpc
    dev = torch.device("cuda:0")
    H, rate = CODES[name]
    g = ldpc.build_graph(torch.from_numpy(np.ascontiguousarray(H)).to(dev))
    C, T = len(g.check_degrees), 12
    rng = np.random.default_rng(3)
    alpha = rng.uniform(0.6, 1.1, size=(T, C)).astype(np.float32)
    beta = rng.uniform(0.0, 0.3, size=(T, C)).astype(np.float32)
    al, be = torch.from_numpy(alpha).to(dev), torch.from_numpy(beta).to(dev)
    cus = torch.cuda.get_device_properties(dev).multi_processor_count
    for B in (1, 2, 3, cus + 1, 4 * cus, 4 * cus + 1, 9 * cus + 5):
        note(f"[small] {name} B={B}")
        llr = wl.bpsk_awgn_llr(None, 1.5 + 5.5 * max(0.0, rate - 0.5), rate, seed=B, n=g.n, batch=B)
        x = torch.from_numpy(llr).to(dev)
        some = slice(max(0, B - 6), B)
        for learned in (False, True):
            def run(flags, out=None):
                if learned:
                    return ldpc.nms_decode(g, x, T, al, be, flags=flags, out=out)
                return ldpc.minsum_decode(g, x, 20, flags=flags, out=out)
            out = ldpc._outputs(B, g.n, dev, True)
            for t, v in zip(out, (7, float("nan"), -7, 9)):
                t.fill_(v)
            run(0, out)
            ref = run(ldpc.LDPC_FORCE_STREAM)
            torch.cuda.synchronize()
            for a, b in zip(out, ref):
                assert torch.equal(a, b), (name, B, learned)
            want = oracle_decode(H, llr[some], T, 0, alpha, beta) if learned else oracle_decode(H, llr[some], 20)
            assert_parity(tuple(t.cpu().numpy()[some] for t in out), want, f"{name} B={B} learned={learned}")


# Smallest and largest n of each kernel for one row and one column degree (a
# multiple of the row degree; 512 threads hold 2, 4 or 6 bits each), and one
# whose threads are not all used.
REGULAR = [(3, 9, 108), (3, 9, 1161), (3, 9, 3069), (3, 12, 108), (3, 12, 1044), (3, 12, 2040), (4, 16, 192),
           (4, 16, 1056), (4, 16, 2032), (4, 8, 104), (4, 8, 1048), (4, 8, 2040), (5, 10, 110), (5, 10, 1030),
           (5, 10, 2040)]


@pytest.mark.parametrize("dv,dc,n", REGULAR)
def test_regular_forms(dv, dc, n):
    """Rows of one degree and columns of one degree: few frames, and more than
    two per resident workgroup (a CU holds at most 32 workgroups)."""
    import torch
    from paper_2507_10424_amd import ldpc
    dev = torch.device("cuda:0")
    H = wl.regular_ldpc(n, n * dv // dc, dv, dc, seed=dv + n)
    g = ldpc.build_graph(torch.from_numpy(np.ascontiguousarray(H)).to(dev))
    T, rate = 9, 1 - dv / dc
    rng = np.random.default_rng(n)
    alpha = rng.uniform(0.6, 1.1, size=(T, 1)).astype(np.float32)
    beta = rng.uniform(0.0, 0.3, size=(T, 1)).astype(np.float32)
    al, be = torch.from_numpy(alpha).to(dev), torch.from_numpy(beta).to(dev)
    cus = torch.cuda.get_device_properties(dev).multi_processor_count
    waves = -(-n // (64 * (6 if dc == 9 else 4)))
    for B in (5, 2 * cus * max(1, 32 // waves) + 700):
        note(f"[regular] ({dv},{dc}) n={n} B={B}")
        llr = wl.bpsk_awgn_llr(None, 2.0 + 5.5 * max(0.0, rate - 0.5), rate, seed=n + B, n=n, batch=B)
        x = torch.from_numpy(llr).to(dev)
        some = slice(B - 4, B)
        for learned in (False, True):
            def run(flags, out=None):
                if learned:
                    return ldpc.nms_decode(g, x, T, al, be, flags=flags, out=out)
                return ldpc.minsum_decode(g, x, 14, flags=flags, out=out)
            out = ldpc._outputs(B, n, dev, True)
            for t, v in zip(out, (7, float("nan"), -7, 9)):
                t.fill_(v)
            run(0, out)
            ref = run(ldpc.LDPC_FORCE_STREAM)
            torch.cuda.synchronize()
            for a, b in zip(out, ref):
                assert torch.equal(a, b), (B, learned)
            want = oracle_decode(H, llr[some], T, 0, alpha, beta) if learned else oracle_decode(H, llr[some], 14)
            assert_parity(tuple(t.cpu().numpy()[some] for t in out), want, f"({dv},{dc}) n={n} B={B} learned={learned}")


def test_regular_forms_leave_forced_paths_and_records_alone():
    """A forced on-chip decode of a graph that no variant of the tuning record
    fits is refused as before, and a record still chooses its own variant."""
    import torch
    from paper_2507_10424_amd import ldpc
    dev = torch.device("cuda:0")
    H = wl.regular_ldpc(1510, 755, 5, 10, seed=1)
    g = ldpc.build_graph(torch.from_numpy(H).to(dev))
    x = torch.from_numpy(wl.bpsk_awgn_llr(None, 2.0, 0.5, seed=1, n=1510, batch=40)).to(dev)
    with pytest.raises(ldpc.LdpcError) as e:
        ldpc.minsum_decode(g, x, 5, flags=ldpc.LDPC_FORCE_ONCHIP)
    assert e.value.name == "LDPC_EUNSUPPORTED"
    want = ldpc.minsum_decode(g, x, 5, flags=ldpc.LDPC_FORCE_STREAM)
    assert all(torch.equal(a, b) for a, b in zip(ldpc.minsum_decode(g, x, 5), want))
    H = wl.regular_ldpc(207, 69, 3, 9, seed=1)
    g = ldpc.build_graph(torch.from_numpy(H).to(dev))
    x = torch.from_numpy(wl.bpsk_awgn_llr(None, 4.0, 2 / 3, seed=1, n=207, batch=40)).to(dev)
    plain = ldpc.minsum_decode(g, x, 9)
    for variant in (26, 27):
        ldpc.set_tuning(g, path=1, variant=variant)
        assert ldpc.get_tuning(g)["variant"] == variant
        assert all(torch.equal(a, b) for a, b in zip(ldpc.minsum_decode(g, x, 9), plain))


@pytest.mark.parametrize("dv,dc,n,B", [(3, 6, 102, 9001), (3, 6, 102, 17003), (3, 9, 108, 5000), (4, 8, 2000, 1025),
                                       (4, 8, 2000, 1300), (2, 5, 400, 4999), (2, 5, 400, 9001), (4, 20, 6000, 900)])
def test_batches_of_a_few_frames_per_workgroup(dv, dc, n, B):
    """Between one and three frames per resident workgroup, where the second
    frames are dealt and the third ones drawn, many of them from counters that
    run out at the same time: every frame is decoded once, as in small batches."""
    import torch
    from paper_2507_10424_amd import ldpc
    dev = torch.device("cuda:0")
    H = wl.regular_ldpc(n, n * dv // dc, dv, dc, seed=3)
    g = ldpc.build_graph(torch.from_numpy(np.ascontiguousarray(H)).to(dev))
    rate = 1 - dv / dc
    note(f"[few] ({dv},{dc}) n={n} B={B}")
    x = torch.from_numpy(wl.bpsk_awgn_llr(None, 2.5 + 5.5 * max(0.0, rate - 0.5), rate, seed=B, n=n, batch=B)).to(dev)
    out = ldpc._outputs(B, n, dev, True)
    for t, v in zip(out, (7, float("nan"), -7, 9)):
        t.fill_(v)
    ldpc.minsum_decode(g, x, 20, out=out)
    for k in range(0, B, 250):
        part = ldpc.minsum_decode(g, x[k:k + 250], 20)
        for a, b in zip(out, part):
            assert torch.equal(a[k:k + 250], b), k

"""GPU: batched uneven blocks (rfi_process_batch) and its HIP graph.

A batch of blocks with different beam counts (all four sums-engine classes
and both eigen solvers), channel counts and sub-interval lengths, some with
offsets, a stream state or preserved channels, must give for every block
exactly what rfi_process_block gives for it alone (same kernels' arithmetic,
bit for bit), and the statistic and mask of the oracle. The graph is replayed
several times with eager work between replays; every replay must reproduce
the eager batch.
"""
import numpy as np
import pytest

from gpu_util import say, upload
from oracle import clip, pipeline

pytestmark = pytest.mark.gpu

# (nbeam, nchan, L, nsub, t0)
SHAPES = [(7, 100, 256, 5, 0), (19, 64, 512, 4, 3), (36, 40, 300, 3, 0), (72, 33, 128, 2, 0),
          (19, 200, 128, 6, 0), (12, 64, 1000, 2, 5), (3, 17, 64, 3, 0)]


@pytest.fixture(scope="module")
def dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2512_16278_amd import rfi
    rfi.lib()
    return torch.device("cuda:0")


def _data(nbeam, nchan, nsamp, seed):
    rng = np.random.default_rng(seed)
    x = 128 + 20 * rng.standard_normal((nbeam, nsamp, nchan))
    t = np.arange(nsamp)
    for j in rng.choice(nchan, size=max(1, nchan // 20), replace=False):
        g = rng.uniform(0.5, 1.5, nbeam)
        x[:, :, j] += 12 * g[:, None] * np.sin(2 * np.pi * t / 31.0 + j)[None, :]
    return np.clip(np.rint(x), 0, 255).astype(np.uint8)


def _outputs(nb, nc, nsub, dev):
    import torch
    n = nsub * nc
    return (torch.full((n,), -1.0, dtype=torch.float64, device=dev),
            torch.full((n,), 0xEE, dtype=torch.uint8, device=dev),
            torch.full((n,), 7, dtype=torch.uint8, device=dev),
            torch.zeros(48, dtype=torch.uint8, device=dev))


def _make(dev):
    import torch
    from paper_2512_16278_amd import rfi
    blocks = []
    for i, (nb, nc, L, nsub, t0) in enumerate(SHAPES):
        x = _data(nb, nc, t0 + nsub * L + 7, 300 + i)
        buf = upload(x, dev)
        prot = None
        if i == 4:
            p = np.zeros(nc, np.uint8)
            p[10:20] = 1
            prot = torch.from_numpy(p).to(dev)
        state = torch.zeros(len(bytes(rfi.rfi_stream_state())), dtype=torch.uint8,
                            device=dev) if i == 1 else None
        blocks.append(dict(x=x, buf=buf, blk=rfi.make_block(buf, nc), nb=nb, nc=nc, L=L,
                           nsub=nsub, t0=t0, protect_chan=prot, state=state))
    return blocks


def _single(b, dev, state=None):
    import torch
    from paper_2512_16278_amd import rfi
    stat, status, mask, out = _outputs(b["nb"], b["nc"], b["nsub"], dev)
    p = rfi.process_params(b["L"], b["nsub"], t0=b["t0"])
    ws = torch.empty(rfi.rfi_process_workspace_size(b["nb"], b["nc"], p), dtype=torch.uint8,
                     device=dev)
    rfi.rfi_process_block(b["blk"], p, stat, status, mask, ws, protect_chan=b["protect_chan"],
                          state=state, out=out)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in (stat, status, mask, out)]


def _batch_items(blocks, dev):
    items = []
    for b in blocks:
        stat, status, mask, out = _outputs(b["nb"], b["nc"], b["nsub"], dev)
        items.append(dict(blk=b["blk"], t0=b["t0"], L=b["L"], nsub=b["nsub"], stat=stat,
                          status=status, mask=mask, out=out, protect_chan=b["protect_chan"],
                          state=b["state"]))
    return items


def test_batch_equals_single_blocks_and_oracle(dev):
    import torch
    from paper_2512_16278_amd import rfi
    blocks = _make(dev)
    ref = []
    for b in blocks:
        st = None
        if b["state"] is not None:
            st = torch.zeros_like(b["state"])
        say("batch: single block", b["nb"], b["nc"], b["L"], b["nsub"])
        ref.append(_single(b, dev, st) + [None if st is None else st.cpu().numpy()])
    items = _batch_items(blocks, dev)
    bt = rfi.Batch(items)
    ws = torch.empty(bt.workspace_size(), dtype=torch.uint8, device=dev)
    say("batch: rfi_process_batch of", len(items))
    bt.run(ws)
    torch.cuda.synchronize()
    for b, it, r in zip(blocks, items, ref):
        got = [it[k].cpu().numpy() for k in ("stat", "status", "mask", "out")]
        for u, v in zip(got, r[:4]):
            assert np.array_equal(u, v), (b["nb"], b["nc"])
        if r[4] is not None:
            assert np.array_equal(b["state"].cpu().numpy(), r[4])
    for b, it in zip(blocks, items):
        cr = pipeline.cells(b["x"], b["L"], b["nsub"], t0=b["t0"])
        ok = pipeline.eligible_cells(cr.degenerate, None if b["protect_chan"] is None
                                     else b["protect_chan"].cpu().numpy())
        res = clip.clip_iterative(cr.stat.ravel(), ok.ravel())
        assert np.abs(it["stat"].cpu().numpy() - cr.stat.ravel()).max() <= 1e-9, b["nb"]
        assert np.array_equal(it["mask"].cpu().numpy().astype(bool), res.mask), b["nb"]


def test_batch_beam_stage(dev):
    """Per-beam outputs in a batch (Sec. 3.3 last paragraph): items with v1
    and a beam mask (per-lane and tridiagonal solver classes, a preserved-
    channel item), items without; each item's v1 and beam mask equal those
    of rfi_process_block for that block alone with the same outputs, bit for
    bit, and so do stat, status and mask; a beam mask without v1 is refused.
    The graph of the batch reproduces them."""
    import torch
    from paper_2512_16278_amd import rfi
    blocks = _make(dev)
    items = _batch_items(blocks, dev)
    for b, it in zip(blocks, items):
        b["state"] = None
        it["state"] = None
    want = [0, 1, 2, 3, 4]                       # 7, 19, 36, 72 beams and a preserved-channel item
    for i in want:
        b = blocks[i]
        n = b["nsub"] * b["nc"]
        items[i]["v1"] = torch.full((b["nb"], n), -9.0, dtype=torch.float32, device=dev)
        items[i]["beam_mask"] = torch.full((b["nb"], n), 7, dtype=torch.uint8, device=dev)
    bt = rfi.Batch(items, kappa_v=1.0)
    ws = torch.empty(bt.workspace_size(), dtype=torch.uint8, device=dev)
    say("batch: beam stage")
    bt.run(ws)
    torch.cuda.synchronize()
    got = {i: (items[i]["v1"].cpu().numpy(), items[i]["beam_mask"].cpu().numpy()) for i in want}
    for i in want:
        b = blocks[i]
        n = b["nsub"] * b["nc"]
        stat, status, mask, out = _outputs(b["nb"], b["nc"], b["nsub"], dev)
        v1 = torch.empty((b["nb"], n), dtype=torch.float32, device=dev)
        bm = torch.empty((b["nb"], n), dtype=torch.uint8, device=dev)
        p = rfi.process_params(b["L"], b["nsub"], t0=b["t0"], kappa_v=1.0, beam_mask=bm)
        pws = torch.empty(rfi.rfi_process_workspace_size(b["nb"], b["nc"], p), dtype=torch.uint8,
                          device=dev)
        rfi.rfi_process_block(b["blk"], p, stat, status, mask, pws,
                              protect_chan=b["protect_chan"], v1=v1, out=out)
        torch.cuda.synchronize()
        assert np.array_equal(got[i][0], v1.cpu().numpy()), b["nb"]
        assert np.array_equal(got[i][1], bm.cpu().numpy()), b["nb"]
        assert np.array_equal(items[i]["mask"].cpu().numpy(), mask.cpu().numpy())
        assert set(np.unique(got[i][1])) <= {0, 1}
    # the graph of the same batch reproduces the beam outputs
    g = bt.graph(ws)
    for i in want:
        items[i]["beam_mask"].fill_(5)
    g.launch()
    torch.cuda.synchronize()
    for i in want:
        assert np.array_equal(items[i]["beam_mask"].cpu().numpy(), got[i][1])
    g.close()
    items[0]["v1"] = None                        # a beam mask without v1
    bad = rfi.Batch(items, kappa_v=1.0)
    assert bad.workspace_size() == 0
    with pytest.raises(rfi.RfiError):
        bad.run(ws)


def test_batch_graph_replays(dev):
    import torch
    from paper_2512_16278_amd import rfi
    blocks = [b for b in _make(dev)]
    for b in blocks:
        b["state"] = None
    items = _batch_items(blocks, dev)
    bt = rfi.Batch(items)
    ws = torch.empty(bt.workspace_size(), dtype=torch.uint8, device=dev)
    bt.run(ws)
    torch.cuda.synchronize()
    eager = [[it[k].cpu().numpy() for k in ("stat", "status", "mask", "out")] for it in items]
    say("batch: graph")
    g = bt.graph(ws)
    for rep in range(3):
        for it in items:                               # eager work between replays
            it["stat"].fill_(-3.0)
            it["mask"].fill_(9)
            it["status"].fill_(0xAB)
        junk = torch.randn(1 << 20, device=dev).sum()
        torch.cuda.synchronize()
        g.launch()
        torch.cuda.synchronize()
        assert float(junk) == float(junk)
        for it, e in zip(items, eager):
            got = [it[k].cpu().numpy() for k in ("stat", "status", "mask", "out")]
            for u, v in zip(got, e):
                assert np.array_equal(u, v), rep
    g.close()


# items whose classes take the packed sums engine, several beam counts to an instance and one long
# item in each, which is cut in time (nbeam, nchan, L, nsub, t0)
PACKED = [(19, 1024, 40, 30, 0), (17, 1000, 33, 20, 2), (16, 64, 1000, 1, 0),
          (36, 500, 64, 11, 0), (39, 333, 50, 12, 1), (37, 64, 3000, 1, 0),
          (68, 200, 90, 12, 0), (71, 100, 70, 30, 5), (70, 40, 900, 2, 0),
          (72, 300, 210, 15, 0), (72, 40, 1000, 1, 3)]


def test_batch_packed_classes(dev):
    """Classes large enough for the packed sums engine: every block as the whole-block call gives
    it alone, bit for bit, eager and in a graph replayed with eager work in between."""
    import torch
    from gpu_util import sums_class
    from paper_2512_16278_amd import rfi
    classes = {}
    for shape in PACKED:
        classes.setdefault(sums_class(shape[0], 1 << 40, 900).key, []).append(shape)
    assert sorted(len(v) for v in classes.values()) == [2, 3, 3, 3]
    for of in classes.values():
        cells, longest = sum(s[1] * s[3] for s in of), max(s[2] for s in of)
        assert all(sums_class(s[0], cells, longest).engine == 2 for s in of)
    blocks = []
    for i, (nb, nc, L, nsub, t0) in enumerate(PACKED):
        buf = upload(_data(nb, nc, t0 + nsub * L, 500 + i), dev)
        blocks.append(dict(buf=buf, blk=rfi.make_block(buf, nc), nb=nb, nc=nc, L=L, nsub=nsub,
                           t0=t0, protect_chan=None, state=None))
    ref = [_single(b, dev) for b in blocks]
    items = _batch_items(blocks, dev)
    bt = rfi.Batch(items)
    ws = torch.empty(bt.workspace_size(), dtype=torch.uint8, device=dev)

    def check(what):
        torch.cuda.synchronize()
        for b, it, r in zip(blocks, items, ref):
            for k, u in zip(("stat", "status", "mask", "out"), r):
                assert np.array_equal(it[k].cpu().numpy(), u), (what, b["nb"], k)
            it["stat"].fill_(-3.0)
            it["mask"].fill_(9)

    say("batch: packed classes")
    ws.fill_(0x5A)                                      # sums that are not zeroed would show
    bt.run(ws)
    check("eager")
    say("batch: packed classes, graph")
    g = bt.graph(ws)
    for rep in range(3):
        junk = torch.randn(1 << 20, device=dev).sum()
        g.launch()
        check(rep)
        assert float(junk) == float(junk)
    g.close()


def test_batch_empty_and_errors(dev):
    import torch
    from paper_2512_16278_amd import rfi
    bt = rfi.Batch([])
    assert bt.workspace_size() > 0
    bt.run(torch.empty(256, dtype=torch.uint8, device=dev))
    b = _make(dev)[0]
    stat, status, mask, out = _outputs(b["nb"], b["nc"], b["nsub"], dev)
    bad = rfi.Batch([dict(blk=b["blk"], L=b["L"], nsub=b["nsub"] + 50, stat=stat, status=status,
                          mask=mask)])
    assert bad.workspace_size() == 0
    with pytest.raises(rfi.RfiError):
        bad.run(torch.empty(256, dtype=torch.uint8, device=dev))


def _run_batch(blocks, dev, tune=None):
    import torch
    from paper_2512_16278_amd import rfi
    items = _batch_items(blocks, dev)
    bt = rfi.Batch(items, tune=tune)
    ws = torch.empty(bt.workspace_size(), dtype=torch.uint8, device=dev)
    bt.run(ws)
    torch.cuda.synchronize()
    return [[it[k].cpu().numpy() for k in ("stat", "status", "mask", "out")] for it in items]


def _table(entries):
    from paper_2512_16278_amd import rfi
    t = rfi.rfi_tune_table()
    t.n = len(entries)
    for i, e in enumerate(entries):
        for k, v in e.items():
            setattr(t.e[i], k, v)
    return t


CLASSES = [(2, 15), (16, 31), (32, 47), (48, 63), (64, 79)]


def test_forced_launch_choices_are_bit_exact(dev):
    """Every sums-engine choice (tile variant, ring depth, XCD group size) and
    every per-lane workgroup size computes the same bits as the defaults."""
    from paper_2512_16278_amd import rfi
    blocks = _make(dev)
    for b in blocks:
        b["state"] = None
    ref = _run_batch(blocks, dev)
    L = rfi.lib()
    for lo, hi in CLASSES:
        nb = next((b["nb"] for b in blocks if lo <= b["nb"] <= hi), None)
        if nb is None:
            continue
        for tile in range(L.rfi_ccm_tile_variants(nb)):
            for stages in (2, 3, 4):
                for gb in (0, 256, 4096):
                    say("forced", lo, hi, "tile", tile, "stages", stages, "group", gb)
                    t = _table([dict(nbeam_lo=lo, nbeam_hi=hi, ccm_tile=tile, ccm_stages=stages,
                                     ccm_group_bytes=gb)])
                    got = _run_batch(blocks, dev, t)
                    for g, r in zip(got, ref):
                        for u, v in zip(g, r):
                            assert np.array_equal(u, v), (lo, tile, stages, gb)
    # per-lane workgroup sizes of the default per-lane solver; the 16-31 class
    # holds 19-beam blocks only (per-lane solvers apply)
    small = [b for b in blocks if b["nb"] <= 20]
    want = [r for b, r in zip(blocks, ref) if b["nb"] <= 20]
    for wg in (64, 128):
        t = _table([dict(nbeam_lo=2, nbeam_hi=15, eig_solver=rfi.RFI_EIG_LANE_TRI, eig_wg=wg),
                    dict(nbeam_lo=16, nbeam_hi=31, eig_solver=rfi.RFI_EIG_LANE_TRI, eig_wg=wg)])
        got = _run_batch(small, dev, t)
        for g, r in zip(got, want):
            for u, v in zip(g, r):
                assert np.array_equal(u, v), wg
    # the Jacobi per-lane solver at two workgroup sizes: the same bits as each
    # other, and within 1e-12 of the default solver's statistic
    jac = []
    for wg in (64, 256):
        t = _table([dict(nbeam_lo=2, nbeam_hi=15, eig_solver=rfi.RFI_EIG_LANE, eig_wg=wg),
                    dict(nbeam_lo=16, nbeam_hi=31, eig_solver=rfi.RFI_EIG_LANE, eig_wg=wg)])
        jac.append(_run_batch(small, dev, t))
    for g0, g1, r in zip(jac[0], jac[1], want):
        for u, v in zip(g0, g1):
            assert np.array_equal(u, v)
        assert np.abs(g0[0] - r[0]).max() <= 1e-12


def test_tuned_batch_matches_oracle_and_graph(dev):
    import torch
    from paper_2512_16278_amd import rfi
    blocks = _make(dev)
    for b in blocks:
        b["state"] = None
    items = _batch_items(blocks, dev)
    bt = rfi.Batch(items)
    ws = torch.empty(bt.workspace_size(), dtype=torch.uint8, device=dev)
    say("tune: rfi_tune_batch")
    table = bt.tune(ws)
    ents = rfi.tune_table_dict(table)
    present = sorted({next(i for i, (lo, hi) in enumerate(CLASSES) if lo <= b["nb"] <= hi)
                      for b in blocks})
    assert [(e["nbeam_lo"], e["nbeam_hi"]) for e in ents] == [CLASSES[i] for i in present]
    for e in ents:
        assert 0 < e["ms_tuned"] <= e["ms_default"] + 1e-9, e
        assert 0 <= e["ccm_tile"] < 3 and e["ccm_stages"] in (0, 2, 3, 4)
        assert e["ccm_group_bytes"] in (0, 256, 512, 2048, 4096, 8192)
        assert e["eig_solver"] in (0, rfi.RFI_EIG_LANE, rfi.RFI_EIG_WAVE, rfi.RFI_EIG_TRIDIAG,
                                   rfi.RFI_EIG_LANE_TRI)
        if e["eig_solver"] in (rfi.RFI_EIG_LANE, rfi.RFI_EIG_LANE_TRI):
            assert e["nbeam_hi"] <= 31 and e["eig_wg"] in (64, 128, 256)
    tuned = rfi.Batch(items, tune=table)
    ws2 = torch.empty(tuned.workspace_size(), dtype=torch.uint8, device=dev)
    tuned.run(ws2)
    torch.cuda.synchronize()
    eager = [[it[k].cpu().numpy() for k in ("stat", "status", "mask", "out")] for it in items]
    for b, it in zip(blocks, items):
        cr = pipeline.cells(b["x"], b["L"], b["nsub"], t0=b["t0"])
        ok = pipeline.eligible_cells(cr.degenerate, None if b["protect_chan"] is None
                                     else b["protect_chan"].cpu().numpy())
        res = clip.clip_iterative(cr.stat.ravel(), ok.ravel())
        assert np.abs(it["stat"].cpu().numpy() - cr.stat.ravel()).max() <= 1e-9, b["nb"]
        assert np.array_equal(it["mask"].cpu().numpy().astype(bool), res.mask), b["nb"]
    g = tuned.graph(ws2)
    for rep in range(2):
        for it in items:
            it["stat"].fill_(-3.0)
            it["mask"].fill_(9)
        torch.cuda.synchronize()
        g.launch()
        torch.cuda.synchronize()
        for it, e in zip(items, eager):
            got = [it[k].cpu().numpy() for k in ("stat", "status", "mask", "out")]
            for u, v in zip(got, e):
                assert np.array_equal(u, v), rep
    g.close()

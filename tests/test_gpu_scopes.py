"""GPU: clip scopes (Sec. 3.3: outliers are masked as a function of frequency
and time) and the histogram Gaussian fit, through rfi_flag_scoped, against the
oracle's clip_scoped on the same statistic.

* moment fit: the combined mask, and every per-channel, per-sub-interval and
  global summary (mu, sigma, thr bit-equal; iterations; nflag) identical;
* histogram fit: the GPU's log() and the oracle's may differ in the last
  place, so mu and sigma agree to 1e-12 relative and the masks are identical
  (no cell lies within 1e-9 of its threshold in these data).
"""
import numpy as np
import pytest

from gpu_util import say
from oracle import clip

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2512_16278_amd import rfi
    rfi.lib()
    return torch.device("cuda:0")


def _stat(rng, K, F):
    s = 0.075 + 0.002 * rng.standard_normal((K, F))
    s[3, :] += 0.01 + 0.02 * rng.uniform(size=F)          # broadband burst
    for j in rng.choice(F, size=max(2, F // 50), replace=False):
        s[:, j] += rng.uniform(0.005, 0.3)                 # persistent channel RFI
    out = rng.choice(K * F, size=K * F // 100, replace=False)
    s.ravel()[out] += rng.uniform(0.003, 0.5, size=out.size)
    return np.clip(s, 1 / 19, 1.0)


def _stats(buf, n):
    from paper_2512_16278_amd import rfi
    raw = buf.cpu().numpy().tobytes()
    return [rfi.flag_stats_from_bytes(raw[48 * i: 48 * (i + 1)]) for i in range(n)]


def _cmp(g, r, exact):
    assert g["iterations"] == r.iterations and bool(g["converged"]) == r.converged
    assert g["nflag"] == r.nflag
    for k in ("mu", "sigma", "thr"):
        a, b = g[k], getattr(r, k)
        if np.isnan(b):
            assert np.isnan(a)
        elif exact:
            assert a == b, k
        else:
            assert abs(a - b) <= 1e-12 * abs(b), (k, a, b)


@pytest.mark.parametrize("fit", ["moments", "histogram"])
@pytest.mark.parametrize("K,F", [(37, 513), (99, 1024)])
def test_scopes_match_oracle(dev, K, F, fit):
    import torch
    from paper_2512_16278_amd import rfi
    rng = np.random.default_rng(K * 7 + F)
    s = _stat(rng, K, F)
    status = np.zeros((K, F), np.uint8)
    status.ravel()[rng.choice(K * F, 20, replace=False)] = rfi.RFI_CELL_DEGENERATE
    prot = (rng.uniform(size=F) < 0.02).astype(np.uint8)
    elig = (status == 0) & ~prot.astype(bool)[None, :]
    st = torch.from_numpy(s.ravel().copy()).to(dev)
    stt = torch.from_numpy(status.ravel().copy()).to(dev)
    pr = torch.from_numpy(prot).to(dev)
    fcode = rfi.RFI_FIT_MOMENTS if fit == "moments" else rfi.RFI_FIT_HISTOGRAM
    for scopes in (2, 4, 6, 7, 1):
        mask = torch.full((K * F,), 9, dtype=torch.uint8, device=dev)
        out = torch.zeros(48, dtype=torch.uint8, device=dev)
        co = torch.zeros(48 * F, dtype=torch.uint8, device=dev)
        so = torch.zeros(48 * K, dtype=torch.uint8, device=dev)
        say("scopes", K, F, fit, scopes)
        rfi.rfi_flag_scoped(K, F, st, stt, mask, scopes=scopes, fit=fcode, protect_chan=pr,
                            out=out, chan_out=co, sub_out=so)
        torch.cuda.synchronize()
        ref = clip.clip_scoped(s, elig, 3.0, 50, scopes, fit)
        m = mask.cpu().numpy().reshape(K, F)
        assert set(np.unique(m)) <= {0, 1}
        assert np.array_equal(m.astype(bool), ref.mask), (scopes, fit)
        exact = fit == "moments"
        if scopes & 1:
            _cmp(_stats(out, 1)[0], ref.glob, exact)
        if scopes & 2:
            for j, g in enumerate(_stats(co, F)):
                _cmp(g, ref.chan[j], exact)
        if scopes & 4:
            for k, g in enumerate(_stats(so, K)):
                _cmp(g, ref.sub[k], exact)
    # the scopes catch what the global clip misses: a moderate burst row and
    # channel-wise outliers are flagged by the union
    ref_g = clip.clip_scoped(s, elig, 3.0, 50, 1, fit).mask
    ref_u = clip.clip_scoped(s, elig, 3.0, 50, 7, fit).mask
    assert ref_u.sum() >= ref_g.sum()


@pytest.mark.parametrize("fit", ["moments", "histogram"])
@pytest.mark.parametrize("K,F", [(4, 5), (128, 9), (129, 64), (512, 31), (513, 33), (5, 512),
                                 (4, 4096), (4, 16384), (4, 16387)])
def test_scopes_segment_lengths(dev, K, F, fit):
    """Segment lengths at the ends of each way of clipping one (128 and 512 cells in registers,
    16384 in LDS, longer ones re-read; the whole block in LDS or over many workgroups), with a
    mask at an odd address, against the oracle; then the histogram clip capped at one fit."""
    import torch
    from paper_2512_16278_amd import rfi
    rng = np.random.default_rng(K * 31 + F)
    s = _stat(rng, K, F)
    status = np.zeros((K, F), np.uint8)
    status.ravel()[rng.choice(K * F, 3, replace=False)] = rfi.RFI_CELL_DEGENERATE
    elig = status == 0
    st = torch.from_numpy(s.ravel().copy()).to(dev)
    stt = torch.from_numpy(status.ravel().copy()).to(dev)
    fcode = rfi.RFI_FIT_MOMENTS if fit == "moments" else rfi.RFI_FIT_HISTOGRAM
    for scopes, max_iter in ((7, 50), (1, 1)):
        mask = torch.full((K * F + 3,), 9, dtype=torch.uint8, device=dev)
        out = torch.zeros(48, dtype=torch.uint8, device=dev)
        co = torch.zeros(48 * F, dtype=torch.uint8, device=dev)
        so = torch.zeros(48 * K, dtype=torch.uint8, device=dev)
        say("segments", K, F, fit, scopes)
        rfi.rfi_flag_scoped(K, F, st, stt, mask[3:], scopes=scopes, fit=fcode, max_iter=max_iter,
                            out=out, chan_out=co, sub_out=so)
        torch.cuda.synchronize()
        ref = clip.clip_scoped(s, elig, 3.0, max_iter, scopes, fit)
        assert (mask[:3] == 9).all()
        assert np.array_equal(mask[3:].cpu().numpy().reshape(K, F).astype(bool), ref.mask)
        exact = fit == "moments"
        _cmp(_stats(out, 1)[0], ref.glob, exact)
        if scopes == 7:
            for j, g in enumerate(_stats(co, F)):
                _cmp(g, ref.chan[j], exact)
            for k, g in enumerate(_stats(so, K)):
                _cmp(g, ref.sub[k], exact)


@pytest.mark.parametrize("fit", ["moments", "histogram"])
@pytest.mark.parametrize("K,F", [(1023, 9), (1024, 9), (1025, 9), (7, 700), (7, 1024), (7, 1025)])
def test_scopes_longest_in_registers(dev, K, F, fit):
    """Segments around the longest that one wavefront holds in registers (1024 cells)."""
    test_scopes_segment_lengths(dev, K, F, fit)


@pytest.mark.parametrize("K,F", [(5, 100), (9, 2048)])
def test_largest_max_iter(dev, K, F):
    """max_iter up to the largest int32: as a cap that the clip does not reach (one launch and
    four, the histogram fit in one workgroup and over many)."""
    import torch
    from paper_2512_16278_amd import rfi
    rng = np.random.default_rng(K + F)
    st = torch.from_numpy(_stat(rng, K, F).ravel().copy()).to(dev)
    stt = torch.zeros(K * F, dtype=torch.uint8, device=dev)

    def clipped(max_iter, fit):
        mask = torch.full((K * F,), 9, dtype=torch.uint8, device=dev)
        out = torch.zeros(48, dtype=torch.uint8, device=dev)
        say("max_iter", K, F, max_iter, fit)
        if fit is None:
            rfi.rfi_flag(K, F, st, stt, mask, max_iter=max_iter, out=out)
        else:
            rfi.rfi_flag_scoped(K, F, st, stt, mask, scopes=1, fit=fit, max_iter=max_iter, out=out)
        torch.cuda.synchronize()
        return mask.cpu().numpy(), _stats(out, 1)[0]

    for fit in (None, rfi.RFI_FIT_MOMENTS, rfi.RFI_FIT_HISTOGRAM):
        m0, s0 = clipped(200, fit)
        assert s0["converged"] and s0["iterations"] < 200 and 0 < m0.sum() < K * F
        for most in (2 ** 31 - 2, 2 ** 31 - 1):
            m1, s1 = clipped(most, fit)
            assert np.array_equal(m0, m1) and s0 == s1, (most, fit)

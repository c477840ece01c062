"""The work that the speed of this library is measured on, through its public entry points.

listed() names the workloads, draw() gives further ones of the same ranges, prepare() builds
what a caller holds before the call (device-resident beams, plans, workspaces, output buffers),
run() is one pass as a caller's program makes it, exact() is the same answer in plain 64-bit
NumPy / PyTorch, and work() the bytes and operations a pass cannot do without.

Data: the seeded synthetic observations of paper_2512_16278_amd.synth (noise, narrow-band and
broadband interference, single-beam pulses), written on the GPU. Shapes: the FAST 19-beam
receiver (4096 channels, 49.152 us samples, sub-intervals of 0.05 s to 10 s), the uneven mix of
7 / 19 / 36 / 72 beams and 1024 / 4096 / 8192 channels, and ragged ones of the same ranges.
"""
from __future__ import annotations

import math
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

from paper_2512_16278_amd import rfi, synth

KAPPA = 3.0
STATS_BYTES = 48          # sizeof(rfi_flag_stats): 3 doubles, 2 int32, 2 int64
LAM, RATIO, ITERMAX = 1e5, 0.05, 100


def listed():
    return [
        # a short stretch of a narrow band: the call a quick look makes, bound by launches
        dict(name="block_tiny", kind="block", nbeam=19, nchan=64, L=1024, nsub=16),
        # ten seconds of the 19-beam receiver at 0.1 s: the survey's block
        dict(name="block_fast", kind="block", nbeam=19, nchan=4096, L=2048, nsub=99),
        # the paper's default 1.00 s sub-intervals with its final product, the per-beam mask,
        # and some preserved channels
        dict(name="block_1s_beams", kind="block", nbeam=19, nchan=4096, L=20345, nsub=10,
             v1=True, beam_mask=True, protect=True),
        # 2.00 s sub-intervals (past the int32 bound of the sums), odd length
        dict(name="block_2s_long", kind="block", nbeam=19, nchan=4096, L=40690, nsub=3),
        # a phased-array feed of 36 beams, ragged channel count, all eigenvalues kept
        dict(name="block_paf36", kind="block", nbeam=36, nchan=1000, L=1024, nsub=39,
             eigvals=True, v1=True, beam_mask=True),
        # a phased-array feed of 72 beams at short sub-intervals
        dict(name="block_paf72", kind="block", nbeam=72, nchan=1024, L=512, nsub=40),
        # FP64 Jacobi: the reference precision, on a part of the band
        dict(name="block_fp64", kind="block", nbeam=19, nchan=1024, L=2048, nsub=10,
             precision=64),
        # uneven blocks of several receivers in one call
        dict(name="batch_uneven", kind="batch", graph=False,
             shapes="7x1024x512x39,19x4096x1024x9,36x1024x4096x4,72x1024x1024x9,19x8192x512x7,"
                    "7x4096x4096x4,36x1024x512x17,72x1024x4096x2"),
        # serving: streams of several receivers, blocks that end inside a sub-interval
        dict(name="serve_mix", kind="serve", slots=8,
             shapes="7x1024x512x24,19x4096x1024x12,36x1024x1024x8,72x1024x1024x6"),
        # an analysis of the shortest sub-intervals (0.05 s): the separate calls, every
        # eigenvalue and vector, clips per channel and per sub-interval
        dict(name="stages_50ms", kind="stages", nbeam=19, nchan=1024, L=1017, nsub=60),
        # bandpass fit and raw-moment statistic of one second at 0.1 s
        dict(name="bandpass_raw", kind="bandpass", nbeam=19, nchan=4096, L=2034, nsub=10),
        # the clip alone on the survey block's statistic, histogram fit, every scope
        dict(name="scopes_hist", kind="scopes", nsub=99, nchan=4096, fit=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _beams(rng):
    return rng.choice([7, 19, 19, 36, 72, rng.randint(4, 20), rng.randint(21, 79)])


def _fit_nsub(rng, nbeam, nchan, L, most_bytes, most_cells):
    top = min(most_bytes // (nbeam * nchan * L), most_cells // nchan, 200)
    return _log(rng, 1, top) if top > 1 else 1


def draw(rng):
    kind = rng.choice(["block", "block", "block", "block", "long", "batch", "serve", "stages",
                       "bandpass", "scopes"])
    if kind == "block":
        nbeam = _beams(rng)
        nchan = _log(rng, 64, 4096)
        L = _log(rng, 512, 20345)
        fp64 = rng.random() < 0.2
        cells = 10240 if fp64 else (40960 if nbeam > 20 else 400000)
        v1 = rng.random() < 0.3
        return dict(kind="block", nbeam=nbeam, nchan=min(nchan, cells), L=L,
                    nsub=_fit_nsub(rng, nbeam, nchan, L, 4 << 30, cells),
                    v1=v1, beam_mask=v1 and rng.random() < 0.7, eigvals=rng.random() < 0.2,
                    protect=rng.random() < 0.3, precision=64 if fp64 else 32)
    if kind == "long":
        nbeam, nchan, L = rng.choice([7, 19, 36]), _log(rng, 256, 4096), _log(rng, 33026, 203450)
        return dict(kind="block", nbeam=nbeam, nchan=nchan, L=L,
                    nsub=_fit_nsub(rng, nbeam, nchan, L, 8 << 30, 8192))
    if kind in ("batch", "serve"):
        shapes = []
        for _ in range(rng.randint(3, 8 if kind == "batch" else 4)):
            nbeam, nchan, L = _beams(rng), _log(rng, 256, 4096), _log(rng, 512, 4096)
            nsub = max(2, _fit_nsub(rng, nbeam, nchan, L, 1 << 30, 9216 if nbeam > 20 else 40960))
            shapes.append("%dx%dx%dx%d" % (nbeam, nchan, L, nsub))
        more = dict(graph=rng.random() < 0.5) if kind == "batch" else dict(slots=rng.choice([1, 8]))
        return dict(kind=kind, shapes=",".join(shapes), **more)
    if kind in ("stages", "bandpass"):
        nbeam, nchan, L = rng.choice([7, 13, 19]), _log(rng, 256, 4096), _log(rng, 1017, 8138)
        return dict(kind=kind, nbeam=nbeam, nchan=nchan, L=L,
                    nsub=_fit_nsub(rng, nbeam, nchan, L, 3 << 30,
                                   65536 if kind == "stages" else 40960))
    return dict(kind="scopes", nsub=_log(rng, 8, 99), nchan=_log(rng, 64, 4096),
                fit=rng.randint(0, 1))


# --- inputs --------------------------------------------------------------------------------

def _shapes(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["shapes"].split(",")]


def _observe(seed, nbeam, nchan, nsamp, L):
    """(storage, per-beam device tensors) of a seeded observation of nsamp samples, the beams
    placed as rfi.alloc_beams places them."""
    spec = synth.mixed_spec(seed, nbeam, nchan, L, (nsamp + 0.5) * synth.TSAMP)
    assert spec.nsamp == nsamp
    raw, beams = rfi.alloc_beams(nbeam, nsamp, (nchan + 15) // 16 * 16)
    ds = rfi.DeviceSynth(spec)
    for b in range(nbeam):
        ds.fill(beams[b], b)
    torch.cuda.synchronize()
    return raw, beams


def _protect(seed, nchan):
    p = np.zeros(nchan, dtype=np.uint8)
    p[np.random.default_rng(seed + 5).choice(nchan, size=max(1, nchan // 50), replace=False)] = 1
    return p


def _dev(n, dtype):
    return torch.empty(n, dtype=dtype, device="cuda")


def _cell_outputs(ncell):
    return dict(stat=_dev(ncell, torch.float64), status=_dev(ncell, torch.uint8),
                mask=_dev(ncell, torch.uint8))


def _statistic(seed, nsub, nchan):
    """A 19-beam block's statistic as the clip meets it: a narrow skewed bulk, channels of
    persistent interference, one sub-interval with a broadband burst."""
    g = torch.Generator(device="cuda").manual_seed(seed)

    def u(*n):
        return torch.rand(n, generator=g, device="cuda", dtype=torch.float64)

    s = 0.0625 + 0.0022 * torch.randn((nsub, nchan), generator=g, device="cuda",
                                      dtype=torch.float64).abs() + 0.002 * u(nsub, nchan)
    hot = u(nchan) < 0.02
    s[:, hot] += 0.4 * u(nsub, int(hot.sum())) * u(int(hot.sum()))
    s[int(u(1) * nsub)] += 0.3 * u(nchan)
    return s.reshape(-1)


class _Serving:
    """A session with one open stream per shape; closed with its owner."""

    def __init__(self, shapes, slots):
        self.session = rfi.Session(max_inflight=slots)
        self.sids = [self.session.open_stream(nb, F, L, kappa=KAPPA) for nb, F, L, _ in shapes]

    def __del__(self):
        self.session.close()


def _cut(L, nsub):
    """Samples of the first of a stream's two blocks: it ends inside a sub-interval."""
    return L * (nsub // 2) + L // 3


def prepare(case, seed):
    kind = case["kind"]
    if kind == "scopes":
        nsub, nchan = case["nsub"], case["nchan"]
        ncell = nsub * nchan
        return dict(case=case, stat=_statistic(seed, nsub, nchan),
                    status=torch.zeros(ncell, dtype=torch.uint8, device="cuda"),
                    mask=_dev(ncell, torch.uint8),
                    out=_dev((1, STATS_BYTES), torch.uint8),
                    chan=_dev((nchan, STATS_BYTES), torch.uint8),
                    sub=_dev((nsub, STATS_BYTES), torch.uint8),
                    ws=rfi.flag_workspace(nsub, nchan))
    if kind == "batch":
        items, keep = [], []
        for i, (nb, F, L, nsub) in enumerate(_shapes(case)):
            raw, beams = _observe(seed + 101 * i, nb, F, L * nsub, L)
            keep.append((raw, beams))
            items.append(dict(blk=rfi.make_block(beams, F), L=L, nsub=nsub,
                              out=_dev((1, STATS_BYTES), torch.uint8), **_cell_outputs(nsub * F)))
        batch = rfi.Batch(items, kappa=KAPPA)
        ws = _dev(batch.workspace_size(), torch.uint8)
        return dict(case=case, items=items, keep=keep, batch=batch, ws=ws,
                    graph=batch.graph(ws) if case["graph"] else None)
    if kind == "serve":
        shapes = _shapes(case)
        blocks, keep = [], []
        for i, (nb, F, L, nsub) in enumerate(shapes):
            raw, beams = _observe(seed + 101 * i, nb, F, L * nsub, L)
            keep.append((raw, beams))
            n1 = _cut(L, nsub)
            blocks.append((rfi.make_block([b[:n1] for b in beams], F),
                           rfi.make_block([b[n1:] for b in beams], F)))
        return dict(case=case, serving=_Serving(shapes, case["slots"]), blocks=blocks, keep=keep)
    nb, F, L, nsub = case["nbeam"], case["nchan"], case["L"], case["nsub"]
    ncell = nsub * F
    raw, beams = _observe(seed, nb, F, L * nsub, L)
    st = dict(case=case, keep=(raw, beams), blk=rfi.make_block(beams, F),
              out=_dev((1, STATS_BYTES), torch.uint8), **_cell_outputs(ncell))
    if kind == "block":
        st["v1"] = _dev((nb, ncell), torch.float32) if case.get("v1") else None
        st["eigvals"] = _dev((nb, ncell), torch.float32) if case.get("eigvals") else None
        st["beam_mask"] = _dev((nb, ncell), torch.uint8) if case.get("beam_mask") else None
        st["protect"] = (torch.from_numpy(_protect(seed, F)).cuda() if case.get("protect")
                         else None)
        st["p"] = rfi.process_params(L, nsub, kappa=KAPPA, beam_mask=st["beam_mask"],
                                     eig_precision=case.get("precision", 32))
        st["ws"] = _dev(rfi.rfi_process_workspace_size(nb, F, st["p"]), torch.uint8)
        return st
    st["sum_x"] = _dev((nb, ncell), torch.int32)
    st["sum_xy"] = _dev((nb * (nb + 1) // 2, ncell), torch.int32)
    st["count"] = _dev(nsub, torch.int32)
    st["ws"] = rfi.flag_workspace(nsub, F)
    if kind == "stages":
        st["v1"], st["eigvals"] = _dev((nb, ncell), torch.float32), _dev((nb, ncell), torch.float32)
        st["chan"] = _dev((F, STATS_BYTES), torch.uint8)
        st["sub"] = _dev((nsub, STATS_BYTES), torch.uint8)
    else:
        st["z"] = _dev((nb, ncell), torch.float64)
        st["passes"] = _dev((nsub, nb), torch.int32)
        st["bws"] = _dev(rfi.rfi_bandpass_workspace_size(nb, F, nsub), torch.uint8)
    return st


# --- one pass ------------------------------------------------------------------------------

def _fit(buf):
    """The fits (mu, sigma, thr) and the counts of rfi_flag_stats records."""
    return dict(fit=buf.view(torch.float64)[:, :3], counts=buf.view(torch.int64)[:, 3:6])


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "block":
        rfi.rfi_process_block(st["blk"], st["p"], st["stat"], st["status"], st["mask"], st["ws"],
                              protect_chan=st["protect"], eigvals=st["eigvals"], v1=st["v1"],
                              out=st["out"])
        return dict(stat=st["stat"], status=st["status"], mask=st["mask"], v1=st["v1"],
                    eigvals=st["eigvals"], beam_mask=st["beam_mask"], **_fit(st["out"]))
    if kind == "batch":
        if st["graph"] is not None:
            st["graph"].launch()
        else:
            st["batch"].run(st["ws"])
        return [dict(stat=it["stat"], status=it["status"], mask=it["mask"], **_fit(it["out"]))
                for it in st["items"]]
    if kind == "serve":
        sv = st["serving"]
        tickets = [sv.session.submit(sid, pair[half]) for half in (0, 1)
                   for sid, pair in zip(sv.sids, st["blocks"])]
        got = []
        for t in tickets:
            r = sv.session.wait(t)
            if r.status != rfi.RFI_OK:
                raise RuntimeError("block failed (%d)" % r.status)
            stat, status, mask = rfi.result_arrays(sv.session, r)
            got.append(dict(stat=stat, status=status, mask=mask,
                            fit=np.array([r.flag.mu, r.flag.sigma, r.flag.thr]),
                            counts=np.array([r.flag.iterations, r.flag.nflag, r.flag.nfit])))
            sv.session.release(t)
        return got
    if kind == "scopes":
        rfi.rfi_flag_scoped(case["nsub"], case["nchan"], st["stat"], st["status"], st["mask"],
                            scopes=7, fit=case["fit"], kappa=KAPPA, out=st["out"],
                            chan_out=st["chan"], sub_out=st["sub"], workspace=st["ws"])
        return dict(mask=st["mask"], all=_fit(st["out"]), chan=_fit(st["chan"]),
                    sub=_fit(st["sub"]))
    nb, F, L, nsub = case["nbeam"], case["nchan"], case["L"], case["nsub"]
    rfi.rfi_ccm_accumulate(st["blk"], 0, L, nsub, st["sum_x"], st["sum_xy"], st["count"])
    if kind == "stages":
        rfi.rfi_eig_batched(nb, nsub, F, st["sum_x"], st["sum_xy"], st["count"], st["stat"],
                            st["status"], eigvals=st["eigvals"], v1=st["v1"])
        rfi.rfi_flag_scoped(nsub, F, st["stat"], st["status"], st["mask"], scopes=7, kappa=KAPPA,
                            out=st["out"], chan_out=st["chan"], sub_out=st["sub"],
                            workspace=st["ws"])
        return dict(sum_x=st["sum_x"], sum_xy=st["sum_xy"], stat=st["stat"], status=st["status"],
                    mask=st["mask"], eigvals=st["eigvals"], v1=st["v1"], all=_fit(st["out"]),
                    chan=_fit(st["chan"]), sub=_fit(st["sub"]))
    rfi.rfi_bandpass_arpls(nb, nsub, F, st["sum_x"], st["count"], st["z"], workspace=st["bws"],
                           passes=st["passes"], lam=LAM, ratio=RATIO, itermax=ITERMAX)
    rfi.rfi_eig_noncentred(nb, nsub, F, st["sum_x"], st["sum_xy"], st["count"], st["z"],
                           st["stat"], st["status"])
    rfi.rfi_flag(nsub, F, st["stat"], st["status"], st["mask"], kappa=KAPPA, out=st["out"],
                 workspace=st["ws"])
    return dict(z=st["z"], passes=st["passes"], stat=st["stat"], status=st["status"],
                mask=st["mask"], **_fit(st["out"]))


# --- the same in 64 bits -------------------------------------------------------------------

def _sums64(beams, nchan, L, nsub):
    """Exact sums S [nsub, nchan, n] and S2 [nsub, nchan, n, n] in FP64."""
    n = len(beams)
    S = np.empty((nsub, nchan, n))
    S2 = np.empty((nsub, nchan, n, n))
    step = max(1, (2 << 30) // (8 * n * nchan))
    for k in range(nsub):
        s = torch.zeros((nchan, n), dtype=torch.float64, device="cuda")
        s2 = torch.zeros((nchan, n, n), dtype=torch.float64, device="cuda")
        for t in range(k * L, (k + 1) * L, step):
            e = min(t + step, (k + 1) * L)
            x = torch.stack([b[t:e, :nchan] for b in beams])        # [n, T, F]
            x = x.permute(2, 0, 1).to(torch.float64).contiguous()   # [F, n, T]
            s += x.sum(dim=2)
            s2 += torch.bmm(x, x.transpose(1, 2).contiguous())
        S[k], S2[k] = s.cpu().numpy(), s2.cpu().numpy()
    return S, S2


def _pearson(S, S2, L):
    N = L * S2 - S[..., :, None] * S[..., None, :]
    d = np.sqrt(np.einsum("...ii->...i", N))
    r = N / (d[..., :, None] * d[..., None, :])
    i = np.arange(r.shape[-1])
    r[..., i, i] = 1.0
    return r


def _spread(fn, a, parts=32):
    with ThreadPoolExecutor(16) as pool:
        return list(pool.map(fn, np.array_split(a, min(parts, len(a)))))


def _eigen(r, vectors):
    """(statistic, eigenvalues by falling magnitude, dominant vectors or None) of [cells, n, n]."""
    if vectors:
        got = _spread(np.linalg.eigh, r)
        w = np.concatenate([g[0] for g in got])
        v = np.concatenate([g[1] for g in got])
    else:
        w, v = np.concatenate(_spread(np.linalg.eigvalsh, r)), None
    order = np.argsort(-np.abs(w), axis=1, kind="stable")
    w = np.take_along_axis(w, order, axis=1)
    stat = w[:, 0] ** 2 / np.einsum("cij,cij->c", r, r)
    if v is not None:
        v = np.take_along_axis(v, order[:, None, :1], axis=2)[:, :, 0]
        v = v * np.where(v.sum(axis=1) < 0, -1.0, 1.0)[:, None]
    return stat, w, v


def _hist_fit(x, mu, sg):
    if len(x) < 8 or not sg > 0:
        return mu, sg
    f = np.floor((x - (mu - 4 * sg)) / (sg / 8))
    c = np.bincount(f[(f >= 0) & (f < 64)].astype(int), minlength=64).astype(float)
    use = c > 0
    if use.sum() < 3:
        return mu, sg
    z = (np.arange(64) + 0.5) / 8 - 4
    z, c = z[use], c[use]
    A = np.stack([np.ones_like(z), z, z * z], axis=1)
    wt = c * c
    _, b, c2 = np.linalg.solve(A.T @ (wt[:, None] * A), A.T @ (wt * np.log(c)))
    if not c2 < 0:
        return mu, sg
    return mu - b / (2 * c2) * sg, math.sqrt(-1 / (2 * c2)) * sg


def _clip(x, fit=0, before=()):
    """(mu, sigma, thr) of the last fit and the cells left, clipping x (pooled with the values
    `before`) at mu + KAPPA sigma until nothing new is masked."""
    live, mu, sg, thr, T = x, math.nan, math.nan, math.nan, math.inf
    for _ in range(50):
        if len(live) + len(before) == 0:
            break
        pool = np.concatenate([live, *before]) if len(before) else live
        mu = pool.mean()
        sg = math.sqrt(((pool - mu) ** 2).mean())
        if fit:
            mu, sg = _hist_fit(pool, mu, sg)
        thr = mu + KAPPA * sg
        T = min(T, thr)
        kept = live[live <= T]
        if len(kept) == len(live):
            break
        live = kept
    return np.array([mu, sg, thr]), live


def _clips(stat, nsub, nchan, fit):
    s = stat.reshape(nsub, nchan)
    return dict(all=dict(fit=_clip(stat, fit)[0][None]),
                chan=dict(fit=np.stack([_clip(s[:, j], fit)[0] for j in range(nchan)])),
                sub=dict(fit=np.stack([_clip(s[k], fit)[0] for k in range(nsub)])))


def _solve_penta(w, y, lam):
    """(diag(w) + lam D'D) z = w y for the rows of w and y, in extended precision."""
    n, F = y.shape
    d0, d1, d2 = (np.zeros(F, np.longdouble) for _ in range(3))
    for r in range(F - 2):
        d0[r:r + 3] += (1, 4, 1)
        d1[r:r + 2] += (-2, -2)
        d2[r] += 1
    a = w + lam * d0
    l1, l2, D, u = (np.zeros((F, n), np.longdouble) for _ in range(4))
    for j in range(F):
        D[j] = a[:, j]
        u[j] = w[:, j] * y[:, j]
        if j >= 1:
            e = lam * d1[j - 1]
            if j >= 2:
                e = e - l1[j - 2] * D[j - 2] * l2[j - 2]
            l1[j - 1] = e / D[j - 1]
            D[j] -= l1[j - 1] ** 2 * D[j - 1]
            u[j] -= l1[j - 1] * u[j - 1]
        if j >= 2:
            D[j] -= l2[j - 2] ** 2 * D[j - 2]
            u[j] -= l2[j - 2] * u[j - 2]
        if j + 2 < F:
            l2[j] = lam * d2[j] / D[j]
    z = np.zeros((F + 2, n), np.longdouble)
    for j in range(F - 1, -1, -1):
        z[j] = u[j] / D[j] - l1[j] * z[j + 1] - l2[j] * z[j + 2]
    return z[:F].T


def _arpls(y):
    z = np.array(y)
    w = np.ones_like(y)
    todo = np.arange(len(y))
    for _ in range(ITERMAX):
        zt = _solve_penta(w[todo], y[todo], LAM)
        z[todo] = zt
        keep = []
        for i, s in enumerate(todo):
            d = y[s] - zt[i]
            neg = d[d < 0]
            if len(neg) < 2:
                continue
            m, sd = neg.mean(), neg.std(ddof=1)
            if not sd > 0:
                continue
            wt = 1 / (1 + np.exp(2 * (d - (2 * sd - m)) / sd))
            if np.linalg.norm(w[s] - wt) / np.linalg.norm(w[s]) >= RATIO:
                w[s] = wt
                keep.append(s)
        todo = np.array(keep, dtype=int)
        if not len(todo):
            break
    return z


def exact(case, seed):
    kind = case["kind"]
    if kind == "scopes":
        stat = _statistic(seed, case["nsub"], case["nchan"]).cpu().numpy()
        return dict(mask=None, **_clips(stat, case["nsub"], case["nchan"], case["fit"]))
    if kind in ("batch", "serve"):
        got, halves = [], ([], [])
        for i, (nb, F, L, nsub) in enumerate(_shapes(case)):
            raw, beams = _observe(seed + 101 * i, nb, F, L * nsub, L)
            stat = _eigen(_pearson(*_sums64(beams, F, L, nsub), L).reshape(-1, nb, nb), False)[0]
            del raw, beams
            if kind == "batch":
                got.append(dict(stat=stat, fit=_clip(stat)[0][None]))
                continue
            before = []
            n1 = _cut(L, nsub) // L * F
            for half, s in zip(halves, (stat[:n1], stat[n1:])):
                fit, left = _clip(s, before=before)
                before.append(left)
                half.append(dict(stat=s, fit=fit))
        return got or halves[0] + halves[1]
    nb, F, L, nsub = case["nbeam"], case["nchan"], case["L"], case["nsub"]
    raw, beams = _observe(seed, nb, F, L * nsub, L)
    S, S2 = _sums64(beams, F, L, nsub)
    del raw, beams
    if kind == "bandpass":
        y = (S / L).transpose(2, 0, 1).astype(np.longdouble)                 # [n, nsub, F]
        z = _arpls(y.reshape(nb * nsub, F)).reshape(nb, nsub, F)
        zc = z.transpose(1, 2, 0)
        M = (S2 - zc[..., None, :] * S[..., :, None] - zc[..., :, None] * S[..., None, :] +
             L * zc[..., :, None] * zc[..., None, :]) / L
        stat = _eigen(M.astype(np.float64).reshape(-1, nb, nb), False)[0]
        return dict(z=z.astype(np.float64).reshape(nb, -1), stat=stat, fit=_clip(stat)[0][None])
    vectors = kind == "stages" or bool(case.get("v1"))
    stat, w, v = _eigen(_pearson(S, S2, L).reshape(-1, nb, nb), vectors)
    if kind == "stages":
        return dict(stat=stat, eigvals=np.ascontiguousarray(w.T), v1=np.ascontiguousarray(v.T),
                    **_clips(stat, nsub, F, 0))
    live = stat
    if case.get("protect"):
        live = stat.reshape(nsub, F)[:, _protect(seed, F) == 0].reshape(-1)
    return dict(stat=stat, v1=np.ascontiguousarray(v.T) if case.get("v1") else None,
                eigvals=np.ascontiguousarray(w.T) if case.get("eigvals") else None,
                fit=_clip(live)[0][None])


# --- what a pass cannot do without ------------------------------------------------------------

def _cell_work(n, cells, L):
    """Bytes and operations of `cells` cells: the samples read once, statistic, status and mask
    written; a multiply and an add per pair and sample, and the eigenvalue reduction."""
    return n * L * cells + 10 * cells, (n * (n + 1) * L + 4 * n ** 3 // 3) * cells


def work(case):
    kind = case["kind"]
    if kind == "scopes":
        n = case["nsub"] * case["nchan"]
        return dict(bytes=10 * n, flops=6 * n)
    if kind in ("batch", "serve"):
        per = [_cell_work(nb, F * nsub, L) for nb, F, L, nsub in _shapes(case)]
        return dict(bytes=sum(b for b, _ in per), flops=sum(f for _, f in per))
    nb, cells = case["nbeam"], case["nchan"] * case["nsub"]
    b, f = _cell_work(nb, cells, case["L"])
    if kind == "stages":
        b += (nb + nb * (nb + 1) // 2) * 4 * cells + 8 * nb * cells
    elif kind == "bandpass":
        b += 8 * nb * cells
    else:
        b += (4 * bool(case.get("v1")) + 4 * bool(case.get("eigvals")) +
              bool(case.get("beam_mask"))) * nb * cells
    return dict(bytes=b, flops=f)

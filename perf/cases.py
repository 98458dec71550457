"""The work that performance is measured on: calls through the package's public entry points,
from one small dedispersion and search to the whole survey, with the options, odd sizes and
input paths (resident, batched, decimated ranges, streamed from pinned host memory) that a
user's program has.

Inputs are seeded synthetic filterbanks as the package's own workloads have them: N(128, 16)
noise in uint8 with dispersed pulses. Sizes are those of the tiny (128 channels x 32768
samples), streamed (128 channels in 2^18-sample chunks), survey (4096 channels x 2^20
samples, 3000 trials), batched (1024 to 4096 channels, uneven) and serving (2^17-sample
chunks) workloads, and odd ones between them.
"""

import numpy as np
import torch

import paper_2101_00941_amd as aa

K_DM = 4.148808e3
TSAMP = 64e-6
POW2_32 = "1,2,4,8,16,32"
POW2_256 = "1,2,4,8,16,32,64,128,256"
ODD_WIDTHS = "1,3,5,9,17,33,100"

# bands: (centre of the highest channel, total bandwidth) in MHz
BANDS = {"tiny": (1500.0, 100.0), "survey": (1450.0, 300.0)}


def listed():
    return [
        # the smallest whole search: latency and launches count
        dict(name="tiny_search", kind="search", band="tiny", nchan=128, nsamp=32768, dms="uniform", ndm=100,
             widths=POW2_32, tune=False, best=False, block=32768),
        # one chunk of the 128-channel stream, resident, on a plan tuned for it
        dict(name="chunk_128ch_tuned", kind="search", band="tiny", nchan=128, nsamp=(1 << 18) + 3072, dms="uniform",
             ndm=100, widths=POW2_32, tune=True, best=False, block=32768),
        # odd everything: channels, samples, trials, widths, a small stat block, and the best-S/N plane
        dict(name="ragged_best", kind="search", band="survey", nchan=1001, nsamp=77777, dms="uniform", ndm=333,
             widths=ODD_WIDTHS, tune=False, best=True, block=4096),
        # a serving request: one 2^17-sample chunk of a 4096-channel beam and its delay tail
        dict(name="serving_chunk", kind="search", band="survey", nchan=4096, nsamp=(1 << 17) + 16384, dms="doubling",
             ndm=1500, widths=POW2_256, tune=False, best=False, block=32768),
        # the survey: the whole resident signal, every trial
        dict(name="survey", kind="search", band="survey", nchan=4096, nsamp=1 << 20, dms="doubling", ndm=3000,
             widths=POW2_256, tune=False, best=False, block=32768),
        # a quarter of the survey with per-range time decimation
        dict(name="ranges", kind="ranges", band="survey", nchan=4096, nsamp=1 << 18, dms="doubling", ndm=3000,
             widths=POW2_256, block=32768),
        # uneven beams in one persistent launch
        dict(name="batch", kind="batch", band="survey", nbeams=5, nchan=2048, nsamp=200000, dms="doubling", ndm=1200,
             widths=POW2_256, block=32768),
        # the search alone over a plane that is already there
        dict(name="plane_search", kind="plane", nchan=4096, n_dd=225000, ndm=3000, widths=POW2_256, clip=False,
             noalloc=False, block=32768),
        # the search with outlier-clipped statistics and the boxcar hierarchy
        dict(name="plane_robust", kind="plane", nchan=1024, n_dd=100003, ndm=1000, widths=POW2_256, clip=True,
             noalloc=False, block=8192),
        # the allocation-free search of a tight serving loop
        dict(name="noalloc_search", kind="plane", nchan=128, n_dd=32000, ndm=100, widths=POW2_32, clip=False,
             noalloc=True, block=32768),
        # one halving of a quarter of the survey's input
        dict(name="decimate", kind="decimate", nchan=4096, nsamp=(1 << 18) + 4),
        # host data streamed in 2^18-sample chunks through the pipeline
        dict(name="stream_128ch", kind="stream", band="tiny", nchan=128, chunk=1 << 18, nchunks=4, nstreams=2,
             dms="uniform", ndm=100, widths=POW2_32, block=32768),
    ]


def _logint(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "search", "ranges", "batch", "plane", "plane", "decimate", "stream"])
    if kind == "search":
        band = rng.choice(["tiny", "survey", "survey"])
        nchan = _logint(rng, 64, 4096)
        ndm = _logint(rng, 20, 3000)
        dms = rng.choice(["uniform", "doubling"])
        widths = rng.choice([POW2_32, POW2_256, ODD_WIDTHS])
        nsamp = _logint(rng, 4096, 1 << 18) + _span(band, nchan, dms, ndm) + 1100
        # at most an eighth of the survey's work, and of the time its inputs take to make
        while nchan * ndm * nsamp > 4096 * 3000 * (1 << 17):
            ndm = max(20, ndm // 2)
        return dict(kind=kind, band=band, nchan=nchan, nsamp=nsamp, dms=dms, ndm=ndm, widths=widths,
                    tune=nchan * ndm <= 60000 and rng.random() < 0.4, best=rng.random() < 0.25,
                    block=rng.choice([4096, 32768]))
    if kind == "ranges":
        return dict(kind=kind, band="survey", nchan=rng.choice([512, 1024, 2048, 4096]),
                    nsamp=rng.randint(1 << 17, 1 << 18), dms="doubling", ndm=rng.randint(1100, 3000), widths=POW2_256,
                    block=32768)
    if kind == "batch":
        return dict(kind=kind, band="survey", nbeams=rng.randint(2, 8), nchan=rng.choice([512, 1024, 2048]),
                    nsamp=rng.randint(70000, 200000), dms="doubling", ndm=rng.randint(200, 1200), widths=POW2_256,
                    block=32768)
    if kind == "plane":
        noalloc = rng.random() < 0.4
        return dict(kind=kind, nchan=rng.choice([128, 1024, 4096]),
                    n_dd=_logint(rng, 2000, 60000 if noalloc else 200000), ndm=_logint(rng, 16, 1000 if noalloc else 3000),
                    widths=rng.choice([POW2_32, POW2_256, ODD_WIDTHS]), clip=rng.random() < 0.4, noalloc=noalloc,
                    block=rng.choice([4096, 32768]))
    if kind == "decimate":
        return dict(kind=kind, nchan=_logint(rng, 64, 4096), nsamp=_logint(rng, 1 << 14, 1 << 18) + rng.randint(0, 15))
    return dict(kind="stream", band="tiny", nchan=rng.choice([64, 128, 256]), chunk=32768 * rng.randint(2, 8),
                nchunks=rng.randint(2, 4), nstreams=rng.choice([1, 2, 4]), dms="uniform", ndm=rng.randint(50, 150),
                widths=POW2_32, block=32768)


# ---- descriptions ------------------------------------------------------------------


def _widths(case):
    return [int(w) for w in case["widths"].split(",")]


def _dms(kind, n):
    """n ascending trials: DM 0, 1, 2, ... or the survey's plan, whose step doubles from range to range."""
    if kind == "uniform":
        return np.arange(n, dtype=np.float64)
    out, start = [], 0.0
    for step, count in ((1 / 16, 512), (1 / 8, 512), (1 / 4, 512), (1 / 2, 512), (1.0, 384), (2.0, 1 << 20)):
        take = min(count, n - len(out))
        out += [start + step * i for i in range(take)]
        start += step * count
        if len(out) == n:
            break
    return np.asarray(out, dtype=np.float64)


def _shifts(band, nchan, dm):
    """Delay in samples of every channel against the top one, for one trial (float64, rounded half up)."""
    f_top, width = BANDS[band]
    f = f_top - np.arange(nchan, dtype=np.float64) * (width / nchan)
    inv = 1.0 / (f * f) - 1.0 / (f_top * f_top)
    return np.floor((K_DM * dm) * inv / TSAMP + 0.5).astype(np.int64)


def _span(band, nchan, dms, ndm):
    return int(_shifts(band, nchan, float(_dms(dms, ndm)[-1]))[-1])


def _plan_args(case, nchan=None, nsamp=None, ndm=None):
    nchan = nchan or case["nchan"]
    f_top, width = BANDS[case["band"]]
    return (nchan, nsamp or case["nsamp"], f_top, width / nchan, TSAMP, _dms(case["dms"], ndm or case["ndm"]),
            _widths(case), 6.0, case["block"])


def _filterbank(band, nchan, nsamp, dm_max, seed, pitch):
    """uint8 [nchan, pitch] on the GPU: N(128, 16) noise and six dispersed pulses per 2^18 samples."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.zeros((nchan, pitch), dtype=torch.uint8, device="cuda")
    rows = max(1, (1 << 28) // nsamp)
    for r in range(0, nchan, rows):
        n = min(rows, nchan - r)
        v = torch.randn((n, nsamp), generator=g, device="cuda", dtype=torch.float16)
        x[r:r + n, :nsamp] = v.mul_(16).add_(128).round_().clamp_(0, 255).to(torch.uint8)
    rng = np.random.default_rng(seed)
    c = torch.arange(nchan, device="cuda")[:, None]
    for _ in range(max(2, 6 * nsamp >> 18)):
        s = torch.from_numpy(_shifts(band, nchan, rng.uniform(0.05, 0.75) * max(dm_max, 1.0))).cuda()
        w = int(rng.integers(1, 17))
        t0 = int(rng.integers(0, max(1, nsamp - int(s[-1]) - w - 64)))
        i = (t0 + s)[:, None] + torch.arange(w, device="cuda")[None, :]
        i = i.clamp_(max=nsamp - 1)
        x[c, i] = (x[c, i].to(torch.int16) + int(rng.integers(4, 16))).clamp_(max=255).to(torch.uint8)
    return x


def _pitch(n):
    return (n + 255) // 256 * 256


# rows of a candidate table on the host
BATCH_CAP, STREAM_CAP = 1 << 14, 1 << 12


def _table(c, rows):
    """A candidate list in a table of `rows` entries, as bytes."""
    out = np.zeros(rows, dtype=c.dtype)
    out[:len(c)] = c[:rows]
    return out.view(np.uint8)


def _cand(cap):
    return torch.zeros(cap * 24, dtype=torch.uint8, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")


# ---- what a user's program has in hand -----------------------------------------------


def prepare(case, seed):
    return {"search": _prepare_search, "ranges": _prepare_ranges, "batch": _prepare_batch, "plane": _prepare_plane,
            "decimate": _prepare_decimate, "stream": _prepare_stream}[case["kind"]](case, seed)


def _prepare_search(case, seed):
    plan = aa.Plan(*_plan_args(case))
    x = _filterbank(case["band"], case["nchan"], case["nsamp"], plan.dms[-1], seed, plan.in_pitch)
    out = torch.zeros((case["ndm"], plan.out_pitch), dtype=torch.int32, device="cuda")
    if case["tune"]:
        plan.autotune(x, n_in=case["nsamp"], out=out, reps=3)
    work = torch.empty(plan.work_bytes(plan.n_start), dtype=torch.uint8, device="cuda")
    cap = 1 << 16
    cand, count = _cand(cap)
    return dict(case=case, plan=plan, x=x, out=out, work=work, cap=cap, cand=cand, count=count)


def _prepare_ranges(case, seed):
    first, factor = [], []
    for r, f in enumerate((0, 512, 1024, 1536, 2048, 2432)):
        if f < case["ndm"]:
            first.append(f)
            factor.append(1 << r)
    args = _plan_args(case)
    plan = aa.RangePlan(*args[:8], first, factor, stat_block=case["block"])
    x = _filterbank(case["band"], case["nchan"], case["nsamp"], args[5][-1], seed, _pitch(case["nsamp"]))
    cap = 1 << 16
    work = torch.empty(plan.work_bytes(case["nsamp"], cap), dtype=torch.uint8, device="cuda")
    cand, count = _cand(cap)
    return dict(case=case, plan=plan, x=x, work=work, cap=cap, cand=cand, count=count)


def _beams(case):
    """(channels, samples, trials) of each beam: uneven, as independent pointings are."""
    out = []
    for b in range(case["nbeams"]):
        ndm = max(50, case["ndm"] * (b % 3 + 1) // 3)
        nchan = case["nchan"] if b % 2 == 0 else case["nchan"] // 2
        tail = _span(case["band"], nchan, case["dms"], ndm) + 512
        out.append((nchan, max(tail + 4096, case["nsamp"] * (4 - b % 4) // 4 + 37 * b), ndm))
    return out


def _prepare_batch(case, seed):
    beams, need = [], 0
    for b, (nchan, nsamp, ndm) in enumerate(_beams(case)):
        plan = aa.Plan(*_plan_args(case, nchan, nsamp, ndm))
        x = _filterbank(case["band"], nchan, nsamp, plan.dms[-1], seed + 7919 * b, plan.in_pitch)
        beams.append((plan, x, nsamp))
        need += ndm * plan.out_pitch * 4 + plan.work_bytes(plan.n_start) + 1024
    work = torch.empty(need + (1 << 16), dtype=torch.uint8, device="cuda")
    return dict(case=case, beams=beams, variant=beams[0][0].variant, work=work)


def _prepare_plane(case, seed):
    widths = _widths(case)
    extra = dict(clip_sigma=3.0, clip_iters=3, boxcar_full_width=16) if case["clip"] else {}
    # a plan of ndm trials at (almost) one DM: the search needs its rows, widths and threshold only
    plan = aa.Plan(case["nchan"], case["n_dd"], 1450.0, 300.0 / case["nchan"], TSAMP,
                   np.arange(case["ndm"]) * 1e-9, widths, 6.0, case["block"], **extra)
    g = torch.Generator(device="cuda").manual_seed(seed)
    pitch = (case["n_dd"] + 63) // 64 * 64
    dd = torch.zeros((case["ndm"], pitch), dtype=torch.int32, device="cuda")
    rows = max(1, (1 << 28) // pitch)
    for r in range(0, case["ndm"], rows):
        n = min(rows, case["ndm"] - r)
        v = torch.randn((n, case["n_dd"]), generator=g, device="cuda", dtype=torch.float32)
        dd[r:r + n, :case["n_dd"]] = v.mul_(16 * case["nchan"] ** 0.5).add_(128 * case["nchan"]).round_().to(torch.int32)
    rng = np.random.default_rng(seed)
    for _ in range(8):   # pulses over a few trials
        d, t, w = (int(rng.integers(0, n)) for n in (case["ndm"], max(1, case["n_dd"] - 300), 40))
        dd[max(0, d - 3):d + 4, t:min(t + w + 1, case["n_dd"])] += int(60 * case["nchan"] ** 0.5)
    work = torch.empty(plan.work_bytes(plan.n_start), dtype=torch.uint8, device="cuda")
    cap = 1 << 16
    cand, count = _cand(cap)
    return dict(case=case, plan=plan, dd=dd, work=work, cap=cap, cand=cand, count=count)


def _prepare_decimate(case, seed):
    x = _filterbank("survey", case["nchan"], case["nsamp"], 100.0, seed, _pitch(case["nsamp"]))
    out = torch.zeros((case["nchan"], _pitch(case["nsamp"] // 2)), dtype=torch.uint8, device="cuda")
    return dict(case=case, x=x, out=out)


def _prepare_stream(case, seed):
    total = case["chunk"] * case["nchunks"]
    plan = aa.Plan(*_plan_args(case, nsamp=total))
    x = _filterbank(case["band"], case["nchan"], total, plan.dms[-1], seed, total)
    chunks = []
    for k in range(case["nchunks"]):
        h = torch.empty((case["nchan"], case["chunk"]), dtype=torch.uint8, pin_memory=True)
        h.copy_(x[:, k * case["chunk"]:(k + 1) * case["chunk"]])
        chunks.append(h)
    pipe = aa.Pipeline(nstreams=case["nstreams"], max_beams=1, max_chunk=case["chunk"], hbm_budget=4 << 30)
    state = dict(case=case, plan=plan, pipe=pipe, beam=pipe.add_beam(plan), chunks=chunks)
    _run_stream(state)   # the stream has been running: its delay tail is on the device
    return state


# ---- one pass ------------------------------------------------------------------------


def run(state):
    return {"search": _run_search, "ranges": _run_ranges, "batch": _run_batch, "plane": _run_plane,
            "decimate": _run_decimate, "stream": _run_stream}[state["case"]["kind"]](state)


def _run_search(s):
    plan = s["plan"]
    dd = plan.dedisperse(s["x"], n_in=s["case"]["nsamp"], out=s["out"])
    cand, count, best = plan.single_pulse(dd, cap=s["cap"], work=s["work"], cand=s["cand"], count=s["count"],
                                          want_best=s["case"]["best"])
    res = dict(plane=dd, cand=cand, count=count)
    if best is not None:
        res["best"] = best[:, :plan.n_start]
    return res


def _run_ranges(s):
    cand, count = s["plan"].run(s["x"], n_in=s["case"]["nsamp"], cap=s["cap"], work=s["work"], cand=s["cand"],
                                count=s["count"])
    return dict(cand=cand, count=count)


def _run_batch(s):
    cands, counts, _ = aa.batch_run(s["beams"], variant=s["variant"], work=s["work"], cap=BATCH_CAP)
    return dict(cand=[_table(c, BATCH_CAP) for c in cands], counts=counts)


def _run_plane(s):
    if s["case"]["noalloc"]:
        cand, count, _ = s["plan"].single_pulse_noalloc(s["dd"], s["cand"], s["count"])
    else:
        cand, count, _ = s["plan"].single_pulse(s["dd"], cap=s["cap"], work=s["work"], cand=s["cand"], count=s["count"])
    return dict(cand=cand, count=count)


def _run_decimate(s):
    return aa.decimate2(s["x"], n_in=s["case"]["nsamp"], out=s["out"])


def _run_stream(s):
    """Every chunk once more, as the next part of an endless stream; starts are relative to their chunk's first."""
    for k, h in enumerate(s["chunks"]):
        s["pipe"].submit(s["beam"], h, tag=k + 1)
    got = {}
    for _ in s["chunks"]:
        r = s["pipe"].poll()
        got[r["tag"]] = r
    res = []
    for k in sorted(got):
        r = got[k]
        r["cand"]["t"] -= r["t_begin"]
        res.append([r["status"], r["t_end"] - r["t_begin"], r["n_true"], _table(r["cand"], STREAM_CAP)])
    return res


# ---- what a pass cannot do without -----------------------------------------------------


def _search_work(nchan, nsamp, ndm, n_out, nw, best):
    """The input once, the plane written once and read once; one add per channel, trial and output,
    one sum, threshold and comparison per width, trial and output."""
    return dict(bytes=nchan * nsamp + 8 * ndm * n_out + (4 * ndm * n_out if best else 0),
                flops=nchan * ndm * n_out + 3 * nw * ndm * n_out)


def work(case):
    kind = case["kind"]
    if kind == "search":
        n_out = case["nsamp"] - _span(case["band"], case["nchan"], case["dms"], case["ndm"])
        return _search_work(case["nchan"], case["nsamp"], case["ndm"], n_out, len(_widths(case)), case["best"])
    if kind == "ranges":
        w = dict(bytes=case["nchan"] * case["nsamp"], flops=0)
        edges = [f for f in (0, 512, 1024, 1536, 2048, 2432) if f < case["ndm"]] + [case["ndm"]]
        for r, (a, b) in enumerate(zip(edges, edges[1:])):
            n = (case["nsamp"] - _span(case["band"], case["nchan"], case["dms"], b)) >> r
            v = _search_work(case["nchan"], case["nsamp"] >> r if r else 0, b - a, n, len(_widths(case)), False)
            w = dict(bytes=w["bytes"] + v["bytes"], flops=w["flops"] + v["flops"])
        return w
    if kind == "batch":
        w = dict(bytes=0, flops=0)
        for nchan, nsamp, ndm in _beams(case):
            n_out = nsamp - _span(case["band"], nchan, case["dms"], ndm)
            v = _search_work(nchan, nsamp, ndm, n_out, len(_widths(case)), False)
            w = dict(bytes=w["bytes"] + v["bytes"], flops=w["flops"] + v["flops"])
        return w
    if kind == "plane":
        n = case["ndm"] * case["n_dd"]
        return dict(bytes=4 * n, flops=3 * len(_widths(case)) * n)
    if kind == "decimate":
        return dict(bytes=case["nchan"] * (case["nsamp"] + case["nsamp"] // 2), flops=case["nchan"] * case["nsamp"])
    n = case["chunk"] * case["nchunks"]
    return _search_work(case["nchan"], n, case["ndm"], n, len(_widths(case)), False)


# ---- 64-bit values ---------------------------------------------------------------------


def exact(case, seed):
    if case["kind"] == "decimate":
        n = case["nsamp"] // 2
        x = _filterbank("survey", case["nchan"], case["nsamp"], 100.0, seed, _pitch(case["nsamp"])).to(torch.int64)
        out = torch.zeros((case["nchan"], _pitch(n)), dtype=torch.int64, device="cuda")
        out[:, :n] = (x[:, 0:2 * n:2] + x[:, 1:2 * n:2] + 1) >> 1
        return out
    if case["kind"] != "search" or case["nchan"] * case["ndm"] > 400000:
        return None
    nchan, nsamp, dms = case["nchan"], case["nsamp"], _dms(case["dms"], case["ndm"])
    x = _filterbank(case["band"], nchan, nsamp, dms[-1], seed, _pitch(nsamp))
    n_out = nsamp - _span(case["band"], nchan, case["dms"], case["ndm"])
    plane = torch.zeros((case["ndm"], (n_out + 63) // 64 * 64), dtype=torch.int64, device="cuda")
    for d, dm in enumerate(dms):
        row = plane[d, :n_out]
        for c, s in enumerate(_shifts(case["band"], nchan, float(dm)).tolist()):
            row += x[c, s:s + n_out]
    res = dict(plane=plane, cand=None, count=None)
    if case["best"]:
        widths, B = _widths(case), case["block"]
        T = n_out - widths[-1] + 1
        dd = plane[:, :n_out].to(torch.float64)
        pre = torch.nn.functional.pad(dd.cumsum(1), (1, 0))
        best = torch.empty((case["ndm"], T), dtype=torch.float64, device="cuda")
        for a in range(0, T, B):
            b = min(a + B, T)
            mu = dd[:, a:b].mean(1, keepdim=True)
            sd = (dd[:, a:b] - mu).square().mean(1, keepdim=True).sqrt()
            v = torch.stack([(pre[:, a + w:b + w] - pre[:, a:b] - w * mu) / (sd * w ** 0.5) for w in widths])
            best[:, a:b] = torch.where(sd > 0, v.amax(0), torch.zeros_like(mu))
        res["best"] = best
    return res

"""What a user of the library has it do, as cases that can be timed.

Each case is a dict of plain values.  `prepare` makes what a program holds
before the call (samples on the GPU, or in pinned host memory for the serving
loop; the plan, search, filterbank or server handle), `run` is one pass
through the public entry points, `work` what the pass cannot do without, and
`exact` the same outputs in 64 bits from torch alone.

Frequencies are those of the observatory's pulsar backend throughout: 16 MHz
of band at 326.5 MHz, 16 Msps of complex int8 (32 Msps of real int8 pairs on
the two-channel path).
"""
import math

import numpy as np
import torch

import paper_1503_01405_amd as P

F0, BW = 326.5, 16.0
FS = BW * 1e6
K_DM = 1.0 / 2.41e-4          # s MHz^2 per unit DM
SMEAR = 61_100                # samples of smear per unit DM, about
CHUNK = 1 << 24               # samples generated at a time


# ------------------------------------------------------------------ cases
def listed():
    return [
        # One short segment through the entry that allocates nothing (a
        # caller under graph capture or in a control loop): latency.
        dict(name="segment_2e12", kind="segment", nfft=1 << 12, dm=0.03, form="fp32", nbins=64,
             period=0.0021, nsamp=40_001, decim=16),
        # A quick-look call on a plan: a few short blocks of a nearby pulsar,
        # ragged length, several sub-integrations, fine time resolution.
        dict(name="quicklook_2e14", kind="stream", nfft=1 << 14, dm=0.1, form="mixed_valu", nbins=64,
             period=0.0053, nsamp=300_007, calls=1, subint=65_536, decim=4, taper=0.0),
        # The small workload of the benchmark's test strategy: half a second
        # at DM 1, blocks that overlap by a quarter.
        dict(name="half_second_2e18", kind="stream", nfft=1 << 18, dm=1.0, form="fp32", nbins=256,
             period=0.0891, nsamp=8_000_000, calls=1, subint=0, decim=16, taper=0.0),
        # A live stream in 1 s pieces, the overlap carried between calls, one
        # profile a second.
        dict(name="live_1s_2e20", kind="stream", nfft=1 << 20, dm=8.0, form="half", nbins=512,
             period=0.033, nsamp=96_000_000, calls=6, subint=16_000_000, decim=16, taper=0.0),
        # The production workload: 60 s at DM 50, blocks of 2^23 that
        # overlap by half, 1024 bins per 10 s and the 1 us series, in the
        # plain form and in the two float16 ones.
        dict(name="production_fp32", kind="stream", nfft=1 << 23, dm=50.0, form="fp32", nbins=1024,
             period=0.0891, nsamp=960_000_000, calls=1, subint=160_000_000, decim=16, taper=0.0),
        dict(name="production_half", kind="stream", nfft=1 << 23, dm=50.0, form="half", nbins=1024,
             period=0.0891, nsamp=960_000_000, calls=1, subint=160_000_000, decim=16, taper=0.0),
        dict(name="production_mixed", kind="stream", nfft=1 << 23, dm=50.0, form="mixed", nbins=1024,
             period=0.0891, nsamp=960_000_000, calls=1, subint=160_000_000, decim=16, taper=0.0),
        # The largest blocks: the greatest DM the backend takes in real time.
        dict(name="long_dm130_2e26", kind="stream", nfft=1 << 26, dm=130.0, form="fp32", nbins=1024,
             period=0.714, nsamp=300_000_000, calls=1, subint=0, decim=16, taper=0.1),
        # The receiver's own samples: two real channels, 30 s.
        dict(name="real_2e24", kind="real", nfft=1 << 24, dm=50.0, form="mixed_valu", nbins=1024,
             period=0.0891, nsamp=960_000_000, subint=320_000_000, decim=32, taper=0.0, sideband="lsb"),
        # A DM search of a 10 s stream over 128 trials.
        dict(name="search_128", kind="search", ntrials=128, dm_step=0.5, nfft_min=1 << 20, nfft_max=1 << 23,
             form="half", nbins=512, period=0.0891, nsamp=160_000_000),
        # The filterbank mode over 60 s.
        dict(name="aid_1024ch", kind="aid", nchan=1024, nint=4, dm=50.0, nbins=1024, period=0.0891,
             nsamp=960_000_000),
        # A session of the serving loop: streams admitted, fed 1 s blocks
        # from pinned host memory, closed, their profiles taken.
        dict(name="serve_4x3", kind="serve", streams=4, blocks=3, form="half", nbins=512, subint=8_000_000,
             block=16_000_000, mix=6),
    ]


def _spread(rng, lo, hi):
    """A whole number, even over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["stream"] * 9 + ["segment"] * 2 + ["real"] * 2 + ["search", "aid", "aid", "serve"])
    period = math.exp(rng.uniform(math.log(0.002), math.log(2.0)))
    nbins = rng.choice([64, 100, 128, 256, 300, 512, 1000, 1024])
    if kind == "segment":
        nfft = 1 << rng.randint(10, 20)
        return dict(kind=kind, nfft=nfft, dm=rng.uniform(0.15, 0.95) * nfft / 2 / SMEAR,
                    form=rng.choice(["fp32", "mixed_valu"]), nbins=nbins, period=period,
                    nsamp=_spread(rng, 2 * nfft, 24 * nfft) | 1, decim=rng.choice([1, 2, 4, 8, 16, 16]))
    if kind == "stream":
        nfft = 1 << rng.choice(list(range(12, 26)) + [20, 21, 22, 23, 23, 24])
        nsamp = _spread(rng, 2 * nfft, min(64 * nfft, 400_000_000)) | 1
        calls = rng.choice([1, 1, 2, 5])
        return dict(kind=kind, nfft=nfft, dm=rng.uniform(0.15, 0.95) * nfft / 2 / SMEAR,
                    form=rng.choice(["fp32", "half", "half", "mixed", "mixed_valu"]), nbins=nbins, period=period,
                    nsamp=nsamp, calls=calls, subint=rng.choice([0, max(64, nsamp // 5), max(64, nsamp // 3)]),
                    decim=rng.choice([1, 2, 4, 8, 16, 16, 16]), taper=rng.choice([0.0, 0.0, 0.1, 0.3]))
    if kind == "real":
        nfft = 1 << rng.randint(13, 25)
        nsamp = 2 * _spread(rng, nfft, min(32 * nfft, 400_000_000))
        return dict(kind=kind, nfft=nfft, dm=rng.uniform(0.15, 0.95) * nfft / 4 / SMEAR,
                    form=rng.choice(["fp32", "mixed_valu"]), nbins=nbins, period=period, nsamp=nsamp,
                    subint=rng.choice([0, 2 * (nsamp // 8)]), decim=rng.choice([2, 4, 8, 16, 32, 32]),
                    taper=rng.choice([0.0, 0.0, 0.2]), sideband=rng.choice(["lsb", "usb"]))
    if kind == "search":
        return dict(kind=kind, ntrials=rng.choice([8, 17, 32, 64]), dm_step=rng.choice([0.25, 0.5, 0.9]),
                    nfft_min=1 << rng.randint(18, 20), nfft_max=1 << 23,
                    form=rng.choice(["half", "half", "mixed", "mixed_valu", "fp32"]), nbins=nbins, period=period,
                    nsamp=_spread(rng, 20_000_000, 100_000_000) | 1)
    if kind == "aid":
        return dict(kind=kind, nchan=1 << rng.randint(6, 12), nint=rng.choice([1, 2, 4, 5, 16]),
                    dm=rng.uniform(0.0, 100.0), nbins=nbins, period=period,
                    nsamp=_spread(rng, 8_000_000, 400_000_000) | 1)
    return dict(kind="serve", streams=rng.randint(2, 6), blocks=rng.randint(1, 4),
                form=rng.choice(["half", "fp32", "mixed_valu"]), nbins=nbins, subint=rng.choice([0, 8_000_000]),
                block=rng.choice([8_000_000, 16_000_000]), mix=rng.randint(2, 1 << 20))


# ----------------------------------------------------------------- inputs
def _noise(seed, nsamp, period, fs, amp=20.0):
    """int8 pairs, N(0, 20^2) with a Gaussian pulse (FWHM 1 ms, peak 3 times
    the noise power) once a period, on the GPU."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    out = torch.empty((nsamp, 2), dtype=torch.int8, device="cuda")
    sigma = 1e-3 / 2.3548
    for a in range(0, nsamp, CHUNK):
        n = min(CHUNK, nsamp - a)
        t = (torch.arange(a, a + n, device="cuda", dtype=torch.float64) / (fs * period)) % 1.0
        g = torch.exp(-0.5 * ((t - 0.5) * period / sigma) ** 2).float()
        x = torch.randn((n, 2), generator=gen, device="cuda") * (amp * torch.sqrt(1.0 + 3.0 * g))[:, None]
        out[a:a + n] = x.round_().clamp_(-128, 127).to(torch.int8)
    return out.view(-1)


def _serve_streams(case):
    """(dm, period, nfft) of the session's streams: DMs over 0.5-120 and
    periods over 2 ms-2 s, the block length the smallest power of two from
    2^16 to 2^23 whose half holds the smear."""
    rng = np.random.RandomState(case["mix"])
    got = []
    for _ in range(case["streams"]):
        dm = float(np.exp(rng.uniform(np.log(0.5), np.log(120.0))))
        period = float(np.exp(rng.uniform(np.log(0.002), np.log(2.0))))
        nfft = 1 << 16
        while nfft < (1 << 23) and _geometry(dm, nfft, check=False)[1] > nfft // 2:
            nfft <<= 1
        got.append((dm, period, nfft))
    return got


class _Handle:
    """Destroys its handle with itself, as a program's owner object does."""

    def __init__(self, h, destroy):
        self.h, self.destroy = h, destroy

    def __del__(self):
        self.destroy(self.h)


def prepare(case, seed):
    k = case["kind"]
    if k in ("segment", "stream", "search", "aid"):
        x = _noise(seed, case["nsamp"], case.get("period"), FS)
    if k == "segment":
        _, _, hop = _geometry(case["dm"], case["nfft"])
        nout = _blocks(case["nsamp"], case["nfft"], hop) * hop
        return dict(case=case, x=x, profile=torch.empty(case["nbins"], device="cuda"),
                    series=torch.empty(nout // case["decim"], device="cuda"))
    if k == "stream":
        plan = P.Plan(F0, BW, case["dm"], case["nfft"], case["nbins"], case["period"], precision=case["form"],
                      subint_nsamp=case["subint"], decim=case["decim"], taper_alpha=case["taper"])
        return dict(case=case, plan=plan, pieces=[x[2 * a:2 * b] for a, b in _pieces(case)])
    if k == "real":
        # the pulse is in both channels' noise alike; A and B are the halves
        x = _noise(seed, case["nsamp"], case["period"], 2 * FS)
        plan = P.Plan(F0, BW, case["dm"], case["nfft"], case["nbins"], case["period"], precision=case["form"],
                      subint_nsamp=case["subint"], decim=case["decim"], taper_alpha=case["taper"],
                      sideband=case["sideband"])
        return dict(case=case, plan=plan, pieces=[x])
    if k == "search":
        h = P.pond_search_create(F0, BW, _dms(case), case["nbins"], case["period"], case["nfft_min"],
                                 case["nfft_max"], P.FORMS[case["form"]])
        return dict(case=case, x=x, search=_Handle(h, P.pond_search_destroy),
                    profiles=torch.empty((case["ntrials"], case["nbins"]), device="cuda"))
    if k == "aid":
        h = P.pond_aid_create(F0, BW, case["dm"], case["nchan"], case["nint"], case["nbins"], case["period"])
        n = P.pond_aid_geometry(h, case["nsamp"])["n_series"]
        return dict(case=case, x=x, aid=_Handle(h, P.pond_aid_destroy),
                    profile=torch.empty(case["nbins"], device="cuda"), series=torch.empty(n, device="cuda"))
    streams = _serve_streams(case)
    descs, hosts = [], []
    for i, (dm, period, nfft) in enumerate(streams):
        d = P.pond_stream_desc(F0, BW, dm, period, nfft, case["subint"], case["block"], case["nbins"],
                               P.FORMS[case["form"]])
        n = case["block"] * case["blocks"]
        host = torch.empty(2 * n, dtype=torch.int8, pin_memory=True)
        host.copy_(_noise(seed * 64 + i, n, period, FS))
        descs.append(d)
        hosts.append([host[2 * a:2 * (a + case["block"])] for a in range(0, n, case["block"])])
    return dict(case=case, descs=descs, hosts=hosts, server=_Handle(P.pond_server_create(64 << 30, 16),
                                                                    P.pond_server_destroy))


def _dms(case):
    return [i * case["dm_step"] for i in range(case["ntrials"])]


def _pieces(case):
    """The sample ranges of a stream's calls: as even as whole samples go."""
    n, c = case["nsamp"], case["calls"]
    at = [n * i // c for i in range(c + 1)]
    return list(zip(at, at[1:]))


# -------------------------------------------------------------------- run
def run(state):
    case = state["case"]
    k = case["kind"]
    if k == "segment":
        r = P.pond_dedisperse_segment_noalloc(F0, BW, case["dm"], case["nfft"], case["nbins"], case["period"],
                                              P.FORMS[case["form"]], state["x"], case["nsamp"], case["decim"],
                                              state["profile"], state["series"], state["series"].numel())
        if r < 0:
            raise P.PondError(r, "segment")
        return dict(profile=state["profile"], series=state["series"])
    if k in ("stream", "real"):
        plan, got = state["plan"], []
        for x in state["pieces"]:
            got.append(plan.process(x))
        return dict(profiles=[p for p, _ in got], series=[s for _, s in got], last=plan.flush())
    if k == "search":
        r = P.pond_search_run(state["search"].h, state["x"], case["nsamp"], state["profiles"])
        if r < 0:
            raise P.PondError(r, "search")
        return state["profiles"]
    if k == "aid":
        r = P.pond_aid_run(state["aid"].h, state["x"], case["nsamp"], state["profile"], state["series"],
                           state["series"].numel())
        if r < 0:
            raise P.PondError(r, "aid")
        return dict(profile=state["profile"], series=state["series"])
    srv, ids, left = state["server"].h, [], 0
    for d in state["descs"]:
        ids.append(P.pond_server_open(srv, d))
    for j in range(case["blocks"]):
        for i, blocks in zip(ids, state["hosts"]):
            if P.pond_server_submit(srv, i, blocks[j], case["block"]) < 0:
                raise RuntimeError("submit")
            left += 1
    while left:
        left -= sum(c["ticket"] >= 0 for c in P.pond_server_poll(srv, 64, wait=True))
    out = []
    for i in ids:
        if P.pond_server_close(srv, i) != P.POND_OK:
            raise RuntimeError("close")
        out.append(P.pond_server_take_profiles(srv, i, case["nbins"]))
    return out


# ------------------------------------------------------------------- work
def _transforms(nsamp, nfft, hop, pairs=1.0):
    """Operations of the block transforms (forward, and `pairs` inverses),
    the filter and the detection."""
    nb = _blocks(nsamp, nfft, hop)
    return nb * (5.0 * nfft * math.log2(nfft) * (1 + pairs) + pairs * (6.0 * nfft + 3.0 * hop))


def work(case):
    k = case["kind"]
    if k in ("segment", "stream"):
        _, _, hop = _geometry(case["dm"], case["nfft"])
        nout = _blocks(case["nsamp"], case["nfft"], hop) * hop
        nprof = 1 + (nout // case["subint"] if case.get("subint") else 0)
        return dict(bytes=2 * case["nsamp"] + 4 * (nout // case["decim"]) + 4 * nprof * case["nbins"],
                    flops=_transforms(case["nsamp"], case["nfft"], hop))
    if k == "real":
        n = case["nfft"] // 2
        _, _, hop = _geometry(case["dm"], n)
        nout = 2 * hop * _blocks(case["nsamp"] // 2, n, hop)
        return dict(bytes=2 * case["nsamp"] + 4 * (nout // case["decim"]),
                    flops=_transforms(case["nsamp"] // 2, n, hop))
    if k == "search":
        flops = 0.0
        groups = {}
        for dm in _dms(case):
            n, _ = _trial(case, dm)
            groups[n] = groups.get(n, 0) + 1
        for n, c in groups.items():
            flops += _transforms(case["nsamp"], n, n // 2, pairs=c)
        return dict(bytes=2 * case["nsamp"] + 4 * case["ntrials"] * case["nbins"], flops=flops)
    if k == "aid":
        n = case["nsamp"] // (case["nchan"] * case["nint"])
        return dict(bytes=2 * case["nsamp"] + 4 * n,
                    flops=n * case["nchan"] * case["nint"] * (5.0 * math.log2(case["nchan"]) + 4.0))
    flops = 0.0
    for dm, _, nfft in _serve_streams(case):
        _, _, hop = _geometry(dm, nfft)
        flops += _transforms(case["block"] * case["blocks"], nfft, hop)
    return dict(bytes=2.0 * case["block"] * case["blocks"] * case["streams"], flops=flops)


# ------------------------------------------------------------------ exact
def _geometry(dm, nfft, check=True):
    """(n_front, discard, hop) of a block: the samples the filter smears in
    front and behind are dropped, their number rounded up."""
    lo, hi = F0 - BW / 2, F0 + BW / 2
    front = math.ceil(K_DM * dm * (1.0 / (F0 * F0) - 1.0 / (hi * hi)) * FS)
    back = math.ceil(K_DM * dm * (1.0 / (lo * lo) - 1.0 / (F0 * F0)) * FS)
    s = front + back
    if s == 0:
        return 0, 0, nfft
    p2 = 1 << max(4, (s - 1).bit_length())
    discard = p2 if p2 <= nfft // 2 else (s + 15) // 16 * 16
    if check and nfft - discard <= 0:
        raise ValueError("block shorter than the smear")
    return front, discard, nfft - discard


def _blocks(nsamp, nfft, hop):
    return 0 if nsamp < nfft else (nsamp - nfft) // hop + 1


def _turns(f, dm):
    return dm * f * f / (2.41e-10 * F0 * F0 * (F0 + f))


def _taper(f, alpha):
    if alpha <= 0:
        return torch.ones_like(f)
    flat, edge = (1 - alpha) * BW / 2, alpha * BW / 2
    af = f.abs()
    return torch.where(af <= flat, torch.ones_like(f),
                       0.5 * (1 + torch.cos(math.pi * torch.clamp(af - flat, max=edge) / edge)))


def _filter(nfft, dm, alpha):
    k = torch.arange(nfft, device="cuda", dtype=torch.float64)
    f = torch.where(k < nfft // 2, k, k - nfft) * (BW / nfft)
    t = _turns(f, dm)
    return torch.polar(_taper(f, alpha), -2 * math.pi * (t - torch.round(t)))


class _Fold:
    """Power per (sub-integration, bin) in 64 bits: consecutive samples of one
    bin are one difference of a running sum."""

    def __init__(self, nbins, inv_pfs, front, subint):
        self.nbins, self.inv_pfs, self.front, self.subint = nbins, inv_pfs, front, subint
        self.sums, self.counts = {}, {}

    def add(self, p, m0):
        m = torch.arange(m0, m0 + p.numel(), device=p.device)
        x = (m + self.front).double() * self.inv_pfs
        turn = torch.floor(x)
        b = ((x - turn) * self.nbins).to(torch.int64).clamp_(max=self.nbins - 1)
        sub = m // self.subint if self.subint > 0 else torch.zeros_like(m)
        change = (b[1:] != b[:-1]) | (turn[1:] != turn[:-1]) | (sub[1:] != sub[:-1])
        ends = torch.cat([change.nonzero().view(-1), torch.tensor([p.numel() - 1], device=p.device)])
        run = torch.cumsum(p, 0)[ends]
        cell = torch.cat([run[:1], run[1:] - run[:-1]])
        size = torch.cat([ends[:1] + 1, ends[1:] - ends[:-1]])
        for s in range(int(sub[0]), int(sub[-1]) + 1):
            at = sub[ends] == s
            if s not in self.sums:
                self.sums[s] = torch.zeros(self.nbins, dtype=torch.float64, device=p.device)
                self.counts[s] = torch.zeros(self.nbins, dtype=torch.float64, device=p.device)
            self.sums[s].index_add_(0, b[ends][at], cell[at])
            self.counts[s].index_add_(0, b[ends][at], size[at].double())

    def profile(self, s):
        return self.sums[s] / self.counts[s].clamp(min=1)


def _complex(x):
    v = x.view(-1, 2).double()
    return torch.complex(v[:, 0].contiguous(), v[:, 1].contiguous())


def _stream_exact(x, dm, nfft, nbins, period, subint, decim, taper, ends, hop=None):
    """Outputs of a stream fed up to the samples `ends`, call by call."""
    front, _, h = _geometry(dm, nfft)
    hop = hop or h
    H = _filter(nfft, dm, taper)
    fold = _Fold(nbins, 1.0 / (period * FS), front, subint)
    profiles, series, nb, carry = [], [], 0, None
    for end in ends:
        first, rows = nb * hop, []
        while nb < _blocks(end, nfft, hop):
            y = torch.fft.ifft(torch.fft.fft(_complex(x[2 * nb * hop:2 * (nb * hop + nfft)])) * H)[front:front + hop]
            p = y.real ** 2 + y.imag ** 2
            fold.add(p, nb * hop)
            if decim:
                rows.append(p.view(-1, decim).sum(1))
            nb += 1
        s0, s1 = (first // subint, nb * hop // subint) if subint > 0 else (0, 0)
        done = [fold.profile(s) for s in range(s0, s1)]
        profiles.append(torch.stack(done) if done else torch.empty((0, nbins), dtype=torch.float64))
        series.append(torch.cat(rows) if rows else torch.empty(0, dtype=torch.float64))
    out, s = nb * hop, (nb * hop // subint if subint > 0 else 0)
    last = fold.profile(s)[None] if out > s * subint else torch.empty((0, nbins), dtype=torch.float64)
    return dict(profiles=profiles, series=series, last=last)


def _trial(case, dm):
    front, discard, _ = _geometry(dm, case["nfft_max"])
    return max(case["nfft_min"], min(case["nfft_max"], 2 * discard)), front


def _real_exact(case, x):
    n2 = case["nfft"]
    n = n2 // 2
    front, _, hop = _geometry(case["dm"], n)
    fb = torch.arange(n + 1, device="cuda", dtype=torch.float64) * (BW / n)
    f = BW / 2 - fb if case["sideband"] == "lsb" else fb - BW / 2
    t = _turns(f, case["dm"])
    sign = 1 if case["sideband"] == "lsb" else -1
    M = torch.polar(_taper(f, case["taper"]), sign * 2 * math.pi * (t - torch.round(t)))
    M[0], M[-1] = M[0].real.clone(), M[-1].real.clone()
    subint = case["subint"]
    fold = _Fold(case["nbins"], 1.0 / (case["period"] * FS * 2.0), 2 * front, subint)
    nb, rows = _blocks(case["nsamp"] // 2, n, hop), []
    for b in range(nb):
        v = x[4 * b * hop:4 * b * hop + 2 * n2].view(-1, 2).double().sum(1)
        p = torch.fft.irfft(torch.fft.rfft(v) * M, n=n2)[2 * front:2 * (front + hop)] ** 2
        fold.add(p, 2 * b * hop)
        rows.append(p.view(-1, case["decim"]).sum(1))
    out = 2 * nb * hop
    s = out // subint if subint else 0
    empty = torch.empty((0, case["nbins"]), dtype=torch.float64)
    return dict(profiles=[torch.stack([fold.profile(i) for i in range(s)]) if s else empty],
                series=[torch.cat(rows) if rows else torch.empty(0, dtype=torch.float64)],
                last=fold.profile(s)[None] if out > s * subint else empty)


def _search_exact(case, x):
    trials = [(dm,) + _trial(case, dm) for dm in _dms(case)]
    folds = [_Fold(case["nbins"], 1.0 / (case["period"] * FS), front, 0) for _, _, front in trials]
    for n in sorted({t[1] for t in trials}):
        hop = n // 2
        for b in range(_blocks(case["nsamp"], n, hop)):
            X = torch.fft.fft(_complex(x[2 * b * hop:2 * (b * hop + n)]))
            for (dm, nt, front), fold in zip(trials, folds):
                if nt == n:
                    y = torch.fft.ifft(X * _filter(n, dm, 0.0))[front:front + hop]
                    fold.add(y.real ** 2 + y.imag ** 2, b * hop)
    zero = torch.zeros(case["nbins"], dtype=torch.float64, device="cuda")
    return torch.stack([f.profile(0) if f.sums else zero for f in folds])


def _aid_exact(case, x):
    C, nint = case["nchan"], case["nint"]
    n = case["nsamp"] // (C * nint)
    F = torch.empty((n, C), dtype=torch.float64, device="cuda")
    step = max(1, CHUNK // (C * nint))
    for a in range(0, n, step):
        m = min(step, n - a)
        X = torch.fft.fft(_complex(x[2 * a * C * nint:2 * (a + m) * C * nint]).view(m * nint, C), dim=1)
        F[a:a + m] = (X.real ** 2 + X.imag ** 2).view(m, nint, C).sum(1)
    ts = C * nint / FS
    f = F0 + np.fft.fftfreq(C, d=1.0 / BW)
    d = np.floor(K_DM * case["dm"] * (1.0 / (f * f) - 1.0 / (F0 * F0)) / ts + 0.5).astype(np.int64)
    dmin = int(d.min())
    nout = n - int(d.max() - dmin)
    if nout <= 0:
        return dict(profile=torch.zeros(case["nbins"], dtype=torch.float64),
                    series=torch.empty(0, dtype=torch.float64))
    s = torch.zeros(nout, dtype=torch.float64, device="cuda")
    for c in range(C):
        s += F[int(d[c]) - dmin:int(d[c]) - dmin + nout, c]
    xph = (torch.arange(nout, device="cuda") - dmin).double() * float(C * nint) * (1.0 / (case["period"] * FS))
    b = ((xph - torch.floor(xph)) * case["nbins"]).to(torch.int64).clamp_(max=case["nbins"] - 1)
    sums = torch.zeros(case["nbins"], dtype=torch.float64, device="cuda").index_add_(0, b, s)
    counts = torch.bincount(b, minlength=case["nbins"])
    return dict(profile=sums / counts.clamp(min=1), series=s)


def exact(case, seed):
    k = case["kind"]
    if k == "serve":
        out = []
        for i, (dm, period, nfft) in enumerate(_serve_streams(case)):
            n = case["block"] * case["blocks"]
            x = _noise(seed * 64 + i, n, period, FS)
            r = _stream_exact(x, dm, nfft, case["nbins"], period, case["subint"], 0, 0.0, [n])
            out.append(torch.cat([r["profiles"][0].to("cuda"), r["last"].to("cuda")]))
        return out
    x = _noise(seed, case["nsamp"], case["period"], FS if k != "real" else 2 * FS)
    if k == "segment":
        r = _stream_exact(x, case["dm"], case["nfft"], case["nbins"], case["period"], 0, case["decim"], 0.0,
                          [case["nsamp"]])
        return dict(profile=r["last"][0] if r["last"].numel() else torch.zeros(case["nbins"], dtype=torch.float64),
                    series=r["series"][0])
    if k == "stream":
        return _stream_exact(x, case["dm"], case["nfft"], case["nbins"], case["period"], case["subint"],
                             case["decim"], case["taper"], [b for _, b in _pieces(case)])
    if k == "real":
        return _real_exact(case, x)
    if k == "search":
        return _search_exact(case, x)
    return _aid_exact(case, x)

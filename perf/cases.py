"""The work that programs have this library do, as cases that can be timed.

A case is a dict of plain values:
  path      the entry points: "process" (a batch of device events, unpack + cluster in one call),
            "host" (the same from and to pageable host memory), "plain" (unpack, then cluster, one
            event), "hits" (clusters to global hits), "ingest" (page-locked host events, pipelined
            in batches), "serve" (events submitted to the server and polled)
  n_fed     FEDs of the detector part (96 channels x 256 strips each); 440 is the full detector
  n_events  events of one pass
  occ_lo, occ_hi   per-event occupancy, log-uniform in this range (hits per strip)
  wide      False: hits of up to 8 strips, noise U[3, 6], 0.1 % bad strips; True: up to 32
            strips, noise U[2, 10], 1 % bad (FEDs of 8 KB at 6 % occupancy)
  modules   clusters run on across the channels of a module
  status    per-channel status bytes are asked for
  batch     events per pipelined batch ("ingest")

The inputs have the distributions of the repository's synthetic generator, drawn on the GPU from
the seed: hit widths min(Geometric, cap), LogNormal charges, Gaussian noise, 8-bit ADCs, and a
front end that keeps a strip when its ADC exceeds twice its noise.
"""
import math

import numpy as np
import torch

import paper_2101_11489_amd as sc

CH, STRIPS, APV = 96, 256, 128
T_SEED, T_CHANNEL, T_CLUSTER = 3.0, 2.0, 5.0


def _case(name, path, n_fed, n_events, occ_lo, occ_hi=None, wide=False, modules=False, status=False,
          batch=0):
    return {"name": name, "path": path, "n_fed": n_fed, "n_events": n_events, "occ_lo": occ_lo,
            "occ_hi": occ_hi or occ_lo, "wide": wide, "modules": modules, "status": status,
            "batch": batch}


def listed():
    return [
        # one event of a detector part: the smallest call, all latency
        _case("one-50fed", "process", 50, 1, 0.01),
        # one full-detector event as soon as it is there
        _case("one-full", "process", 440, 1, 0.015, status=True),
        # the same for a program whose data and results are in ordinary host memory
        _case("one-full-host", "host", 440, 1, 0.015, status=True),
        # the two steps alone, with the dense strip array between them
        _case("plain-full", "plain", 440, 1, 0.015, status=True),
        # a small batch of a detector part
        _case("batch20-50fed", "process", 50, 20, 0.01),
        # a batch of ordinary full-detector events
        _case("batch20-full", "process", 440, 20, 0.015),
        # the batched workload: occupancies of a whole run in one launch
        _case("batch64-full", "process", 440, 64, 0.005, 0.05),
        # the busiest events: FEDs larger than the default LDS stage
        _case("stress64-full", "process", 440, 64, 0.06, wide=True),
        # module rows, an odd number of events and of FEDs
        _case("modules13-431fed", "process", 431, 13, 0.005, 0.05, modules=True, status=True),
        # global hits of a batch's clusters
        _case("hits32-full", "hits", 440, 32, 0.005, 0.05),
        # a readout ring in page-locked host memory, processed in batches
        _case("ingest64-full", "ingest", 440, 64, 0.005, 0.05, batch=16),
        # events handed to the server one by one
        _case("serve24-full", "serve", 440, 24, 0.005, 0.06),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    path = rng.choice(["process", "process", "process", "process", "host", "plain", "hits",
                       "ingest", "serve"])
    wide = path == "process" and rng.random() < 0.25
    n_fed = int(round(_log(rng, 9, 440)))
    lo = _log(rng, 0.004, 0.05)
    hi = min(0.06, lo * rng.choice([1.0, 2.0, 5.0]))
    if wide:
        lo = hi = _log(rng, 0.02, 0.06)
    most = {"process": 64, "host": 6, "plain": 1, "hits": 32, "ingest": 64, "serve": 24}[path]
    n_events = int(round(_log(rng, 1, most)))
    c = _case("", path, n_fed, n_events, round(lo, 5), round(hi, 5), wide,
              modules=path in ("process", "plain") and rng.random() < 0.25,
              status=path in ("process", "host", "plain") and rng.random() < 0.4,
              batch=rng.choice([3, 8, 16]) if path == "ingest" else 0)
    del c["name"]
    return c


# ---- inputs ------------------------------------------------------------------------------------

def _calibration(case, gen, dev):
    n = case["n_fed"] * CH * STRIPS
    lo, hi = (2.0, 10.0) if case["wide"] else (3.0, 6.0)
    noise = torch.empty(n, device=dev).uniform_(lo, hi, generator=gen)
    gain = torch.empty(n // APV, device=dev).normal_(1.0, 0.05, generator=gen)
    bad = torch.rand(n, device=dev, generator=gen) < (0.01 if case["wide"] else 0.001)
    return noise, gain, bad


def _event(case, gen, dev, noise, gain):
    """ADC of every strip and whether the front end keeps it."""
    n = noise.numel()
    u = torch.rand(1, device=dev, generator=gen).item()
    occ = case["occ_lo"] * (case["occ_hi"] / case["occ_lo"]) ** u
    start = torch.nonzero(torch.rand(n, device=dev, generator=gen) < occ).reshape(-1)
    p, cap = (0.25, 32) if case["wide"] else (0.5, 8)
    h = start.numel()
    width = torch.empty(h, device=dev).geometric_(p, generator=gen).clamp_(max=cap).long()
    charge = torch.empty(h, device=dev).log_normal_(math.log(90.0), 0.5, generator=gen)
    share = torch.round(charge / width * 1024.0).int()   # whole numbers: their sum has no order
    hit = torch.repeat_interleave(width)
    within = torch.arange(hit.numel(), device=dev) - (torch.cumsum(width, 0) - width)[hit]
    strip = start[hit] + within
    keep = strip // STRIPS == start[hit] // STRIPS
    deposit = torch.zeros(n, dtype=torch.int32, device=dev)
    deposit.scatter_add_(0, strip[keep], share[hit[keep]])
    z = torch.empty(n, device=dev).normal_(generator=gen)
    x = gain.repeat_interleave(APV) * (deposit.float() / 1024.0) + noise * z
    adc = torch.round(x).clamp_(0, 255).to(torch.uint8)
    return adc, adc.float() > 2.0 * noise


def _encode(adc, kept, n_fed):
    """Zero-suppressed bytes of the kept strips, and the FED offsets."""
    dev, n_ch = adc.device, n_fed * CH
    m = kept.view(n_ch, STRIPS)
    prev = torch.zeros_like(m)
    prev[:, 1:] = m[:, :-1]
    first = m & ~prev
    first[:, 255] |= m.all(dim=1)   # a run carries at most 255 strips
    cost = (m.to(torch.int32) + 2 * first.to(torch.int32)).reshape(-1)
    end = torch.cumsum(cost, 0, dtype=torch.int64)
    chan_end = end.view(n_ch, STRIPS)[:, -1]
    payload = torch.diff(chan_end, prepend=chan_end.new_zeros(1))
    rec_end = chan_end + 2 * torch.arange(1, n_ch + 1, device=dev)
    zs = torch.zeros(int(rec_end[-1]), dtype=torch.uint8, device=dev)
    at = rec_end - payload - 2
    zs[at] = (payload & 255).to(torch.uint8)
    zs[at + 1] = (payload >> 8).to(torch.uint8)
    digi = torch.nonzero(kept).reshape(-1)
    pos = end[digi] - 1 + 2 * (digi // STRIPS + 1)
    zs[pos] = adc[digi]
    heads = torch.nonzero(first.reshape(-1)[digi]).reshape(-1)
    count = torch.diff(heads, append=heads.new_full((1,), digi.numel()))
    zs[pos[heads] - 2] = (digi[heads] % STRIPS).to(torch.uint8)
    zs[pos[heads] - 1] = count.to(torch.uint8)
    fed = torch.zeros(n_fed + 1, dtype=torch.int64, device=dev)
    fed[1:] = rec_end.view(n_fed, CH)[:, -1]
    return zs, fed


def _modules(n_fed, seed):
    """Rows of 2 or 3 channels inside blocks of 24, on barrel layers (for hits and module rows)."""
    rng = np.random.default_rng(seed)
    sizes = []
    for _ in range(n_fed * (CH // 24)):
        left = 24
        while left:
            k = left if left in (2, 3) else 2 if left == 4 else int(rng.integers(2, 4))
            sizes.append(k)
            left -= k
    sizes = np.array(sizes)
    m = sizes.size
    layer, phi = rng.integers(0, 10, m), rng.uniform(0.0, 2.0 * math.pi, m)
    z, tilt = rng.uniform(-100.0, 100.0, m), rng.uniform(-0.1, 0.1, m)
    r = np.linspace(25.0, 110.0, 10)[layer]

    class Geometry:
        channel_module = np.repeat(np.arange(m), sizes).astype(np.uint32)
        channel_first = ((np.arange(sizes.sum()) - np.repeat(np.cumsum(sizes) - sizes, sizes))
                         * STRIPS).astype(np.uint32)
        module_strips = (sizes * STRIPS).astype(np.uint32)
        origin = np.stack([r * np.cos(phi), r * np.sin(phi), z], axis=1).astype(np.float32)
        u_dir = np.stack([-np.sin(phi) * np.cos(tilt), np.cos(phi) * np.cos(tilt), np.sin(tilt)],
                         axis=1).astype(np.float32)
        pitch = np.array([0.0080] * 4 + [0.0120] * 3 + [0.0183] * 3)[layer].astype(np.float32)
    return Geometry


def _generator(seed, dev):
    gen = torch.Generator(device=dev)
    gen.manual_seed(0x2CE1 + int(seed))
    return gen


def _caps(case):
    """Capacities of one event's outputs: what the busiest events of such a run need, and a margin."""
    strips, occ = case["n_fed"] * CH * STRIPS, case["occ_hi"]
    return (int(strips * (1.15 * occ + 0.003)) + 512,
            int(strips * ((4.6 if case["wide"] else 2.6) * occ + 0.006)) + 1024)


class _Slice(sc.Output):
    """One event's part of buffers that the whole batch shares."""

    def __init__(self, cl, adc, status, device):
        self.device, self.cl, self.adc, self.chan_status = device, cl, adc, status
        ptr = (lambda x: 0 if x is None else x.ctypes.data) if not device else \
            (lambda x: 0 if x is None else x.data_ptr())
        self.cs = sc.ScClusters(ptr(cl), len(cl), 0, ptr(adc), len(adc), 0, ptr(status),
                                sc.SC_MEM_DEVICE if device else sc.SC_MEM_HOST)


class _Out:
    """The output buffers of a batch, and the outputs that share them."""

    def __init__(self, case, device=True):
        n, n_fed, status = case["n_events"], case["n_fed"], case["status"]
        cc, ca = _caps(case)
        rows, adcs = n * cc, n * ca
        if device:
            self.cl = torch.zeros((rows, 4), dtype=torch.int32, device="cuda")
            self.adc = torch.zeros(adcs, dtype=torch.int16, device="cuda")
            self.status = torch.zeros((n, n_fed * CH), dtype=torch.uint8, device="cuda") if status else None
            self.fields, self.bary = self.cl[:, :3], self.cl.view(torch.float32)[:, 3]
        else:
            self.cl = np.zeros(rows, dtype=sc.CLUSTER_DTYPE)
            self.adc = np.zeros(adcs, dtype=np.uint16)
            self.status = np.zeros((n, n_fed * CH), dtype=np.uint8) if status else None
            self.fields, self.bary = self.cl.view(np.int32).reshape(-1, 4)[:, :3], self.cl["barycenter"]
        self.outs = [_Slice(self.cl[i * cc:(i + 1) * cc], self.adc[i * ca:(i + 1) * ca],
                            self.status[i] if status else None, device) for i in range(n)]

    def result(self, counts):
        return {"clusters": self.fields, "bary": self.bary, "adc": self.adc,
                "status": self.status, "counts": counts}


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = _generator(seed, dev)
    noise, gain, bad = _calibration(case, gen, dev)
    n_fed, path = case["n_fed"], case["path"]
    geo = _modules(n_fed, seed)
    ctx = sc.Context(noise.cpu().numpy(), gain.cpu().numpy(), bad.to(torch.uint8).cpu().numpy(),
                     T_SEED, T_CHANNEL, T_CLUSTER)
    if case["modules"]:
        ctx.set_modules(geo.channel_module)
    events = []
    for _ in range(case["n_events"]):
        adc, kept = _event(case, gen, dev, noise, gain)
        zs, fed = _encode(adc, kept, n_fed)
        if path in ("host", "ingest"):
            events.append(sc.Event(zs.cpu().numpy(), fed.cpu().numpy().view(np.uint64)))
        else:
            events.append(sc.Event(zs, fed))
    if path == "ingest":
        events = sc.pack_pinned(events)
    out = _Out(case, device=path != "host")
    s = {"case": case, "ctx": ctx, "events": events, "out": out}
    if path == "plain":
        s["dense"] = ctx.dense_buffer()
        s["status"] = torch.zeros(n_fed * CH, dtype=torch.uint8, device=dev) if case["status"] else None
    if path == "hits" or (path == "process" and case["n_events"] > 1):
        b = ctx.batch(events, out.outs)
        s["batch"] = b
        words = np.frombuffer(b.c_out, dtype=np.uint32).reshape(b.n, -1)
        s["counts"] = words[:, 3:8:4]   # n_cl, n_adc of every event, as the library writes them
    if path == "hits":
        ctx.set_geometry(geo)
        ctx.process_batch(s["batch"])
        s["hits"] = torch.zeros((case["n_events"], _caps(case)[0], 4), dtype=torch.float32, device=dev)
        s["parts"] = [h[:o.n_cl] for h, o in zip(s["hits"], out.outs)]
    return s


def run(s):
    path, ctx, out = s["case"]["path"], s["ctx"], s["out"]
    if path == "process" and "batch" in s:
        ctx.process_batch(s["batch"])
        return out.result(s["counts"])
    if path in ("process", "host"):
        ctx.process_events(s["events"], out.outs)
    elif path == "plain":
        ctx.unpack(s["events"][0], s["dense"], s["status"])
        ctx.cluster(s["dense"], out.outs[0])
        return dict(out.result([out.outs[0].n_cl, out.outs[0].n_adc]), dense=s["dense"],
                    status=s["status"])
    elif path == "hits":
        ctx.cluster_hits(out.outs, s["parts"])
        return s["hits"]
    elif path == "ingest":
        ctx.process_pipelined(s["events"], out.outs, s["case"]["batch"])
    elif path == "serve":
        tickets = [ctx.submit(e, o) for e, o in zip(s["events"], out.outs)]
        for t in tickets:
            ctx.poll(t)
    return out.result(np.array([(o.n_cl, o.n_adc) for o in out.outs]))


# ---- the definition, in 64 bits ------------------------------------------------------------------

def _clusters(adc, kept, noise, gain, bad, joins):
    """(strip of each cluster's first member, width, charge, barycenter) of one event: runs of
    strips above T_CHANNEL x noise with one above T_SEED x noise and a charge of at least
    T_CLUSTER x sqrt(sum of squared noise), the FP32 roundings of the thresholds included."""
    n, dev = adc.numel(), adc.device
    a = torch.where(kept, adc, torch.zeros_like(adc)).float()
    good = ~bad & (gain.repeat_interleave(APV) > 0)
    active = good & (a > T_CHANNEL * noise)
    seed = active & (a > T_SEED * noise)
    at = torch.nonzero(active).reshape(-1)
    last = torch.full_like(at, -2)
    last[1:] = at[:-1]
    new = (at != last + 1) | ((at % STRIPS == 0) & ~joins[at // STRIPS])
    run = torch.cumsum(new.long(), 0) - 1
    head = at[new]
    n_run = head.numel()
    k = at - head[run]
    zero = torch.zeros(n_run, dtype=torch.float64, device=dev)
    s = zero.clone()
    for i in range(int(k.max()) + 1 if at.numel() else 0):
        sel = torch.nonzero(k == i).reshape(-1)
        r, v = run[sel], noise[at[sel]].double()
        s[r] = (v * v + s[r]).float().double()
    q = torch.zeros(n_run, dtype=torch.int64, device=dev).scatter_add_(0, run, adc[at].long())
    seeds = torch.zeros_like(q).scatter_add_(0, run, seed[at].long())
    width = torch.zeros_like(q).scatter_add_(0, run, torch.ones_like(at))
    ok = (seeds > 0) & (q.double() >= (T_CLUSTER * torch.sqrt(s).float().double()).float().double())
    c = torch.round((adc[at].double() / gain[at // APV].double()).float()).clamp(max=65535).long()
    charge = torch.zeros_like(q).scatter_add_(0, run, c)
    twice = torch.zeros_like(q).scatter_add_(0, run, (2 * (at - head[run] // STRIPS * STRIPS) + 1) * c)
    mid = (head % STRIPS).double() + width.double() / 2
    bary = torch.where(charge > 0, twice.double() / (2.0 * charge.double().clamp(min=1.0)), mid)
    return head[ok], width[ok], charge[ok], bary[ok]


def _joins(case, geo, dev):
    m = torch.from_numpy(geo.channel_module.astype(np.int64)).to(dev)
    j = torch.zeros(m.numel(), dtype=torch.bool, device=dev)
    if case["modules"]:
        j[1:] = m[1:] == m[:-1]
        j[::CH] = False
    return j


def exact(case, seed):
    dev = torch.device("cuda")
    gen = _generator(seed, dev)
    noise, gain, bad = _calibration(case, gen, dev)
    n_fed = case["n_fed"]
    geo = _modules(n_fed, seed)
    joins = _joins(case, geo, dev)
    parts = []
    for _ in range(case["n_events"]):
        adc, kept = _event(case, gen, dev, noise, gain)
        head, _, _, bary = _clusters(adc, kept, noise, gain, bad, joins)
        rows = torch.zeros((_caps(case)[0], 4 if case["path"] == "hits" else 1), dtype=torch.float64,
                           device=dev)
        if case["path"] == "hits":
            ch = head // STRIPS
            mod = torch.from_numpy(geo.channel_module.astype(np.int64)).to(dev)[ch]
            table = lambda x: torch.from_numpy(np.asarray(x).astype(np.float64)).to(dev)  # noqa: E731
            u = (table(geo.channel_first)[ch] + bary - table(geo.module_strips)[mod] / 2) * table(geo.pitch)[mod]
            xyz = table(geo.origin)[mod] + u[:, None] * table(geo.u_dir)[mod]
            rows[:len(u)] = torch.cat([xyz, u[:, None]], dim=1)
        else:
            rows[:len(bary), 0] = bary
        parts.append(rows)
    if case["path"] == "hits":
        return torch.stack(parts)
    return {"bary": torch.cat(parts)[:, 0], "clusters": None, "adc": None, "status": None, "counts": None}


# ---- what a pass cannot do without -----------------------------------------------------------------

def work(case):
    """From a sample of the case's events on a few FEDs: each ZS byte, FED offset and calibration
    entry of a strip with a digi read once, each record, ADC and status byte written once."""
    dev, feds = torch.device("cpu"), min(4, case["n_fed"])
    few = dict(case, n_fed=feds)
    gen = _generator(1, dev)
    noise, gain, bad = _calibration(few, gen, dev)
    joins = _joins(few, _modules(feds, 1), dev)
    touched = torch.zeros(noise.numel(), dtype=torch.bool)
    zs_bytes = digis = clusters = members = 0
    samples = min(8, case["n_events"])
    for _ in range(samples):
        adc, kept = _event(few, gen, dev, noise, gain)
        touched |= kept
        zs_bytes += _encode(adc, kept, feds)[0].numel()
        digis += int(kept.sum())
        head, width, _, _ = _clusters(adc, kept, noise, gain, bad, joins)
        clusters += head.numel()
        members += int(width.sum())
    per = case["n_events"] * case["n_fed"] / (samples * feds)
    zs_bytes, digis, clusters, members = (per * v for v in (zs_bytes, digis, clusters, members))
    n_ch = case["n_fed"] * CH
    density = float(touched.float().mean())
    strips = n_ch * STRIPS * (1.0 - (1.0 - density) ** (case["n_events"] / samples))
    calib = 4.125 * strips + 8.0 * n_ch
    if case["path"] == "hits":
        return {"bytes": 32.0 * clusters + 8.0 * n_ch, "flops": 9.0 * clusters}
    n_bytes = zs_bytes + 8.0 * (case["n_fed"] + 1) * case["n_events"] + calib + 16.0 * clusters + 2.0 * members
    if case["status"]:
        n_bytes += case["n_events"] * n_ch
    if case["path"] == "plain":
        n_bytes += 2.0 * n_ch * STRIPS
    return {"bytes": n_bytes, "flops": 8.0 * digis + 8.0 * members + 12.0 * clusters}

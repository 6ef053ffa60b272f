"""Performance cases of the library: what its users run, through the public
Python entry points of ``paper_2101_05012_amd``.

Five kinds of work, each a ``kind`` of case:

  align      ABEA of a batch of reads.  ``form`` is how the program calls it:
             "device" (``Aligner.align_device`` on device-resident reads, one
             launch per batch), "graph" (a captured batch replayed, a pool of
             wavefronts taking reads from the device queue), "host"
             (``Aligner.align``, host arrays in and out)
  serve      reads handed to a running ``Server``, results collected by polling
  detect     raw samples to events (``Aligner.detect_events_device``)
  meth       per-site methylation scores of an aligned batch
             (``Aligner.methylation_device``)
  pipeline   raw samples to site scores (``pipeline.call_methylation``)

Inputs follow ``synth``'s recipes (pore model, event counts per k-mer, dwell
times, noise), drawn on the device so that the largest batches take seconds.
A case fixes the sizes (read lengths, events per k-mer, dwell times); the seed
draws the sequences, the signal and the scaling.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2101_05012_amd import abea, pipeline, synth

EVENTS_PER_KMER = (1.0 - synth.SKIP_PROB) * synth.EVENTS_PER_KMER_MEAN
DWELL = synth.SAMPLE_RATE_HZ / synth.BASES_PER_S
CHUNK_KMERS = 1 << 25  # k-mers drawn at a time


def _align(name, n, lengths, lo, hi, median=0, W=100, k=6, form="device", trim=False, scale_events=False,
           workers_per_simd=0):
    return {"name": name, "kind": "align", "n": n, "lengths": lengths, "lo": lo, "hi": hi, "median": median, "W": W,
            "k": k, "form": form, "trim": trim, "scale_events": scale_events, "workers_per_simd": workers_per_simd}


def _other(name, kind, n, lengths, lo, hi, median=0, k=6, W=100):
    return {"name": name, "kind": kind, "n": n, "lengths": lengths, "lo": lo, "hi": hi, "median": median, "W": W,
            "k": k}


def listed():
    return [
        # the smallest batch: 64 reads of 1 kb, one launch (a sequencer's
        # first seconds, amplicons); latency and launch count
        _align("align-64x1kb", 64, "uniform", 1000, 1000),
        # reads arriving at a basecalling server, collected as they finish
        _other("serve-64x8kb", "serve", 64, "lognormal", 200, 30_000, 8000),
        # an ordinary batch of a whole-genome run, resident on the device
        _align("align-4000x5kb", 4000, "lognormal", 200, 100_000, 5000),
        # the same with open-pore and adaptor events at the ends: trim states
        _align("align-4000x5kb-trim", 4000, "lognormal", 200, 100_000, 5000, trim=True),
        # the C caller's entry point: host buffers in and out, events scaled
        # to the model
        _align("align-host-1000x5kb", 1000, "lognormal", 200, 50_000, 5000, form="host", scale_events=True),
        # a large job of very uneven reads in the persistent form
        _align("align-20000-uneven", 20000, "mixed", 500, 200_000, form="graph", workers_per_simd=4),
        # the same job shape at twice the band width (four slots per lane)
        _align("align-10000-uneven-w200", 10000, "mixed", 500, 200_000, W=200, form="graph", workers_per_simd=3),
        # ultra-long reads: few, each up to 1 Mb
        _align("align-100-ultralong", 100, "uniform", 200_000, 1_000_000, form="graph", workers_per_simd=4),
        # event detection of a handful of reads, and of an ordinary batch
        _other("detect-16x5kb", "detect", 16, "lognormal", 200, 20_000, 5000),
        _other("detect-4000x5kb", "detect", 4000, "lognormal", 200, 100_000, 5000),
        # methylation scores of an ordinary aligned batch
        _other("meth-4000x5kb", "meth", 4000, "lognormal", 200, 100_000, 5000),
        # the three steps chained, raw signal to site scores
        _other("pipeline-1000x5kb", "pipeline", 1000, "lognormal", 200, 50_000, 5000),
    ]


def draw(rng):
    def spread(a, b):  # log-uniform integer
        return max(a, min(b, int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))))

    kind = rng.choice(["align"] * 6 + ["serve", "detect", "detect", "meth", "pipeline"])
    if kind == "align":
        form = rng.choice(["device", "device", "graph", "host"])
        n = spread(1, {"device": 4000, "graph": 10_000, "host": 1000}[form])
        W = rng.choice([100, 100, rng.randint(30, 300)])
        k = rng.choice([5, 6, 6, 9])
        top = spread(2000, 200_000 if n <= 2000 else 50_000)
        lengths = rng.choice(["lognormal", "uniform"])
        c = _align("", n, lengths, 200, top, max(500, top // 20), W, k, form, trim=rng.random() < 0.25,
                   scale_events=rng.random() < 0.25, workers_per_simd=4 if form == "graph" else 0)
        most = 25_000_000_000 if form != "host" else 1_000_000_000  # cells
    else:
        n = spread(1, {"serve": 128, "detect": 4000, "meth": 4000, "pipeline": 1000}[kind])
        top = spread(2000, {"serve": 30_000, "detect": 100_000, "meth": 100_000, "pipeline": 50_000}[kind])
        k = rng.choice([5, 6, 6]) if kind in ("meth", "pipeline") else 6
        c = _other("", kind, n, "lognormal", 200, top, max(500, top // 12), k)
        most = 10_000_000_000
    while c["n"] > 1 and c["n"] * _mean_length(c) * (1 + EVENTS_PER_KMER) * c["W"] > most:
        c["n"] //= 2
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs


def _mean_length(c):
    if c["lengths"] == "uniform":
        return 0.5 * (c["lo"] + c["hi"])
    if c["lengths"] == "mixed":
        return 0.7 * 2750 + 0.3 * 110_000
    return min(c["median"] * math.exp(0.5), 0.7 * c["hi"])


def _lengths(c, rng):
    n = c["n"]
    if c["lengths"] == "uniform":
        return rng.integers(c["lo"], c["hi"] + 1, n)
    if c["lengths"] == "mixed":  # 70% of 0.5-5 kb, 30% of 20-200 kb
        short = rng.random(n) < 0.7
        return np.where(short, rng.integers(500, 5001, n), rng.integers(20_000, 200_001, n))
    return np.clip(np.round(np.exp(rng.normal(math.log(c["median"]), 1.0, n))), c["lo"], c["hi"]).astype(np.int64)


def _offsets(counts):
    o = np.zeros(len(counts) + 1, np.uint64)
    np.cumsum(np.asarray(counts, np.uint64), out=o[1:])
    return o


def _ranks(n_kmers, k, gen):
    """Ranks of consecutive k-mers of one random sequence (a read takes a run
    of them)."""
    b = torch.randint(0, 4, (n_kmers + k - 1,), generator=gen, device="cuda", dtype=torch.int32)
    r = torch.zeros(n_kmers, dtype=torch.int32, device="cuda")
    for t in range(k):
        r = r * 4 + b[t : t + n_kmers]
    return r


def _chunks(ko):
    """Runs of reads of about CHUNK_KMERS k-mers."""
    lo, n = 0, len(ko) - 1
    while lo < n:
        hi = int(np.searchsorted(ko, ko[lo] + np.uint64(CHUNK_KMERS), side="right")) - 1
        hi = min(n, max(hi, lo + 1))
        yield lo, hi
        lo = hi


def _common(c, seed):
    size = [c["n"], c["lo"], c["hi"], c["median"]]
    sizes = torch.Generator(device="cuda").manual_seed(sum(v * m for v, m in zip(size, (1, 7919, 104729, 1299709))))
    rng = np.random.default_rng([int(seed), 17])
    gen = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 11)
    model = synth.pore_model(c["k"])
    nk = np.maximum(_lengths(c, np.random.default_rng(size)) - c["k"] + 1, 1)
    ko = _offsets(nk)
    scale = torch.from_numpy(rng.uniform(0.9, 1.1, c["n"]).astype(np.float32)).cuda()
    shift = torch.from_numpy(rng.uniform(-5.0, 5.0, c["n"]).astype(np.float32)).cuda()
    return rng, gen, sizes, model, nk, ko, scale, shift


def _levels(c, model, meth):
    lv = torch.from_numpy(model.level_mean).cuda()
    sd = torch.from_numpy(model.level_stdv).cuda()
    ml = torch.from_numpy(synth.methylated_model(model).level_mean).cuda() if meth else lv
    return lv, ml, sd


def _reads(c, seed, meth=False, ends=False, path=False):
    """Reads with events: (model, DeviceBatch, path pairs and their offsets or
    None).  ``ends``: open-pore and adaptor events around each read;
    ``path``: the alignment that emitted the events, as pairs."""
    rng, gen, sizes, model, nk, ko, scale, shift = _common(c, seed)
    lv, ml, sd = _levels(c, model, meth)
    ranks = _ranks(int(ko[-1]), c["k"], gen)
    is_meth = torch.from_numpy(rng.random(c["n"]) < 0.5).cuda()
    means, ne, pairs, npairs = [], [], [], []
    q = 1.0 / synth.EVENTS_PER_KMER_MEAN
    for lo, hi in _chunks(ko):
        k0, k1 = int(ko[lo]), int(ko[hi])
        read = torch.repeat_interleave(torch.arange(lo, hi, device="cuda"), torch.from_numpy(nk[lo:hi]).cuda())
        u = torch.rand(k1 - k0, generator=sizes, device="cuda")
        cnt = 1 + torch.floor(torch.log1p(-u) / math.log1p(-q)).to(torch.int64).clamp_(0, 200)
        cnt[torch.rand(k1 - k0, generator=sizes, device="cuda") < synth.SKIP_PROB] = 0
        first = torch.from_numpy((ko[lo:hi] - ko[lo]).astype(np.int64)).cuda()
        cnt[first] = cnt[first].clamp(min=1)  # a read starts with an event of its first k-mer
        km = torch.repeat_interleave(torch.arange(k1 - k0, device="cuda"), cnt)
        rk = ranks[k0:k1].long()
        level = torch.where(is_meth[read], ml[rk], lv[rk]) * scale[read] + shift[read]
        m = level[km] + sd[rk][km] * torch.randn(km.shape[0], generator=gen, device="cuda")
        cum = torch.cumsum(cnt, 0)
        last = torch.from_numpy((ko[lo + 1 : hi + 1] - ko[lo]).astype(np.int64) - 1).cuda()
        nr = torch.diff(cum[last], prepend=torch.zeros(1, dtype=torch.int64, device="cuda"))
        if path:
            # a k-mer without events is entered by a skip from its predecessor's last event
            rows = cnt.clamp(min=1)
            pk = torch.repeat_interleave(torch.arange(k1 - k0, device="cuda"), rows)
            ro = torch.cumsum(rows, 0) - rows
            within = torch.arange(pk.shape[0], device="cuda") - ro[pk]
            before = cum - cnt  # events of the chunk before the k-mer
            e = before[pk] + within - (cnt[pk] == 0).long()
            base_e = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), cum[last][:-1]])
            rr = read[pk] - lo
            pairs.append(torch.stack([e - base_e[rr], pk - first[rr]], 1).to(torch.int32))
            pr = torch.cumsum(rows, 0)[last]
            npairs.append(torch.diff(pr, prepend=torch.zeros(1, dtype=torch.int64, device="cuda")))
        if ends:
            m, nr = _with_ends(m, nr, gen, sizes)
        means.append(m)
        ne.append(nr)
        del read, km, rk, level, cnt, u, cum
    n_e = torch.cat(ne).cpu().numpy()
    eo = _offsets(n_e)
    mean = torch.cat(means) if len(means) > 1 else means[0]
    del means
    ev = torch.empty((mean.shape[0], 3), dtype=torch.float32, device="cuda")
    ev[:, 0] = mean
    ev[:, 1].uniform_(0.5, 3.0, generator=gen)
    ev[:, 2].exponential_(400.0, generator=gen)
    db = abea.DeviceBatch(c["n"], ev, ranks, scale, shift, eo, ko)
    if not path:
        return model, db, None, None
    po = torch.from_numpy(_offsets(torch.cat(npairs).cpu().numpy()).view(np.int64)).cuda()
    return model, db, torch.cat(pairs), po


def _with_ends(m, nr, gen, sizes):
    n = nr.shape[0]
    lead = torch.randint(0, synth.MAX_OPEN_PORE_EVENTS + 1, (n,), generator=sizes, device="cuda")
    adapt = torch.randint(0, synth.MAX_ADAPTOR_EVENTS + 1, (n,), generator=sizes, device="cuda")
    tail = torch.randint(0, synth.MAX_OPEN_PORE_EVENTS + 1, (n,), generator=sizes, device="cuda")
    total = lead + adapt + nr + tail
    read = torch.repeat_interleave(torch.arange(n, device="cuda"), total)
    at = torch.arange(read.shape[0], device="cuda") - (torch.cumsum(total, 0) - total)[read]
    opened = synth.OPEN_PORE_MEAN + synth.OPEN_PORE_SD * torch.randn(read.shape[0], generator=gen, device="cuda")
    adaptor = 60.0 + 70.0 * torch.rand(read.shape[0], generator=gen, device="cuda")
    inside = (at >= (lead + adapt)[read]) & (at < (lead + adapt + nr)[read])
    out = torch.where((at >= lead[read]) & (at < (lead + adapt)[read]), adaptor, opened)
    out[inside] = m  # the read's own events, in order
    return out, total


def _raw(c, seed, meth=False):
    """Raw reads: (model, DeviceRawBatch, ranks, kmer_offset, scale, shift)."""
    rng, gen, sizes, model, nk, ko, scale, shift = _common(c, seed)
    lv, ml, sd = _levels(c, model, meth)
    ranks = _ranks(int(ko[-1]), c["k"], gen)
    is_meth = torch.from_numpy(rng.random(c["n"]) < 0.5).cuda()
    pa_scale = torch.from_numpy((rng.uniform(*synth.RAW_RANGE_PA, c["n"]) / synth.RAW_DIGITISATION).astype(np.float32)).cuda()
    offset = torch.from_numpy(rng.uniform(*synth.RAW_OFFSET, c["n"]).astype(np.float32)).cuda()
    raw, ns = [], []
    for lo, hi in _chunks(ko):
        k0, k1 = int(ko[lo]), int(ko[hi])
        read = torch.repeat_interleave(torch.arange(lo, hi, device="cuda"), torch.from_numpy(nk[lo:hi]).cuda())
        half = DWELL / synth.DWELL_GAMMA_SHAPE
        g = -half * (torch.log1p(-torch.rand(k1 - k0, generator=sizes, device="cuda"))
                     + torch.log1p(-torch.rand(k1 - k0, generator=sizes, device="cuda")))  # Gamma(2)
        dwell = g.round().clamp(1, 2000).to(torch.int64)
        km = torch.repeat_interleave(torch.arange(k1 - k0, device="cuda"), dwell)
        rk = ranks[k0:k1].long()
        level = torch.where(is_meth[read], ml[rk], lv[rk]) * scale[read] + shift[read]
        pa = level[km] + sd[rk][km] * torch.randn(km.shape[0], generator=gen, device="cuda")
        rd = read[km]
        raw.append((pa / pa_scale[rd] - offset[rd]).round().clamp(-32768, 32767).to(torch.int16))
        last = torch.from_numpy((ko[lo + 1 : hi + 1] - ko[lo]).astype(np.int64) - 1).cuda()
        cum = torch.cumsum(dwell, 0)[last]
        ns.append(torch.diff(cum, prepend=torch.zeros(1, dtype=torch.int64, device="cuda")))
        del read, km, rk, level, pa, rd
    so = _offsets(torch.cat(ns).cpu().numpy())
    samples = torch.cat(raw) if len(raw) > 1 else raw[0]
    return model, abea.DeviceRawBatch(c["n"], samples, offset, pa_scale, so), ranks, ko, scale, shift


def _result(n, cap):
    z = lambda s, t: torch.zeros(s, dtype=t, device="cuda")  # noqa: E731
    return abea.DeviceResult(z((max(cap, 1), 2), torch.int32), cap, z(n + 1, torch.int64), z(n, torch.float32),
                             z(n, torch.int32), z(n, torch.int64))


def _host(db):
    return synth.Batch(db.events.cpu().numpy(), db.event_offset, db.ranks.cpu().numpy().view(np.uint32),
                       db.kmer_offset, db.scale.cpu().numpy(), db.shift.cpu().numpy())


# ------------------------------------------------------------- prepare, run


def prepare(case, seed):
    c = case
    kind = c["kind"]
    s = {"case": c}
    if kind in ("align", "serve"):
        model, db, _, _ = _reads(c, seed, ends=c.get("trim", False))
        workers = 0
        wpg = 1
        if c.get("workers_per_simd"):
            props = torch.cuda.get_device_properties(0)
            workers = c["workers_per_simd"] * 4 * props.multi_processor_count
            wpg = 4
        al = abea.Aligner(model.level_mean, model.level_stdv, c["k"], W=c["W"], workers=workers, waves_per_group=wpg,
                          scale_events=c.get("scale_events", False), trim=c.get("trim", False))
        s["al"] = al
        if kind == "serve":
            s["batch"] = _host(db)
            s["tags"] = np.arange(c["n"], dtype=np.uint64)
            s["first"] = db.event_offset + db.kmer_offset  # a read's place in the collected pairs
            s["server"] = abea.Server(al, slots=8, max_batch_reads=256, max_batch_events=1 << 21,
                                      max_batch_kmers=1 << 20, host_staging_bytes=256 << 20)
        elif c["form"] == "host":
            s["batch"] = _host(db)
        else:
            s["db"] = db
            s["dres"] = _result(c["n"], db.capacity)
            if c["form"] == "graph":
                s["graph"] = al.graph(db, s["dres"])
    elif kind == "detect":
        model, draw_, _, _, _, _ = _raw(c, seed)
        s["al"] = abea.Aligner(model.level_mean, model.level_stdv, c["k"])
        s["raw"] = draw_
        s["events"] = torch.zeros((max(draw_.n_samples, 1), 3), dtype=torch.float32, device="cuda")
        s["offset"] = torch.zeros(c["n"] + 1, dtype=torch.int64, device="cuda")
    elif kind == "meth":
        model, db, pairs, po = _reads(c, seed, meth=True, path=True)
        al = abea.Aligner(model.level_mean, model.level_stdv, c["k"])
        mm = synth.methylated_model(model)
        al.set_methylated_model(mm.level_mean, mm.level_stdv)
        n, K = c["n"], int(db.kmer_offset[-1])
        s.update(al=al, db=db)
        s["dres"] = abea.DeviceResult(pairs, int(pairs.shape[0]), po, torch.zeros(n, device="cuda"),
                                      torch.zeros(n, dtype=torch.int32, device="cuda"),
                                      torch.zeros(n, dtype=torch.int64, device="cuda"))
        s["llr"] = torch.zeros(K, dtype=torch.float32, device="cuda")
        s["n_ev"] = torch.zeros(K, dtype=torch.int32, device="cuda")
    else:
        model, draw_, ranks, ko, scale, shift = _raw(c, seed, meth=True)
        al = abea.Aligner(model.level_mean, model.level_stdv, c["k"], W=c["W"])
        mm = synth.methylated_model(model)
        al.set_methylated_model(mm.level_mean, mm.level_stdv)
        S, K = draw_.n_samples, int(ko[-1])
        s.update(al=al, raw=draw_, ranks=ranks, ko=ko, scale=scale, shift=shift)
        # the output buffers a program keeps between batches
        s["bufs"] = {"ev": torch.zeros((S, 3), dtype=torch.float32, device="cuda"),
                     "eo": torch.zeros(c["n"] + 1, dtype=torch.int64, device="cuda"),
                     "llr": torch.zeros(K, dtype=torch.float32, device="cuda"),
                     "nev": torch.zeros(K, dtype=torch.int32, device="cuda"),
                     "dres": _result(c["n"], S + K)}
    return s


def _aligned(r):
    return {"pairs": r.pairs, "pair_offset": r.pair_offset, "log_likelihood": r.log_likelihood, "status": r.status,
            "cells": r.cells}


def run(state):
    s = state
    c = s["case"]
    kind = c["kind"]
    if kind == "align":
        if c["form"] == "host":
            r = s["al"].align(s["batch"])
            # r.pairs is the used part of the buffer that the call filled
            return {"pairs": r.pairs if r.pairs.base is None else r.pairs.base, "pair_offset": r.pair_offset.view(np.int64), "log_likelihood": r.log_likelihood,
                    "status": r.status, "cells": r.cells.view(np.int64)}
        if c["form"] == "graph":
            s["graph"].launch()
        else:
            s["al"].align_device(s["db"], s["dres"])
        return _aligned(s["dres"])
    if kind == "serve":
        n = c["n"]
        s["server"].submit(s["batch"], 0, n, s["tags"])
        got, done = [], 0
        pairs = np.zeros((int(s["first"][n]), 2), np.int32)
        while done < n:
            comp, p = s["server"].poll(timeout_us=2000)
            for x in comp:
                o = int(x["pair_offset"])
                m, at = int(x["n_pairs"]), int(s["first"][int(x["tag"])])
                pairs[at : at + m] = p[o : o + m]
            got.append(comp)
            done += comp.shape[0]
        comp = np.concatenate(got)
        comp = comp[np.argsort(comp["tag"])]
        return {"pairs": pairs, "n_pairs": comp["n_pairs"].astype(np.int64),
                "log_likelihood": comp["log_likelihood"].copy(), "status": comp["status"].copy(),
                "cells": comp["cells"].astype(np.int64)}
    if kind == "detect":
        s["al"].detect_events_device(s["raw"], s["events"], s["offset"])
        return {"events": s["events"], "offset": s["offset"]}
    if kind == "meth":
        s["al"].methylation_device(s["db"], s["dres"], s["llr"], s["n_ev"])
        return {"llr": s["llr"], "n_ev": s["n_ev"]}
    r = pipeline.call_methylation(s["al"], s["raw"], s["ranks"], s["ko"], s["scale"], s["shift"], bufs=s["bufs"])
    return {"event_offset": r.event_offset.view(np.int64), "events": r.events, "llr": r.llr, "n_ev": r.n_ev,
            **_aligned(r.dres)}


# -------------------------------------------------------------------- work


def work(case):
    """The inputs read once and the outputs written once, and 11 operations per
    band cell (emission 4, moves 5, maximum 2), from the mean read."""
    c = case
    n = c["n"]
    nk = n * _mean_length(c)
    ne = nk * EVENTS_PER_KMER
    bands = nk + ne
    path = 1.05 * ne  # one cell per event, and the skipped k-mers
    sites = nk / 16.0
    align_b = 12 * ne + 4 * nk + 8 * path + 40 * n
    align_f = 11.0 * c["W"] * bands
    ns = nk * DWELL
    detect_b = 2 * ns + 12 * ne + 24 * n
    detect_f = 40.0 * ns
    meth_b = 12 * ne + 4 * nk + 8 * path + 8 * nk
    meth_f = sites * c["k"] * (c["k"] * EVENTS_PER_KMER) * 22.0
    if c["kind"] in ("align", "serve"):
        return {"bytes": align_b, "flops": align_f}
    if c["kind"] == "detect":
        return {"bytes": detect_b, "flops": detect_f}
    if c["kind"] == "meth":
        return {"bytes": meth_b, "flops": meth_f}
    return {"bytes": detect_b + align_b + meth_b, "flops": detect_f + align_f + meth_f}


# ------------------------------------------------------------------- exact


def exact(case, seed):
    c = case
    if c["kind"] == "detect":
        return _exact_detect(c, seed)
    if c["kind"] == "meth":
        return _exact_meth(c, seed)
    if c["kind"] == "align" and not c["trim"] and not c["scale_events"] and c["hi"] <= 2000 and c["n"] * c["W"] <= 16_000:
        return _exact_align(c, seed)
    return None


def _transitions(ne, nk):
    skip = math.log(1e-10)
    stay = np.log(1.0 - 1.0 / (ne / nk + 1.0))
    step = np.log(1.0 - math.exp(skip) - np.exp(stay))
    return skip, stay, step


def _exact_align(c, seed):
    """Log-likelihoods: band moves and path decided in float32, as the
    alignment defines them, the path's score summed in float64."""
    f4 = np.float32
    model, db, _, _ = _reads(c, seed)
    n, W = c["n"], c["W"]
    ev = db.events[:, 0].cpu().numpy()
    rk = db.ranks.cpu().numpy()
    eo, ko = db.event_offset.astype(np.int64), db.kmer_offset.astype(np.int64)
    ne, nk = np.diff(eo), np.diff(ko)
    X = np.zeros((n, ne.max()), f4)
    R = np.zeros((n, nk.max()), np.int64)
    for r in range(n):
        X[r, : ne[r]] = ev[eo[r] : eo[r + 1]]
        R[r, : nk[r]] = rk[ko[r] : ko[r + 1]]
    sc, sh = db.scale.cpu().numpy(), db.shift.cpu().numpy()
    mu64 = model.level_mean.astype(np.float64)[R] * sc[:, None].astype(np.float64) + sh[:, None]
    mu = mu64.astype(f4)
    sd = model.level_stdv.astype(np.float64)[R]
    cc64, hh64 = -math.log(math.sqrt(2 * math.pi)) - np.log(sd), 0.5 / sd**2
    cc, hh = cc64.astype(f4), hh64.astype(f4)
    skip, stay, step = _transitions(ne.astype(np.float64), nk.astype(np.float64))
    lp = [np.full(n, skip), stay, step]
    lp64 = [v[:, None] for v in lp]
    lp32 = [v.astype(f4)[:, None] for v in lp]
    ar, off = np.arange(n)[:, None], np.arange(W)[None, :]
    NI = f4(-np.inf)
    H = W // 2

    def padded(dt):
        return np.full((n, W + 4), NI, dt)

    def at(S, d):  # offsets shifted by d (per read), -inf outside the band
        j = off + 2 + d
        return S[ar, np.clip(j, 0, W + 3)]

    P2, P1, Q2, Q1 = padded(f4), padded(f4), padded(np.float64), padded(np.float64)
    P2[:, H + 2] = 0
    Q2[:, H + 2] = 0
    K2 = np.full((n, 1), -1 - H)
    K1 = K2 + 1
    end = np.full(n, np.nan)
    for i in range(2, int((ne + nk).max()) + 1):
        lo, hi = P1[:, 2], P1[:, W + 1]
        both = np.isneginf(lo) & np.isneginf(hi)
        K = K1 + np.where(both, i % 2 == 1, lo < hi)[:, None]
        k = K + off
        e = i - 2 - k
        ok = (k >= 0) & (k < nk[:, None]) & (e >= 0) & (e < ne[:, None])
        kc, ec = np.clip(k, 0, R.shape[1] - 1), np.clip(e, 0, X.shape[1] - 1)
        x = X[ar, ec]
        d = x - mu[ar, kc]
        em = cc[ar, kc] - (d * d) * hh[ar, kc]
        d64 = x.astype(np.float64) - mu64[ar, kc]
        em64 = cc64[ar, kc] - d64 * d64 * hh64[ar, kc]
        a = (at(P2, K - K2 - 1) + lp32[2]) + em
        b = (at(P1, K - K1) + lp32[1]) + em
        g = at(P1, K - K1 - 1) + lp32[0]
        a64 = at(Q2, K - K2 - 1) + lp64[2] + em64
        b64 = at(Q1, K - K1) + lp64[1] + em64
        g64 = at(Q1, K - K1 - 1) + lp64[0]
        m = np.maximum(np.maximum(a, b), g)
        m64 = np.where(a == m, a64, np.where(b == m, b64, g64))
        P2, P1, Q2, Q1, K2, K1 = P1, padded(f4), Q1, padded(np.float64), K1, K
        P1[:, 2 : W + 2] = np.where(ok, m, NI)
        Q1[:, 2 : W + 2] = np.where(ok, m64, -np.inf)
        at_end = np.nonzero(ne + nk == i)[0]
        if at_end.size:
            j = nk[at_end] - 1 - K[at_end, 0]
            inside = (j >= 0) & (j < W)
            end[at_end] = np.where(inside, Q1[at_end, np.clip(j, 0, W - 1) + 2], -np.inf)
    return {"pairs": None, "pair_offset": None, "log_likelihood": end, "status": None, "cells": None}


def _exact_detect(c, seed):
    """Events: change points as the detector defines them (integer window
    sums, float32 statistic), means and deviations in float64."""
    _, raw, _, _, _, _ = _raw(c, seed)
    x = raw.samples.long()
    S = x.shape[0]
    so = torch.from_numpy(raw.sample_offset.astype(np.int64)).cuda()
    n = torch.diff(so)
    zero = torch.zeros(1, dtype=torch.int64, device="cuda")
    P = torch.cat([zero, torch.cumsum(x, 0)])
    Q = torch.cat([zero, torch.cumsum(x * x, 0)])
    del x
    read = torch.repeat_interleave(torch.arange(c["n"], device="cuda"), n)
    j = torch.arange(S, device="cuda") - so[read]
    left = n[read] - j  # samples from the boundary to the read's end
    flag = j == 0
    for w, t in ((3, 1.5), (8, 5.0)):
        T = torch.full((S + 2 * w,), -1.0, dtype=torch.float32, device="cuda")
        ok = ((j >= w) & (left >= w)).nonzero()[:, 0]
        sl, sr = P[ok] - P[ok - w], P[ok + w] - P[ok]
        V = w * (Q[ok + w] - Q[ok - w]) - sl * sl - sr * sr
        D = (sr - sl).float()
        T[w + ok] = torch.where(V == 0, torch.where(D != 0, math.inf, 0.0).float(),
                                (D * D) * float(w) / V.double().float())
        del sl, sr, V, D, ok
        peak = T[w : w + S] > float(np.float32(t) * np.float32(t))
        for m in range(1, w):
            peak &= (T[w : w + S] > T[w - m : w - m + S]) & (T[w : w + S] >= T[w + m : w + m + S])
        flag |= peak
        del T, peak
    del j, left
    b = flag.nonzero()[:, 0]
    e = torch.cat([b[1:], torch.full((1,), S, device="cuda")])
    r = read[b]
    ln = (e - b).double()
    s, q = (P[e] - P[b]), (Q[e] - Q[b])
    sc, off = raw.pa_scale.double()[r], raw.offset.double()[r]
    out = torch.zeros((max(S, 1), 3), dtype=torch.float64, device="cuda")
    out[: b.shape[0], 0] = (s.double() / ln + off) * sc
    out[: b.shape[0], 1] = torch.sqrt(((e - b) * q - s * s).double()) / ln * sc
    out[: b.shape[0], 2] = ln
    return {"events": out, "offset": None}


def _exact_meth(c, seed):
    """Site scores: the best path of each window under both models, in
    float64."""
    model, db, pairs, po = _reads(c, seed, meth=True, path=True)
    mm = synth.methylated_model(model)
    k, n = c["k"], c["n"]
    ko = torch.from_numpy(db.kmer_offset.astype(np.int64)).cuda()
    eo = torch.from_numpy(db.event_offset.astype(np.int64)).cuda()
    K = int(ko[-1])
    ne, nk = torch.diff(eo).double(), torch.diff(ko).double()
    skip = math.log(1e-10)
    stay = torch.log(1.0 - 1.0 / (ne / nk + 1.0))
    step = torch.log(1.0 - math.exp(skip) - torch.exp(stay))
    kread = torch.repeat_interleave(torch.arange(n, device="cuda"), torch.diff(ko))
    pread = torch.repeat_interleave(torch.arange(n, device="cuda"), torch.diff(po))
    g = pairs[:, 1].long() + ko[pread]
    ends = torch.ones_like(g, dtype=torch.bool)
    ends[:-1] = g[1:] != g[:-1]
    starts = torch.ones_like(ends)
    starts[1:] = ends[:-1]
    klast = torch.zeros(K, dtype=torch.int64, device="cuda")
    kfirst = torch.zeros(K, dtype=torch.int64, device="cuda")
    klast[g[ends]] = pairs[ends, 0].long()
    kfirst[g[starts]] = pairs[starts, 0].long()
    del g, ends, starts, pread
    rk = db.ranks.long()
    site = (((rk >> (2 * (k - 1))) & 3) == 1) & (((rk >> (2 * (k - 2))) & 3) == 2)
    at = site.nonzero()[:, 0]
    r = kread[at]
    i = at - ko[r]
    j0 = (i - (k - 1)).clamp(min=0)
    e0, e1 = kfirst[ko[r] + j0], klast[at]
    score = []
    for m in (mm, model):
        lm = torch.from_numpy(m.level_mean).cuda().double()
        ls = torch.from_numpy(m.level_stdv).cuda().double()
        mu, cc, hh = [], [], []
        for t in range(k):
            q = rk[(ko[r] + j0 + t).clamp(max=K - 1)]
            mu.append(lm[q] * db.scale[r].double() + db.shift[r].double())
            cc.append(-math.log(math.sqrt(2 * math.pi)) - torch.log(ls[q]))
            hh.append(0.5 / ls[q] ** 2)
        col = [torch.full_like(mu[0], -math.inf) for _ in range(k)]
        for d in range(int((e1 - e0).max()) + 1 if at.numel() else 0):
            live = e0 + d <= e1
            x = db.events[(eo[r] + e0 + d).clamp(max=db.events.shape[0] - 1), 0].double()
            diag = torch.full_like(x, 0.0 if d == 0 else -math.inf)
            lf = torch.full_like(x, -math.inf)
            for t in range(k):
                em = cc[t] - (x - mu[t]) ** 2 * hh[t]
                v = torch.maximum(torch.maximum(diag + step[r], col[t] + stay[r]) + em, lf + skip)
                diag, lf = col[t], v
                col[t] = torch.where(live, v, col[t])
        last = (i - j0)[:, None]
        score.append(torch.gather(torch.stack(col, 1), 1, last)[:, 0] if at.numel() else mu[0])
    llr = torch.full((K,), math.nan, dtype=torch.float64, device="cuda")
    llr[at] = score[0] - score[1]
    return {"llr": llr, "n_ev": None}

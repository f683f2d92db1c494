"""Performance cases of the SPIIR library, through its public entry points.

A case is one block of strain filtered by a bank (or by a batch of banks) that
a search program keeps on the GPU.  ``prepare`` makes what such a program has in
hand before the block arrives: the bank with its tables and plan, the strain
block and the output buffers.  ``run`` is the call that the program makes per
block; each pass takes the block as the next one of the stream, so the filter
states carry on from pass to pass.

Fields of a case:
  entry      block (spiir_process_block), batch (spiir_process_batch over
             `streams` banks, each with a caller workspace), graph (a recorded
             batch, its input refilled before each replay) or peaks
             (spiir_process_peaks without z)
  templates  templates per bank; streams: banks, one per detector
  bands      1 = single rate; rate: base rate in Hz
  layout     equal (`hi` filters in every segment), uniform (`lo`..`hi` filters
             per template and band) or uneven (`lo`..`hi` filters per template,
             log-uniform, over 1..`bands` of its bands)
  seconds    the delays run up to seconds * rate samples of each band
  n          samples per block; a batch takes three quarters of it from the
             second stream and half of it from the third
  precision  fp32 or fp32_compensated
  split      0 = the library's default, -1 = the time split it chooses by itself
"""
import math

import numpy as np
import torch

from paper_1702_02256_amd import serving, spiir, workloads

SHORTEST = 64   # samples of the shortest block drawn
LARGEST = 6e9   # filter-samples of the largest case drawn


def _case(name, entry, templates, bands, rate, layout, lo, hi, seconds, n, precision, split=0, streams=1):
    return {"name": name, "entry": entry, "templates": templates, "streams": streams, "bands": bands, "rate": rate,
            "layout": layout, "lo": lo, "hi": hi, "seconds": seconds, "n": n, "precision": precision, "split": split}


def listed():
    return [
        # one template looked at by hand: the smallest call, all latency
        _case("one template", "block", 1, 1, 4096, "equal", 128, 128, 0.5, 4096, "fp32"),
        # a few templates of a follow-up, blocks and filter counts of no round size
        _case("single rate, small and odd", "block", 37, 1, 2048, "equal", 301, 301, 2.0, 1001, "fp32"),
        # the single-rate bank of the paper's first comparison, 1 s blocks
        _case("single rate, 1024 x 512", "block", 1024, 1, 2048, "equal", 512, 512, 2.0, 2048, "fp32"),
        # a low-latency search: the bank of one node's share, blocks of 1/8 s
        _case("low latency, 1/8 s", "block", 160, 7, 4096, "uniform", 40, 300, 0.5, 576, "fp32_compensated"),
        # a small multi-rate bank on one GPU, with the split that the library picks for it
        _case("small multi-rate, split", "block", 128, 7, 4096, "uniform", 40, 300, 0.5, 4096, "fp32_compensated", split=-1),
        # the trigger search: peaks only, z is not written
        _case("triggers", "peaks", 512, 7, 4096, "uniform", 40, 300, 0.5, 4096, "fp32_compensated"),
        # a quarter of the multi-rate bank: does not fill the GPU
        _case("multi-rate, 1024", "block", 1024, 7, 4096, "uniform", 40, 300, 0.5, 4096, "fp32"),
        # stored data filtered again: one call over 8 s
        _case("stored data, 8 s", "block", 48, 5, 4096, "uniform", 40, 300, 0.5, 32768, "fp32_compensated"),
        # the multi-rate bank, 1 s blocks
        _case("multi-rate, 4096", "block", 4096, 7, 4096, "uniform", 40, 300, 0.5, 4096, "fp32_compensated"),
        # templates of very different lengths, the recorded launch sequence replayed
        _case("uneven, recorded", "graph", 8192, 7, 4096, "uneven", 16, 1024, 0.5, 4096, "fp32"),
        # serving: the same bank on three detectors, blocks of uneven length in one batch
        _case("serving batch", "batch", 5461, 7, 4096, "uniform", 40, 300, 0.5, 4096, "fp32_compensated", streams=3),
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        bands = rng.choice((1, 1, 3, 5, 7, 7))
        unit = 1 << (bands - 1)
        layout = "equal" if bands == 1 else rng.choice(("uniform", "uniform", "uneven"))
        hi = logint(60, 600) if layout == "equal" else 1024 if layout == "uneven" else rng.randint(120, 300)
        lo = hi if layout == "equal" else 16 if layout == "uneven" else rng.randint(20, 100)
        entry = rng.choice(("block", "block", "block", "batch", "graph", "peaks"))
        split = -1 if entry == "block" and rng.random() < 0.25 else 0
        case = {"entry": entry, "templates": logint(1, 4096), "streams": rng.randint(2, 3) if entry == "batch" else 1,
                "bands": bands, "rate": rng.choice((2048, 4096)), "layout": layout, "lo": lo, "hi": hi,
                "seconds": rng.choice((0.25, 0.5, 1.0)), "n": unit * max(1, round(logint(SHORTEST, 16384) / unit)),
                "precision": rng.choice(("fp32", "fp32_compensated")), "split": split}
        if _filter_samples(case) <= LARGEST:
            return case


def _lengths(case):
    """Samples of each stream's block: whole multiples of the lowest band's step."""
    unit = 1 << (case["bands"] - 1)
    return [max(unit, case["n"] * s // 4 // unit * unit) for s in (4, 3, 2)[: case["streams"]]]


# ---------------------------------------------------------------- tables

_kept = {}  # the tables and the planned bank of the case in use, as a search program keeps them


def _counts(case):
    rng = np.random.default_rng([71, case["templates"], case["bands"], case["lo"], case["hi"]])
    T, H, lo, hi = case["templates"], case["bands"], case["lo"], case["hi"]
    if case["layout"] == "equal":
        return np.full((T, H), hi, np.int32)
    if case["layout"] == "uniform":
        return rng.integers(lo, hi + 1, size=(T, H)).astype(np.int32)
    out = np.zeros((T, H), np.int32)
    total = np.exp(rng.uniform(math.log(lo), math.log(hi), T)).round().astype(int)
    for t in range(T):
        used = np.sort(rng.permutation(H)[: int(rng.integers(1, H + 1))])
        out[t, used] = rng.multinomial(max(int(total[t]) - len(used), 0), np.full(len(used), 1 / len(used))) + 1
    return out


def _filter_samples(case):
    per_band = _counts(case).sum(axis=0, dtype=np.int64)
    return sum(int(per_band[h]) * (n >> h) for n in _lengths(case) for h in range(case["bands"]))


def _tables(case):
    key = tuple((k, case[k]) for k in ("templates", "bands", "rate", "layout", "lo", "hi", "seconds"))
    if _kept.get("tables key") != key:
        _kept.clear()
        nf = _counts(case)
        H, M = case["bands"], int(nf.sum())
        rng = np.random.default_rng([72, M, H])
        a1 = rng.uniform(0.9, 0.9999, M) * np.exp(1j * rng.uniform(0.0, 2.0 * np.pi, M))
        b0 = (rng.standard_normal(M) + 1j * rng.standard_normal(M)) * 1e-3
        dmax = np.array([max(int(case["seconds"] * (case["rate"] >> h)) - 1, 0) for h in range(H)])
        top = np.repeat(np.broadcast_to(dmax, nf.shape).ravel(), nf.ravel())
        delay = rng.integers(0, top + 1).astype(np.int32)
        taps = (workloads.down_taps(32), workloads.up_taps(32)) if H > 1 else (np.ones(1), np.ones(1))
        _kept["tables"] = workloads.BankTables(base_rate=case["rate"], n_filters=nf, a1=a1, b0=b0, delay=delay,
                                               h_down=taps[0], h_up=taps[1])
        _kept["tables key"] = key
    return _kept["tables"]


def _strain(case, seed, stream):
    g = torch.Generator().manual_seed(1_000_003 * seed + stream)
    return torch.randn(_lengths(case)[stream], generator=g)


# ---------------------------------------------------------------- the calls


def _bank(case):
    """A bank of the case with zero state: planned once, then cloned (the paper's
    search runs one template bank on every detector)."""
    tables = _tables(case)
    kw = {"precision": case["precision"], "time_chunks": case["split"]}
    if case["entry"] == "batch":
        kw.update(workspace=spiir.WORKSPACE_CALLER, **serving.BATCHED_BANK_SHAPE)
    key = (case["n"], tuple(sorted(kw.items())))
    if _kept.get("bank key") != key:
        _kept["bank"] = spiir.Bank(tables, case["n"], **kw)
        _kept["bank key"] = key
    return _kept["bank"].clone()


def prepare(case, seed):
    T = case["templates"]
    state = {"entry": case["entry"], "banks": [], "x": [], "z": []}
    for s, n in enumerate(_lengths(case)):
        state["banks"].append(_bank(case))
        state["x"].append(_strain(case, seed, s).cuda())
        if case["entry"] == "peaks":
            state["peaks"] = spiir.peaks_empty(T)
            # three times the rms of z: 2e-6 (|b0|^2) times 35 (a filter's mean gain) per filter
            state["threshold"] = 3 * math.sqrt(70e-6 * _tables(case).total_filters / T)
        else:
            state["z"].append(torch.empty((T, n), dtype=torch.complex64, device="cuda"))
    if case["entry"] == "batch":
        state["requests"] = [(b, x, z, spiir.workspace_empty(b.workspace_bytes))
                             for b, x, z in zip(state["banks"], state["x"], state["z"])]
    if case["entry"] == "graph":
        state["input"] = torch.empty_like(state["x"][0])
        state["graph"] = spiir.Graph([(state["banks"][0], state["input"], state["z"][0])])
    return state


def run(state):
    entry, bank, x = state["entry"], state["banks"][0], state["x"][0]
    if entry == "peaks":
        bank.process_peaks(x, None, state["peaks"], state["threshold"])
        p = state["peaks"]
        return {"peak2": p[:, 0].view(torch.float32), "index": p[:, 1], "n_above": p[:, 2]}
    if entry == "graph":
        state["input"].copy_(x)
        state["graph"].launch()
    elif entry == "batch":
        spiir.spiir_process_batch(state["requests"])
    else:
        bank.process_block(x, state["z"][0])
    return state["z"]


def work(case):
    """Tables and states once per bank (a1, b0 and the state as complex64, the
    delay, the state back), the strain in, z (or the peaks) out; 12 flops per
    filter-sample, the resamplers' multiply-adds."""
    nf = _counts(case)
    H, T = case["bands"], case["templates"]
    out = 0
    flops = 12 * _filter_samples(case)
    for n in _lengths(case):
        out += 4 * n + (12 * T if case["entry"] == "peaks" else 8 * T * n) + 36 * int(nf.sum())
        flops += sum(64 * (n >> h) for h in range(1, H)) + T * sum(66 * (n >> h) for h in range(H - 1))
    return {"bytes": out, "flops": flops}


# ---------------------------------------------------------------- 64 bits


def _padded(case, band):
    """a1, b0 and delay of one band as [templates, most filters], zeros beyond a template's own."""
    t = _tables(case)
    m, off = t.n_filters[:, band].astype(np.int64), t.offsets()[:, band]
    at = off[:, None] + np.arange(max(int(m.max()), 1))[None, :]
    used = np.arange(at.shape[1])[None, :] < m[:, None]
    at = np.where(used, at, 0)
    a, b, d = np.where(used, t.a1[at], 0), np.where(used, t.b0[at], 0), np.where(used, t.delay[at], 0)
    return [torch.from_numpy(v).cuda() for v in (a, b, d.astype(np.int64))]


def exact(case, seed):
    """The block from zero state in float64: the recurrence sample by sample, the
    sum over a template's filters, the halving and doubling FIRs written out."""
    t, H, T = _tables(case), case["bands"], case["templates"]
    hd, hu = torch.from_numpy(np.array(t.h_down)).cuda(), torch.from_numpy(np.array(t.h_up)).cuda()
    answers = []
    for s, n in enumerate(_lengths(case)):
        x = _strain(case, seed, s).double().cuda()
        xs = [x]
        for _ in range(1, H):
            full = torch.nn.functional.conv1d(torch.nn.functional.pad(xs[-1], (len(hd) - 1, 0))[None, None],
                                              hd.flip(0)[None, None])[0, 0]
            xs.append(full[::2].contiguous())
        acc = None
        for h in range(H - 1, -1, -1):
            a, b, d = _padded(case, h)
            nh, dmax = n >> h, int(d.max())
            xp = torch.nn.functional.pad(xs[h], (dmax, 0))
            back = dmax - d
            y = torch.zeros_like(a)
            z = torch.empty((T, nh), dtype=torch.complex128, device="cuda")
            for k in range(nh):
                y.mul_(a).addcmul_(b, xp[k:k + dmax + 1][back].to(torch.complex128))
                z[:, k] = y.sum(1)
            if acc is not None:
                for j in range(len(hu)):  # acc_h[k] += h_up[j] v[k - j], v[2m] = acc_{h+1}[m]
                    z[:, j::2] += hu[j] * acc[:, : len(range(j, nh, 2))]
            acc = z
        answers.append(acc)
    if case["entry"] == "peaks":
        return {"peak2": (answers[0].real ** 2 + answers[0].imag ** 2).max(1).values, "index": None, "n_above": None}
    return answers

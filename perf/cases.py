"""The work that users of the phasing library have it do, as cases that can be timed.

Families (each case names one; sizes, storage types and options are its other fields):

  read_job     fragments -> read graph -> solve -> haplotypes, the whole read-based method
  read_solve   a read graph in hand, one whole bSB solve with its readout
  read_steps   a read graph in hand, the first part of a schedule, state kept (checkpoint)
  read_trace   the energy of every replica all along a schedule (convergence view)
  snp_job      fragments -> SNP graph -> solve -> haplotypes, the whole SNP-based method
  snp_steps    an SNP graph in hand, with or without Pore-C contacts, the first part of a
               schedule, state kept
  snp_refine   an SNP graph in hand, the adaptive multi-round refinement
  batch_solve  the blocks of a sample, graphs in hand, one solve of all of them
  batch_job    the blocks of a sample from fragments to haplotypes

Inputs are synthetic reads of the shapes that the paper's data have: a planted haplotype,
reads of either haplotype over consecutive SNPs, independent allele flips, uniform Phred
qualities.  SNP graphs are built in fixed point (deterministic), as a pipeline that has to
give the same answer twice does.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2603_25762_amd as qh

DEV = "cuda"


def listed():
    return [
        # the smallest job: one region of 60 reads, plain FP32, latency of everything
        dict(name="tiny_read_job", family="read_job", reads=60, snps=200, span=40, dtype="f32", replicas=16,
             steps=1000),
        # the MHC read graph of the paper's read-based runs, whole solve of many samples
        dict(name="mhc_read_solve", family="read_solve", reads=8000, snps=12000, span=45, dtype="bf16",
             replicas=256, steps=2000),
        # a checkpointed part of a schedule on a ragged, mid-sized read graph in plain FP32
        dict(name="read_f32_steps", family="read_steps", reads=1501, snps=2300, span=45, dtype="f32", replicas=64,
             steps=1000, upto=250, discrete=False),
        # the energy all along a run (solver comparison), a readout every 50 steps
        dict(name="read_trace", family="read_trace", reads=3000, snps=4500, span=45, dtype="f16", replicas=64,
             steps=1000, every=50),
        # one region by the SNP-based method with its adaptive settings, end to end
        dict(name="region_snp_job", family="snp_job", snps=2001, gap=1430.0, read_len=20000.0, coverage=30.0,
             dtype="f16"),
        # the multi-round refinement of an MHC-sized, densely linked SNP graph
        dict(name="mhc_snp_refine", family="snp_refine", snps=7768, gap=515.0, read_len=20000.0, coverage=50.0,
             dtype="f32", rounds=3, steps=1000, replicas=128),
        # a chromosome's solver steps, 16-bit couplings, state kept
        dict(name="chrom_snp_steps", family="snp_steps", snps=250000, gap=1430.0, read_len=20000.0, coverage=30.0,
             contacts=0, dtype="f16", replicas=64, steps=3000, upto=300, discrete=False),
        # the same with 600,000 long-range Pore-C contacts
        dict(name="chrom_porec_steps", family="snp_steps", snps=250000, gap=1430.0, read_len=20000.0, coverage=30.0,
             contacts=600000, dtype="bf16", replicas=64, steps=4000, upto=200, discrete=False),
        # a chromosome by the SNP-based method with its adaptive settings, end to end
        dict(name="chrom_snp_job", family="snp_job", snps=250000, gap=1430.0, read_len=20000.0, coverage=30.0,
             dtype="bf16"),
        # the benchmark's batch: 3,000 uneven blocks, dense FP8 read graphs and BF16 SNP graphs
        dict(name="batch_solve", family="batch_solve", blocks=3000, lo=50, hi=5000, read_share=0.5,
             read_dtype="fp8", snp_dtype="bf16", replicas=32, steps=500),
        # a smaller sample's blocks from fragments to haplotypes
        dict(name="batch_job", family="batch_job", blocks=300, lo=50, hi=5000, read_share=0.5, read_dtype="fp8",
             snp_dtype="bf16", replicas=32, steps=500),
        # a few small blocks only (a targeted panel), where one launch serves hardly any work
        dict(name="panel_batch_solve", family="batch_solve", blocks=24, lo=50, hi=900, read_share=0.5,
             read_dtype="f16", snp_dtype="f16", replicas=64, steps=500),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["read_job", "read_solve", "read_steps", "read_trace", "snp_job", "snp_steps", "snp_refine",
                         "batch_solve", "batch_job"])
    if family == "read_job":
        reads = _log(rng, 50, 8000)
        return dict(family=family, reads=reads, snps=max(150, int(reads * rng.uniform(0.3, 3.0))),
                    span=rng.randint(20, 60), dtype=rng.choice(["f32", "f16", "bf16", "fp8"]),
                    replicas=rng.choice([16, 32, 64]), steps=rng.randint(300, 1000))
    if family in ("read_solve", "read_trace"):
        reads = _log(rng, 500, 8000)
        c = dict(family=family, reads=reads, snps=int(reads * rng.uniform(1.0, 2.0)), span=rng.randint(30, 60),
                 dtype=rng.choice(["f16", "bf16", "fp8", "f32"]), replicas=rng.choice([32, 64, 128, 256]),
                 steps=rng.randint(500, 2000))
        if family == "read_trace":
            c["every"] = rng.randint(20, 100)
        return c
    if family == "read_steps":
        reads = _log(rng, 200, 8000)
        return dict(family=family, reads=reads, snps=int(reads * rng.uniform(1.0, 2.0)), span=rng.randint(20, 60),
                    dtype=rng.choice(["f32", "f32", "f16", "bf16"]), replicas=rng.choice([16, 32, 64, 128]),
                    steps=rng.randint(500, 2000), upto=rng.randint(50, 250), discrete=False)
    if family == "snp_job":
        return dict(family=family, snps=_log(rng, 200, 200000), gap=rng.uniform(500.0, 1500.0),
                    read_len=rng.uniform(15000.0, 25000.0), coverage=float(rng.randint(20, 50)),
                    dtype=rng.choice(["f32", "f16", "bf16"]))
    if family == "snp_steps":
        snps = _log(rng, 1000, 250000)
        return dict(family=family, snps=snps, gap=rng.uniform(800.0, 1500.0), read_len=rng.uniform(15000.0, 25000.0),
                    coverage=30.0, contacts=rng.choice([0, 0, int(snps * rng.uniform(0.5, 2.4))]),
                    dtype=rng.choice(["f32", "f16", "bf16"]), replicas=rng.choice([64, 64, 128]),
                    steps=rng.randint(1000, 4000), upto=rng.randint(50, 200), discrete=rng.random() < 0.15)
    if family == "snp_refine":
        return dict(family=family, snps=_log(rng, 1000, 20000), gap=rng.uniform(500.0, 1500.0), read_len=20000.0,
                    coverage=float(rng.randint(20, 50)), dtype=rng.choice(["f32", "f16", "bf16"]),
                    rounds=rng.randint(2, 5), steps=500, replicas=rng.choice([64, 128]))
    blocks = _log(rng, 16, 1500 if family == "batch_solve" else 300)
    lo = rng.choice([50, 50, 200])
    d16 = rng.choice(["f16", "bf16"])
    return dict(family=family, blocks=blocks, lo=lo, hi=rng.randint(800, 5000),
                read_share=rng.choice([0.0, 0.5, 0.5, 1.0]), read_dtype=rng.choice(["fp8", "fp8", d16]), snp_dtype=d16,
                replicas=rng.choice([16, 32, 32, 64]), steps=rng.randint(200, 500))


# ------------------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) & 0x7FFFFFFFFFFF)


def _observe(g, first, count, truth, err, q_lo, q_hi):
    """Fragments over the consecutive SNPs [first, first + count), on the GPU: each from
    either planted haplotype, alleles flipped at rate err, uniform Phred qualities."""
    first = torch.as_tensor(first, dtype=torch.int64, device=DEV)
    count = torch.as_tensor(count, dtype=torch.int64, device=DEV)
    ptr = torch.zeros(first.numel() + 1, dtype=torch.int64, device=DEV)
    ptr[1:] = torch.cumsum(count, 0)
    total = int(ptr[-1])
    snp = torch.repeat_interleave(first - ptr[:-1], count, output_size=total) + torch.arange(total, device=DEV)
    origin = torch.randint(0, 2, (first.numel(),), generator=g, device=DEV, dtype=torch.uint8)
    flip = (torch.rand(total, generator=g, device=DEV) < err).to(torch.uint8)
    allele = truth[snp] ^ torch.repeat_interleave(origin, count, output_size=total) ^ flip
    phred = torch.randint(q_lo, q_hi + 1, (total,), generator=g, device=DEV, dtype=torch.uint8)
    return ptr, snp, allele, phred


def _haplotypes(g, n_snp):
    truth = torch.randint(0, 2, (n_snp,), generator=g, device=DEV, dtype=torch.uint8)
    h1 = torch.randint(0, 2, (n_snp,), generator=g, device=DEV, dtype=torch.uint8)
    return truth, h1


def _reads(case, seed):
    """Reads of about `span` consecutive SNPs from uniform starts, sorted by their first SNP."""
    rng = np.random.default_rng([seed, 1])
    g = _gen(seed)
    n, m = case["snps"], case["span"]
    truth, h1 = _haplotypes(g, n)
    count = np.clip(np.round(rng.lognormal(math.log(m) - 0.08, 0.4, case["reads"])), 2, min(n, 4 * m)).astype(np.int64)
    first = (rng.random(case["reads"]) * (n - count + 1)).astype(np.int64)
    o = np.lexsort((count, first))
    ptr, snp, allele, phred = _observe(g, first[o], count[o], truth, 0.05, 10, 40)
    return dict(frag_ptr=ptr, snp=snp.int(), allele=allele, phred=phred, init_h1=h1)


def _spans(rng, pos, n_reads, read_len, lo, hi):
    """First SNP and SNP count of reads with lognormal lengths inside [lo, hi) (bp)."""
    ln = np.minimum(rng.lognormal(math.log(read_len) - 0.045, 0.3, n_reads), hi - lo - 1)
    st = lo + rng.random(n_reads) * (hi - lo - ln)
    a = np.searchsorted(pos, st)
    c = np.searchsorted(pos, st + ln) - a
    ok = c >= 2
    return a[ok], c[ok]


def _snp_reads(case, seed):
    """Long reads over SNPs with exponential gaps; contacts are fragments of two far SNPs."""
    rng = np.random.default_rng([seed, 2])
    g = _gen(seed)
    n = case["snps"]
    pos = np.cumsum(rng.exponential(case["gap"], n) + 1.0)
    truth, h1 = _haplotypes(g, n)
    n_reads = max(2, int(round(case["coverage"] * pos[-1] / case["read_len"])))
    first, count = _spans(rng, pos, n_reads, case["read_len"], 0.0, pos[-1] + 1.0)
    o = np.lexsort((count, first))
    ptr, snp, allele, phred = _observe(g, first[o], count[o], truth, 0.06, 7, 40)
    d = dict(frag_ptr=ptr, snp=snp.int(), allele=allele, phred=phred, init_h1=h1)
    m = int(case.get("contacts", 0))
    if m:
        # contact distance with density d^-1.1 over 100 kb to a third of the region; anchors
        # with a rank^-0.6 propensity, so that a few hub SNPs collect many contacts
        rank = np.empty(n)
        rank[rng.permutation(n)] = np.arange(1, n + 1)
        cdf = np.cumsum(rank ** -0.6)
        u = np.minimum(np.searchsorted(cdf, rng.random(m) * cdf[-1]), n - 1)
        ea, eb = 1e5 ** -0.1, max(2e5, min(1e8, pos[-1] / 3)) ** -0.1
        dist = (ea + rng.random(m) * (eb - ea)) ** -10.0
        v = np.clip(np.searchsorted(pos, pos[u] + np.where(rng.random(m) < 0.5, -dist, dist)), 0, n - 1)
        key = np.unique(np.minimum(u, v)[u != v] * n + np.maximum(u, v)[u != v])
        pair = torch.from_numpy(np.stack([key // n, key % n], 1)).to(DEV).reshape(-1)
        k = key.size
        org = torch.randint(0, 2, (k,), generator=g, device=DEV, dtype=torch.uint8).repeat_interleave(2)
        flip = (torch.rand(2 * k, generator=g, device=DEV) < 0.06).to(torch.uint8)
        f = ptr.numel() - 1
        d["frag_ptr"] = torch.cat([ptr, ptr[-1] + 2 * torch.arange(1, k + 1, device=DEV)])
        d["snp"] = torch.cat([d["snp"], pair.int()])
        d["allele"] = torch.cat([allele, truth[pair] ^ org ^ flip])
        d["phred"] = torch.cat([phred, torch.randint(7, 41, (2 * k,), generator=g, device=DEV, dtype=torch.uint8)])
        d["alpha"] = torch.cat([torch.ones(f, dtype=torch.float64, device=DEV),
                                torch.from_numpy(rng.uniform(0.1, 0.5, k)).to(DEV)])
    return d


def _batch(case, seed):
    """Specs of the sample's blocks: log-uniform vertex counts, a share of read blocks (reads of
    20-60 SNPs over 200) and SNP blocks (30x of 20 kb reads, 1,430 bp gaps), drawn together."""
    rng = np.random.default_rng([seed, 3])
    g = _gen(seed)
    nb = case["blocks"]
    # the block sizes belong to the case: another seed draws other reads over the same blocks
    size = np.round(np.exp(np.random.default_rng(nb).uniform(math.log(case["lo"]), math.log(case["hi"]), nb)))
    size = size.astype(np.int64)
    is_read = np.arange(nb) % 2 == 0 if case["read_share"] == 0.5 else np.full(nb, case["read_share"] > 0.5)
    n_snp = np.where(is_read, 200, size)
    base = np.concatenate([[0], np.cumsum(n_snp)])
    # the SNPs of all blocks on one axis, every block a stretch of its own
    pos = np.cumsum(rng.exponential(1430.0, int(base[-1])) + 1.0)
    lo, hi = pos[base[:-1]], pos[base[1:] - 1]
    n_reads = np.where(is_read, size, np.maximum(2, np.round(30.0 * (hi - lo) / 20000.0))).astype(np.int64)
    blk = np.repeat(np.arange(nb), n_reads)
    m = blk.size
    ln = np.minimum(rng.lognormal(math.log(20000.0) - 0.045, 0.3, m), (hi - lo)[blk] * 0.999)
    st = lo[blk] + rng.random(m) * ((hi - lo)[blk] - ln)
    p = torch.from_numpy(pos).to(DEV)
    first = torch.searchsorted(p, torch.from_numpy(st).to(DEV))
    count = torch.searchsorted(p, torch.from_numpy(st + ln).to(DEV)) - first
    rd = torch.from_numpy(is_read[blk]).to(DEV)
    rc = torch.randint(20, 61, (m,), generator=g, device=DEV)
    rf = (torch.rand(m, generator=g, device=DEV, dtype=torch.float64) * (201 - rc)).long()
    b = torch.from_numpy(blk).to(DEV)
    first = torch.where(rd, rf + torch.from_numpy(base[:-1]).to(DEV)[b], first)
    count = torch.where(rd, rc, count)
    keep = count >= 2
    first, count, b = first[keep], count[keep], b[keep]
    o = torch.argsort(first * 65536 + count, stable=True)          # blocks are stretches of one axis: in order too
    first, count, b = first[o], count[o], b[o]
    truth, h1 = _haplotypes(g, int(base[-1]))
    ptr, snp, allele, phred = _observe(g, first, count, truth, 0.055, 10, 40)
    snp = (snp - torch.repeat_interleave(torch.from_numpy(base[:-1]).to(DEV)[b], count)).int()
    frags = torch.bincount(b, minlength=nb).cpu().numpy()
    f0 = np.concatenate([[0], np.cumsum(frags)])
    # every block's own fragment pointers (from 0), one after another
    fb = torch.from_numpy(f0).to(DEV)
    start = ptr[fb[:-1]]
    rows = torch.from_numpy(np.repeat(np.arange(nb), frags + 1)).to(DEV)
    at = torch.arange(rows.numel(), device=DEV) - rows
    local = ptr[at] - start[rows]
    o0 = ptr[fb].cpu().numpy()
    specs = []
    for i in range(nb):
        a, z = int(o0[i]), int(o0[i + 1])
        d = dict(frag_ptr=local[f0[i] + i:f0[i + 1] + i + 1], snp=snp[a:z], allele=allele[a:z], phred=phred[a:z],
                 init_h1=h1[base[i]:base[i + 1]])
        d.update(dict(kind="read_signed", dtype=case["read_dtype"]) if is_read[i] else
                 dict(kind="snp_llr", dtype=case["snp_dtype"], deterministic=True))
        specs.append(d)
    return specs


def _graph(case, reads):
    if case["family"].startswith("read"):
        return qh.build_graph(**reads, kind="read_signed", dtype=case["dtype"])
    return qh.build_graph(**reads, kind="snp_llr", dtype=case["dtype"], deterministic=True,
                          band_limit=64 if case.get("contacts") else 0)


def prepare(case, seed):
    family = case["family"]
    s = dict(case=case, seed=seed)
    if family.startswith("batch"):
        s["specs"] = _batch(case, seed)
        if family == "batch_solve":
            s["graphs"] = qh.build_graphs(s.pop("specs"))
        return s
    s["reads"] = _reads(case, seed) if family.startswith("read") else _snp_reads(case, seed)
    if not family.endswith("job"):
        s["graph"] = _graph(case, s.pop("reads"))
    if family.endswith("steps"):
        n = s["graph"].info()["n"]
        s["x"] = torch.zeros((n, case["replicas"]), dtype=torch.float32, device=DEV)
        s["y"] = torch.zeros((n, case["replicas"]), dtype=torch.float32, device=DEV)
    return s


# ------------------------------------------------------------------------------ one pass

def _answers(r):
    return {k: r[k] for k in ("best_spins", "cuts", "best_cut", "selected_cut")}


def run(state):
    case, seed, family = state["case"], state["seed"], state["case"]["family"]
    if family.startswith("batch"):
        graphs = state["graphs"] if family == "batch_solve" else qh.build_graphs(state["specs"])
        r = qh.bsb_solve_batched(graphs, case["replicas"], case["steps"], seed=seed, use_graph=True)
        out = _answers(r)
        if family == "batch_job":
            out["h1"], out["block"], _ = qh.phase_batched(graphs, r["best_spins"])
        return out
    if family.endswith("job"):
        g = _graph(case, state["reads"])
        if family == "read_job":
            r = qh.bsb_solve(g, case["replicas"], case["steps"], seed=seed)
        else:
            a = qh.adaptive_schedule(g)
            r = qh.bsb_solve(g, a["replicas"], a["steps"], seed=seed)
        out = _answers(r)
        out["h1"], out["block"] = qh.phase(g, r["best_spins"])
        return out
    g = state["graph"]
    if family == "read_solve":
        return _answers(qh.bsb_solve(g, case["replicas"], case["steps"], seed=seed))
    if family == "read_trace":
        t = qh.energy_trace(g, case["replicas"], case["steps"], case["every"], seed=seed)
        return dict(energy=t["energy"], best=t["best"])
    if family == "snp_refine":
        r = qh.refine(g, case["replicas"], case["steps"], max_rounds=case["rounds"], seed=seed)
        cuts = r["round_cuts"] + [0.0] * (case["rounds"] - r["rounds"])      # rounds that flipped nothing: 0
        return dict(h1=r["h1"], block=r["block"], flips=r["flips"], round_cuts=np.array(cuts), rounds=r["rounds"])
    qh.bsb_solve(g, case["replicas"], case["steps"], seed=seed, step_end=case["upto"], x=state["x"], y=state["y"],
                 discrete=case["discrete"], readout=False)
    return dict(x=state["x"], y=state["y"])


# ------------------------------------------------------------------------------ the work of a pass

def _linked(case):
    """Couplings per vertex: reads that share a SNP with a read, SNPs that share a read with a SNP."""
    if case["family"].startswith("read"):
        return min(2.0 * case["span"] * case["reads"] / case["snps"], case["reads"] - 1.0)
    return min(2.9 * case["read_len"] / case["gap"], case["snps"] - 1.0) + 2.0 * case.get("contacts", 0) / case["snps"]


_BYTES = {"f32": 4, "f16": 2, "bf16": 2, "fp8": 1}
_TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def work(case):
    """Couplings (or fragments) read once, results written once; one multiply-add per coupling,
    replica and step."""
    family = case["family"]
    if family.startswith("batch"):
        # log-uniform sizes: mean and mean square; a read pair shares a SNP with chance 0.36
        span = math.log(case["hi"] / case["lo"])
        m1 = (case["hi"] - case["lo"]) / span
        m2 = (case["hi"] ** 2 - case["lo"] ** 2) / (2 * span)
        reads = case["blocks"] * case["read_share"]
        snps = case["blocks"] - reads
        nnz_r, nnz_s = 0.36 * m2 * reads, 40.0 * m1 * snps
        obs = 40.0 * m1 * reads + 20.0 * m1 * snps
        n = m1 * case["blocks"]
        held = nnz_r * _BYTES[case["read_dtype"]] + nnz_s * _BYTES[case["snp_dtype"]]
        return dict(bytes=(held if family == "batch_solve" else 6.0 * obs) + n,
                    flops=2.0 * (nnz_r + nnz_s) * case["replicas"] * case["steps"])
    n = case["reads"] if family.startswith("read") else case["snps"]
    nnz = _linked(case) * n
    replicas, steps = case.get("replicas", 128), case.get("upto", case.get("steps", 500 if n < 5000 else 1000))
    obs = case["span"] * n if family.startswith("read") else case["coverage"] * n
    out = 8.0 * n * replicas if family.endswith("steps") else 6.0 * n
    given = 6.0 * obs if family.endswith("job") else nnz * _BYTES[case["dtype"]]
    return dict(bytes=given + out, flops=2.0 * nnz * replicas * steps * case.get("rounds", 1))


# ------------------------------------------------------------------------------ in 64 bits

def _draws(seed, n, replicas):
    """x0, y0 ~ U(-0.1, 0.1) from SplitMix64, draw 2 (r n + i) + {0, 1}, held in 32 bits."""
    k = 2 * (np.arange(replicas, dtype=np.uint64)[None, :] * np.uint64(n) + np.arange(n, dtype=np.uint64)[:, None])

    def u(c):
        z = np.uint64(seed) + (c + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
        return 0.2 * ((z >> np.uint64(11)).astype(np.float64) * 2.0 ** -53) - 0.1

    with np.errstate(over="ignore"):
        x, y = u(k), u(k + np.uint64(1))
    return (torch.from_numpy(a.astype(np.float32)).to(DEV).double() for a in (x, y))


def _read_couplings(case, seed):
    d = _reads(case, seed)
    n = case["reads"]
    row = torch.repeat_interleave(torch.arange(n, device=DEV), torch.diff(d["frag_ptr"]))
    m = torch.zeros((n, case["snps"]), dtype=torch.float64, device=DEV)
    m[row, d["snp"].long()] = torch.where(d["allele"] == d["init_h1"][d["snp"].long()], 1.0, -1.0).double()
    j = m @ m.t()
    j.fill_diagonal_(0.0)
    return j, float((j * j).sum())


def _snp_couplings(case, seed):
    """J = -w, w_uv = -sum alpha l / (|S| - 1) over the fragments that hold both SNPs."""
    d = _snp_reads(case, seed)
    n, snp = case["snps"], d["snp"].long()
    count = torch.diff(d["frag_ptr"])
    frag = torch.repeat_interleave(torch.arange(count.numel(), device=DEV), count)
    q = 1.0 - 10.0 ** (-d["phred"].double() / 10.0)
    sign = torch.where(d["allele"] == d["init_h1"][snp], 1.0, -1.0).double()
    alpha = d.get("alpha")
    keys, vals = [], []
    for k in range(1, int(count.max())):
        a = torch.nonzero(frag[k:] == frag[:-k]).flatten()
        b = a + k
        cis = q[a] * q[b] + (1.0 - q[a]) * (1.0 - q[b])
        w = sign[a] * sign[b] * torch.log10(cis / (q[a] + q[b] - 2.0 * q[a] * q[b])) / (count[frag[a]] - 1).double()
        w = w if alpha is None else w * alpha[frag[a]]
        key, inv = torch.unique(snp[a] * n + snp[b], return_inverse=True)
        keys.append(key)
        vals.append(torch.zeros(key.numel(), dtype=torch.float64, device=DEV).index_add_(0, inv, w))
    key, inv = torch.unique(torch.cat(keys), return_inverse=True)
    w = torch.zeros(key.numel(), dtype=torch.float64, device=DEV).index_add_(0, inv, torch.cat(vals))
    u, v = key // n, key % n
    square = 2.0 * float((w * w).sum())
    w = w.to(_TORCH[case["dtype"]]).double()        # the couplings as the storage type holds them
    j = torch.sparse_coo_tensor(torch.stack([torch.cat([u, v]), torch.cat([v, u])]), torch.cat([w, w]), (n, n))
    return j.coalesce().to_sparse_csr(), square


def exact(case, seed):
    """The state after the first part of a schedule, stepped in 64 bits from the fragments'
    couplings, rounded to the storage type that the case asks for.  Whole runs end in spins
    that have no such value: two runs whose arithmetic differs in the last bit may pick
    different samples."""
    family = case["family"]
    if not family.endswith("steps"):
        return None
    replicas = case["replicas"]
    n = case["reads"] if family == "read_steps" else case["snps"]
    if n * float(replicas) * case["upto"] * (n if family == "read_steps" else 200) > 4e12:
        return None                  # over a few tens of seconds in 64 bits
    j, square = (_read_couplings if family == "read_steps" else _snp_couplings)(case, seed)
    c0 = 0.5 / math.sqrt(square / (n - 1))
    x, y = _draws(seed, n, replicas)
    for k in range(case["upto"]):
        p = k / (case["steps"] - 1)
        z = j @ (torch.where(x >= 0, 1.0, -1.0).double() if case["discrete"] else x)
        y = y + (-(1.0 - p) * x + c0 * z) * 0.5
        x = x + y * 0.5
        wall = x.abs() > 1.0
        x = x.clamp(-1.0, 1.0)
        y = torch.where(wall, 0.0, y)
    return dict(x=x, y=y)

"""GPU-vs-oracle parity of the gfx950 library, called through its C ABI.

Every expected value comes from ``oracle/`` (or the paper): graph weights
(bit-exact for integer kinds, <= 1e-12 of the summed |terms| for the SNP
log-likelihood weights), stored number formats (bit-exact against the oracle's
software rounding), one bSB step (<= 1e-5 of the step's own magnitude), the
FP64 readout (exact for integer weights), phasing (exact), and the final best
cut of a whole solve (<= 0.1 % below the FP64 oracle, equal switch error).
"""
import ctypes
import json

import numpy as np
import pytest
import torch

import oracle
import paper_2603_25762_amd as qh
import synth
from oracle import metrics, quant
from gpu_helpers import (COPY_ABS, COPY_UNIT, cpu, device_reads, f32, far_mask, gpu_graph, oracle_graph,
                         snp_abs_terms, step_bounds, step_with_rounded_copy)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    qh.load()
    yield
    torch.cuda.synchronize()


FMT = {"f32": None, "f16": "f16", "bf16": "bf16", "fp8": "f16"}


def stored_J(J, dtype):
    if dtype == "f32":
        return quant.round_to("f32", J)
    if dtype == "fp8":
        scale, q = quant.rowscale_e4m3(J)
        return scale[:, None] * q
    return quant.round_to(dtype, J)


# ----------------------------------------------------------------------------- graphs

READ_CASES = {
    "tiny": lambda: synth.read_tiny(),
    "ragged300": lambda: synth.read_small(5, n_snp=400, n_reads=300, span=(10, 60)),
    "sparse_many_comps": lambda: synth.read_small(6, n_snp=2000, n_reads=130, span=(3, 12)),
    # reads plus Pore-C contact fragments, which the read-based method merges unweighted
    "porec_merged": lambda: synth.snp_porec(43, n_snp=600, n_edges=500, zipf_s=1.0),
}


@pytest.mark.parametrize("kind", ["read_signed", "read_conflict"])
@pytest.mark.parametrize("case", list(READ_CASES))
def test_read_graph_bit_exact(kind, case):
    w = READ_CASES[case]()
    g = gpu_graph(w, kind)
    go = oracle_graph(w, kind)
    info = g.info()
    assert info["n"] == go.n and info["integer_weights"] == 1
    assert np.array_equal(cpu(g.export_rows(0, go.n)), go.dense())
    comp, nc = oracle.components(go)
    assert info["n_comp"] == nc
    assert np.array_equal(cpu(g.components()), comp)
    assert info["nnz"] == go.nnz
    assert info["c0_auto"] == pytest.approx(oracle.c0(go), rel=1e-15)
    if case == "porec_merged":
        # Pore-C fragments join the read graph without their down-weighting factor
        assert np.any(w.alpha != 1.0)
        g1 = gpu_graph(w, kind, with_alpha=False)
        assert torch.equal(g1.export_rows(0, go.n), g.export_rows(0, go.n))


def _oracle_read_row(w, kind, p):
    """Row p of the oracle's read graph from the oracle run on read p and the reads sharing a
    SNP with it (an entry (p, q) depends on reads p and q alone), mapped back to all reads."""
    fp, snp = w.frag_ptr, w.snp
    owner = np.repeat(np.arange(len(fp) - 1), np.diff(fp))
    qs = np.unique(owner[np.isin(snp, snp[fp[p]:fp[p + 1]])])
    lens = np.diff(fp)[qs]
    sub_fp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    take = np.concatenate([np.arange(fp[q], fp[q + 1]) for q in qs])
    M = oracle.encode(snp[take], w.allele[take], w.init_h1)
    go = oracle.read_graph(w.n_snp, sub_fp, snp[take], M, "signed" if kind == "read_signed" else "conflict")
    i = int(np.searchsorted(qs, p))
    row = np.zeros(len(fp) - 1)
    b, e = go.row_ptr[i], go.row_ptr[i + 1]
    row[qs[go.col[b:e]]] = go.val[b:e]
    return row


@pytest.mark.parametrize("n_reads,kind", [(20000, "read_signed"), (40000, "read_conflict")])
def test_read_graph_large_fragment_counts(n_reads, kind):
    """Eqs. (2)-(3) past the row kernel's small-LDS case: 20,000 reads need 80 KB of LDS per
    row (the large-LDS launch), 40,000 go past its limit to the per-SNP kernel with global
    atomics.  Sampled rows of the FP64 master equal the oracle's bit for bit (each from the
    oracle on the reads that share a SNP with the row's read); at 20,000 reads the whole
    oracle graph also gives the nonzero count and the components."""
    w = synth.read_small(61, n_snp=4000, n_reads=n_reads, span=(2, 6))
    g = gpu_graph(w, kind)
    n = g.info()["n"]
    assert n == n_reads and g.info()["integer_weights"] == 1
    rng = np.random.default_rng(5)
    for r in sorted({0, 1, n // 3, n // 2, n - 2, n - 1, *rng.integers(0, n, 24).tolist()}):
        assert np.array_equal(cpu(g.export_rows(r, r + 1))[0], _oracle_read_row(w, kind, r)), r
    if n_reads <= 20000:
        go = oracle_graph(w, kind)
        assert g.info()["nnz"] == go.nnz
        comp, nc = oracle.components(go)
        assert g.info()["n_comp"] == nc
        assert np.array_equal(cpu(g.components()), comp)
    g.free()


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16", "fp8"])
def test_dense_stored_values_bit_exact(dtype):
    w = synth.read_small(9, n_snp=300, n_reads=200, span=(20, 60))
    g = gpu_graph(w, "read_signed", dtype)
    J = oracle_graph(w).dense()
    S = cpu(g.export_rows(0, g.info()["n"], stored=True))
    assert np.array_equal(S, stored_J(J, dtype))
    tiles = g.info()["dense_tiles"]
    assert 0 < tiles <= 4 * 4


@pytest.fixture(scope="module")
def mhc():
    w = synth.read_mhc()
    M = oracle.encode(w.snp, w.allele, w.init_h1)
    W, _ = oracle.read_graph_dense(w.n_snp, w.frag_ptr, w.snp, M, "signed")
    return w, W


def test_read_graph_mhc_scale_sampled_rows(mhc):
    """Full MHC-scale read graph (8,000 reads): sampled rows, master and FP16 copy."""
    w, W = mhc
    g = gpu_graph(w, "read_signed", "f16")
    n = g.info()["n"]
    assert n == W.shape[0]
    rows = sorted(set([0, 1, 63, 64, 65, n // 2, n - 65, n - 64, n - 2, n - 1] +
                      list(np.random.default_rng(0).integers(0, n, 40))))
    for r in rows:
        assert np.array_equal(cpu(g.export_rows(r, r + 1))[0], W[r].astype(np.float64)), r
        assert np.array_equal(cpu(g.export_rows(r, r + 1, stored=True))[0],
                              quant.round_to("f16", W[r].astype(np.float64))), r
    assert g.info()["nnz"] == int(np.count_nonzero(W))


SNP_CASES = {
    "snp2000": dict(make=lambda: synth.snp_small(3, n_snp=2000), k=10, band=0),
    "snp2000_k5": dict(make=lambda: synth.snp_small(4, n_snp=2000), k=5, band=0),
    "snp_q_low": dict(make=lambda: synth.snp_small(12, n_snp=800, q=(2, 12)), k=10, band=0),
    "porec3000": dict(make=lambda: synth.snp_porec(41, n_snp=3000, n_edges=3000, zipf_s=1.0), k=10,
                      band=100),
    # eight fragments of 500-1,336 SNPs: longer than the builder's per-wave LDS staging
    "snp_long_reads": dict(make=lambda: synth.snp_small(13, n_snp=1500, coverage=4.0, read_mean=80000.0,
                                                        gap_mean=100.0), k=2, band=0),
    "snp_long_reads_band": dict(make=lambda: synth.snp_small(13, n_snp=1500, coverage=4.0, read_mean=80000.0,
                                                             gap_mean=100.0), k=2, band=50),
}


@pytest.mark.parametrize("case", list(SNP_CASES))
def test_snp_graph_normwise(case):
    c = SNP_CASES[case]
    w = c["make"]()
    g = gpu_graph(w, "snp_llr", "f32", linkage_k=c["k"], band_limit=c["band"])
    go = oracle_graph(w, "snp_llr", c["k"])
    D = cpu(g.export_rows(0, go.n))
    T = snp_abs_terms(w, c["k"])
    assert np.all(np.abs(D - go.dense()) <= 1e-12 * T)
    comp, nc = oracle.components(go)
    assert g.info()["n_comp"] == nc
    assert np.array_equal(cpu(g.components()), comp)
    if c["band"]:
        assert g.info()["longrange_nnz"] > 0


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_skyline_stored_values_bit_exact(dtype):
    w = synth.snp_porec(42, n_snp=1500, n_edges=1500, zipf_s=1.0)
    g = gpu_graph(w, "snp_llr", dtype, band_limit=100)
    S = cpu(g.export_rows(0, g.info()["n"], stored=True))
    J = oracle_graph(w, "snp_llr").dense()
    tol = 1e-12 * snp_abs_terms(w)
    lo, hi = quant.round_to(dtype, J - tol), quant.round_to(dtype, J + tol)
    if dtype == "bf16":
        # BF16 storage flushes magnitudes below 2^(E - 31), E = exponent of the largest weight
        thr = 2.0 ** (np.floor(np.log2(np.abs(J).max())) - 31)
        lo = np.where(np.abs(J) + tol < thr, 0.0, lo)
        hi = np.where(np.abs(J) - tol < thr, np.where(np.abs(J) + tol < thr, 0.0, hi), hi)
        maybe = (np.abs(J) - tol < thr) & (np.abs(J) + tol >= thr)
        assert np.all(np.where(maybe, (S == 0) | (S == lo) | (S == hi), True))
        lo = np.where(maybe, S, lo)
        hi = np.where(maybe, S, hi)
    sure = lo == hi          # the master's last-bit freedom cannot move the rounding
    assert sure.mean() > 0.999
    assert np.array_equal(S[sure], lo[sure])
    assert np.all((S[~sure] == lo[~sure]) | (S[~sure] == hi[~sure]))


# ----------------------------------------------------------------------------- one step

def _one_step_case(g, J, dtype, R, rng_seed, product_format, steps=100, k=37, plan=0, discrete=False,
                   field=False, lr_band=None):
    n = J.shape[0]
    rng = np.random.default_rng(rng_seed)
    x0 = f32(rng.uniform(-1.0, 1.0, (n, R)))
    y0 = f32(rng.uniform(-0.6, 0.6, (n, R)))
    # deformation field: a few units of the typical coupling sum, zero on some rows
    h = f32(rng.normal(0.0, 1.0, n) * max(1.0, float(np.abs(J).sum(axis=1).mean()))) if field else None
    if field:
        h[::7] = 0.0
    pump = np.linspace(0.0, 1.0, steps).astype(np.float32)
    c0 = 0.4 / max(1.0, float(np.sqrt((J ** 2).sum() / max(n - 1, 1))))
    c0 = float(np.float32(c0))
    p = float(pump[k])
    dt = 0.5
    x = torch.tensor(x0, dtype=torch.float32, device="cuda").contiguous()
    y = torch.tensor(y0, dtype=torch.float32, device="cuda").contiguous()
    qh.bsb_solve(g, R, steps, dt=dt, c0=c0, pump=torch.tensor(pump, device="cuda"), init=False,
                 x=x, y=y, step_begin=k, step_end=k + 1, readout=False, plan=plan, discrete=discrete,
                 field=None if h is None else torch.tensor(h, dtype=torch.float32, device="cuda"))
    xg, yg = cpu(x).astype(np.float64), cpu(y).astype(np.float64)
    xu, yu = step_with_rounded_copy(J, x0, y0, p, dt, c0, 1.0, product_format, walls=False, discrete=discrete,
                                    field=h, lr_band=lr_band)
    xo, yo = step_with_rounded_copy(J, x0, y0, p, dt, c0, 1.0, product_format, walls=True, discrete=discrete,
                                    field=h, lr_band=lr_band)
    if discrete:
        xq = np.ones_like(x0)
    else:
        xq = x0 if product_format is None else quant.round_to(product_format, x0)
    mag = np.abs(J) @ np.abs(xq)
    if h is not None:
        mag = mag + np.abs(h)[:, None]
    tol_x, tol_y = step_bounds(mag, x0, y0, p, dt, c0)
    ambiguous = np.abs(np.abs(xu) - 1.0) <= tol_x
    ok = ~ambiguous
    assert ok.mean() > 0.9
    assert np.all(np.abs(xg - xo)[ok] <= tol_x[ok])
    assert np.all(np.abs(yg - yo)[ok] <= tol_y[ok])
    assert np.all(np.abs(xg) <= 1.0)
    assert np.all(yg[np.abs(xg) == 1.0][~ambiguous[np.abs(xg) == 1.0]] == 0.0)


@pytest.mark.parametrize("plan", [1, 2, 0])       # per-step kernel; persistent kernel; autotuned
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16", "fp8"])
@pytest.mark.parametrize("R", [16, 32, 64, 128])
def test_dense_one_step(dtype, R, plan):
    if plan == 2 and dtype == "f32":
        pytest.skip("the persistent plan is offered for 16- and 8-bit dense storage")
    w = synth.read_small(13, n_snp=300, n_reads=150, span=(20, 60))     # 3 row tiles, ragged tail
    g = gpu_graph(w, "read_signed", dtype)
    J = stored_J(oracle_graph(w).dense(), dtype)
    _one_step_case(g, J, dtype, R, 100 + R, FMT[dtype], plan=plan)


@pytest.mark.parametrize("plan", [1, 2])
@pytest.mark.parametrize("dtype", ["f16", "bf16", "fp8"])
def test_dense_one_step_against_unrounded_oracle(dtype, plan):
    """The 16-bit copy of x that the 16/8-bit dense products multiply, bounded against the
    oracle's unrounded step (stored J, FP64, x itself in the product): rounding x_j to the
    copy's format moves it by at most u |x_j| + a (u = 2^-11 for binary16, used by F16 and FP8
    tiles; 2^-8 for bfloat16; a = 2^-25 below binary16's normal range), so the coupling sum
    moves by at most sum_j |J_ij| (u |x_j| + a), y by c0 dt times that and x by a0 dt times
    y's bound, on top of the FP32 step tolerance."""
    w = synth.read_small(13, n_snp=300, n_reads=150, span=(20, 60))
    g = gpu_graph(w, "read_signed", dtype)
    J = stored_J(oracle_graph(w).dense(), dtype)
    n, R, k, steps, dt = J.shape[0], 64, 37, 100, 0.5
    fmt = FMT[dtype]
    rng = np.random.default_rng(321)
    x0 = f32(rng.uniform(-1.0, 1.0, (n, R)))
    y0 = f32(rng.uniform(-0.6, 0.6, (n, R)))
    pump = np.linspace(0.0, 1.0, steps).astype(np.float32)
    c0 = float(np.float32(0.4 / max(1.0, float(np.sqrt((J ** 2).sum() / (n - 1))))))
    p = float(pump[k])
    x = torch.tensor(x0, dtype=torch.float32, device="cuda").contiguous()
    y = torch.tensor(y0, dtype=torch.float32, device="cuda").contiguous()
    qh.bsb_solve(g, R, steps, dt=dt, c0=c0, pump=torch.tensor(pump, device="cuda"), init=False, x=x, y=y,
                 step_begin=k, step_end=k + 1, readout=False, plan=plan)
    xg, yg = cpu(x).astype(np.float64), cpu(y).astype(np.float64)
    xu, yu = oracle.bsb_step_dense(J, x0, y0, p, dt, c0, 1.0, walls=False)
    xo, yo = oracle.bsb_step_dense(J, x0, y0, p, dt, c0, 1.0, walls=True)
    tol_x, tol_y = step_bounds(np.abs(J) @ np.abs(x0), x0, y0, p, dt, c0)
    copy = c0 * dt * (np.abs(J) @ (COPY_UNIT[fmt] * np.abs(x0) + COPY_ABS[fmt]))
    tol_y = tol_y + copy
    tol_x = tol_x + dt * copy
    ok = np.abs(np.abs(xu) - 1.0) > tol_x        # entries not within the tolerance of a wall
    assert ok.mean() > 0.9
    assert np.all(np.abs(yg - yo)[ok] <= tol_y[ok])
    assert np.all(np.abs(xg - xo)[ok] <= tol_x[ok])
    # the bound is not vacuous: the copy's effect is visible and of the size it predicts
    dev = np.abs(yg - yo)[ok]
    assert dev.max() > 1e-3 * copy[ok].max()


@pytest.mark.parametrize("plan", [1, 2])
@pytest.mark.parametrize("dtype", ["f32", "f16", "fp8"])
@pytest.mark.parametrize("R", [32, 64])
def test_dense_one_step_discrete(dtype, R, plan):
    """Discrete variant: the coupling takes sgn(x_j) (sgn(0) = +1), on every dense path."""
    if plan == 2 and dtype == "f32":
        pytest.skip("the persistent plan is offered for 16- and 8-bit dense storage")
    w = synth.read_small(13, n_snp=300, n_reads=150, span=(20, 60))
    g = gpu_graph(w, "read_signed", dtype)
    J = stored_J(oracle_graph(w).dense(), dtype)
    _one_step_case(g, J, dtype, R, 700 + R, None, plan=plan, discrete=True)


@pytest.mark.parametrize("plan", [3, 4, 5])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_skyline_one_step_discrete(dtype, plan):
    w = synth.snp_porec(43, n_snp=2500, n_edges=4000, zipf_s=1.0)
    g = gpu_graph(w, "snp_llr", dtype, band_limit=100)
    assert g.info()["longrange_nnz"] > 0
    J = stored_J(oracle_graph(w, "snp_llr").dense(), dtype)
    _one_step_case(g, J, dtype, 64, 800, None, plan=plan, discrete=True)


@pytest.mark.parametrize("plan", [1, 2])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16", "fp8"])
def test_dense_one_step_field(dtype, plan):
    """Deformation field h on the dense paths: y' = y + (-(a0 - p) x + c0 (J x + h)) dt."""
    if plan == 2 and dtype == "f32":
        pytest.skip("the persistent plan is offered for 16- and 8-bit dense storage")
    w = synth.read_small(13, n_snp=300, n_reads=150, span=(20, 60))
    g = gpu_graph(w, "read_signed", dtype)
    J = stored_J(oracle_graph(w).dense(), dtype)
    _one_step_case(g, J, dtype, 64, 900, FMT[dtype], plan=plan, field=True)
    _one_step_case(g, J, dtype, 32, 901, None, plan=plan, discrete=True, field=True)


@pytest.mark.parametrize("plan", [3, 4, 5])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_skyline_one_step_field(dtype, plan):
    """The field on the SNP step kernels, with long-range rows (chunk partials) present (16-bit
    storage: the long-range entries multiply the binary16 copy of x)."""
    w = synth.snp_porec(43, n_snp=2500, n_edges=4000, zipf_s=1.0)
    g = gpu_graph(w, "snp_llr", dtype, band_limit=100)
    assert g.info()["longrange_nnz"] > 0
    J = stored_J(oracle_graph(w, "snp_llr").dense(), dtype)
    _one_step_case(g, J, dtype, 64, 902, None, plan=plan, field=True, lr_band=None if dtype == "f32" else 100)


def test_field_solves_match_oracle_plans_and_batches():
    """Whole solves under a field: the oracle's cut within 0.1 %; h = 0 is the plain solve
    bit for bit; every dense plan, the band kernels and the batched plans agree bit for
    bit with the per-step solve of each graph."""
    rng = np.random.default_rng(5)
    w = synth.read_tiny()
    g = gpu_graph(w, "read_signed", "f16")
    go = oracle_graph(w)
    n = g.info()["n"]
    h = f32(rng.normal(0.0, 2.0, n))
    ht = torch.tensor(h, dtype=torch.float32, device="cuda")
    ro = oracle.solve(go, 16, 1000, 0.5, seed=11, integer=True, field=h)
    rg = qh.bsb_solve(g, 16, 1000, seed=11, field=ht)
    assert _gap(ro["best_cut"], float(cpu(rg["best_cut"])[0])) <= 1e-3
    # h = 0 is no field
    for gg, plan in ((g, 1), (gpu_graph(synth.snp_small(61, n_snp=400), "snp_llr", "bf16"), 4)):
        m = gg.info()["n"]
        xa = torch.empty((m, 32), dtype=torch.float32, device="cuda")
        xb = torch.empty_like(xa)
        qh.bsb_solve(gg, 32, 200, seed=3, x=xa, readout=False, plan=plan)
        qh.bsb_solve(gg, 32, 200, seed=3, x=xb, readout=False, plan=plan,
                     field=torch.zeros(m, dtype=torch.float32, device="cuda"))
        assert torch.equal(xa, xb)
    # dense plans: per-step, persistent (both synchronisations), captured graph
    wm = synth.read_mhc(seed=78, n_snp=1500, n_reads=1000, region=500_000)
    gm = gpu_graph(wm, "read_signed", "f16")
    nm = gm.info()["n"]
    hm = torch.tensor(f32(rng.normal(0.0, 3.0, nm)), dtype=torch.float32, device="cuda")
    outs = []
    for plan, sync, ug in ((1, 0, False), (2, 1, False), (2, 2, False), (1, 0, True)):
        x = torch.empty((nm, 64), dtype=torch.float32, device="cuda")
        y = torch.empty((nm, 64), dtype=torch.float32, device="cuda")
        r = qh.bsb_solve(gm, 64, 300, seed=31, x=x, y=y, plan=plan, persistent_sync=sync, use_graph=ug, field=hm)
        outs.append((x, y, r))
    x0 = torch.empty((nm, 64), dtype=torch.float32, device="cuda")
    qh.bsb_solve(gm, 64, 300, seed=31, x=x0, plan=1)
    assert not torch.equal(x0, outs[0][0])            # the field changes the run
    for o in outs[1:]:
        assert torch.equal(outs[0][0], o[0]) and torch.equal(outs[0][1], o[1])
        assert torch.equal(outs[0][2]["best_cut"], o[2]["best_cut"])
    # SNP band kernels: rows = band FMA bit for bit, band MFMA to rounding
    wp = synth.snp_porec(43, n_snp=2500, n_edges=4000, zipf_s=1.0)
    gp = gpu_graph(wp, "snp_llr", "f32", band_limit=100)
    npv = gp.info()["n"]
    hp = torch.tensor(f32(rng.normal(0.0, 1.0, npv)), dtype=torch.float32, device="cuda")
    xs = {}
    for plan in (3, 4, 5):
        xs[plan] = torch.empty((npv, 64), dtype=torch.float32, device="cuda")
        qh.bsb_solve(gp, 64, 200, seed=4, x=xs[plan], readout=False, plan=plan, field=hp)
    assert torch.equal(xs[3], xs[4])
    assert float((xs[3] - xs[5]).abs().max()) <= 1e-2
    # batched: packed field, each block equal to its single solve
    blocks = [synth.read_small(50, n_snp=200, n_reads=40), synth.snp_small(60, n_snp=350), w]
    kinds = ["read_signed", "snp_llr", "read_signed"]
    gs = [gpu_graph(b, k, d) for b, k, d in zip(blocks, kinds, ["fp8", "bf16", "f16"])]
    ns = [gg.info()["n"] for gg in gs]
    hb = torch.tensor(f32(rng.normal(0.0, 2.0, sum(ns))), dtype=torch.float32, device="cuda")
    for plan in (1, 2):
        rb = qh.bsb_solve_batched(gs, 32, 300, seed=9, return_state=True, plan=plan, field=hb)
        off = rb["vertex_offset"]
        for b, gg in enumerate(gs):
            lo, hi = int(off[b]), int(off[b + 1])
            xs1 = torch.empty(ns[b], 32, dtype=torch.float32, device="cuda")
            rs = qh.bsb_solve(gg, 32, 300, seed=9, plan=1, x=xs1, field=hb[lo:hi].contiguous())
            assert torch.equal(rb["x"][lo * 32:hi * 32], xs1.reshape(-1)), (plan, b)
            assert torch.equal(rb["best_cut"][b:b + 1], rs["best_cut"]), (plan, b)
    with pytest.raises(ValueError):
        qh.bsb_solve(g, 16, 10, field=ht[:-1])
    with pytest.raises(TypeError):
        qh.bsb_solve(g, 16, 10, field=ht.double())


def test_refine_deformation_matches_oracle():
    """Adaptive deformation in the library's refinement equals the oracle's: on weights
    gauge-flipped around a good partition, rough two-step rounds (no greedy pass) cut
    negatively, so deformed re-solves run; the number run, the rounds, the applied cuts
    and the flip counters agree, and the weights are restored."""
    w = synth.snp_small(24, n_snp=800)
    go = oracle_graph(w, "snp_llr")
    s0 = oracle.solve(go, 16, 600, 0.5, seed=1)["best"]
    g = gpu_graph(w, "snp_llr", "f32")
    n = g.info()["n"]
    qh.flip_crossing(g, torch.tensor(s0, dtype=torch.int8, device="cuda"))
    g2 = oracle.flip_crossing(go, s0)
    master = cpu(g.export_rows(0, n))
    ro = oracle.refine(g2, w.init_h1, 16, 2, 0.5, seed=3, max_rounds=3, greedy_pass=False, deform=0.5,
                       deform_tries=4)
    rr = qh.refine(g, 16, 2, seed=3, max_rounds=3, greedy=False, deform=0.5, deform_tries=4)
    assert np.array_equal(cpu(g.export_rows(0, n)), master)
    assert ro["deformed"] >= 1
    assert rr["deformed"] == ro["deformed"] and rr["rounds"] == ro["rounds"]
    assert np.allclose(rr["round_cuts"], ro["round_cuts"], rtol=1e-9, atol=1e-9)
    assert np.array_equal(cpu(rr["flips"]), ro["flips"])
    # full-length rounds: the flip counters carry exactly the applied cuts
    rr = qh.refine(g, 16, 300, seed=3, max_rounds=4, deform=0.5, deform_tries=2)
    assert np.array_equal(cpu(g.export_rows(0, n)), master)
    comp, nc = oracle.components(g2)
    S = np.where(cpu(rr["flips"]) % 2 == 1, -1, 1).astype(np.int8)
    assert oracle.cuts(g2, comp, nc, S).sum() == pytest.approx(sum(rr["round_cuts"]), rel=1e-9, abs=1e-9)
    with pytest.raises(qh.QhapError) as e:
        qh.refine(g, 16, 10, deform=-1.0, deform_tries=1)
    assert e.value.status == qh.Status.EINVAL


def test_discrete_whole_solves_match_oracle_and_plans():
    """Discrete variant end to end: cut gap to the oracle's discrete solve, persistent =
    per-step bit for bit, batched = single bit for bit."""
    w = synth.read_tiny()
    g = gpu_graph(w, "read_signed", "f16")
    ro = oracle.solve(oracle_graph(w), 16, 1000, 0.5, seed=11, integer=True, discrete=True)
    rs = qh.bsb_solve(g, 16, 1000, seed=11, discrete=True)
    assert _gap(ro["best_cut"], float(cpu(rs["best_cut"])[0])) <= 1e-3
    wm = synth.read_mhc(seed=78, n_snp=1500, n_reads=1000, region=500_000)
    gm = gpu_graph(wm, "read_signed", "f16")
    n = gm.info()["n"]
    outs = []
    for plan, sync in ((1, 0), (2, 1), (2, 2)):
        x = torch.empty((n, 64), dtype=torch.float32, device="cuda")
        y = torch.empty((n, 64), dtype=torch.float32, device="cuda")
        r = qh.bsb_solve(gm, 64, 300, seed=31, x=x, y=y, plan=plan, discrete=True, persistent_sync=sync)
        outs.append((x, y, r))
    for o in outs[1:]:
        assert torch.equal(outs[0][0], o[0]) and torch.equal(outs[0][1], o[1])
        assert torch.equal(outs[0][2]["best_cut"], o[2]["best_cut"])
    ws = synth.snp_small(61, n_snp=400)
    gs_ = gpu_graph(ws, "snp_llr", "bf16")
    rb = qh.bsb_solve_batched([g, gs_], 32, 300, seed=9, discrete=True)
    for b, gg in enumerate((g, gs_)):
        r1 = qh.bsb_solve(gg, 32, 300, seed=9, discrete=True, plan=1)
        assert torch.equal(rb["best_cut"][b:b + 1], r1["best_cut"])
        lo, hi = int(rb["vertex_offset"][b]), int(rb["vertex_offset"][b + 1])
        assert torch.equal(rb["best_spins"][lo:hi], r1["best_spins"])


@pytest.mark.parametrize("dtype", ["f16", "bf16", "fp8"])
@pytest.mark.parametrize("R", [16, 64, 256])
def test_persistent_equals_per_step_bit_exact(dtype, R):
    """The persistent plan runs the same MFMA sequence and update as the per-step kernel,
    so 300 steps of both must agree bit for bit (state and readout), with either way of
    passing x between workgroups (cache-wide fences, device-coherent accesses)."""
    w = synth.read_mhc(seed=78, n_snp=1500, n_reads=1000, region=500_000)
    g = gpu_graph(w, "read_signed", dtype)
    n = g.info()["n"]
    out = []
    # one fused kernel per step; persistent with fences; persistent with coherent accesses
    for plan, sync in ((1, 0), (2, 1), (2, 2)):
        x = torch.empty((n, R), dtype=torch.float32, device="cuda")
        y = torch.empty((n, R), dtype=torch.float32, device="cuda")
        r = qh.bsb_solve(g, R, 300, seed=31, x=x, y=y, plan=plan, persistent_sync=sync)
        if plan == 2:
            info = g.plan_info(R)
            assert info["plan_used"] == 2 and info["persistent_sync"] == sync
        out.append((x, y, r))
    xa, ya, ra = out[0]
    for xb, yb, rb in out[1:]:
        assert torch.equal(xa, xb) and torch.equal(ya, yb)
        assert torch.equal(ra["best_spins"], rb["best_spins"]) and torch.equal(ra["best_cut"], rb["best_cut"])


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16", "fp8"])
def test_replica_tiles_bit_exact(dtype):
    """The per-step dense kernel with 64, 32 or 16 replicas per workgroup computes every
    replica's product and update identically; the autotuned plan equals them too."""
    w = synth.read_mhc(seed=79, n_snp=1500, n_reads=900, region=500_000)
    g = gpu_graph(w, "read_signed", dtype)
    n, R = g.info()["n"], 128
    out = []
    for tile, depth in ((64, 2), (64, 4), (32, 0), (16, 0)):
        x = torch.empty((n, R), dtype=torch.float32, device="cuda")
        y = torch.empty((n, R), dtype=torch.float32, device="cuda")
        r = qh.bsb_solve(g, R, 200, seed=5, x=x, y=y, plan=1, replica_tile=tile, tiles_in_flight=depth)
        out.append((x, y, r))
    x = torch.empty((n, R), dtype=torch.float32, device="cuda")
    y = torch.empty((n, R), dtype=torch.float32, device="cuda")
    out.append((x, y, qh.bsb_solve(g, R, 200, seed=5, x=x, y=y, plan=0)))
    info = g.plan_info(R)
    assert info["replica_tile"] in (16, 32, 64) and info["us_per_step"][0] > 0
    assert info["tiles_in_flight"] in (2, 4)
    xa, ya, ra = out[0]
    for xb, yb, rb in out[1:]:
        assert torch.equal(xa, xb) and torch.equal(ya, yb)
        assert torch.equal(ra["cuts"], rb["cuts"]) and torch.equal(ra["best_spins"], rb["best_spins"])
    with pytest.raises(qh.QhapError) as e:
        qh.bsb_solve(g, 32, 10, replica_tile=16)
    assert e.value.status == qh.Status.EINVAL
    with pytest.raises(qh.QhapError) as e:
        qh.bsb_solve(g, 64, 10, tiles_in_flight=3)
    assert e.value.status == qh.Status.EINVAL
    with pytest.raises(qh.QhapError) as e:
        qh.bsb_solve(g, 64, 10, persistent_sync=3)
    assert e.value.status == qh.Status.EINVAL


@pytest.mark.parametrize("plan", [0, 3, 4, 5])   # autotuned; per row; band FMA (R % 64 == 0); band MFMA
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("R", [16, 32, 64, 128])
def test_skyline_one_step(dtype, R, plan):
    w = synth.snp_small(14, n_snp=1500)
    g = gpu_graph(w, "snp_llr", dtype)
    J = stored_J(oracle_graph(w, "snp_llr").dense(), dtype)
    _one_step_case(g, J, dtype, R, 200 + R, None, plan=plan)


@pytest.mark.parametrize("case", ["snp", "porec", "snp_large", "porec_wide", "snp_tiny"])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_band_kernel_equals_row_kernel_bit_exact(dtype, case):
    """Band blocks add exact zeros around each row's range in the same ascending column
    order as the per-row kernel, so 200 steps of both agree bit for bit.  BF16 band values
    are stored as binary16 of value x 2^s when one power of two makes all of them exact
    there (the kernels multiply the band sums by 2^-s; BF16 storage flushes magnitudes 2^31
    below the largest, so this always holds unless the scale leaves the float range), else
    as BF16: "snp_large" scales every fragment weight by 1e5 (past the binary16 range),
    "porec_wide" shrinks the Pore-C contacts in the band by 1e-12 (flushed), "snp_tiny"
    scales every weight by 1e-35 (the scale would be 2^128: the band stays BF16)."""
    if case in ("snp", "snp_large", "snp_tiny"):
        w, band = synth.snp_small(26, n_snp=1700), 0
        if case == "snp_large":
            if dtype == "f16":
                pytest.skip("weights past the binary16 range")
            w.alpha = w.alpha * 1e5
        if case == "snp_tiny":
            if dtype == "f16":
                pytest.skip("weights below the binary16 range")
            w.alpha = w.alpha * 1e-35
    elif case == "porec_wide":
        w, band = synth.snp_porec(45, n_snp=2000, n_edges=2500, zipf_s=1.0), 0
        w.alpha = np.where(w.alpha < 1.0, w.alpha * 1e-12, w.alpha)
    else:
        w, band = synth.snp_porec(45, n_snp=2000, n_edges=2500, zipf_s=1.0), 100
    g = gpu_graph(w, "snp_llr", dtype, band_limit=band)
    want_band = {"f32": 0, "f16": 1, "bf16": 2 if case == "snp_tiny" else 1}[dtype]
    assert g.info()["band_dtype"] == want_band
    n, R = g.info()["n"], 128
    out = []
    for plan in (4, 3):          # band blocks on FMAs; per-row kernel
        x = torch.empty((n, R), dtype=torch.float32, device="cuda")
        y = torch.empty((n, R), dtype=torch.float32, device="cuda")
        r = qh.bsb_solve(g, R, 200, seed=33, x=x, y=y, plan=plan)
        out.append((x, y, r))
    (xa, ya, ra), (xb, yb, rb) = out
    assert torch.equal(xa, xb) and torch.equal(ya, yb)
    assert torch.equal(ra["best_spins"], rb["best_spins"]) and torch.equal(ra["best_cut"], rb["best_cut"])


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_band_mfma_whole_solve_and_tuner(dtype):
    """Band blocks on MFMAs over a whole solve: the final cut tracks the oracle's, the
    autotuner reports both band kernels, and plans 4 and 5 agree to FP32 rounding."""
    w = synth.snp_small(27, n_snp=1800)
    g = gpu_graph(w, "snp_llr", dtype)
    go = oracle_graph(w, "snp_llr")
    ro = oracle.solve(go, 64, 600, 0.5, seed=3)
    r5 = qh.bsb_solve(g, 64, 600, seed=3, plan=5)
    assert g.plan_info(64)["skyline_kernel"] == 5
    assert _gap(ro["best_cut"], float(cpu(r5["best_cut"])[0])) <= 1e-3
    n = g.info()["n"]
    xs = []
    for plan in (4, 5):
        x = torch.empty((n, 64), dtype=torch.float32, device="cuda")
        y = torch.empty((n, 64), dtype=torch.float32, device="cuda")
        qh.bsb_solve(g, 64, 3, seed=3, x=x, y=y, plan=plan, readout=False)
        xs.append(cpu(x))
    assert np.allclose(xs[0], xs[1], rtol=0, atol=1e-5)
    g2 = gpu_graph(w, "snp_llr", dtype)
    qh.bsb_solve(g2, 64, 100, seed=3, plan=0, readout=False)
    info = g2.plan_info(64)
    assert info["skyline_kernel"] in (4, 5) and min(info["skyline_us"]) > 0
    gd = gpu_graph(synth.read_tiny())
    with pytest.raises(qh.QhapError) as e:      # skyline plans on a dense graph
        qh.bsb_solve(gd, 16, 10, plan=5)
    assert e.value.status == qh.Status.EINVAL


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("R", [32, 64])
def test_longrange_hub_one_step(dtype, R):
    """Long-range rows, hub rows among them (chunk partials from the packet kernel for R = 64,
    per chunk for R = 32); 16-bit storage gathers the binary16 copy of x."""
    w = synth.snp_porec(43, n_snp=2500, n_edges=4000, zipf_s=1.0)
    g = gpu_graph(w, "snp_llr", dtype, band_limit=100)
    assert g.info()["longrange_nnz"] > 0
    J = stored_J(oracle_graph(w, "snp_llr").dense(), dtype)
    _one_step_case(g, J, dtype, R, 300 + R, None, lr_band=None if dtype == "f32" else 100)


@pytest.mark.parametrize("plan", [3, 4, 5])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_longrange_copy_against_unrounded_oracle(dtype, plan):
    """The binary16 copy of x that 16-bit SNP graphs gather for their long-range entries,
    bounded against the oracle's unrounded step (stored J, FP64): rounding x_j to binary16
    moves it by at most 2^-11 |x_j| + 2^-25, so row i's coupling sum moves by at most
    sum over its long-range j of |J_ij| (2^-11 |x_j| + 2^-25), y by c0 dt times that and x by
    a0 dt times y's bound, on top of the FP32 step tolerance; band entries take x itself."""
    w = synth.snp_porec(43, n_snp=2500, n_edges=4000, zipf_s=1.0)
    g = gpu_graph(w, "snp_llr", dtype, band_limit=100)
    J = stored_J(oracle_graph(w, "snp_llr").dense(), dtype)
    n, R, k, steps, dt = J.shape[0], 64, 37, 100, 0.5
    rng = np.random.default_rng(654)
    x0 = f32(rng.uniform(-1.0, 1.0, (n, R)))
    y0 = f32(rng.uniform(-0.6, 0.6, (n, R)))
    pump = np.linspace(0.0, 1.0, steps).astype(np.float32)
    c0 = float(np.float32(0.4 / max(1.0, float(np.sqrt((J ** 2).sum() / (n - 1))))))
    p = float(pump[k])
    x = torch.tensor(x0, dtype=torch.float32, device="cuda").contiguous()
    y = torch.tensor(y0, dtype=torch.float32, device="cuda").contiguous()
    qh.bsb_solve(g, R, steps, dt=dt, c0=c0, pump=torch.tensor(pump, device="cuda"), init=False, x=x, y=y,
                 step_begin=k, step_end=k + 1, readout=False, plan=plan)
    xg, yg = cpu(x).astype(np.float64), cpu(y).astype(np.float64)
    xu, yu = oracle.bsb_step_dense(J, x0, y0, p, dt, c0, 1.0, walls=False)
    xo, yo = oracle.bsb_step_dense(J, x0, y0, p, dt, c0, 1.0, walls=True)
    tol_x, tol_y = step_bounds(np.abs(J) @ np.abs(x0), x0, y0, p, dt, c0)
    Jfar = np.where(far_mask(n, 100), np.abs(J), 0.0)
    assert Jfar.sum() > 0
    copy = c0 * dt * (Jfar @ (COPY_UNIT["f16"] * np.abs(x0) + COPY_ABS["f16"]))
    tol_y = tol_y + copy
    tol_x = tol_x + dt * copy
    ok = np.abs(np.abs(xu) - 1.0) > tol_x        # entries not within the tolerance of a wall
    assert ok.mean() > 0.9
    assert np.all(np.abs(yg - yo)[ok] <= tol_y[ok])
    assert np.all(np.abs(xg - xo)[ok] <= tol_x[ok])


@pytest.mark.parametrize("plan", [2, 1])
def test_mhc_scale_one_step_f16(mhc, plan):
    """One step at the full MHC-scale shape and the benchmark's launch (R = 256, FP16):
    plan 2 requires the persistent kernel the benchmark uses, plan 1 the per-step kernel."""
    w, W = mhc
    g = gpu_graph(w, "read_signed", "f16")
    _one_step_case(g, W.astype(np.float64), "f16", 256, 7, "f16", steps=2000, k=999, plan=plan)


# ----------------------------------------------------------------------------- init, resume, graphs

def test_init_bit_exact():
    w = synth.read_small(15, n_snp=200, n_reads=70)
    g = gpu_graph(w)
    n = g.info()["n"]
    for R in (16, 64):
        x = torch.empty((n, R), dtype=torch.float32, device="cuda")
        y = torch.empty((n, R), dtype=torch.float32, device="cuda")
        qh.bsb_solve(g, R, 1, seed=12345, init=True, x=x, y=y, step_begin=1, step_end=1, readout=False)
        xo, yo = oracle.init_state(12345, n, R)
        assert np.array_equal(cpu(x), xo.astype(np.float32))
        assert np.array_equal(cpu(y), yo.astype(np.float32))


RESUME_CASES = [("read_signed", "f32"), ("read_signed", "f16"), ("read_signed", "fp8"), ("snp_llr", "f32"),
                ("snp_llr", "bf16")]


@pytest.mark.parametrize("kind,dtype", RESUME_CASES)
def test_resume_and_graph_replay_bit_identical(kind, dtype):
    w = synth.read_small(16, n_snp=300, n_reads=140) if kind != "snp_llr" else synth.snp_small(16, n_snp=900)
    g = gpu_graph(w, kind, dtype)
    n, R, steps = g.info()["n"], 64, 200
    def run(**kw):
        x = torch.empty((n, R), dtype=torch.float32, device="cuda")
        y = torch.empty((n, R), dtype=torch.float32, device="cuda")
        r = qh.bsb_solve(g, R, steps, seed=5, x=x, y=y, **kw)
        return x, y, r
    xa, ya, ra = run()
    xb, yb, _ = run(step_end=120, readout=False)
    xb2 = xb.clone(); yb2 = yb.clone()
    qh.bsb_solve(g, R, steps, init=False, x=xb2, y=yb2, step_begin=120, step_end=200, readout=False)
    assert torch.equal(xa, xb2) and torch.equal(ya, yb2)
    # captured step loop, replayed several times with eager work in between
    for rep in range(3):
        torch.cuda.synchronize()
        junk = torch.randn(1000, device="cuda").sum()
        xc, yc, rc = run(use_graph=True)
        torch.cuda.synchronize()
        assert torch.equal(xa, xc) and torch.equal(ya, yc), rep
        assert torch.equal(ra["best_spins"], rc["best_spins"]) and torch.equal(ra["best_cut"], rc["best_cut"])
        del junk


# ----------------------------------------------------------------------------- readout

def _readout_case(w, kind, R, seed, exact):
    g = gpu_graph(w, kind, "f32")
    go = oracle_graph(w, kind)
    n = go.n
    rng = np.random.default_rng(seed)
    x0 = f32(np.where(rng.random((n, R)) < 0.5, -0.5, 0.5))
    x0[rng.random((n, R)) < 0.05] = 0.0          # sgn(0) = +1
    y0 = np.zeros((n, R))
    x = torch.tensor(x0, dtype=torch.float32, device="cuda")
    y = torch.tensor(y0, dtype=torch.float32, device="cuda")
    res = qh.bsb_solve(g, R, 1, init=False, x=x, y=y, step_begin=1, step_end=1, readout=True, greedy=True,
                       all_spins=True, per_component=True)
    s = oracle.signs(x0)
    comp, nc = oracle.components(go)
    cut = oracle.cuts(go, comp, nc, s)
    best, br = oracle.select(comp, nc, s, cut)
    sel = float(sum(cut[br[c], c] for c in range(nc)))
    gbest, rounds = oracle.greedy(go, best, oracle.greedy_eps(go, exact))
    final = float(oracle.cuts(go, comp, nc, gbest).sum())
    assert np.array_equal(cpu(res["all_spins"]), s)
    if exact:
        assert np.array_equal(cpu(res["cut_rc"])[:, :nc], cut)
        assert np.array_equal(cpu(res["cuts"]), cut.sum(axis=1))
        assert np.array_equal(cpu(res["best_replica"])[:nc], br)
        assert cpu(res["selected_cut"])[0] == sel
        assert np.array_equal(cpu(res["best_spins"]), gbest)
        assert cpu(res["best_cut"])[0] == final
        assert int(cpu(res["greedy_rounds"])[0]) == rounds
    else:
        scale = np.abs(go.val).sum()
        assert np.allclose(cpu(res["cut_rc"])[:, :nc], cut, rtol=0, atol=1e-12 * scale)
        assert cpu(res["selected_cut"])[0] == pytest.approx(sel, abs=1e-12 * scale)
        assert cpu(res["best_cut"])[0] == pytest.approx(final, abs=1e-9 * scale)


@pytest.mark.parametrize("R", [16, 64, 256])
def test_readout_integer_exact(R):
    _readout_case(synth.read_small(17, n_snp=600, n_reads=250, span=(5, 40)), "read_signed", R, R, True)


def test_readout_conflict_many_components():
    _readout_case(synth.read_small(18, n_snp=3000, n_reads=200, span=(3, 15)), "read_conflict", 32, 3, True)


def test_readout_float_weights():
    _readout_case(synth.snp_small(19, n_snp=1200), "snp_llr", 64, 4, False)


# ----------------------------------------------------------------------------- phasing

def test_phase_vote_exact():
    w = synth.read_small(20, n_snp=500, n_reads=260, span=(5, 50), error=0.08)
    g = gpu_graph(w)
    go = oracle_graph(w)
    comp, nc = oracle.components(go)
    rng = np.random.default_rng(1)
    s = np.where(w.origin == 0, 1, -1).astype(np.int8)
    s[rng.random(s.shape[0]) < 0.2] *= -1
    h1, blk = qh.phase(g, torch.tensor(s, device="cuda"))
    M = oracle.encode(w.snp, w.allele, w.init_h1)
    ho, bo = oracle.phase_vote(w.n_snp, w.frag_ptr, w.snp, M, s, comp, w.init_h1)
    assert np.array_equal(cpu(h1), ho) and np.array_equal(cpu(blk), bo)


def test_phase_parity_exact():
    w = synth.snp_small(21, n_snp=1500)
    g = gpu_graph(w, "snp_llr")
    go = oracle_graph(w, "snp_llr")
    comp, nc = oracle.components(go)
    s = np.where(np.random.default_rng(2).random(go.n) < 0.4, 1, -1).astype(np.int8)
    h1, blk = qh.phase(g, torch.tensor(s, device="cuda"))
    ho, bo = oracle.phase_parity(comp, nc, s, w.init_h1)
    assert np.array_equal(cpu(h1), ho) and np.array_equal(cpu(blk), bo)


def test_phase_batched_equals_per_graph_phase():
    """qh_phase_batched over a list of read and SNP graphs (one and zero fragments, long-range
    rows, many components among them), with random spins packed as a batched solve packs
    them: every graph's slice of h1 and block equals qh_phase on that graph, bit for bit; and
    on the spins of a batched solve, every block's haplotype equals its qh_phase."""
    batch = synth.batched_blocks(93, n_blocks=40, n_lo=20, n_hi=600)
    gs = [gpu_graph(w, "read_signed" if i % 2 == 0 else "snp_llr", w.solve["dtype"])
          for i, w in enumerate(batch.blocks)]
    gs.append(gpu_graph(synth.read_tiny(), "read_conflict"))
    gs.append(gpu_graph(synth.snp_porec(45, n_snp=2000, n_edges=2500, zipf_s=1.0), "snp_llr", "bf16",
                        band_limit=64))
    for nf in (1, 0):
        w = synth.read_small(25, n_snp=50, n_reads=1, span=(5, 10))
        fp = w.frag_ptr[: nf + 1].copy()
        gs.append(qh.build_graph(qh.to_device(fp), qh.to_device(w.snp[: fp[-1]].copy()),
                                 qh.to_device(w.allele[: fp[-1]].copy()), qh.to_device(w.phred[: fp[-1]].copy()),
                                 qh.to_device(w.init_h1)))
    ns = [g.info()["n"] for g in gs]
    vo = np.concatenate([[0], np.cumsum(ns)]).astype(np.int64)
    rng = np.random.default_rng(17)
    spins = torch.tensor(rng.choice(np.array([-1, 1], dtype=np.int8), size=max(int(vo[-1]), 1)), device="cuda")
    h1, blk, so = qh.phase_batched(gs, spins)
    assert len(so) == len(gs) + 1 and int(so[-1]) == sum(g.n_snp for g in gs)
    for b, g in enumerate(gs):
        sb = spins[int(vo[b]):int(vo[b + 1])] if ns[b] else torch.ones(1, dtype=torch.int8, device="cuda")
        h1b, blkb = qh.phase(g, sb)
        assert torch.equal(h1[int(so[b]):int(so[b + 1])], h1b), b
        assert torch.equal(blk[int(so[b]):int(so[b + 1])], blkb), b
    # the spins of a batched solve
    r = qh.bsb_solve_batched(gs[:40], 32, 200, seed=4)
    h1, blk, so = qh.phase_batched(gs[:40], r["best_spins"])
    off = r["vertex_offset"]
    for b, g in enumerate(gs[:40]):
        h1b, blkb = qh.phase(g, r["best_spins"][int(off[b]):int(off[b + 1])])
        assert torch.equal(h1[int(so[b]):int(so[b + 1])], h1b) and torch.equal(blk[int(so[b]):int(so[b + 1])], blkb)
    arr = (ctypes.c_void_p * 2)(gs[0].handle.value, None)       # a null graph in the list
    rc = qh.load().qh_phase_batched(arr, 2, spins.data_ptr(), h1.data_ptr(), blk.data_ptr(), None)
    assert rc == qh.Status.EINVAL


def test_flip_crossing_matches_oracle():
    w = synth.snp_small(22, n_snp=1000)
    g = gpu_graph(w, "snp_llr", "f32")
    go = oracle_graph(w, "snp_llr")
    s = np.where(np.random.default_rng(3).random(go.n) < 0.5, 1, -1).astype(np.int8)
    qh.flip_crossing(g, torch.tensor(s, device="cuda"))
    D = cpu(g.export_rows(0, go.n))
    Do = oracle.flip_crossing(go, s).dense()
    assert np.all(np.abs(D - Do) <= 1e-12 * snp_abs_terms(w))
    S = cpu(g.export_rows(0, go.n, stored=True))
    assert np.array_equal(S, quant.round_to("f32", D))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_refine_gauge_identity_restore_and_single_round(dtype):
    """Eqs. (15)-(17) in the library: the flip counters' partition has, on the original
    weights (cut by the oracle), exactly the sum of the per-round cuts; the graph is
    restored bit for bit; one round equals the parity phasing of one solve."""
    w = synth.snp_small(24, n_snp=1500)
    g = gpu_graph(w, "snp_llr", dtype)
    go = oracle_graph(w, "snp_llr")
    n = go.n
    master, stored = cpu(g.export_rows(0, n)), cpu(g.export_rows(0, n, stored=True))
    rr = qh.refine(g, 32, 600, seed=1, max_rounds=15)
    assert np.array_equal(cpu(g.export_rows(0, n)), master)
    assert np.array_equal(cpu(g.export_rows(0, n, stored=True)), stored)
    assert rr["rounds"] >= 1 and all(c > 0 for c in rr["round_cuts"])
    comp, nc = oracle.components(go)
    S = np.where(cpu(rr["flips"]) % 2 == 1, -1, 1).astype(np.int8)
    total = oracle.cuts(go, comp, nc, S).sum()
    assert total == pytest.approx(sum(rr["round_cuts"]), rel=1e-9)
    # the oracle's refinement at the same schedule reaches the same total within 0.1 %
    ro = oracle.refine(go, w.init_h1, 32, 600, 0.5, seed=1, max_rounds=15)
    assert _gap(sum(ro["round_cuts"]), total) <= 1e-3
    # one round is the single-round parity phasing of the round-0 solve
    r1 = qh.refine(g, 32, 600, seed=1, max_rounds=1)
    rs = qh.bsb_solve(g, 32, 600, seed=1)
    h1, blk = qh.phase(g, rs["best_spins"])
    assert torch.equal(r1["h1"], h1) and torch.equal(r1["block"], blk)
    assert r1["round_cuts"][0] == pytest.approx(float(cpu(rs["best_cut"])[0]), rel=1e-12)


@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_refine_adaptive_schedule_planted_twin(dtype):
    """The size-adaptive settings end to end on an error-free planted twin (500 steps below
    5,000 vertices, 128 replicas, at most 15 rounds, deformation on) against the oracle's
    refinement with the same settings, seed and deformation: the applied round cuts agree in
    total within 0.1 % and the switch errors are equal."""
    w = synth.snp_small(8, n_snp=900, error=0.0)
    g = gpu_graph(w, "snp_llr", dtype)
    rr = qh.refine_adaptive(g, seed=2, deform=0.5, deform_tries=2)
    sc = rr["schedule"]
    assert sc["steps"] == 500 and sc["replicas"] == 128 and sc["max_rounds"] == 15
    assert sc["size"] == g.info()["largest_component"]
    assert 1 <= rr["rounds"] <= 15
    ro = oracle.refine(oracle_graph(w, "snp_llr"), w.init_h1, sc["replicas"], sc["steps"], seed=2,
                       max_rounds=sc["max_rounds"], deform=0.5, deform_tries=2)
    assert _gap(sum(ro["round_cuts"]), sum(rr["round_cuts"])) <= 1e-3
    assert metrics.switch_error(cpu(rr["h1"]), w.truth, cpu(rr["block"])) == \
        metrics.switch_error(ro["h1"], w.truth, ro["block"])


def test_refine_planted_twin_and_errors():
    w = synth.snp_small(8, n_snp=600, error=0.0)
    g = gpu_graph(w, "snp_llr", "f32")
    rr = qh.refine(g, 32, 600, seed=5)
    assert metrics.switch_error(cpu(rr["h1"]), w.truth, cpu(rr["block"])) == 0.0
    gr = gpu_graph(synth.read_tiny())
    with pytest.raises(qh.QhapError) as e:
        qh.refine(gr, 16, 10)
    assert e.value.status == qh.Status.EUNSUPPORTED
    with pytest.raises(qh.QhapError) as e:
        qh.refine(g, 32, 10, max_rounds=0)
    assert e.value.status == qh.Status.EINVAL


# ----------------------------------------------------------------------------- whole solves

def _gap(oracle_cut, gpu_cut):
    return (oracle_cut - gpu_cut) / abs(oracle_cut)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16", "fp8"])
def test_read_tiny_final_cut_and_switch_error(dtype):
    """Read-based tiny workload: R = 16, 1,000 steps, dt = 0.5, linear pump."""
    w = synth.read_tiny()
    g = gpu_graph(w, "read_signed", dtype)
    go = oracle_graph(w)
    ro = oracle.solve(go, 16, 1000, 0.5, seed=11, integer=True)
    rg = qh.bsb_solve(g, 16, 1000, dt=0.5, seed=11)
    assert _gap(ro["best_cut"], float(cpu(rg["best_cut"])[0])) <= 1e-3
    M = oracle.encode(w.snp, w.allele, w.init_h1)
    ho, bo = oracle.phase_vote(w.n_snp, w.frag_ptr, w.snp, M, ro["best"], ro["comp"], w.init_h1)
    hg, bg = qh.phase(g, rg["best_spins"])
    assert metrics.switch_error(cpu(hg), w.truth, cpu(bg)) == metrics.switch_error(ho, w.truth, bo)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16", "fp8"])
def test_read_midsize_final_cut(dtype):
    w = synth.read_mhc(seed=77, n_snp=2400, n_reads=1600, region=800_000)
    g = gpu_graph(w, "read_signed", dtype)
    go = oracle_graph(w)
    ro = oracle.solve(go, 64, 1000, 0.5, seed=3, integer=True)
    rg = qh.bsb_solve(g, 64, 1000, dt=0.5, seed=3, use_graph=True)
    assert _gap(ro["best_cut"], float(cpu(rg["best_cut"])[0])) <= 1e-3
    M = oracle.encode(w.snp, w.allele, w.init_h1)
    ho, bo = oracle.phase_vote(w.n_snp, w.frag_ptr, w.snp, M, ro["best"], ro["comp"], w.init_h1)
    hg, bg = qh.phase(g, rg["best_spins"])
    assert metrics.switch_error(cpu(hg), w.truth, cpu(bg)) <= metrics.switch_error(ho, w.truth, bo)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_snp_final_cut(dtype):
    w = synth.snp_small(23, n_snp=2000)
    g = gpu_graph(w, "snp_llr", dtype)
    go = oracle_graph(w, "snp_llr")
    ro = oracle.solve(go, 64, 1000, 0.5, seed=4)
    rg = qh.bsb_solve(g, 64, 1000, dt=0.5, seed=4, use_graph=True)
    assert _gap(ro["best_cut"], float(cpu(rg["best_cut"])[0])) <= 1e-3
    comp, nc = oracle.components(go)
    ho, bo = oracle.phase_parity(comp, nc, ro["best"], w.init_h1)
    hg, bg = qh.phase(g, rg["best_spins"])
    assert metrics.switch_error(cpu(hg), w.truth, cpu(bg)) <= metrics.switch_error(ho, w.truth, bo)


@pytest.mark.parametrize("n_snp,dtype", [(600, "f16"), (1500, "f32"), (1500, "f16")])
def test_snp_planted_twin_switch_error_equals_oracle(n_snp, dtype):
    """Error-free reads: the GPU's switch error equals the FP64 oracle's at the same
    schedule (on long SNP chains bSB can keep domain walls; both sides then agree)."""
    w = synth.snp_small(24, n_snp=n_snp, error=0.0)
    g = gpu_graph(w, "snp_llr", dtype)
    go = oracle_graph(w, "snp_llr")
    rg = qh.bsb_solve(g, 32, 600, dt=0.5, seed=1)
    ro = oracle.solve(go, 32, 600, 0.5, seed=1)
    comp, nc = oracle.components(go)
    ho, bo = oracle.phase_parity(comp, nc, ro["best"], w.init_h1)
    hg, bg = qh.phase(g, rg["best_spins"])
    se_o = metrics.switch_error(ho, w.truth, bo)
    assert metrics.switch_error(cpu(hg), w.truth, cpu(bg)) == se_o
    assert _gap(ro["best_cut"], float(cpu(rg["best_cut"])[0])) <= 1e-3


def test_porec_final_cut():
    w = synth.snp_porec(44, n_snp=2500, n_edges=3000, zipf_s=1.0)
    g = gpu_graph(w, "snp_llr", "bf16", band_limit=100)
    go = oracle_graph(w, "snp_llr")
    ro = oracle.solve(go, 64, 800, 0.5, seed=6)
    rg = qh.bsb_solve(g, 64, 800, dt=0.5, seed=6)
    assert _gap(ro["best_cut"], float(cpu(rg["best_cut"])[0])) <= 1e-3


@pytest.mark.parametrize("threads", [0, 1, 5])
def test_build_graphs_equals_single_builds(threads):
    """qh_build_graphs (host threads, a stream each) returns the graphs that qh_build_graph
    builds one by one: equal info, FP64 master and stored rows bit for bit, equal components
    (deterministic builds: the default SNP build sums Eq. 14 terms with atomics, whose order,
    and so the last bit, may change from one build to the next).  A malformed block fails
    the whole call with its index, and no graph is returned."""
    blocks = [synth.read_small(70 + b, n_snp=200, n_reads=30 + 25 * b) for b in range(6)] + \
             [synth.snp_small(80 + b, n_snp=120 + 150 * b) for b in range(6)] + [synth.read_tiny()] + \
             [synth.snp_porec(45, n_snp=2000, n_edges=2500, zipf_s=1.0)]
    kinds = ["read_signed"] * 6 + ["snp_llr"] * 6 + ["read_conflict", "snp_llr"]
    dtypes = ["fp8", "f16", "bf16", "f32", "fp8", "f16", "bf16", "f16", "f32", "bf16", "f16", "f32", "f32", "bf16"]
    specs = []
    for b, (w, k, dt) in enumerate(zip(blocks, kinds, dtypes)):
        d = device_reads(w)
        specs.append(dict(frag_ptr=d["frag_ptr"], snp=d["snp"], allele=d["allele"], phred=d["phred"],
                          init_h1=d["init_h1"], kind=k, dtype=dt, alpha=d["alpha"], deterministic=True,
                          band_limit=64 if b == 13 else 0))
    # degenerate graphs among them: one fragment, and none
    for nf in (1, 0):
        w = synth.read_small(25, n_snp=50, n_reads=1, span=(5, 10))
        fp = w.frag_ptr[: nf + 1].copy()
        specs.append(dict(frag_ptr=qh.to_device(fp), snp=qh.to_device(w.snp[: fp[-1]].copy()),
                          allele=qh.to_device(w.allele[: fp[-1]].copy()),
                          phred=qh.to_device(w.phred[: fp[-1]].copy()), init_h1=qh.to_device(w.init_h1)))
    many = qh.build_graphs(specs, threads=threads)
    assert len(many) == len(specs)
    assert many[13].info()["longrange_nnz"] > 0 and many[-1].info()["n"] == 0 and many[-2].info()["n"] == 1
    for b, (sp, gm) in enumerate(zip(specs, many)):
        g1 = qh.build_graph(**sp)
        assert g1.info() == gm.info(), b
        n = g1.info()["n"]
        if n:
            assert torch.equal(g1.export_rows(0, n), gm.export_rows(0, n)), b
            assert torch.equal(g1.export_rows(0, n, stored=True), gm.export_rows(0, n, stored=True)), b
            assert torch.equal(g1.components(), gm.components()), b
        g1.free()
    for g in many:
        g.free()
    # many small blocks: every worker recycles its temporaries many times over
    batch = synth.batched_blocks(91, n_blocks=240, n_lo=20, n_hi=300)
    specs2 = []
    for i, w in enumerate(batch.blocks):
        d = device_reads(w)
        k = "read_signed" if i % 2 == 0 else "snp_llr"
        specs2.append(dict(frag_ptr=d["frag_ptr"], snp=d["snp"], allele=d["allele"], phred=d["phred"],
                           init_h1=d["init_h1"], kind=k, dtype=w.solve["dtype"], alpha=d["alpha"],
                           deterministic=True))
    many = qh.build_graphs(specs2, threads=threads)
    for b, (sp, gm) in enumerate(zip(specs2, many)):
        g1 = qh.build_graph(**sp)
        assert g1.info() == gm.info(), b
        n = g1.info()["n"]
        assert torch.equal(g1.export_rows(0, n, stored=True), gm.export_rows(0, n, stored=True)), b
        assert torch.equal(g1.components(), gm.components()), b
        g1.free()
        gm.free()
    bad = dict(specs[7])
    snp = bad["snp"].clone()
    snp[0] = bad["init_h1"].numel()           # a SNP index past the last SNP
    bad["snp"] = snp
    with pytest.raises(qh.QhapError) as e:
        qh.build_graphs(specs[:7] + [bad] + specs[8:], threads=threads)
    assert e.value.status == qh.Status.EINVAL and "graph 7" in str(e.value)


@pytest.mark.parametrize("R,plan", [(16, 1), (32, 1), (64, 1), (16, 2), (32, 2), (64, 2), (32, 0)])
def test_batched_matches_single_solves(R, plan):
    """Uneven blocks of every storage and dtype, per-step (1), whole-block (2) or autotuned
    (0) plan: each block's state, replica cuts, selection and greedy result equal its
    single-graph solve bit for bit."""
    blocks = [synth.read_small(50 + b, n_snp=200, n_reads=40 + 30 * b) for b in range(4)] + \
             [synth.snp_small(60 + b, n_snp=150 + 200 * b) for b in range(3)] + [synth.read_tiny()]
    kinds = ["read_signed"] * 4 + ["snp_llr"] * 3 + ["read_signed"]
    dtypes = ["fp8", "f16", "bf16", "f32", "bf16", "f16", "f32", "f16"]
    gs = [gpu_graph(w, k, d) for w, k, d in zip(blocks, kinds, dtypes)]     # reads dense, SNPs skyline
    steps = 300
    rb = qh.bsb_solve_batched(gs, R, steps, seed=9, return_state=True, plan=plan)
    assert rb["plan_used"] == plan or (plan == 0 and rb["plan_used"] in (1, 2))
    off = rb["vertex_offset"]
    for b, (w, k, g) in enumerate(zip(blocks, kinds, gs)):
        n = g.info()["n"]
        xs = torch.empty(n, R, dtype=torch.float32, device="cuda")
        ys = torch.empty(n, R, dtype=torch.float32, device="cuda")
        rs = qh.bsb_solve(g, R, steps, seed=9, plan=1, x=xs, y=ys)
        lo, hi = int(off[b]), int(off[b + 1])
        assert hi - lo == n
        assert torch.equal(rb["x"][lo * R:hi * R], xs.reshape(-1)), b
        assert torch.equal(rb["y"][lo * R:hi * R], ys.reshape(-1)), b
        assert torch.equal(rb["cuts"][b * R:(b + 1) * R], rs["cuts"]), b
        assert torch.equal(rb["selected_cut"][b:b + 1], rs["selected_cut"]), b
        assert torch.equal(rb["best_spins"][lo:hi], rs["best_spins"]), b
        assert torch.equal(rb["best_cut"][b:b + 1], rs["best_cut"]), b
    # and the single solves track the oracle
    for b in (0, 4):
        go = oracle_graph(blocks[b], kinds[b])
        ro = oracle.solve(go, R, steps, 0.5, seed=9, integer=(kinds[b] != "snp_llr"))
        rs = qh.bsb_solve(gs[b], R, steps, seed=9)
        assert _gap(ro["best_cut"], float(cpu(rs["best_cut"])[0])) <= 1e-3, b


def test_batched_graph_replay_equals_per_step_plan():
    """use_graph = 1: the per-step plan's launches captured once and replayed.  Every replay
    (with eager solves and syncs in between, and a recapture for another seed) gives the
    per-step plan's results bit for bit; the whole-block plan refuses it."""
    blocks = [synth.read_small(50 + b, n_snp=200, n_reads=40 + 30 * b) for b in range(3)] + \
             [synth.snp_small(60 + b, n_snp=150 + 200 * b) for b in range(2)]
    kinds = ["read_signed"] * 3 + ["snp_llr"] * 2
    dtypes = ["fp8", "f16", "f32", "bf16", "f16"]
    gs = [gpu_graph(w, k, d) for w, k, d in zip(blocks, kinds, dtypes)]
    for seed in (9, 9, 10, 9):
        ref = qh.bsb_solve_batched(gs, 32, 200, seed=seed, plan=1, return_state=True)
        torch.cuda.synchronize()
        rg = qh.bsb_solve_batched(gs, 32, 200, seed=seed, use_graph=True, return_state=True)
        assert rg["plan_used"] == 1
        for k in ("x", "y", "cuts", "best_spins", "best_cut", "selected_cut"):
            assert torch.equal(rg[k], ref[k]), (seed, k)
        qh.bsb_solve(gs[0], 32, 50, seed=1)      # eager work between replays
    with pytest.raises(qh.QhapError) as e:
        qh.bsb_solve_batched(gs, 32, 20, plan=2, use_graph=True)
    assert e.value.status == qh.Status.EUNSUPPORTED


def test_batched_errors_and_empty_batch():
    w = synth.snp_porec(43, n_snp=2500, n_edges=4000, zipf_s=1.0)
    g_lr = gpu_graph(w, "snp_llr", "f32", band_limit=100)
    assert g_lr.info()["longrange_nnz"] > 0
    g_ok = gpu_graph(synth.read_tiny())
    with pytest.raises(qh.QhapError) as e:      # long-range couplings need the single-graph path
        qh.bsb_solve_batched([g_ok, g_lr], 32, 10)
    assert e.value.status == qh.Status.EUNSUPPORTED
    with pytest.raises(qh.QhapError) as e:
        qh.bsb_solve_batched([g_ok], 128, 10)
    assert e.value.status == qh.Status.EUNSUPPORTED
    with pytest.raises(qh.QhapError) as e:
        qh.bsb_solve_batched([g_ok, g_ok], 32, 10)
    assert e.value.status == qh.Status.EINVAL
    with pytest.raises(qh.QhapError) as e:
        qh.bsb_solve_batched([g_ok], 32, 10, plan=3)
    assert e.value.status == qh.Status.EINVAL
    r = qh.bsb_solve_batched([], 32, 10)
    assert r["vertex_offset"].tolist() == [0]


# ----------------------------------------------------------------------------- errors, edges

def test_error_paths():
    w = synth.read_tiny()
    g = gpu_graph(w)
    with pytest.raises(qh.QhapError) as e:
        qh.bsb_solve(g, 48, 10)
    assert e.value.status == qh.Status.EINVAL
    with pytest.raises(qh.QhapError) as e:
        qh.bsb_solve(g, 16, 10, step_begin=5, step_end=20)
    assert e.value.status == qh.Status.EINVAL
    d = {k: qh.to_device(v) for k, v in w.arrays().items()}
    with pytest.raises(qh.QhapError) as e:     # SNP index beyond n_snp
        qh.build_graph(d["frag_ptr"], d["snp"], d["allele"], d["phred"], d["init_h1"][:100])
    assert e.value.status == qh.Status.EINVAL
    with pytest.raises(qh.QhapError) as e:
        qh.build_graph(d["frag_ptr"], d["snp"], d["allele"], d["phred"], d["init_h1"], kind="read_signed",
                       storage="skyline")
    assert e.value.status == qh.Status.EUNSUPPORTED
    with pytest.raises(qh.QhapError) as e:
        qh.build_graph(d["frag_ptr"], d["snp"], d["allele"], d["phred"], d["init_h1"], kind="snp_llr",
                       dtype="fp8")
    assert e.value.status == qh.Status.EUNSUPPORTED
    bad = d["snp"].clone()
    bad[5], bad[6] = bad[6].item(), bad[5].item()        # not ascending inside fragment 0
    for kind in ("read_signed", "snp_llr"):
        with pytest.raises(qh.QhapError) as e:
            qh.build_graph(d["frag_ptr"], bad, d["allele"], d["phred"], d["init_h1"], kind=kind)
        assert e.value.status == qh.Status.EINVAL
    al = d["allele"].clone()
    al[17] = 2                                           # allele outside {0, 1}
    with pytest.raises(qh.QhapError) as e:
        qh.build_graph(d["frag_ptr"], d["snp"], al, d["phred"], d["init_h1"])
    assert e.value.status == qh.Status.EINVAL
    fp = d["frag_ptr"].clone()
    fp[3] = fp[4] + 1                                    # frag_ptr decreases at fragment 3
    with pytest.raises(qh.QhapError) as e:
        qh.build_graph(fp, d["snp"], d["allele"], d["phred"], d["init_h1"])
    assert e.value.status == qh.Status.EINVAL
    for i, v in ((0, 1), (-1, -1)):                      # frag_ptr[0] != 0; a negative count
        fp = d["frag_ptr"].clone()
        fp[i] = v
        with pytest.raises(qh.QhapError) as e:
            qh.build_graph(fp, d["snp"], d["allele"], d["phred"], d["init_h1"])
        assert e.value.status == qh.Status.EINVAL
    n = g.info()["n"]
    x = torch.zeros((n, 16), device="cuda")
    x[3, 2] = float("nan")
    y = torch.zeros((n, 16), device="cuda")
    with pytest.raises(qh.QhapError) as e:
        qh.bsb_solve(g, 16, 1, init=False, x=x, y=y, step_begin=1, step_end=1)
    assert e.value.status == qh.Status.ENUMERIC


@pytest.mark.parametrize("kind,dtype", [("read_signed", "fp8"), ("snp_llr", "bf16")])
def test_device_memory_cap(kind, dtype):
    """max_device_bytes: a graph that fits is built unchanged at exactly its footprint; one
    byte less, or a tiny cap, fails with ENOMEM and keeps nothing; a negative cap is EINVAL."""
    w = synth.snp_porec(43, n_snp=600, n_edges=500, zipf_s=1.0) if kind == "snp_llr" else synth.read_tiny()
    d = device_reads(w)
    # (deterministic SNP weights: with FP64 atomics a cancelling entry may come out as an
    # exact zero in one build and as residue in the next, which changes nnz and the footprint)
    kw = dict(kind=kind, dtype=dtype, alpha=d["alpha"], band_limit=100 if kind == "snp_llr" else 0,
              deterministic=kind == "snp_llr")
    g = qh.build_graph(d["frag_ptr"], d["snp"], d["allele"], d["phred"], d["init_h1"], **kw)
    need = g.info()["device_bytes"]
    assert need > 0
    g2 = qh.build_graph(d["frag_ptr"], d["snp"], d["allele"], d["phred"], d["init_h1"], max_device_bytes=need, **kw)
    assert g2.info()["device_bytes"] == need
    assert torch.equal(g2.export_rows(0, g.info()["n"]), g.export_rows(0, g.info()["n"]))
    for cap, status in ((need - 1, qh.Status.ENOMEM), (4096, qh.Status.ENOMEM), (-1, qh.Status.EINVAL)):
        with pytest.raises(qh.QhapError) as e:
            qh.build_graph(d["frag_ptr"], d["snp"], d["allele"], d["phred"], d["init_h1"], max_device_bytes=cap,
                           **kw)
        assert e.value.status == status, cap
    # the library still works after the refusals
    r = qh.bsb_solve(g, 16 if kind != "snp_llr" else 64, 50, seed=1)
    assert np.isfinite(float(cpu(r["best_cut"])[0]))


@pytest.mark.parametrize("kind,dtype", [("read_signed", "f16"), ("snp_llr", "f32")])
def test_best_energy_matches_eq5(kind, dtype):
    """best_energy is the Ising energy E(s) = -1/2 s'Js of the returned spins (Eq. 5), here
    evaluated by the oracle's dense J in FP64; total_weight is -1/2 sum J."""
    w = synth.read_small(13, n_snp=300, n_reads=150, span=(20, 60)) if kind == "read_signed" else \
        synth.snp_small(14, n_snp=800)
    g = gpu_graph(w, kind, dtype)
    J = oracle_graph(w, kind).dense()
    assert g.info()["total_weight"] == pytest.approx(-0.5 * J.sum(), rel=1e-12)
    r = qh.bsb_solve(g, 32, 300, seed=4)
    s = cpu(r["best_spins"]).astype(np.float64)
    e = -0.5 * s @ J @ s
    assert float(cpu(r["best_energy"])[0]) == pytest.approx(e, rel=1e-10, abs=1e-9)
    assert float(cpu(r["best_energy"])[0]) == pytest.approx(g.info()["total_weight"] - 2 * float(cpu(r["best_cut"])[0]),
                                                            rel=1e-14, abs=1e-12)


def test_energy_trace_resumes_one_schedule():
    """energy_trace is one solve read out every 100 steps: its last row is the energy (Eq. 5)
    of every replica after a straight solve of the same schedule, bit for bit, and its first
    rows match the oracle's energies of the same steps' signs."""
    w = synth.read_tiny()
    g = gpu_graph(w, "read_signed", "f32")
    tr = qh.energy_trace(g, 16, 300, 100, seed=7)
    assert tr["steps"] == [100, 200, 300] and tr["energy"].shape == (3, 16)
    r = qh.bsb_solve(g, 16, 300, seed=7, greedy=False, plan=1)
    W = g.info()["total_weight"]
    assert np.array_equal(tr["energy"][-1], W - 2.0 * cpu(r["cuts"]))
    go = oracle_graph(w)
    J = go.dense()
    x, y = oracle.init_state(7, go.n, 16)
    oracle.bsb_run(go, x, y, oracle.pump_linear(300), 0.5, oracle.c0(go), 1.0, 0, 100)
    s = np.where(x >= 0, 1.0, -1.0)
    e = -0.5 * np.einsum("ir,ij,jr->r", s, J, s)
    assert np.allclose(tr["energy"][0], e, rtol=0, atol=1e-9)
    assert tr["best"][-1] <= tr["best"][0]


EVAL_CASES = {
    # (workload, kind, dtype, R, steps, m, plan)
    "read_f32": (lambda: synth.read_tiny(), "read_signed", "f32", 16, 300, 70, 1),
    "read_f16_persistent": (lambda: synth.read_mhc(seed=78, n_snp=1500, n_reads=1000, region=500_000),
                            "read_signed", "f16", 64, 200, 45, 2),
    "read_fp8_step": (lambda: synth.read_small(16, n_snp=300, n_reads=140), "read_signed", "fp8", 32, 150, 40, 1),
    "snp_f16_band": (lambda: synth.snp_small(19, n_snp=1200), "snp_llr", "f16", 64, 200, 60, 4),
    "porec_bf16": (lambda: synth.snp_porec(45, n_snp=2000, n_edges=2500, zipf_s=1.0), "snp_llr", "bf16", 64, 120,
                   50, 0),
}


@pytest.mark.parametrize("case", list(EVAL_CASES))
def test_eval_every_matches_the_readout_definition(case):
    """Readouts every m steps (eval_every): the trajectory is the straight solve's (final
    state bit-identical); the energy row of readout e is -1/2 s'Js (Eq. 5, oracle's FP64
    dense J) of the signs after that readout's step, which a straight solve ending there
    returns; best_spins (no greedy) and selected_cut are the oracle's best-so-far merge of
    those readouts' signs (merge_best), exactly."""
    make, kind, dtype, R, steps, m, plan = EVAL_CASES[case]
    w = make()
    g = gpu_graph(w, kind, dtype, band_limit=64 if case.startswith("porec") else 0)
    n = g.info()["n"]
    go = oracle_graph(w, kind)
    J = go.dense()
    comp, nc = oracle.components(go)
    xe = torch.empty((n, R), dtype=torch.float32, device="cuda")
    r = qh.bsb_solve(g, R, steps, seed=9, greedy=False, plan=plan, eval_every=m, energy=True, x=xe,
                     per_component=True)
    marks = list(range(m, steps, m)) + [steps]
    E = cpu(r["energy"])
    assert E.shape == (len(marks), R)
    sets = []
    for e, k1 in enumerate(marks):
        xs = torch.empty((n, R), dtype=torch.float32, device="cuda")
        rs = qh.bsb_solve(g, R, steps, seed=9, greedy=False, plan=plan, step_end=k1, all_spins=True, x=xs)
        sp = cpu(rs["all_spins"])
        sets.append(sp)
        sd = sp.astype(np.float64)
        ref = -0.5 * np.einsum("ir,ij,jr->r", sd, J, sd)
        scale = max(1.0, float(np.abs(J).sum()))
        assert np.allclose(E[e], ref, rtol=0, atol=1e-12 * scale), e
        if k1 == steps:
            assert torch.equal(xs, xe)          # readouts do not disturb the trajectory
    best, best_c, best_r = oracle.merge_best(go, comp, nc, sets)
    assert np.array_equal(cpu(r["best_spins"]), best)
    assert np.array_equal(cpu(r["best_replica"]), best_r)
    assert float(cpu(r["selected_cut"])[0]) == pytest.approx(float(best_c.sum()), rel=1e-12, abs=1e-9)
    W = g.info()["total_weight"]
    assert np.array_equal(E[-1], W - 2.0 * cpu(r["cuts"]))


def test_eval_every_rejects_bad_combinations():
    g = gpu_graph(synth.read_tiny(), "read_signed", "f32")
    for kw in (dict(eval_every=-1), dict(eval_every=10, use_graph=True), dict(eval_every=10, readout=False)):
        with pytest.raises(qh.QhapError) as e:
            qh.bsb_solve(g, 16, 50, **kw)
        assert e.value.status == qh.Status.EINVAL, kw


def test_eval_every_whole_solve_tracks_the_oracle():
    """A whole solve with readouts every 100 steps against the oracle's at the same schedule
    (FP32 read graph): best cut within 0.1 %, and never below the plain solve's selected cut."""
    w = synth.read_small(13, n_snp=300, n_reads=150, span=(20, 60))
    g = gpu_graph(w, "read_signed", "f32")
    go = oracle_graph(w)
    r = qh.bsb_solve(g, 32, 500, seed=4, eval_every=100)
    ro = oracle.solve(go, 32, 500, 0.5, seed=4, integer=True, eval_every=100)
    cut = float(cpu(r["best_cut"])[0])
    assert (ro["best_cut"] - cut) / abs(ro["best_cut"]) <= 1e-3
    rp = qh.bsb_solve(g, 32, 500, seed=4)
    assert float(cpu(r["selected_cut"])[0]) >= float(cpu(rp["selected_cut"])[0])


def test_flip_crossing_refreshes_total_weight():
    """Eq. (15) flips the sign of every crossing edge: total_weight (-1/2 sum J) follows, and
    best_energy of a solve on the flipped graph is -1/2 s'Js with the flipped J (the
    oracle's flip_crossing)."""
    w = synth.snp_small(22, n_snp=1000)
    g = gpu_graph(w, "snp_llr", "f32")
    go = oracle_graph(w, "snp_llr")
    rng = np.random.default_rng(3)
    s = np.where(rng.random(go.n) < 0.5, 1, -1).astype(np.int8)
    qh.flip_crossing(g, qh.to_device(s))
    Jf = oracle.flip_crossing(go, s).dense()
    assert g.info()["total_weight"] == pytest.approx(-0.5 * Jf.sum(), rel=1e-12, abs=1e-9)
    r = qh.bsb_solve(g, 64, 200, seed=6)
    b = cpu(r["best_spins"]).astype(np.float64)
    assert float(cpu(r["best_energy"])[0]) == pytest.approx(-0.5 * b @ Jf @ b, rel=1e-10, abs=1e-8)


def test_deterministic_snp_build():
    """deterministic = 1: fixed-point sums give the same SNP weights bit for bit on every
    build (and so the same solve), within 2^-40 per Eq. (14) term of the oracle's FP64 sum."""
    w = synth.snp_porec(43, n_snp=1200, n_edges=1500, zipf_s=1.0)
    d = device_reads(w)
    kw = dict(kind="snp_llr", dtype="bf16", alpha=d["alpha"], band_limit=100, deterministic=True)
    g1 = qh.build_graph(d["frag_ptr"], d["snp"], d["allele"], d["phred"], d["init_h1"], **kw)
    g2 = qh.build_graph(d["frag_ptr"], d["snp"], d["allele"], d["phred"], d["init_h1"], **kw)
    n = g1.info()["n"]
    assert g1.info()["longrange_nnz"] > 0
    m1, m2 = g1.export_rows(0, n), g2.export_rows(0, n)
    assert torch.equal(m1, m2)
    assert torch.equal(g1.export_rows(0, n, stored=True), g2.export_rows(0, n, stored=True))
    J = oracle_graph(w, "snp_llr").dense()
    diff = np.abs(cpu(m1) - J)
    # each entry sums at most a few hundred terms, each rounded by at most 2^-41; entries
    # that are not FP64 cancellation residue keep their place
    assert diff.max() <= 1e3 * 2.0 ** -41
    assert np.all(cpu(m1)[np.abs(J) > 1e-9] != 0)
    r1 = qh.bsb_solve(g1, 64, 200, seed=2)
    r2 = qh.bsb_solve(g2, 64, 200, seed=2)
    assert torch.equal(r1["best_spins"], r2["best_spins"]) and torch.equal(r1["best_cut"], r2["best_cut"])


def test_autotune_cache_and_explicit_options(tmp_path):
    """qh_autotune on its own: the chosen options, passed explicitly, run the tuned kernels
    with the plan-0 solve's results bit for bit; the cache file holds one JSON line per
    tuning and load_tuned finds the options again by graph shape and replica count."""
    path = str(tmp_path / "tune.jsonl")
    wm = synth.read_mhc(seed=78, n_snp=1500, n_reads=1000, region=500_000)
    cases = [(gpu_graph(wm, "read_signed", "f16"), 64, (1, 2)),
             (gpu_graph(synth.snp_small(14, n_snp=1500), "snp_llr", "f16"), 64, (3, 4, 5))]
    for g, R, plans in cases:
        ch = qh.autotune(g, R, 200, cache_path=path)
        assert ch["plan"] in plans and ch["us_per_step"][0] > 0.0
        opts = {k: ch[k] for k in ("plan", "replica_tile", "tiles_in_flight", "persistent_sync")}
        n = g.info()["n"]
        xa = torch.empty((n, R), dtype=torch.float32, device="cuda")
        xb = torch.empty_like(xa)
        ra = qh.bsb_solve(g, R, 200, seed=3, x=xa)
        rb = qh.bsb_solve(g, R, 200, seed=3, x=xb, **opts)
        assert torch.equal(xa, xb) and torch.equal(ra["best_cut"], rb["best_cut"])
        info = g.plan_info(R)
        if ch["plan"] == 2:
            assert info["plan_used"] == 2 and info["persistent_sync"] == ch["persistent_sync"]
        elif ch["plan"] == 1:
            assert info["plan_used"] == 1 and info["replica_tile"] == ch["replica_tile"]
        else:
            assert info["skyline_kernel"] == ch["plan"]
        assert qh.load_tuned(path, g, R) == opts
    lines = open(path).read().splitlines()
    assert len(lines) == 2 and all(json.loads(line)["replicas"] == 64 for line in lines)
    assert qh.load_tuned(path, cases[0][0], 128) is None


def test_degenerate_graphs():
    # one fragment: no edges, no components; zero fragments
    for nf in (1, 0):
        w = synth.read_small(25, n_snp=50, n_reads=max(nf, 1), span=(5, 10))
        fp = w.frag_ptr[: nf + 1].copy()
        snp = w.snp[: fp[-1]].copy()
        d = dict(frag_ptr=qh.to_device(fp), snp=qh.to_device(snp), allele=qh.to_device(w.allele[: fp[-1]].copy()),
                 phred=qh.to_device(w.phred[: fp[-1]].copy()), init_h1=qh.to_device(w.init_h1))
        g = qh.build_graph(d["frag_ptr"], d["snp"], d["allele"], d["phred"], d["init_h1"])
        inf = g.info()
        assert inf["n"] == nf and inf["n_comp"] == 0 and inf["nnz"] == 0
        r = qh.bsb_solve(g, 16, 20)
        assert float(cpu(r["best_cut"])[0]) == 0.0
        h1, blk = qh.phase(g, r["best_spins"] if nf else torch.ones(1, dtype=torch.int8, device="cuda"))
        assert np.all(cpu(h1) == -1)


def test_release_cached_memory():
    """A freed graph's device blocks stay cached (a rebuild reuses them) until
    qh_release_cached_memory hands them back; a second release finds nothing, and the
    library allocates afresh afterwards."""
    w = synth.read_tiny()
    d = device_reads(w)
    torch.cuda.synchronize()
    qh.release_cached_memory()

    def build():
        return qh.build_graph(d["frag_ptr"], d["snp"], d["allele"], d["phred"], d["init_h1"], kind="read_signed",
                              dtype="fp8")

    g = build()
    need = g.info()["device_bytes"]
    ref = qh.bsb_solve(g, 16, 50, seed=3)["best_cut"].cpu()
    g.free()
    assert qh.release_cached_memory() >= need
    assert qh.release_cached_memory() == 0
    g = build()
    assert torch.equal(qh.bsb_solve(g, 16, 50, seed=3)["best_cut"].cpu(), ref)
    # blocks in use stay: a live graph solves the same after another one's blocks are released
    g2 = build()
    g2.free()
    assert qh.release_cached_memory() >= need
    assert torch.equal(qh.bsb_solve(g, 16, 50, seed=3)["best_cut"].cpu(), ref)
    g.free()


BAND_PLAN_CASES = [
    # n, gap_mean, dtype, R: one workgroup; a remainder row; several workgroups; 16 replicas only;
    # bands wider than the registers hold (every variant reads columns from memory); replica
    # groups that run one after another
    (17, 1430.0, "f32", 16), (50, 1430.0, "bf16", 32), (300, 1430.0, "f16", 64), (1201, 1430.0, "f16", 48 * 4),
    (2001, 1430.0, "f16", 128), (1500, 1430.0, "f32", 32), (900, 60.0, "f16", 16), (1301, 45.0, "f32", 64),
    (9000, 400.0, "bf16", 64), (30011, 1430.0, "f16", 512), (40000, 1430.0, "f32", 256),
]


@pytest.mark.gpu
@pytest.mark.parametrize("n,gap,dtype,R", BAND_PLAN_CASES)
def test_band_plan_equals_per_step(n, gap, dtype, R):
    """Plan 0 on an SNP graph (all steps in one launch where the graph fits) against the
    per-row kernel, one launch per step: the same state bit for bit, over step ranges that
    start from a kept state, with a field, and in the discrete variant."""
    w = synth.snp_small(5, n_snp=n, gap_mean=gap)
    g = gpu_graph(w, "snp_llr", dtype)
    field = torch.linspace(-0.3, 0.3, n, dtype=torch.float32, device="cuda")
    out = []
    for plan in (3, 0):
        x = torch.empty((n, R), dtype=torch.float32, device="cuda")
        y = torch.empty_like(x)
        got = []
        for kw in (dict(step_end=1), dict(step_begin=1, step_end=4, init=False),
                   dict(step_begin=4, step_end=25, init=False, field=field),
                   dict(step_begin=25, step_end=32, init=False, discrete=True)):
            qh.bsb_solve(g, R, 40, seed=9, x=x, y=y, plan=plan, readout=False, **kw)
            got += [x.clone(), y.clone()]
        r = qh.bsb_solve(g, R, 40, seed=9, plan=plan, eval_every=15, energy=True)
        out.append(got + [r["best_spins"], r["cuts"], r["best_cut"], r["energy"]])
    assert g.plan_info(R)["plan_used"] == 2
    for a, b in zip(*out):
        assert torch.equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16", "fp8"])
@pytest.mark.parametrize("reads,snps,span,R,order", [
    (60, 200, (20, 60), 16, "sorted"), (64, 300, (20, 60), 32, "sorted"), (65, 900, (2, 4), 64, "sorted"),
    (700, 4000, (2, 9), 32, "sorted"), (1501, 2300, (20, 60), 64, "sorted"), (1000, 300, (20, 60), 128, "sorted"),
    (3000, 9000, (20, 60), 512, "sorted"), (500, 200, (20, 60), 32, "shuffled"), (700, 200000, (2, 4), 16, "shuffled")])
def test_dense_one_launch_equals_per_step(reads, snps, span, R, order, dtype):
    """Plan 0 on a dense graph (all steps in one launch, 16-row strips of the row tiles on chip)
    against the per-step kernel: the same state bit for bit, from a kept state, with a field and
    in the discrete variant; row tiles without stored tiles, more tiles than the registers hold,
    shuffled reads (700 reads over 200,000 SNPs: row tiles skip column tiles, where a state or
    field of the caller's goes through the per-step kernels)."""
    w = synth.read_small(6, snps, reads, span)
    if order == "shuffled":
        perm = np.random.default_rng(1).permutation(reads)
        cnt = np.diff(w.frag_ptr)
        idx = np.concatenate([np.arange(w.frag_ptr[f], w.frag_ptr[f + 1]) for f in perm])
        w.frag_ptr = np.concatenate([[0], np.cumsum(cnt[perm])]).astype(np.int64)
        w.snp, w.allele, w.phred = w.snp[idx], w.allele[idx], w.phred[idx]
    g = gpu_graph(w, "read_signed", dtype)
    n = g.info()["n"]
    field = torch.linspace(-0.3, 0.3, n, dtype=torch.float32, device="cuda")
    out = []
    for plan in (1, 0):
        x = torch.empty((n, R), dtype=torch.float32, device="cuda")
        y = torch.empty_like(x)
        got = []
        for kw in (dict(step_end=1), dict(step_begin=1, step_end=4, init=False),
                   dict(step_begin=4, step_end=25, init=False, field=field),
                   dict(step_begin=25, step_end=32, init=False, discrete=True)):
            qh.bsb_solve(g, R, 40, seed=9, x=x, y=y, plan=plan, readout=False, **kw)
            got += [x.clone(), y.clone()]
        r = qh.bsb_solve(g, R, 40, seed=9, plan=plan, eval_every=15, energy=True)
        out.append(got + [r["best_spins"], r["cuts"], r["best_cut"], r["energy"]])
    assert g.plan_info(R)["plan_used"] == 2
    for a, b in zip(*out):
        assert torch.equal(a, b)


def _pair_reads(kind, seed=8):
    """Reads of the SNP pair sums' edges: "sorted" 40,000 reads of 2-9 SNPs in order (workgroups of
    16 whose sums fit the LDS table), "shuffled" the same in no order (they do not), "long" reads of
    127-300 SNPs around the 128 that a wave stages, "interleaved" pairs (u, u + 3)."""
    rng = np.random.default_rng(seed)
    n = 420
    if kind == "interleaved":
        first, count, step = np.arange(n - 3), np.full(n - 3, 2), 3
    elif kind == "long":
        count = np.array([127, 128, 129, 190, 300, 2])
        first, step = np.sort(rng.integers(0, n - count.max(), count.size)), 1
    else:
        count, step = rng.integers(2, 10, 40000), 1
        first = rng.integers(0, n - count)
        o = np.argsort(first, kind="stable")
        first, count = (first[o], count[o]) if kind == "sorted" else (first, count)
    w = synth.snp_small(seed, n_snp=n)
    w.frag_ptr = np.concatenate([[0], np.cumsum(count)]).astype(np.int64)
    t = np.arange(w.frag_ptr[-1]) - np.repeat(w.frag_ptr[:-1], count)
    w.snp = (np.repeat(first, count) + step * t).astype(np.int32)
    w.allele = rng.integers(0, 2, w.snp.size).astype(w.allele.dtype)
    w.phred = rng.integers(5, 40, w.snp.size).astype(np.uint8)
    w.alpha = None
    return w


@pytest.mark.parametrize("kind,k,band", [("sorted", 10, 0), ("sorted", 3, 2), ("shuffled", 10, 0),
                                         ("long", 10, 0), ("long", 2, 30), ("interleaved", 10, 0)])
@pytest.mark.parametrize("fixed", [False, True])
def test_snp_pair_sums(kind, k, band, fixed):
    """Eq. (14) sums of grouped, staged and mirrored pairs against the oracle: 1e-12 of the summed
    |terms|, and in fixed-point mode 2^-41 per term of an entry (at most the deepest SNP's reads)."""
    w = _pair_reads(kind)
    g = qh.build_graph(*(qh.to_device(a) for a in (w.frag_ptr, w.snp, w.allele, w.phred, w.init_h1)),
                       kind="snp_llr", dtype="f32", linkage_k=k, band_limit=band, deterministic=fixed)
    go = oracle_graph(w, "snp_llr", k)
    D = cpu(g.export_rows(0, go.n))
    tol = 1e-12 * snp_abs_terms(w, k) + (np.bincount(w.snp).max() * 2.0 ** -41 if fixed else 0.0)
    assert np.all(np.abs(D - go.dense()) <= tol)
    assert np.array_equal(D, D.T)
    # one spin set per component, its sides counted over whole waves and mixed ones
    comp, nc = oracle.components(go)
    s = np.where(np.random.default_rng(2).random(go.n) < 0.4, 1, -1).astype(np.int8)
    h1, blk = qh.phase(g, torch.tensor(s, device="cuda"))
    ho, bo = oracle.phase_parity(comp, nc, s, w.init_h1)
    assert np.array_equal(cpu(h1), ho) and np.array_equal(cpu(blk), bo)


@pytest.mark.parametrize("R", [16, 64])
def test_readout_component_of_many_chunks(R):
    """A component of 282 chunks of 32 vertices: staged sums of several stages."""
    _readout_case(synth.snp_small(23, n_snp=9000), "snp_llr", R, 4, False)


def test_readout_integer_component_of_many_chunks():
    _readout_case(synth.read_small(24, n_snp=2500, n_reads=2300, span=(10, 40)), "read_signed", 32, 5, True)


@pytest.fixture(scope="module")
def team_batch():
    """300 SNP blocks (bf16) and 300 read blocks (fp8) of 20-300 vertices: more teams of a class than
    the chip has workgroups; and larger blocks of every storage and type, whose teams have several
    (700 shuffled reads over 200,000 SNPs: row tiles skip column tiles)."""
    ws, kinds, dtypes = [], [], []
    for i, w in enumerate(synth.batched_blocks(91, n_blocks=600, n_lo=20, n_hi=300).blocks):
        ws.append(w), kinds.append("read_signed" if i % 2 == 0 else "snp_llr"), dtypes.append("fp8" if i % 2 == 0 else "bf16")
    for i, d in enumerate(["f32", "f16", "bf16", "fp8"]):
        ws.append(synth.read_small(30 + i, 400, 1300 - 150 * i, (20, 120))), kinds.append("read_signed"), dtypes.append(d)
    for i, d in enumerate(["f32", "f16", "bf16"]):
        ws.append(synth.snp_small(40 + i, 2500 - 400 * i)), kinds.append("snp_llr"), dtypes.append(d)
    w = synth.read_small(6, 200000, 700, (3, 40))
    perm = np.random.default_rng(1).permutation(700)
    cnt = np.diff(w.frag_ptr)
    idx = np.concatenate([np.arange(w.frag_ptr[f], w.frag_ptr[f + 1]) for f in perm])
    w.frag_ptr = np.concatenate([[0], np.cumsum(cnt[perm])]).astype(np.int64)
    w.snp, w.allele, w.phred = w.snp[idx], w.allele[idx], w.phred[idx]
    ws.append(w), kinds.append("read_signed"), dtypes.append("f16")
    specs = []
    for w, k, t in zip(ws, kinds, dtypes):
        d = device_reads(w)
        specs.append(dict(frag_ptr=d["frag_ptr"], snp=d["snp"], allele=d["allele"], phred=d["phred"],
                          init_h1=d["init_h1"], kind=k, dtype=t, alpha=d["alpha"], deterministic=True))
    gs = qh.build_graphs(specs)
    yield gs
    for g in gs:
        g.free()


@pytest.mark.parametrize("R", [16, 32, 64])
@pytest.mark.parametrize("variant", ["plain", "discrete", "field", "graph", "small"])
def test_batch_teams_equal_per_step(team_batch, R, variant):
    """Plan 0 (blocks as teams of the persistent kernels) against one launch per step: every block's
    state and results, bit for bit."""
    gs = team_batch[-8:] if variant == "small" else team_batch
    n = sum(g.info()["n"] for g in gs)
    kw = dict(discrete=variant == "discrete", return_state=True, seed=5)
    if variant == "field":
        kw["field"] = torch.linspace(-0.3, 0.3, n, dtype=torch.float32, device="cuda")
    a = qh.bsb_solve_batched(gs, R, 31, plan=1, **kw)
    b = qh.bsb_solve_batched(gs, R, 31, plan=0, use_graph=variant == "graph", **kw)
    for k in ("x", "y", "cuts", "selected_cut", "best_spins", "best_cut"):
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("reads,R,dtype", [(64, 64, "f16"), (1600, 256, "f16"), (1600, 256, "f32"), (4100, 256, "fp8")])
def test_default_replica_tile_bit_exact(reads, R, dtype):
    """The per-step dense kernel's replica tile chosen by the fill (16, 32, 32 and 64 replicas)
    against tiles of 64."""
    g = gpu_graph(synth.read_small(9, reads * 3 // 2, reads, (20, 60)), "read_signed", dtype)
    n = g.info()["n"]
    out = []
    for tile in (0, 64):
        x, y = torch.empty((n, R), device="cuda"), torch.empty((n, R), device="cuda")
        qh.bsb_solve(g, R, 40, seed=3, x=x, y=y, plan=1, replica_tile=tile, readout=False)
        out.append((x, y))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("reads,snps,span", [(900, 70, (20, 60)), (130, 600, (250, 260)), (64, 40, (2, 3))])
@pytest.mark.parametrize("kind", ["read_signed", "read_conflict"])
def test_read_rows_list_lengths(reads, snps, span, kind):
    """Read graph rows over coverage lists of several hundred (a wave each), of around 64 with a read
    of more SNPs than one chunk of observations, and short ones."""
    w = synth.read_small(14, snps, reads, span)
    g = gpu_graph(w, kind, "f32")
    go = oracle_graph(w, kind)
    assert np.array_equal(cpu(g.export_rows(0, go.n)), go.dense())
    comp, nc = oracle.components(go)
    assert g.info()["n_comp"] == nc and np.array_equal(cpu(g.components()), comp)


def _one_launch_case(kind, dtype, n, reads, R):
    w = synth.snp_small(5, n_snp=n) if kind == "snp_llr" else synth.read_small(6, n, reads, (20, 60))
    return gpu_graph(w, kind, dtype), 3 if kind == "snp_llr" else 1


@pytest.mark.parametrize("kind,dtype,n,reads,R", [
    ("snp_llr", "f16", 30011, 0, 512), ("snp_llr", "f32", 2001, 0, 128), ("read_signed", "f32", 2300, 1501, 64),
    ("read_signed", "bf16", 9000, 3000, 512), ("read_signed", "fp8", 2300, 1501, 32)])
def test_one_launch_of_one_step(kind, dtype, n, reads, R):
    """Ranges of one step under plan 0, on graphs whose longer ranges run in one launch of several
    workgroups and replica groups: no workgroup's final state may reach a neighbour that still
    reads the initial one.  Steps one by one, a readout after every step and a last range of one step,
    against one launch per step, bit for bit."""
    g, ref = _one_launch_case(kind, dtype, n, reads, R)
    nv = g.info()["n"]
    out = []
    for plan in (ref, 0):
        x = torch.empty((nv, R), dtype=torch.float32, device="cuda")
        y = torch.empty_like(x)
        got = []
        for k in range(6):
            qh.bsb_solve(g, R, 40, seed=9, x=x, y=y, plan=plan, readout=False, init=k == 0, step_begin=k, step_end=k + 1)
            got += [x.clone(), y.clone()]
        for every, end in ((1, 5), (3, 7)):
            r = qh.bsb_solve(g, R, 40, seed=9, plan=plan, step_end=end, eval_every=every, energy=True)
            got += [r["best_spins"], r["cuts"], r["best_cut"], r["energy"]]
        out.append(got)
    for a, b in zip(*out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("steps", [1, 2, 23, 24, 40])
@pytest.mark.parametrize("kind,dtype,n", [("snp_llr", "bf16", 2500), ("read_signed", "fp8", 1300)])
def test_batch_of_few_steps(kind, dtype, n, steps):
    """More teams of several workgroups than the chip holds at once, so that a team's workgroups start at
    different times, and schedules too short for teams, against one launch per step, bit for bit."""
    w = synth.snp_small(41, n_snp=n) if kind == "snp_llr" else synth.read_small(42, 400, n, (20, 120))
    d = device_reads(w)
    gs = qh.build_graphs([dict(frag_ptr=d["frag_ptr"], snp=d["snp"], allele=d["allele"], phred=d["phred"],
                               init_h1=d["init_h1"], kind=kind, dtype=dtype, alpha=d["alpha"], deterministic=True)
                          for _ in range(200)])
    a = qh.bsb_solve_batched(gs, 64, steps, plan=1, return_state=True, seed=5)
    for _ in range(3):
        b = qh.bsb_solve_batched(gs, 64, steps, plan=0, return_state=True, seed=5)
        for k in ("x", "y", "cuts", "best_spins", "best_cut"):
            assert torch.equal(a[k], b[k]), k
    for g in gs:
        g.free()


@pytest.fixture
def wait_error():
    """Every launch of the one-launch plans finds its error word set, as by a wait that gave up."""
    v = ctypes.c_int32.in_dll(qh.load(), "_ZN2qh16force_wait_errorE")
    v.value = 1
    yield v
    v.value = 0


@pytest.mark.parametrize("kind,dtype,n,reads,R", [
    ("snp_llr", "f16", 2001, 0, 128), ("read_signed", "f32", 2300, 1501, 64), ("read_signed", "bf16", 2300, 1501, 64)])
def test_wait_that_gives_up_is_reported(wait_error, kind, dtype, n, reads, R):
    """A wait between workgroups that gives up: EHIP from the call itself when it reads out, from the next
    call with the graph otherwise, and the state is NaN; afterwards the graph solves as before."""
    g, ref = _one_launch_case(kind, dtype, n, reads, R)
    nv = g.info()["n"]
    x, y = (torch.zeros((nv, R), dtype=torch.float32, device="cuda") for _ in range(2))
    for kw in (dict(), dict(eval_every=300), dict(energy=True)):
        with pytest.raises(qh.QhapError) as e:
            qh.bsb_solve(g, R, 1000, seed=9, **kw)
        assert e.value.status == qh.Status.EHIP and "wait" in str(e.value)
    qh.bsb_solve(g, R, 1000, seed=9, x=x, y=y, readout=False)
    torch.cuda.synchronize()
    assert torch.isnan(x).any() and torch.equal(torch.isnan(x), torch.isnan(y))
    wait_error.value = 0
    with pytest.raises(qh.QhapError) as e:
        qh.bsb_solve(g, R, 1000, init=False, x=x, y=y, step_begin=500, readout=False)
    assert e.value.status == qh.Status.EHIP
    a = qh.bsb_solve(g, R, 1000, seed=9, x=x)
    b = qh.bsb_solve(g, R, 1000, seed=9, x=y, plan=ref)
    assert g.plan_info(R)["plan_used"] == 1
    assert torch.equal(x, y) and torch.equal(a["best_cut"], b["best_cut"])


@pytest.mark.parametrize("readout", [True, False])
def test_batch_wait_that_gives_up_is_reported(team_batch, wait_error, readout):
    """The same for the teams of a batch, which synchronises: EHIP with and without a readout."""
    gs = team_batch[-8:]
    with pytest.raises(qh.QhapError) as e:
        qh.bsb_solve_batched(gs, 32, 500, seed=5, readout=readout)
    assert e.value.status == qh.Status.EHIP and "wait" in str(e.value)
    wait_error.value = 0
    a = qh.bsb_solve_batched(gs, 32, 100, seed=5, plan=1)
    b = qh.bsb_solve_batched(gs, 32, 100, seed=5)
    assert torch.equal(a["best_spins"], b["best_spins"]) and torch.equal(a["best_cut"], b["best_cut"])


def test_choice_of_plans_after_a_one_launch_solve():
    """A plan-0 solve in one launch times the per-step kernels briefly and without the persistent plan;
    whatever acts on the choice later (qh_autotune, plan 2's way to synchronise, plan 0 where the
    one-launch plan does not apply) times every candidate, as on a fresh graph."""
    wm = synth.read_mhc(seed=78, n_snp=1500, n_reads=1000, region=500_000)

    def solved(w, R):
        g = gpu_graph(w, "read_signed", "f16")
        qh.bsb_solve(g, R, 100, seed=3)
        info = g.plan_info(R)
        assert info["plan_used"] == 2 and info["us_per_step"][1] == 0 and info["us_persistent_coherent"] == 0
        return g

    def timed(g, R):
        info = g.plan_info(R)
        assert min(info["us_per_step"]) > 0 and info["us_persistent_coherent"] > 0
        return info

    g = solved(wm, 64)
    ch = qh.autotune(g, 64, 200)
    info = timed(g, 64)
    best = min(info["us_per_step"][1], info["us_persistent_coherent"])
    assert ch["plan"] == (2 if best < info["us_per_step"][0] else 1)
    g = solved(wm, 64)
    qh.bsb_solve(g, 64, 100, seed=3, plan=2)
    info = timed(g, 64)
    assert info["persistent_sync"] == (2 if info["us_persistent_coherent"] < info["us_per_step"][1] else 1)
    g = solved(wm, 64)
    qh.bsb_solve(g, 64, 100, seed=3, plan=1)
    timed(g, 64)
    # row tiles that skip column tiles: a field goes through the per-step or the persistent kernel
    w = synth.read_small(6, 200000, 700, (2, 4))
    perm = np.random.default_rng(1).permutation(700)
    cnt = np.diff(w.frag_ptr)
    idx = np.concatenate([np.arange(w.frag_ptr[f], w.frag_ptr[f + 1]) for f in perm])
    w.frag_ptr = np.concatenate([[0], np.cumsum(cnt[perm])]).astype(np.int64)
    w.snp, w.allele, w.phred = w.snp[idx], w.allele[idx], w.phred[idx]
    g = solved(w, 64)
    qh.bsb_solve(g, 64, 100, seed=3, field=torch.zeros(700, dtype=torch.float32, device="cuda"))
    timed(g, 64)


@pytest.mark.parametrize("reads,R,dtype,tile", [(1600, 32, "f16", 16), (1600, 32, "f32", 32), (1600, 16, "fp8", 16),
                                                (13000, 32, "bf16", 32)])
def test_default_tile_outlives_a_plan_0_solve(reads, R, dtype, tile):
    """Fewer than 64 replicas: the per-step kernel's tile is chosen by the fill before and after a
    plan-0 solve, and plan_info reports the tile that ran."""
    g = gpu_graph(synth.read_small(9, reads * 3 // 2, reads, (20, 60)), "read_signed", dtype)
    for plan in (1, 0, 1):
        qh.bsb_solve(g, R, 20, seed=3, plan=plan)
        if plan == 1:
            assert g.plan_info(R)["replica_tile"] == tile


@pytest.mark.parametrize("n,gap,dtype,R", BAND_PLAN_CASES[:9])
def test_band_mfma_equals_per_row_bit_exact(n, gap, dtype, R):
    """Band blocks on MFMAs against the per-row kernel, bit for bit: plan 0 runs ranges too short for one
    launch on either, and a schedule split into ranges has to give the same state however it is
    split."""
    g = gpu_graph(synth.snp_small(5, n_snp=n, gap_mean=gap), "snp_llr", dtype)
    field = torch.linspace(-0.3, 0.3, n, dtype=torch.float32, device="cuda")
    for kw in (dict(step_end=40), dict(step_end=40, field=field), dict(step_end=40, discrete=True)):
        got = []
        for plan in (3, 5, 0):
            x, y = (torch.empty((n, R), dtype=torch.float32, device="cuda") for _ in range(2))
            if plan:
                qh.bsb_solve(g, R, 60, seed=9, x=x, y=y, plan=plan, readout=False, **kw)
            else:
                for a, b in ((0, 1), (1, 3), (3, 6), (6, 11), (11, 17), (17, 40)):
                    qh.bsb_solve(g, R, 60, seed=9, x=x, y=y, readout=False, init=a == 0,
                                 **{**kw, "step_begin": a, "step_end": b})
            got.append((x, y))
        for x, y in got[1:]:
            assert torch.equal(got[0][0], x) and torch.equal(got[0][1], y)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_band_mfma_equals_per_row_bit_exact_long_range(dtype):
    w = synth.snp_porec(43, n_snp=2500, n_edges=4000, zipf_s=1.0)
    g = gpu_graph(w, "snp_llr", dtype, band_limit=100)
    got = []
    for plan in (3, 5):
        x, y = (torch.empty((2500, 64), dtype=torch.float32, device="cuda") for _ in range(2))
        qh.bsb_solve(g, 64, 200, seed=9, x=x, y=y, plan=plan, readout=False)
        got.append((x, y))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


def _segments(lengths, seed=8):
    """SNPs in stretches that no read crosses: one component each, of reads over neighbouring SNPs."""
    rng = np.random.default_rng(seed)
    n = int(sum(lengths))
    last = np.cumsum(lengths) - 1
    first = np.setdiff1d(np.arange(n), last).repeat(3)
    w = synth.snp_small(seed, n_snp=n)
    w.frag_ptr = 2 * np.arange(first.size + 1, dtype=np.int64)
    w.snp = np.stack([first, first + 1], 1).reshape(-1).astype(np.int32)
    w.allele = rng.integers(0, 2, w.snp.size).astype(w.allele.dtype)
    w.phred = rng.integers(5, 40, w.snp.size).astype(np.uint8)
    w.alpha = np.ones(first.size)
    return w


@pytest.mark.parametrize("R", [16, 64])
@pytest.mark.parametrize("lengths", [[2048, 2049, 2, 3, 4300, 40] + [2] * 300 + [2080, 2081], [2] * 1500, [2048], [2049]])
def test_readout_components_around_the_stage(lengths, R):
    """Components of up to 64 chunks of 32 vertices (summed in one go), of 65 and more (staged), in any
    order, alone and in a batch."""
    w = _segments(lengths)
    _readout_case(w, "snp_llr", R, 4, False)
    gs = [gpu_graph(w, "snp_llr", "f32"), gpu_graph(_segments([2, 2100, 5]), "snp_llr", "f32")]
    b = qh.bsb_solve_batched(gs, R, 10, seed=3)
    for i, g in enumerate(gs):
        r = qh.bsb_solve(g, R, 10, seed=3)
        assert torch.equal(b["cuts"][i * R:(i + 1) * R], r["cuts"]) and torch.equal(b["best_cut"][i:i + 1], r["best_cut"])
        assert torch.equal(b["selected_cut"][i:i + 1], r["selected_cut"])


@pytest.mark.parametrize("lengths", [[65536, 3, 500], [3, 65537, 2, 2, 4000], [2] * 40000])
def test_phase_counts_of_large_and_small_components(lengths):
    """The sides of a component are counted by a wave per 64 vertices, or over longer walks where a component
    has more than 65,536."""
    w = _segments(lengths)
    g = gpu_graph(w, "snp_llr", "f32")
    comp, nc = oracle.components(oracle_graph(w, "snp_llr"))
    s = np.where(np.random.default_rng(2).random(comp.size) < 0.4, 1, -1).astype(np.int8)
    h1, blk = qh.phase(g, torch.tensor(s, device="cuda"))
    ho, bo = oracle.phase_parity(comp, nc, s, w.init_h1)
    assert np.array_equal(cpu(h1), ho) and np.array_equal(cpu(blk), bo)


@pytest.fixture
def no_exchange():
    """No device memory for the exchange buffers of the one-launch plans."""
    v = ctypes.c_int64.in_dll(qh.load(), "_ZN2qh14exchange_limitE")
    old, v.value = v.value, 0
    yield v
    v.value = old


@pytest.mark.parametrize("kind,dtype,n,reads,R", [
    ("snp_llr", "f16", 2001, 0, 128), ("read_signed", "f32", 2300, 1501, 64), ("read_signed", "bf16", 2300, 1501, 64)])
def test_no_memory_for_the_exchange(no_exchange, kind, dtype, n, reads, R):
    """A graph whose one-launch plan finds no memory for its buffers solves per step, as it did before that
    plan."""
    g, ref = _one_launch_case(kind, dtype, n, reads, R)
    a = qh.bsb_solve(g, R, 60, seed=9, plan=ref)
    b = qh.bsb_solve(g, R, 60, seed=9)
    if dtype != "bf16":
        assert g.plan_info(R)["plan_used"] == 1
    assert torch.equal(a["best_spins"], b["best_spins"]) and torch.equal(a["cuts"], b["cuts"])


def test_no_memory_for_the_teams_of_a_batch(team_batch, no_exchange):
    gs = team_batch[-8:]
    a = qh.bsb_solve_batched(gs, 32, 40, seed=5, plan=1, return_state=True)
    b = qh.bsb_solve_batched(gs, 32, 40, seed=5, return_state=True)
    for k in ("x", "y", "cuts", "best_spins", "best_cut"):
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("kind,dtype,n,reads", [("snp_llr", "f16", 2001, 0), ("read_signed", "f32", 1500, 1000),
                                                ("read_signed", "f16", 1500, 1000), ("read_signed", "fp8", 12000, 8000)])
def test_plan_0_under_capture_after_a_warm_solve(kind, dtype, n, reads):
    """A caller captures a plan-0 range of a graph that it has solved before: the per-step launches are
    recorded, and every replay gives the eager solve's state, with eager work between the replays."""
    g, _ = _one_launch_case(kind, dtype, n, reads, 64)
    nv = g.info()["n"]
    xe, ye, x, y = (torch.zeros((nv, 64), dtype=torch.float32, device="cuda") for _ in range(4))
    kw = dict(seed=9, step_end=30, readout=False)
    qh.bsb_solve(g, 64, 40, x=xe, y=ye, **kw)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s, capture_error_mode="thread_local"):
        qh.bsb_solve(g, 64, 40, x=x, y=y, **kw)
    for _ in range(3):
        x.zero_(), y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(x, xe) and torch.equal(y, ye)
        qh.bsb_solve(g, 64, 40, seed=4, readout=False)
        torch.cuda.synchronize()


@pytest.fixture(scope="module")
def mixed_batch():
    """Blocks that run as teams, and one of 5,000 reads (FP8) whose row tiles span more than 64 column tiles:
    it runs per step, beside the teams."""
    ws = [synth.read_small(30, 400, 1300, (20, 120)), synth.snp_small(40, 2500), synth.snp_small(41, 300),
          synth.read_small(31, 200, 90, (20, 60)), synth.read_small(9, 60, 5000, (20, 50))]
    kinds = ["read_signed", "snp_llr", "snp_llr", "read_signed", "read_signed"]
    gs = [gpu_graph(w, k, d) for w, k, d in zip(ws, kinds, ["f16", "bf16", "bf16", "f16", "fp8"])]
    yield gs
    for g in gs:
        g.free()


@pytest.mark.parametrize("R", [16, 32, 64])
@pytest.mark.parametrize("graph", [False, True])
def test_batch_rest_beside_the_teams(mixed_batch, R, graph):
    """Which blocks of a batch run as teams, some of several workgroups, and that the others, on the side
    stream beside them, plain or as a captured replay, give the per-step plan's bits; several
    replays with other work between them, another seed, and the same blocks without the large one."""
    gs = mixed_batch
    for seed in (9, 9, 10, 9):
        a = qh.bsb_solve_batched(gs, R, 100, seed=seed, plan=1, return_state=True)
        assert [g.plan_info(R)["plan_used"] for g in gs] == [1] * len(gs)
        torch.cuda.synchronize()
        b = qh.bsb_solve_batched(gs, R, 100, seed=seed, use_graph=graph, return_state=True)
        info = [g.plan_info(R) for g in gs]
        assert [i["plan_used"] for i in info[:4]] == [2] * 4
        assert info[4]["plan_used"] == b["plan_used"] and info[4]["replicas_per_group"] == 0
        assert max(i["workgroups_per_group"] for i in info[:2]) > 1 and info[3]["workgroups_per_group"] == 1
        assert all(i["replicas_per_group"] * i["groups"] == R and i["lds_bytes"] > 0 for i in info[:4])
        for k in ("x", "y", "cuts", "selected_cut", "best_spins", "best_cut"):
            assert torch.equal(a[k], b[k]), (seed, k)
        qh.bsb_solve(gs[0], R, 50, seed=1)
    a = qh.bsb_solve_batched(gs[:4], R, 100, seed=9, plan=1)
    b = qh.bsb_solve_batched(gs[:4], R, 100, seed=9, use_graph=graph)
    assert torch.equal(a["best_spins"], b["best_spins"]) and torch.equal(a["best_cut"], b["best_cut"])


def test_which_blocks_run_as_teams(team_batch):
    """All of team_batch's blocks run as teams, some of them of several workgroups, but the FP32 read block
    (per step beside them) and, with a field, the one whose row tiles skip column tiles."""
    gs = team_batch
    n = sum(g.info()["n"] for g in gs)
    for field, rest in ((None, [600]), (torch.zeros(n, dtype=torch.float32, device="cuda"), [600, 607])):
        qh.bsb_solve_batched(gs, 32, 31, seed=5, field=field)
        info = [g.plan_info(32) for g in gs]
        assert [b for b, i in enumerate(info) if i["replicas_per_group"] == 0] == rest
        assert all(i["plan_used"] == 2 for b, i in enumerate(info) if b not in rest)
        assert sum(i["workgroups_per_group"] > 1 for i in info) >= 7 - len(rest)


@pytest.mark.parametrize("plan", [1, 2])
def test_batched_plan_1_graph_replay_bit_exact(mixed_batch, plan):
    """use_graph with plan 1: every block's steps captured once and replayed, bit for bit."""
    for seed in (9, 9, 10, 9):
        a = qh.bsb_solve_batched(mixed_batch, 32, 60, seed=seed, plan=plan, return_state=True)
        b = qh.bsb_solve_batched(mixed_batch, 32, 60, seed=seed, plan=1, use_graph=True, return_state=True)
        assert b["plan_used"] == 1
        for k in ("x", "y", "cuts", "best_spins", "best_cut"):
            assert torch.equal(a[k], b[k]), (seed, k)
        qh.bsb_solve(mixed_batch[1], 32, 50, seed=1)


@pytest.mark.parametrize("kind,dtype", RESUME_CASES)
def test_captured_step_loop_bit_exact(kind, dtype):
    """use_graph with plan 1: the captured step loop replayed, with the eager steps' bits; a plan-0 solve
    between the replays (another step kernel on SNP graphs) leaves it valid."""
    w = synth.read_small(16, n_snp=300, n_reads=140) if kind != "snp_llr" else synth.snp_small(16, n_snp=900)
    g = gpu_graph(w, kind, dtype)
    n, R = g.info()["n"], 64
    out = []
    for rep in range(5):
        x, y = (torch.empty((n, R), dtype=torch.float32, device="cuda") for _ in range(2))
        r = qh.bsb_solve(g, R, 200, seed=5, x=x, y=y, plan=1, use_graph=rep > 0)
        assert g.plan_info(R)["plan_used"] == 1
        out.append((x, y, r["best_spins"], r["best_cut"], r["cuts"]))
        qh.bsb_solve(g, R, 200, seed=6, plan=0 if rep % 2 else 1)
    for o in out[1:]:
        assert all(torch.equal(a, b) for a, b in zip(out[0], o))


def test_plan_info_of_the_last_solve():
    """The geometry of the plan that the last solve ran, kept over calls that only read out."""
    g = gpu_graph(synth.read_mhc(seed=78, n_snp=1500, n_reads=1000, region=500_000), "read_signed", "f16")
    n = g.info()["n"]
    x, y = (torch.empty((n, 64), dtype=torch.float32, device="cuda") for _ in range(2))

    def info(plan):
        qh.bsb_solve(g, 64, 60, seed=9, x=x, y=y, plan=plan)
        a = g.plan_info(64)
        qh.bsb_solve(g, 64, 60, init=False, x=x, y=y, step_begin=60, step_end=60, plan=plan if plan != 2 else 0)
        assert g.plan_info(64)["plan_used"] == a["plan_used"]
        return a

    p2 = info(2)
    assert p2["plan_used"] == 2 and p2["persistent_sync"] == 1 and p2["workgroups_per_group"] > 1
    one = info(0)
    assert one["plan_used"] == 2 and one["persistent_sync"] == 2
    assert one["replicas_per_group"] * one["groups"] == 64
    assert (one["workgroups_per_group"], one["lds_bytes"]) != (p2["workgroups_per_group"], p2["lds_bytes"])
    assert info(1)["plan_used"] == 1


def test_autotune_picks_a_plan_that_is_fast_over_a_whole_solve():
    """The persistent plan loads the couplings before its first step; the tuner's few steps must not make it
    look slower than the per-step kernel where a whole solve is 1.6 times as fast (1,500 reads, F16, R = 64:
    3.1 against 5.1 ms per 1,000 steps).  The choice may be at most a quarter slower than the other plan."""
    g = gpu_graph(synth.read_small(9, 2250, 1500, (20, 60)), "read_signed", "f16")
    ch = qh.autotune(g, 64, 1000)

    def ms(**opts):
        ts = []
        for _ in range(4):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            qh.bsb_solve(g, 64, 1000, seed=3, readout=False, **opts)
            e1.record()
            e1.synchronize()
            ts.append(e0.elapsed_time(e1))
        return min(ts)

    opts = {k: ch[k] for k in ("plan", "replica_tile", "tiles_in_flight", "persistent_sync")}
    assert ms(**opts) <= 1.25 * min(ms(plan=1), ms(plan=2))


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16", "fp8"])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_non_finite_state_in_a_row_tile_without_couplings(dtype, bad):
    """A caller's state with one non-finite value among 64 reads that share no SNP with any other: it stays in
    its row (no tile of theirs is stored), under plan 0 as in the per-step kernels."""
    w = synth.read_small(6, 400, 200, (20, 60))
    lone = np.arange(128, dtype=np.int32)
    w.frag_ptr = np.concatenate([2 * np.arange(64), 128 + w.frag_ptr]).astype(np.int64)
    w.snp = np.concatenate([lone, w.snp + 128]).astype(np.int32)
    w.allele = np.concatenate([lone % 2, w.allele]).astype(w.allele.dtype)
    w.phred = np.concatenate([np.full(128, 30), w.phred]).astype(np.uint8)
    w.init_h1 = np.concatenate([np.zeros(128), w.init_h1]).astype(w.init_h1.dtype)
    w.alpha = np.ones(264)
    d = device_reads(w)
    g = qh.build_graph(d["frag_ptr"], d["snp"], d["allele"], d["phred"], d["init_h1"], kind="read_signed", dtype=dtype)
    assert g.info()["n"] == 264
    rng = np.random.default_rng(3)
    x0 = torch.tensor(rng.uniform(-0.5, 0.5, (264, 64)), dtype=torch.float32, device="cuda")
    x0[5, 3] = bad
    out = []
    for plan in (1, 0):
        x, y = x0.clone(), torch.zeros_like(x0)
        qh.bsb_solve(g, 64, 40, init=False, x=x, y=y, step_end=20, plan=plan, readout=False)
        out.append((x, y))
    assert torch.isfinite(out[0][1][6:64]).all()
    for a, b in zip(*out):
        assert torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(7.0), b.nan_to_num(7.0))

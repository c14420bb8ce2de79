"""GPU parity of the HIP codec (through the C ABI) against the CPU oracle.

Inputs come from the seeded generator (``synth``) or are designed here; every
expected value comes from ``oracle`` (float64, rounded once to the output
dtype) or from the stored exact fixture.  Nothing the GPU produces is fed to
the oracle.  Every element of every output is compared, at the full sizes
too (the oracle works through the rows in chunks on a thread pool).
"""
from __future__ import annotations

import json
import os
from fractions import Fraction

import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2506_01260_amd as sn
from gpu_helpers import assert_parity, assert_parity_rows, dev, host, host_bits, ids, log

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "tiny_exact.json")

_CACHE: dict = {}


def workload(cfg: int, n: int | None = None, sigma: float | None = None) -> dict:
    key = (cfg, n, sigma)
    if key not in _CACHE:
        log(f"[gen] config {cfg} n={n} sigma={sigma}")
        _CACHE.clear()  # keep host memory bounded: one workload at a time
        _CACHE[key] = synth.make_workload(cfg, n, sigma)
    return _CACHE[key]


def oracle_inputs(w: dict) -> dict:
    """Exact float32 views of the stored inputs (the oracle up-converts the
    rows it uses to float64); decoded once per workload."""
    if "_oracle_inputs" in w:
        return w["_oracle_inputs"]
    dt = w["cfg"].dtype
    if dt == "bf16":
        dec = lambda a: oracle.decode_bf16(a, np.float32)  # noqa: E731
    else:
        dec = lambda a: np.asarray(a, np.float32)  # noqa: E731
    out = {name: dec(w[name]) for name in ("E", "P", "X", "G")}
    out["U"] = dec(w["U"]).astype(np.float64)
    w["_oracle_inputs"] = out
    return out


def host_rows(t: torch.Tensor, sel: np.ndarray) -> np.ndarray:
    return host(t[torch.from_numpy(np.asarray(sel, dtype=np.int64)).cuda()])


def host_f32(t: torch.Tensor) -> np.ndarray:
    """Device tensor -> float32 numpy (bf16 converts exactly)."""
    return t.detach().float().cpu().numpy()


OPS = ("compress", "decompress", "grad_compress", "grad_decompress", "roundtrip")

_OUT: dict = {}


def codec_outputs(w: dict, key) -> dict:
    """The four codec ops of workload w run once on the GPU through the C ABI
    (the launch configuration the benchmark times: whole batch, default
    positions), plus the forward round trip decompress(compress(X)); host
    float32 copies.  The decompress inputs are the generator's coefficients
    C_true (stored in the dtype), the same on both sides."""
    if key in _OUT:
        return _OUT[key]
    _OUT.clear()
    cfg = w["cfg"]
    dt = cfg.dtype
    U = dev(w["U"], dt)
    basis = sn.sn_basis_pack(U)
    X, E, P, G = dev(w["X"], dt), dev(w["E"], dt), dev(w["P"], dt), dev(w["G"], dt)
    tok = ids(w["tok"])
    n = w["tok"].shape[0]
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    Cin_np = synth.store(w["C_true"], dt)
    Cin = dev(Cin_np, dt)
    log(f"[gpu] codec ops N={n} d={cfg.d} k={cfg.k} {dt}")
    out = {"Cin": Cin_np}
    C = sn.sn_compress(basis, X, tok=tok, E=E, P=P, seq_len=cfg.seq, err_flag=flag)
    out["compress"] = host_f32(C)
    out["roundtrip"] = host_f32(sn.sn_decompress(basis, C, tok=tok, E=E, P=P, seq_len=cfg.seq))
    out["decompress"] = host_f32(sn.sn_decompress(basis, Cin, tok=tok, E=E, P=P,
                                                  seq_len=cfg.seq, err_flag=flag))
    out["grad_compress"] = host_f32(sn.sn_grad_compress(basis, G))
    out["grad_decompress"] = host_f32(sn.sn_decompress(basis, Cin))
    torch.cuda.synchronize()
    out["flag"] = int(flag.item())
    del X, E, P, G, C, Cin, basis, U
    torch.cuda.empty_cache()
    _OUT[key] = out
    return out


def check_op(w: dict, out: dict, op: str, tag: str):
    """One op's GPU result against the oracle, every element (row chunks)."""
    cfg = w["cfg"]
    dt = cfg.dtype
    o = oracle_inputs(w)
    tok, seq = w["tok"], cfg.seq
    Cin64 = oracle.decode_bf16(out["Cin"]) if dt == "bf16" else out["Cin"].astype(np.float64)
    assert out["flag"] == 0, "no id is out of range in generated workloads"
    if op == "compress":
        assert_parity_rows(out[op], lambda r: oracle.compress(o["X"], o["U"], tok, o["E"], o["P"],
                                                              seq_len=seq, rows=r),
                           dt, f"{tag} compress")
    elif op == "decompress":
        assert_parity_rows(out[op], lambda r: oracle.decompress(Cin64, o["U"], tok, o["E"],
                                                                o["P"], seq_len=seq, rows=r),
                           dt, f"{tag} decompress")
    elif op == "grad_compress":
        assert_parity_rows(out[op], lambda r: oracle.grad_compress(o["G"], o["U"], rows=r),
                           dt, f"{tag} grad_compress")
    elif op == "grad_decompress":
        assert_parity_rows(out[op], lambda r: oracle.grad_decompress(Cin64, o["U"], rows=r),
                           dt, f"{tag} grad_decompress")
    else:
        # property at any size: the forward round trip loses only the
        # off-subspace residual (plus rounding of C and X_rec to the dtype)
        Xh = o["X"].astype(np.float64)
        Xrt = out[op].astype(np.float64)
        err = np.linalg.norm(Xrt - Xh)
        pos = oracle.default_positions(Xh.shape[0], seq)
        resid = Xh - o["E"][tok] - o["P"][pos]
        off = np.linalg.norm(resid - (resid @ o["U"]) @ o["U"].T)
        scale = np.linalg.norm(Xh)
        slack = (1e-5 if dt == "f32" else 2e-2) * scale
        log(f"[{tag}] round trip |X_rec - X| = {err:.4g}, off-subspace {off:.4g}, |X| {scale:.4g}")
        assert abs(err - off) <= slack


def run_codec(w: dict, tag: str):
    """Forward and gradient codec of workload w on the GPU vs the oracle,
    every element of every op."""
    out = codec_outputs(w, ("run", tag))
    for op in OPS:
        check_op(w, out, op, tag)


# ---------------------------------------------------------------- fixtures

def _golden(d_pad: int, dtype: str):
    g = json.load(open(GOLDEN))
    d = g["d"]
    f = lambda m: np.array([[float(Fraction(v)) for v in r] for r in m])  # noqa: E731

    def pad(a):
        out = np.zeros((a.shape[0], d_pad))
        out[:, :d] = a
        return out

    mats = {n: f(g[n]) for n in ("U", "E", "P", "X", "G")}
    mats = {n: pad(a.T).T if n == "U" else pad(a) for n, a in mats.items()}
    mats["U"] = mats["U"]  # d_pad x k, zero rows past d
    W = np.zeros((d_pad, 6))
    W[:d] = f(g["W"])
    mats["W"] = W
    ex = {n: f(v) for n, v in g["expect"].items()}
    ex["X_rec"] = pad(ex["X_rec"])
    ex["G_rec"] = pad(ex["G_rec"])
    Wp = np.zeros((d_pad, 6))
    Wp[:d] = ex["W_proj"]
    ex["W_proj"] = Wp
    return g, mats, ex


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d_pad", [8, 32, 64])
def test_golden_fixture_exact(dtype, d_pad):
    """Dyadic inputs whose exact results every dtype represents: bit-exact."""
    log(f"[golden] dtype={dtype} d={d_pad}")
    g, m, ex = _golden(d_pad, dtype)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    t = {n: torch.tensor(np.ascontiguousarray(a), dtype=tdt, device="cuda") for n, a in m.items()}
    basis = sn.sn_basis_pack(t["U"])
    tok, pos = ids(np.array(g["tok"])), ids(np.array(g["pos"]))
    C = sn.sn_compress(basis, t["X"], tok=tok, E=t["E"], P=t["P"], pos=pos)
    assert np.array_equal(host(C), ex["C"])
    Xr = sn.sn_decompress(basis, C, tok=tok, E=t["E"], P=t["P"], pos=pos)
    assert np.array_equal(host(Xr), ex["X_rec"])
    Cg = sn.sn_grad_compress(basis, t["G"])
    assert np.array_equal(host(Cg), ex["Cg"])
    assert np.array_equal(host(sn.sn_decompress(basis, Cg)), ex["G_rec"])
    W = t["W"].clone()
    sn.sn_project_weights(basis, W)
    assert np.array_equal(host(W), ex["W_proj"])


# ------------------------------------------------------------ the configs

@pytest.mark.parametrize("sigma", [0.0, 1e-3])
def test_config0_fp32_all_ops(sigma):
    w = workload(0, sigma=sigma)
    run_codec(w, f"cfg0 sigma={sigma}")
    cfg = w["cfg"]
    (rows, cols), = cfg.weights
    Wnp = synth.make_weight(0, 0, rows, cols)
    W = dev(Wnp, "f32")
    basis = sn.sn_basis_pack(dev(w["U"], "f32"))
    sn.sn_project_weights(basis, W)
    ref = oracle.round_to(oracle.project_weights(Wnp.astype(np.float64),
                                                 w["U"].astype(np.float64)), "f32")
    assert_parity(host(W), ref, "f32", "cfg0 project_weights")


def test_config1_bf16_full():
    run_codec(workload(1), "cfg1")


# configs 2 and 4 at full size (config 4 also with 32767 tokens: a short last
# sequence), one test per op so that each stays well inside the time limit;
# the GPU runs the four ops once per workload
_FULL = [(cfg, n, op) for cfg, n in ((2, None), (4, 32768), (4, 32767)) for op in OPS]


@pytest.mark.parametrize("cfg,n,op", _FULL, ids=[f"cfg{c}-N{n or 32768}-{o}" for c, n, o in _FULL])
def test_config_full(cfg, n, op):
    w = workload(cfg, n=n)
    tag = f"cfg{cfg} N={w['tok'].shape[0]}"
    check_op(w, codec_outputs(w, (cfg, n)), op, tag)


def check_projection(before: np.ndarray, after: np.ndarray, U64: np.ndarray, tag: str):
    """Every column of a projected weight against the oracle, plus the
    properties of the projection on the GPU result: U^T W' = U^T W and no
    off-subspace part, per column (bf16 rounding of W' and the stored,
    not exactly orthonormal bf16 U leave ~1e-3 of each column's norm)."""
    assert_parity_rows(after.T, lambda r: oracle.project_weights(before, U64, cols=r).T,
                       "bf16", f"{tag} project_weights (every column)")
    m = before.shape[1]
    step = 4096
    for c0 in range(0, m, step):
        bf = before[:, c0:c0 + step].astype(np.float64)
        af = after[:, c0:c0 + step].astype(np.float64)
        t_before, t_after = U64.T @ bf, U64.T @ af
        dt_col = np.linalg.norm(t_after - t_before, axis=0)
        assert np.all(dt_col <= 1e-2 * np.linalg.norm(t_before, axis=0) + 1e-30), \
            f"{tag}: U^T W changed in columns {np.flatnonzero(dt_col > 1e-2 * np.linalg.norm(t_before, axis=0))[:5] + c0}"
        resid = np.linalg.norm(af - U64 @ t_after, axis=0)
        assert np.all(resid <= 1e-2 * np.linalg.norm(af, axis=0) + 1e-30), \
            f"{tag}: off-subspace part left in columns {np.flatnonzero(resid > 1e-2 * np.linalg.norm(af, axis=0))[:5] + c0}"
    log(f"  {tag}: U^T W kept, no off-subspace part ({m} columns)")


def _basis_of(cfg_id: int):
    b = synth.make_basis(cfg_id)
    return oracle.decode_bf16(b["U"]), sn.sn_basis_pack(dev(b["U"], "bf16"))


def test_project_weights_config2_wo_w2():
    """Config 2's Wo (4096 x 4096) and W2 (4096 x 14336) confined by one
    call, as the optimizer step (and the benchmark) does it; every column."""
    cfg = synth.CONFIGS[2]
    U64, basis = _basis_of(2)
    hosts = [synth.make_weight(2, i, r, c) for i, (r, c) in enumerate(cfg.weights)]
    Ws = [dev(h, "bf16") for h in hosts]
    log("[cfg2] project Wo and W2 in one call")
    sn.sn_project_weights_multi(basis, Ws)
    for i, (h, W) in enumerate(zip(hosts, Ws)):
        check_projection(oracle.decode_bf16(h, np.float32), host_f32(W), U64, f"cfg2 W{i}")


def test_project_weights_config4_wo():
    """Config 4's Wo (8192 x 8192, k = 82); every column."""
    cfg = synth.CONFIGS[4]
    U64, basis = _basis_of(4)
    (r, c), = cfg.weights
    h = synth.make_weight(4, 0, r, c)
    W = dev(h, "bf16")
    log("[cfg4] project Wo")
    sn.sn_project_weights(basis, W)
    check_projection(oracle.decode_bf16(h, np.float32), host_f32(W), U64, "cfg4 Wo")


@pytest.mark.parametrize("group", range(4))
def test_config3_layer_sweep(group):
    """The 32-layer sweep of (Wo, W2), in the benchmark's calls of 16 matrices
    (8 layers) each; this test is call `group`.  Weights are drawn on the
    device (seeded); each matrix is copied to the host before and after, and
    every column of all 16 is compared with the oracle."""
    cfg = synth.CONFIGS[3]
    U64, basis = _basis_of(3)
    mats, names = [], []
    for layer in range(8 * group, 8 * group + 8):
        for i, (r, c) in enumerate(cfg.weights):
            mats.append(synth.device_weight(3, 2 * layer + i, r, c))
            names.append(f"cfg3 L{layer} W{i}")
    before = [host_f32(W) for W in mats]
    log(f"[cfg3] call {group}: layers {8 * group}..{8 * group + 7}, 16 matrices")
    sn.sn_project_weights_multi(basis, mats)
    after = [host_f32(W) for W in mats]
    del mats
    torch.cuda.empty_cache()
    for name, bf, af in zip(names, before, after):
        check_projection(bf, af, U64, name)


# --------------------------------------------------------------- edge cases

def _small(d, k, n, vocab=50, seq=9, dtype="bf16", seed=0, grid=None):
    rng = np.random.default_rng(seed)
    U, _ = np.linalg.qr(rng.standard_normal((d, k)))
    E = rng.standard_normal((vocab, d)) * 0.05
    P = rng.standard_normal((seq, d)) * 0.05
    C = rng.standard_normal((n, k))
    tok = rng.integers(0, vocab, n).astype(np.int32)
    pos = (np.arange(n) % seq).astype(np.int32)
    X = E[tok] + P[pos] + C @ U.T + rng.standard_normal((n, d)) * 0.01
    G = rng.standard_normal((n, d)) * 0.1
    if grid:
        E, P, X = (np.round(a * grid) / grid for a in (E, P, X))
    st = {name: synth.store(a, dtype) for name, a in
          dict(U=U, E=E, P=P, C=C, X=X, G=G).items()}
    f64 = {name: (oracle.decode_bf16(a) if dtype == "bf16" else a.astype(np.float64))
           for name, a in st.items()}
    return st, f64, tok, pos


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d,k,n", [(256, 20, 1), (256, 20, 17), (256, 20, 33), (256, 1, 40),
                                   (256, 16, 31), (256, 17, 50), (256, 33, 16), (256, 82, 45),
                                   (256, 128, 20), (384, 130, 19), (200, 20, 37), (96, 5, 64)])
def test_shapes(dtype, d, k, n):
    log(f"[shapes] {dtype} d={d} k={k} n={n}")
    st, o, tok, pos = _small(d, k, n, dtype=dtype, seed=d + k + n)
    basis = sn.sn_basis_pack(dev(st["U"], dtype))
    E, P, X, G, Cin = (dev(st[x], dtype) for x in ("E", "P", "X", "G", "C"))
    t_tok = ids(tok)
    C = sn.sn_compress(basis, X, tok=t_tok, E=E, P=P, seq_len=9)
    assert_parity(host(C), oracle.round_to(oracle.compress(o["X"], o["U"], tok, o["E"], o["P"],
                                                           seq_len=9), dtype), dtype, "compress")
    Xr = sn.sn_decompress(basis, Cin, tok=t_tok, E=E, P=P, seq_len=9)
    assert_parity(host(Xr), oracle.round_to(oracle.decompress(o["C"], o["U"], tok, o["E"],
                                                              o["P"], seq_len=9), dtype),
                  dtype, "decompress")
    Cg = sn.sn_grad_compress(basis, G)
    assert_parity(host(Cg), oracle.round_to(oracle.grad_compress(o["G"], o["U"]), dtype), dtype,
                  "grad_compress")
    W = G[: min(n, 64)].T.contiguous() if n >= 1 else None   # d x m
    Wn = host(W)
    sn.sn_project_weights(basis, W)
    assert_parity(host(W).T, oracle.round_to(oracle.project_weights(Wn, o["U"]), dtype).T,
                  dtype, "project_weights")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("tables", ["EP", "E", "P", ""])
@pytest.mark.parametrize("d,k,n,pad", [(7, 3, 5, 0), (31, 4, 16, 1), (33, 15, 65, 3), (49, 17, 63, 0),
                                       (95, 49, 64, 5), (161, 33, 4200, 0), (100, 97, 17, 1),
                                       (300, 129, 130, 2), (257, 256, 33, 0)])
def test_generic_kernel_edges(dtype, d, k, n, pad, tables):
    """The float64 matrix-core kernels at the edges of their tiles: widths
    around 16 and 32 columns (and below one unit), column tiles of U that are
    part-filled or split over workgroups, token tiles of every occupancy, few
    and many workgroups, odd row strides.  float32 results are one rounding
    (2^-24 of the value) off the exact sum, up to the sum's own cancellation:
    2^-22 of max(|value|, row rms)."""
    log(f"[generic] {dtype} d={d} k={k} n={n} pad={pad} tables={tables!r}")
    st, o, tok, pos = _small(d, k, n, dtype=dtype, seed=d + k + n)
    basis = sn.sn_basis_pack(dev(st["U"], dtype))

    def padded(a):  # the same values at a row stride of cols + pad
        t = dev(a, dtype)
        buf = torch.full((t.shape[0], t.shape[1] + pad), float("nan"), dtype=t.dtype, device="cuda")
        buf[:, :t.shape[1]] = t
        return buf[:, :t.shape[1]]

    E, P = (padded(st[x]) if x in tables else None for x in "EP")
    oE, oP = (o[x] if x in tables else None for x in "EP")
    where = dict(tok=ids(tok), seq_len=9)
    X, C = padded(st["X"]), padded(st["C"])
    got_c = sn.sn_compress(basis, X, E=E, P=P, **where)
    got_x = sn.sn_decompress(basis, C, E=E, P=P, **where)
    proj = sn.sn_embed_project(basis, E=E, P=P)
    got_p = sn.sn_compress_projected(basis, X, proj, **where)
    ref_c = oracle.compress(o["X"], o["U"], tok, oE, oP, seq_len=9)
    ref_x = oracle.decompress(o["C"], o["U"], tok, oE, oP, seq_len=9)
    for got, ref, what in ((got_c, ref_c, "compress"), (got_p, ref_c, "projected"),
                           (got_x, ref_x, "decompress")):
        assert_parity(host(got), oracle.round_to(ref, dtype), dtype, what)
        if dtype == "f32" and what != "projected":
            tol = 2.0 ** -22 * np.maximum(np.abs(ref), np.sqrt(np.mean(ref * ref, -1, keepdims=True)))
            assert np.all(np.abs(host(got) - ref) <= tol), what


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d,k,n,pad", [(1, 1, 1, 0), (131, 10, 1000, 1), (131, 10, 1001, 1),  # 5 2^18 products
                                       (8, 2, 65536, 0), (8, 2, 65537, 0), (7, 3, 75001, 2),  # 2^19 values
                                       (33, 15, 2701, 3), (49, 17, 1601, 0), (95, 49, 290, 5),
                                       (31, 20, 2129, 1)])
def test_generic_recovery_of_few_and_many_values(dtype, d, k, n, pad):
    """The generic recovery on both sides of the rule that gives each value a
    thread of its own, and past it partial column tiles, ranks and token groups of
    the matrix-core form; rows wider than d stay as they were past it."""
    log(f"[generic recovery] {dtype} d={d} k={k} n={n} pad={pad}")
    st, o, tok, pos = _small(d, k, n, dtype=dtype, seed=d + k + n)
    basis = sn.sn_basis_pack(dev(st["U"], dtype))
    E, P, C = (dev(st[x], dtype) for x in "EPC")
    for t in ("EP", "E", "P", ""):
        out = torch.full((n, d + pad), 7.0, device="cuda", dtype=C.dtype)
        sn.sn_decompress(basis, C, tok=ids(tok), E=E if "E" in t else None,
                         P=P if "P" in t else None, pos=ids(pos), out=out[:, :d])
        assert bool((out[:, d:] == 7.0).all())
        ref = oracle.decompress(o["C"], o["U"], tok, o["E"] if "E" in t else None,
                                o["P"] if "P" in t else None, pos=pos)
        if dtype == "bf16":
            assert_parity(host(out[:, :d]), oracle.round_to(ref, dtype), dtype, f"recovery {t!r}")
        else:  # one rounding of a float64 sum of k + 2 terms
            terms = np.abs(o["C"]) @ np.abs(o["U"]).T + np.abs(ref)
            err = np.abs(host(out[:, :d]) - ref)
            assert np.all(err <= 2.0 ** -24 * np.abs(ref) + 1e-14 * terms + 1e-45), t


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d,k,m,pad", [(7, 3, 5, 0), (31, 4, 64, 1), (33, 17, 65, 3), (161, 33, 1, 0),
                                       (600, 70, 130, 1), (1000, 129, 67, 5), (300, 256, 40, 0)])
def test_generic_weights_edges(dtype, d, k, m, pad):
    """The float64 weight projection at the edges of its tiles: rows around a
    unit of 32, part-filled column tiles of U (one to several per workgroup),
    column blocks of W and row tiles, odd row strides.  float32: T and the
    result are float64 sums rounded once (2^-24), 2^-22 of max(|value|,
    column rms)."""
    log(f"[generic weights] {dtype} d={d} k={k} m={m} pad={pad}")
    st, o, _, _ = _small(d, k, m, dtype=dtype, seed=d + k + m)
    basis = sn.sn_basis_pack(dev(st["U"], dtype))
    buf = torch.full((d, m + pad), float("nan"), device="cuda",
                     dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
    W = buf[:, :m]
    W.copy_(dev(st["G"], dtype).T)
    sn.sn_project_weights(basis, W)
    ref = oracle.project_weights(o["G"].T, o["U"]).T
    assert_parity(host(W).T, oracle.round_to(ref, dtype), dtype, "project_weights")
    assert bool(torch.isnan(buf[:, m:]).all())
    if dtype == "f32":
        tol = 2.0 ** -22 * np.maximum(np.abs(ref), np.sqrt(np.mean(ref * ref, -1, keepdims=True)))
        assert np.all(np.abs(host(W).T - ref) <= tol)


def test_basis_of_more_than_2_29_rows():
    """A basis of 2^29 + 33 rows, whose operand sections take more threads to pack
    than one grid dimension has: its last rows arrive in both."""
    log("[pack] d=2^29+33 k=1, float32")
    d = (1 << 29) + 33
    U = torch.zeros(d, 1, device="cuda")
    U[d - 1], U[d - 40], U[7] = 2.0, 3.0, 4.0
    basis = sn.sn_basis_pack(U)
    C = sn.sn_grad_compress(basis, torch.ones(1, d, device="cuda"))
    assert float(C) == 9.0
    X = sn.sn_decompress(basis, torch.ones(1, 1, device="cuda"))
    assert torch.equal(X[0], U[:, 0])


def test_generic_kernels_past_2_32_threads():
    """Token and column counts whose workgroups take more threads than one grid
    dimension has (float32, d = k = 1, U = 1/2: every result is exact): compress
    and accumulate of 2^30 + 65 tokens, projection of 2^30 + 129 columns."""
    log("[generic] d=k=1, 2^30 + 65 tokens, 2^30 + 129 columns")
    n, m = (1 << 30) + 65, (1 << 30) + 129
    basis = sn.sn_basis_pack(torch.full((1, 1), 0.5, device="cuda"))
    G = torch.ones(n, 1, device="cuda")
    G[n - 70:, 0] = 2.0
    state = sn.sn_grassmann_state(basis)
    Cg = sn.sn_grassmann_accumulate(basis, G, state, want_cg=True)
    energy = float(n - 70 + 4 * 70)
    assert float(state.scalars()[0]) == 0.5625 * energy and float(state.Y()) == 0.5 * energy
    assert bool((Cg == 0.5 * G).all())
    del Cg
    C = sn.sn_compress(basis, G)
    assert bool((C == 0.5 * G).all())
    del C, G
    W = torch.ones(1, m, device="cuda")
    W[0, m - 200:] = 4.0
    sn.sn_project_weights(basis, W)
    assert bool((W[0, :m - 200] == 0.25).all()) and bool((W[0, m - 200:] == 1.0).all())


def test_generic_weights_of_a_million_rows():
    """More row ranges than one grid dimension takes (d = 1100003, k = 250: 34376
    ranges of two 16-row tiles), every element against float64."""
    log("[generic weights] d=1100003 k=250 m=3")
    d, k, m = 1100003, 250, 3
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    U = torch.randn(d, k, generator=g, device="cuda") * d ** -0.5
    W = torch.randn(d, m, generator=g, device="cuda")
    t, step = torch.zeros(k, m, device="cuda", dtype=torch.float64), 1 << 18
    for r in range(0, d, step):
        t += U[r:r + step].double().T.contiguous() @ W[r:r + step].double()
    ref = torch.cat([U[r:r + step].double() @ t for r in range(0, d, step)])
    sn.sn_project_weights(sn.sn_basis_pack(U), W)
    # one rounding (2^-24 of the value) of float64 sums of k terms of about |t| |u|
    assert bool(((W.double() - ref).abs() <= 2.0 ** -22 * ref.abs() + 1e-12).all())


@pytest.mark.parametrize("dtype,d,k,n", [("f32", 7, 3, 1), ("f32", 33, 17, 65), ("f32", 130, 70, 31),
                                         ("f32", 300, 128, 1000), ("bf16", 100, 20, 129)])
def test_generic_subspace_edges(dtype, d, k, n):
    """The float64 subspace accumulation at the edges of its tiles (tokens
    around 32 and 64, part-filled column tiles and pairs): everything is
    float64, so the loss and Y agree to 1e-12 of their terms."""
    log(f"[generic subspace] {dtype} d={d} k={k} n={n}")
    st, o, _, _ = _small(d, k, n, dtype=dtype, seed=d + k + n)
    basis = sn.sn_basis_pack(dev(st["U"], dtype))
    G = dev(st["G"], dtype)
    state = sn.sn_grassmann_state(basis)
    for _ in range(2):
        cg = sn.sn_grassmann_accumulate(basis, G, state, want_cg=True)
    assert torch.equal(cg.float(), sn.sn_grad_compress(basis, G).float())
    c64 = o["G"] @ o["U"]
    loss = float(np.sum((o["G"] - c64 @ o["U"].T) ** 2))
    sc = state.scalars().cpu().numpy()
    assert abs(sc[0] - 2 * loss) <= 1e-12 * 2 * float(np.sum(o["G"] ** 2)) and sc[1] == sc[3] == 2
    err = np.abs(state.Y().cpu().numpy() - 2 * o["G"].T @ c64)
    assert np.all(err <= 1e-12 * 2 * (np.abs(o["G"]).T @ (np.abs(o["G"]) @ np.abs(o["U"]))))


@pytest.mark.parametrize("d,n", [(288, 20), (1600, 300), (416, 9000)])
def test_recovery_keeps_cancelling_sums_off_multiples_of_256(d, n):
    """bf16 recovery of widths that are multiples of 32 but not of 256 adds the
    tables to C U^T before the one rounding, in more than fp32: with a product of
    2^30 that the tables cancel, the small rest survives.  Whole numbers, so the
    results are exact."""
    log(f"[recovery, cancelling] d={d} n={n}")
    k, V = 16, 50
    g = np.random.default_rng(d)
    U, C = np.zeros((d, k), np.float32), np.zeros((n, k), np.float32)
    U[:, 0], U[:, 3] = 2.0 ** 15, g.integers(1, 100, d)
    C[:, 0], C[:, 3] = 2.0 ** 15, 1.0
    basis = sn.sn_basis_pack(dev(synth.store(U, "bf16"), "bf16"))
    table = lambda v: torch.full((V, d), v, dtype=torch.bfloat16, device="cuda")  # noqa: E731
    tok, Cd = ids(g.integers(0, V, n)), dev(synth.store(C, "bf16"), "bf16")
    for E, P in ((table(-2.0 ** 30), None), (None, table(-2.0 ** 30)),
                 (table(-2.0 ** 29), table(-2.0 ** 29))):
        X = sn.sn_decompress(basis, Cd, tok=tok, E=E, P=P, seq_len=V)
        assert np.array_equal(host(X), np.broadcast_to(U[:, 3].astype(np.float64), (n, d)))
    CS = Cd[:1].expand(V, k).contiguous()
    X = sn.sn_embed_lowrank_forward(basis, CS, tok, E=table(-2.0 ** 30))
    assert np.array_equal(host(X), np.broadcast_to(U[:, 3].astype(np.float64), (n, d)))


@pytest.mark.parametrize("d,n", [(96, 20), (1056, 300), (288, 9000)])
def test_compress_keeps_cancelling_sums_off_multiples_of_64(d, n):
    """bf16 compress with tables, widths that are multiples of 32 but not of 64:
    an activation of 2^15 that the embeddings cancel exactly leaves the small
    rest, in more than fp32.  Whole numbers, so the results are exact."""
    log(f"[compress, cancelling] d={d} n={n}")
    k, V = 16, 50
    g = np.random.default_rng(d)
    U, X = np.zeros((d, k), np.float32), np.zeros((n, d), np.float32)
    U[0], U[5] = 2.0 ** 15, g.integers(1, 100, k)
    X[:, 0], X[:, 5] = 2.0 ** 15, 1.0
    basis = sn.sn_basis_pack(dev(synth.store(U, "bf16"), "bf16"))
    tok, Xd = ids(g.integers(0, V, n)), dev(synth.store(X, "bf16"), "bf16")

    def table(v):
        t = np.zeros((V, d), np.float32)
        t[:, 0] = v
        return dev(synth.store(t, "bf16"), "bf16")

    for E, P in ((table(2.0 ** 15), None), (None, table(2.0 ** 15)),
                 (table(2.0 ** 14), table(2.0 ** 14))):
        C = sn.sn_compress(basis, Xd, tok=tok, E=E, P=P, seq_len=V)
        assert np.array_equal(host(C), np.broadcast_to(U[5].astype(np.float64), (n, k)))


@pytest.mark.parametrize("d,k,n,tables", [
    (256, 63, 50, ""), (256, 64, 50, ""), (256, 64, 50, "P"), (256, 16, 8192, ""), (256, 16, 8193, ""),
    (256, 17, 4097, ""), (3072, 33, 4100, ""), (3072, 49, 4100, ""), (1024, 16, 6144, "EP"), (1024, 16, 6145, "EP"),
    (960, 16, 4097, "E"), (3072, 48, 4097, "P"), (3072, 49, 4097, "P")])
def test_compress_on_both_sides_of_the_few_token_rule(d, k, n, tables):
    """Shapes on both sides of each line of the rule that picks the few-token
    compress (at 256 CUs): the rank against the width and one round of
    workgroups, a second round with and without tables."""
    log(f"[few-token rule] d={d} k={k} n={n} tables={tables!r}")
    st, o, tok, pos = _small(d, k, n, dtype="bf16", seed=d + k + n)
    basis = sn.sn_basis_pack(dev(st["U"], "bf16"))
    E, P = (dev(st[x], "bf16") if x in tables else None for x in "EP")
    oE, oP = (o[x] if x in tables else None for x in "EP")
    C = sn.sn_compress(basis, dev(st["X"], "bf16"), tok=ids(tok), E=E, P=P, pos=ids(pos))
    ref = oracle.compress(o["X"], o["U"], tok, oE, oP, pos=pos)
    assert_parity(host(C), oracle.round_to(ref, "bf16"), "bf16", "compress")
    if tables == "":
        G = dev(st["G"], "bf16")
        cg = sn.sn_grassmann_accumulate(basis, G, sn.sn_grassmann_state(basis), want_cg=True)
        assert torch.equal(cg.view(torch.int16), sn.sn_grad_compress(basis, G).view(torch.int16))


@pytest.mark.parametrize("d,k,n,pad", [(96, 8, 77, 0), (544, 128, 100, 0), (1056, 100, 31, 0),
                                       (288, 20, 4200, 0), (320, 20, 300, 3), (512, 70, 129, 4)])
def test_subspace_state_in_float64(d, k, n, pad):
    """bf16 accumulations off the bf16 matrix-core path keep float64 throughout:
    widths that are multiples of 32 but not of 64, and rows that are not 16-byte
    aligned on a basis that has that path.  The loss and Y agree to 1e-12 of
    their terms."""
    log(f"[subspace float64] d={d} k={k} n={n} pad={pad}")
    st, o, _, _ = _small(d, k, n, dtype="bf16", seed=d + k + n)
    basis = sn.sn_basis_pack(dev(st["U"], "bf16"))
    G = torch.full((n, d + pad), float("nan"), dtype=torch.bfloat16, device="cuda")[:, :d]
    G.copy_(dev(st["G"], "bf16"))
    state = sn.sn_grassmann_state(basis)
    cg = sn.sn_grassmann_accumulate(basis, G, state, want_cg=True)
    assert torch.equal(cg.view(torch.int16), sn.sn_grad_compress(basis, G).view(torch.int16))
    c64 = o["G"] @ o["U"]
    loss = float(np.sum((o["G"] - c64 @ o["U"].T) ** 2))
    assert abs(float(state.scalars()[0]) - loss) <= 1e-12 * float(np.sum(o["G"] ** 2))
    err = np.abs(state.Y().cpu().numpy() - o["G"].T @ c64)
    assert np.all(err <= 1e-12 * (np.abs(o["G"]).T @ (np.abs(o["G"]) @ np.abs(o["U"]))))


@pytest.mark.parametrize("tables", ["EP", "E", "P", ""])
@pytest.mark.parametrize("d,k,n", [(32, 7, 5), (64, 16, 33), (96, 33, 1), (480, 40, 17), (544, 128, 100),
                                   (1056, 100, 31), (288, 20, 8200), (256, 65, 4096),
                                   (320, 65, 4097), (256, 40, 8192), (256, 40, 8193)])
def test_few_token_compress_and_narrow_blocks(d, k, n, tables):
    """The few-token compress: fewer units of 64 columns than waves, an odd last
    step of 32, part-filled token tiles, every column-tile count class, and the
    token counts on both sides of its dispatch (one and two rounds of
    workgroups); the decompress of widths around multiples of 256.  The wire coefficients of the
    subspace update stay those of the gradient compress."""
    log(f"[few tokens] d={d} k={k} n={n} tables={tables!r}")
    st, o, tok, pos = _small(d, min(k, d), n, dtype="bf16", seed=d + k + n)
    k = min(k, d)
    basis = sn.sn_basis_pack(dev(st["U"], "bf16"))
    E, P = (dev(st[x], "bf16") if x in tables else None for x in "EP")
    oE, oP = (o[x] if x in tables else None for x in "EP")
    where = dict(tok=ids(tok), pos=ids(pos))
    C = sn.sn_compress(basis, dev(st["X"], "bf16"), E=E, P=P, **where)
    ref_c = oracle.compress(o["X"], o["U"], tok, oE, oP, pos=pos)
    assert_parity(host(C), oracle.round_to(ref_c, "bf16"), "bf16", "compress")
    Xr = sn.sn_decompress(basis, dev(st["C"], "bf16"), E=E, P=P, **where)
    ref_x = oracle.decompress(o["C"], o["U"], tok, oE, oP, pos=pos)
    assert_parity(host(Xr), oracle.round_to(ref_x, "bf16"), "bf16", "decompress")
    if tables == "":
        G = dev(st["G"], "bf16")
        state = sn.sn_grassmann_state(basis)
        cg = sn.sn_grassmann_accumulate(basis, G, state, want_cg=True)
        assert torch.equal(cg.view(torch.int16), sn.sn_grad_compress(basis, G).view(torch.int16))
        c64 = o["G"] @ o["U"]
        loss = float(np.sum((o["G"] - c64 @ o["U"].T) ** 2))
        assert abs(float(state.scalars()[0]) - loss) <= 1e-5 * float(np.sum(o["G"] ** 2))
        # C enters the token contraction as bf16 hi + lo (2^-18 of each value),
        # summed in fp32 in chains of at most 32 steps of 32 tokens (2^-19 of
        # the terms) before float64 takes over
        err = np.abs(state.Y().cpu().numpy() - o["G"].T @ c64)
        assert np.all(err <= 2.0 ** -17 * (np.abs(o["G"]).T @ np.abs(c64)))
    else:
        proj = sn.sn_embed_project(basis, E=E, P=P)
        got = sn.sn_compress_projected(basis, dev(st["X"], "bf16"), proj, **where)
        assert_parity(host(got), oracle.round_to(ref_c, "bf16"), "bf16", "projected")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_tables_optional_and_explicit_positions(dtype):
    d, k, n = 256, 24, 70
    st, o, tok, _ = _small(d, k, n, dtype=dtype, seed=5)
    rng = np.random.default_rng(6)
    pos = rng.integers(0, 9, n).astype(np.int32)      # arbitrary (e.g. context-parallel) positions
    basis = sn.sn_basis_pack(dev(st["U"], dtype))
    E, P, X, Cin = (dev(st[x], dtype) for x in ("E", "P", "X", "C"))
    cases = [("E+P explicit pos", dict(tok=ids(tok), E=E, P=P, pos=ids(pos)),
              dict(tok=tok, E=o["E"], P=o["P"], pos=pos)),
             ("E only", dict(tok=ids(tok), E=E), dict(tok=tok, E=o["E"])),
             ("P only default pos", dict(P=P, seq_len=9), dict(P=o["P"], seq_len=9)),
             ("no tables", {}, {})]
    for name, gk, ok in cases:
        C = sn.sn_compress(basis, X, **gk)
        assert_parity(host(C), oracle.round_to(oracle.compress(o["X"], o["U"], **ok), dtype),
                      dtype, f"compress {name}")
        Xr = sn.sn_decompress(basis, Cin, **gk)
        assert_parity(host(Xr), oracle.round_to(oracle.decompress(o["C"], o["U"], **ok), dtype),
                      dtype, f"decompress {name}")


@pytest.mark.parametrize("n", [187, 184, 183, 511, 512])
def test_decompress_short_last_sequence(n):
    """Default positions of [batch, seq] rows whose last sequence is short
    (seq = 64: 5, 8, 9, 1 and 0 rows missing).  Up to an eighth of a
    sequence missing, the decompress keeps position-major tiles over whole
    sequences and does not store the missing rows; beyond that it takes
    token-major tiles.  Every element against the oracle, rows past N
    untouched, no out-of-range flag."""
    d, k, seq = 256, 20, 64
    log(f"[short last sequence] n={n}")
    st, o, tok, _ = _small(d, k, n, vocab=40, seq=seq, seed=n)
    basis = sn.sn_basis_pack(dev(st["U"], "bf16"))
    E, P, Cin = (dev(st[x], "bf16") for x in ("E", "P", "C"))
    for name, gk, ok in [("E+P", dict(tok=ids(tok), E=E), dict(tok=tok, E=o["E"])),
                         ("P only", {}, {})]:
        big = torch.full((n + 64, d), 3.0, dtype=torch.bfloat16, device="cuda")
        flag = torch.zeros(1, dtype=torch.int32, device="cuda")
        sn.sn_decompress(basis, Cin, P=P, seq_len=seq, out=big[:n], err_flag=flag, **gk)
        ref = oracle.decompress(o["C"], o["U"], P=o["P"], seq_len=seq, **ok)
        assert_parity(host(big[:n]), oracle.round_to(ref, "bf16"), "bf16", f"{name} n={n}")
        assert bool((big[n:] == 3.0).all()), f"{name}: rows past N were written"
        assert int(flag.item()) == 0, f"{name}: out-of-range flag {int(flag.item())}"


@pytest.mark.parametrize("n,batch", [(256, 4), (255, 4), (249, 4), (248, 4), (247, 4),
                                     (512, 8), (511, 8), (504, 8), (503, 8)])
def test_compress_short_last_sequence(n, batch):
    """Default positions of [batch, seq] rows (seq = 64) whose last sequence
    is short by 0, 1, 7, 8 or 9 rows.  Up to an eighth of a sequence missing,
    the compress keeps position-major tiles over whole sequences (the missing
    rows are loaded as the last token's and not stored); beyond that it takes
    token-major tiles.  Every element against the oracle, rows past N of the
    output untouched, no out-of-range flag."""
    d, k, seq = 256, 40, 64
    assert batch * seq - 9 <= n <= batch * seq
    log(f"[compress short last sequence] n={n} batch={batch}")
    st, o, tok, _ = _small(d, k, n, vocab=40, seq=seq, seed=n + 1000)
    basis = sn.sn_basis_pack(dev(st["U"], "bf16"))
    E, P, X = (dev(st[x], "bf16") for x in ("E", "P", "X"))
    for name, gk, ok in [("E+P", dict(tok=ids(tok), E=E), dict(tok=tok, E=o["E"])),
                         ("P only", {}, {})]:
        big = torch.full((n + 16, k), 3.0, dtype=torch.bfloat16, device="cuda")
        flag = torch.zeros(1, dtype=torch.int32, device="cuda")
        sn.sn_compress(basis, X, P=P, seq_len=seq, out=big[:n], err_flag=flag, **gk)
        ref = oracle.compress(o["X"], o["U"], P=o["P"], seq_len=seq, **ok)
        assert_parity(host(big[:n]), oracle.round_to(ref, "bf16"), "bf16", f"{name} n={n}")
        assert bool((big[n:] == 3.0).all()), f"{name}: rows past N were written"
        assert int(flag.item()) == 0, f"{name}: out-of-range flag {int(flag.item())}"


def test_large_positional_table_streamed():
    """Both tables with a positional table over 64 MiB: compress and
    decompress then load P's rows non-temporally (a kernel variant of the
    decompress, a run-time copy policy of the compress).  Every element is
    compared: default positions of two whole sequences (position-major
    tiles) and explicit scattered positions over a ragged batch."""
    d, k, seq = 4096, 40, 8208          # P: 8208 x 4096 bf16 = 67.2 MB > 64 MiB
    n = 2 * seq
    log(f"[streamed P] d={d} k={k} seq={seq} n={n}")
    st, o, tok, _ = _small(d, k, n, vocab=300, seq=seq, seed=11)
    basis = sn.sn_basis_pack(dev(st["U"], "bf16"))
    E, P, X, Cin = (dev(st[x], "bf16") for x in ("E", "P", "X", "C"))
    t_tok = ids(tok)
    C = sn.sn_compress(basis, X, tok=t_tok, E=E, P=P, seq_len=seq)
    assert_parity(host(C), oracle.round_to(oracle.compress(o["X"], o["U"], tok, o["E"], o["P"],
                                                           seq_len=seq), "bf16"),
                  "bf16", "compress, default positions")
    Xr = sn.sn_decompress(basis, Cin, tok=t_tok, E=E, P=P, seq_len=seq)
    assert_parity(host(Xr), oracle.round_to(oracle.decompress(o["C"], o["U"], tok, o["E"], o["P"],
                                                              seq_len=seq), "bf16"),
                  "bf16", "decompress, default positions")
    m = 1001                            # ragged, scattered explicit positions
    pos = np.random.default_rng(12).integers(0, seq, m).astype(np.int32)
    C = sn.sn_compress(basis, X[:m], tok=ids(tok[:m]), E=E, P=P, pos=ids(pos))
    assert_parity(host(C), oracle.round_to(oracle.compress(o["X"][:m], o["U"], tok[:m], o["E"],
                                                           o["P"], pos=pos), "bf16"),
                  "bf16", "compress, explicit positions")
    Xr = sn.sn_decompress(basis, Cin[:m], tok=ids(tok[:m]), E=E, P=P, pos=ids(pos))
    assert_parity(host(Xr), oracle.round_to(oracle.decompress(o["C"][:m], o["U"], tok[:m],
                                                              o["E"], o["P"], pos=pos), "bf16"),
                  "bf16", "decompress, explicit positions")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_strides_and_guard_canaries(dtype):
    """Row strides larger than the row; nothing is written outside the N x k
    (resp. N x d) region of a padded output buffer."""
    d, k, n = 256, 40, 37
    st, o, tok, _ = _small(d, k, n, dtype=dtype, seed=7)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    basis = sn.sn_basis_pack(dev(st["U"], dtype))
    E, P = dev(st["E"], dtype), dev(st["P"], dtype)
    for ldx_pad in (8, 1):
        Xbig = torch.zeros(n, d + ldx_pad, dtype=tdt, device="cuda")
        Xbig[:, :d] = dev(st["X"], dtype)
        X = Xbig[:, :d]
        Cbig = torch.full((n + 3, k + 5), 7.0, dtype=tdt, device="cuda")
        C = Cbig[:n, :k]
        sn.sn_compress(basis, X, tok=ids(tok), E=E, P=P, seq_len=9, out=C)
        assert_parity(host(C), oracle.round_to(oracle.compress(o["X"], o["U"], tok, o["E"],
                                                               o["P"], seq_len=9), dtype),
                      dtype, f"compress ldx=d+{ldx_pad} ldc=k+5")
        cb = host(Cbig)
        assert np.all(cb[n:] == 7.0) and np.all(cb[:, k:] == 7.0), "compress wrote outside C"
        Obig = torch.full((n + 2, d + 16), 7.0, dtype=tdt, device="cuda")
        Xo = Obig[:n, :d + (0 if ldx_pad == 8 else 0)]
        Cin = dev(st["C"], dtype)
        sn.sn_decompress(basis, Cin, tok=ids(tok), E=E, P=P, seq_len=9, out=Xo)
        assert_parity(host(Xo), oracle.round_to(oracle.decompress(o["C"], o["U"], tok, o["E"],
                                                                  o["P"], seq_len=9), dtype),
                      dtype, "decompress into strided output")
        ob = host(Obig)
        assert np.all(ob[n:] == 7.0) and np.all(ob[:, d:] == 7.0), "decompress wrote outside X"


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_out_of_range_ids_are_clamped_and_flagged(dtype):
    d, k, n, vocab = 256, 20, 40, 50
    st, o, tok, _ = _small(d, k, n, vocab=vocab, dtype=dtype, seed=9)
    bad_tok = tok.copy()
    bad_tok[3], bad_tok[20] = vocab + 5, -2
    pos = (np.arange(n) % 9).astype(np.int32)
    bad_pos = pos.copy()
    bad_pos[7] = 100
    basis = sn.sn_basis_pack(dev(st["U"], dtype))
    E, P, X, Cin = (dev(st[x], dtype) for x in ("E", "P", "X", "C"))
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    C = sn.sn_compress(basis, X, tok=ids(bad_tok), E=E, P=P, pos=ids(bad_pos), err_flag=flag)
    torch.cuda.synchronize()
    assert int(flag.item()) == 3
    ct, cp = np.clip(bad_tok, 0, vocab - 1), np.clip(bad_pos, 0, 8)
    assert_parity(host(C), oracle.round_to(oracle.compress(o["X"], o["U"], ct, o["E"], o["P"],
                                                           pos=cp), dtype), dtype,
                  "compress with clamped ids")
    flag.zero_()
    Xr = sn.sn_decompress(basis, Cin, tok=ids(bad_tok), E=E, err_flag=flag)
    torch.cuda.synchronize()
    assert int(flag.item()) == 1
    assert_parity(host(Xr), oracle.round_to(oracle.decompress(o["C"], o["U"], ct, o["E"]),
                                            dtype), dtype, "decompress with clamped ids")


@pytest.mark.parametrize("pattern", ["one id", "all distinct", "two ids", "zipf"])
@pytest.mark.parametrize("n,seq,d", [(512, 64, 512), (500, 50, 512), (1024, 32, 512),
                                     (32768, 4096, 256), (32768, 64, 256), (32769, 32769, 256)])
def test_compress_token_id_patterns(pattern, n, seq, d):
    """The compress copies each distinct T_fixed row of a workgroup once and
    maps every token to its row: ids that all repeat, never repeat, alternate,
    or follow Zipf, in position-major (n = batch x seq, batch 8, 32 or 512)
    and token-major (500 and 32769 tokens) order; at 32768 tokens the
    workgroups hold 128 tokens (two per lane of the id scan), below that 64."""
    k = 40
    vocab = n + 5 if pattern == "all distinct" else 700
    log(f"[id patterns] {pattern} n={n} seq={seq}")
    rng = np.random.default_rng(n + len(pattern))
    U, _ = np.linalg.qr(rng.standard_normal((d, k)))
    E = rng.standard_normal((vocab, d)) * 0.05
    P = rng.standard_normal((seq, d)) * 0.05
    tok = {"one id": np.full(n, 17),
           "all distinct": rng.permutation(vocab)[:n],
           "two ids": np.where(np.arange(n) % 2 == 0, 3, vocab - 1),
           "zipf": np.minimum(rng.zipf(1.1, n), vocab) - 1}[pattern].astype(np.int32)
    pos = (np.arange(n) % seq).astype(np.int32)
    X = E[tok] + P[pos] + rng.standard_normal((n, d)) * 0.05
    st = {nm: synth.store(a, "bf16") for nm, a in dict(U=U, E=E, P=P, X=X).items()}
    f64 = {nm: oracle.decode_bf16(a) for nm, a in st.items()}
    basis = sn.sn_basis_pack(dev(st["U"], "bf16"))
    C = sn.sn_compress(basis, dev(st["X"], "bf16"), tok=ids(tok), E=dev(st["E"], "bf16"),
                       P=dev(st["P"], "bf16"), seq_len=seq)
    ref = oracle.round_to(oracle.compress(f64["X"], f64["U"], tok, f64["E"], f64["P"],
                                          seq_len=seq), "bf16")
    assert_parity(host(C), ref, "bf16", f"compress, {pattern}")


@pytest.mark.parametrize("tables", ["E only", "P only"])
def test_compress_one_table_128_token_workgroups(tables):
    """One gathered table at 32768 tokens (the 128-token workgroups): T_fixed
    alone (distinct-row copies, no positional rows) or P alone
    (position-major positional rows, no T_fixed)."""
    d, k, n, seq, vocab = 256, 40, 32768, 4096, 2000
    log(f"[one table] {tables} n={n}")
    rng = np.random.default_rng(77 if tables == "E only" else 78)
    U, _ = np.linalg.qr(rng.standard_normal((d, k)))
    E = rng.standard_normal((vocab, d)) * 0.05
    P = rng.standard_normal((seq, d)) * 0.05
    tok = (np.minimum(rng.zipf(1.1, n), vocab) - 1).astype(np.int32)
    pos = (np.arange(n) % seq).astype(np.int32)
    use_e, use_p = tables == "E only", tables == "P only"
    X = (E[tok] if use_e else 0) + (P[pos] if use_p else 0) + rng.standard_normal((n, d)) * 0.05
    st = {nm: synth.store(a, "bf16") for nm, a in dict(U=U, E=E, P=P, X=X).items()}
    f64 = {nm: oracle.decode_bf16(a) for nm, a in st.items()}
    basis = sn.sn_basis_pack(dev(st["U"], "bf16"))
    kw = dict(tok=ids(tok), E=dev(st["E"], "bf16")) if use_e else dict(P=dev(st["P"], "bf16"),
                                                                      seq_len=seq)
    C = sn.sn_compress(basis, dev(st["X"], "bf16"), **kw)
    ref = oracle.round_to(oracle.compress(f64["X"], f64["U"], tok if use_e else None,
                                          f64["E"] if use_e else None,
                                          f64["P"] if use_p else None,
                                          seq_len=seq if use_p else None), "bf16")
    assert_parity(host(C), ref, "bf16", f"compress, {tables}")


def test_bit_exact_gather_and_subtract():
    """C = 0 decompresses to exactly E[tok] + P[pos] (bit-exact gathers);
    X = E[tok] + P[pos] (values on a grid where every sum is exact)
    compresses to 0 within the fp32 accumulation bound of the fused
    subtract-and-project."""
    d, k, n = 256, 40, 70
    rng = np.random.default_rng(12)
    U, _ = np.linalg.qr(rng.standard_normal((d, k)))
    E = rng.integers(-64, 64, (30, d)) / 64.0
    P = rng.integers(-64, 64, (9, d)) / 64.0
    tok = rng.integers(0, 30, n).astype(np.int32)
    pos = (np.arange(n) % 9).astype(np.int32)
    for dtype in ("bf16", "f32"):
        st = {nm: synth.store(a, dtype) for nm, a in dict(U=U, E=E, P=P).items()}
        basis = sn.sn_basis_pack(dev(st["U"], dtype))
        Et, Pt = dev(st["E"], dtype), dev(st["P"], dtype)
        tdt = torch.float32 if dtype == "f32" else torch.bfloat16
        Z = torch.zeros(n, k, dtype=tdt, device="cuda")
        Xr = sn.sn_decompress(basis, Z, tok=ids(tok), E=Et)
        assert np.array_equal(host_bits(Xr), host_bits(Et[ids(tok).long()])), "E gather"
        Xr = sn.sn_decompress(basis, Z, P=Pt, seq_len=9)
        assert np.array_equal(host_bits(Xr), host_bits(Pt[ids(pos).long()])), "P gather"
        Xr = sn.sn_decompress(basis, Z, tok=ids(tok), E=Et, P=Pt, seq_len=9)
        assert np.array_equal(host(Xr), E[tok] + P[pos]), "E + P gather"
        # compress of X = E[tok] + P[pos]: the embedding rows cancel X exactly.
        # In exact arithmetic C = 0.  The matrix-core path sums the products of
        # X, -P and -T_fixed with U in one set of fp32 accumulators, so C is
        # zero up to that accumulation's rounding, bounded by
        # d * 2^-24 * sum |terms|; subtracting a wrong row would leave entries
        # of size ~|x| |u| ~ 1e-1.
        X = dev(synth.store(E[tok] + P[pos], dtype), dtype)
        C = host(sn.sn_compress(basis, X, tok=ids(tok), E=Et, P=Pt, seq_len=9))
        Ud = oracle.decode_bf16(st["U"]) if dtype == "bf16" else st["U"].astype(np.float64)
        absum = (np.abs(E[tok] + P[pos]) + np.abs(E[tok]) + np.abs(P[pos])) @ np.abs(Ud)
        assert np.all(np.abs(C) <= d * 2.0 ** -24 * absum), "subtract of the gathered rows"
        log(f"  bit-exact gather, cancelling subtract ok ({dtype}); max |C| {np.abs(C).max():.3g}")


def test_decompress_cancelling_tables():
    """P[pos] = -T_fixed[tok] for every token: the tables cancel exactly and
    X' is C U^T alone, although each table entry is ~64 times the result.
    The sum of three addends must keep the small one (Sec. 4.3.1 recovery)."""
    d, k, seq, batch = 512, 40, 64, 4
    n = seq * batch
    rng = np.random.default_rng(31)
    U, _ = np.linalg.qr(rng.standard_normal((d, k)))
    E = rng.integers(-4096, 4096, (seq, d)) / 64.0
    P = -E
    tok = (np.arange(n) % seq).astype(np.int32)
    Cin = rng.standard_normal((n, k))
    for dtype in ("bf16", "f32"):
        st = {nm: synth.store(a, dtype) for nm, a in dict(U=U, E=E, P=P, C=Cin).items()}
        basis = sn.sn_basis_pack(dev(st["U"], dtype))
        Xr = host(sn.sn_decompress(basis, dev(st["C"], dtype), tok=ids(tok),
                                   E=dev(st["E"], dtype), P=dev(st["P"], dtype), seq_len=seq))
        val = (lambda a: oracle.decode_bf16(a)) if dtype == "bf16" else (
            lambda a: a.astype(np.float64))
        ref = oracle.decompress(val(st["C"]), val(st["U"]), tok=tok, E=val(st["E"]),
                                P=val(st["P"]), seq_len=seq)
        assert_parity(Xr, ref, dtype, f"decompress, cancelling tables ({dtype})")


def test_output_rounding_ties_to_even():
    """Outputs are rounded once, to nearest even: 1 + 2^-8 -> 1, 1 + 3*2^-8 -> 1 + 2^-6."""
    d, k = 64, 8
    U = np.eye(d)[:, :k]
    E = np.ones((2, d))
    E[1] += 2.0 ** -7
    P = np.full((1, d), 2.0 ** -8)
    tok = np.array([0, 1], dtype=np.int32)
    st = {nm: synth.store(a, "bf16") for nm, a in dict(U=U, E=E, P=P).items()}
    basis = sn.sn_basis_pack(dev(st["U"], "bf16"))
    Z = torch.zeros(2, k, dtype=torch.bfloat16, device="cuda")
    Xr = host(sn.sn_decompress(basis, Z, tok=ids(tok), E=dev(st["E"], "bf16"),
                               P=dev(st["P"], "bf16"), seq_len=1))
    ref = oracle.round_bf16(E[tok] + P[[0, 0]])
    assert np.array_equal(Xr, ref)
    assert np.all(Xr[0] == 1.0) and np.all(Xr[1] == 1.0 + 2.0 ** -6)


def test_empty_batch_is_a_no_op():
    st, o, tok, _ = _small(64, 8, 5, dtype="bf16")
    basis = sn.sn_basis_pack(dev(st["U"], "bf16"))
    X = torch.zeros(0, 64, dtype=torch.bfloat16, device="cuda")
    C = sn.sn_compress(basis, X, tok=ids(np.zeros(0, np.int32)), E=dev(st["E"], "bf16"))
    assert C.shape == (0, 8)
    Xr = sn.sn_decompress(basis, torch.zeros(0, 8, dtype=torch.bfloat16, device="cuda"))
    assert Xr.shape == (0, 64)


def test_deterministic_bitwise():
    w = workload(1)
    dt = "bf16"
    basis = sn.sn_basis_pack(dev(w["U"], dt))
    X, E, P, Cin = dev(w["X"], dt), dev(w["E"], dt), dev(w["P"], dt), dev(synth.store(w["C_true"], dt), dt)
    tok = ids(w["tok"])
    c1 = host_bits(sn.sn_compress(basis, X, tok=tok, E=E, P=P, seq_len=w["cfg"].seq))
    c2 = host_bits(sn.sn_compress(basis, X, tok=tok, E=E, P=P, seq_len=w["cfg"].seq))
    assert np.array_equal(c1, c2)
    x1 = host_bits(sn.sn_decompress(basis, Cin, tok=tok, E=E, P=P, seq_len=w["cfg"].seq))
    x2 = host_bits(sn.sn_decompress(basis, Cin, tok=tok, E=E, P=P, seq_len=w["cfg"].seq))
    assert np.array_equal(x1, x2)


@pytest.mark.parametrize("dtype,d,k,widths,pad", [
    ("bf16", 4096, 40, (4096, 14336), 0),      # config 2's Wo and W2 side by side
    # wide calls (one launch per pass over 16384 or more columns), k from 8 to 64
    ("bf16", 256, 8, (16384,), 0),
    ("bf16", 512, 20, (8192, 8192, 2048), 8),  # three segments, strided rows
    ("bf16", 384, 64, (16384, 256), 0),
    ("bf16", 512, 40, (256, 768, 512), 8),     # strided rows
    ("bf16", 512, 40, (300, 512), 0),          # a width not a multiple of 256: one by one
    ("bf16", 512, 100, (256, 512), 0),         # k > 64: one by one
    ("f32", 256, 8, (256, 100), 0)])
def test_project_weights_multi(dtype, d, k, widths, pad):
    log(f"[project multi] {dtype} d={d} k={k} widths={widths} pad={pad}")
    cfg = synth.Config("multi", dtype, d, k, 10, 1, 1, False, 0.0, 1.0)
    b = synth.make_basis(0, cfg)
    U = (oracle.decode_bf16(b["U"], np.float32) if dtype == "bf16" else b["U"]).astype(np.float64)
    basis = sn.sn_basis_pack(dev(b["U"], dtype))
    hosts, Ws = [], []
    for i, m in enumerate(widths):
        Wh = synth.make_weight(0, i, d, m, cfg)
        hosts.append(Wh)
        full = torch.zeros(d, m + pad, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32,
                           device="cuda")
        full[:, :m] = dev(Wh, dtype)
        Ws.append(full[:, :m] if pad else full)
    sn.sn_project_weights_multi(basis, Ws)
    torch.cuda.synchronize()
    for i, (m, Wh) in enumerate(zip(widths, hosts)):
        Wf = oracle.decode_bf16(Wh, np.float32) if dtype == "bf16" else Wh
        got = host_f32(Ws[i])
        assert_parity_rows(got.T, lambda r: oracle.project_weights(Wf, U, cols=r).T, dtype,
                           f"W[{i}] ({d}x{m}) every column")
        if pad:  # the padding columns are untouched
            assert float(Ws[i].as_strided((d, pad), (m + pad, 1), m).abs().max()) == 0.0


def test_id_check_mode_raises_index_error():
    """With id checking on, a call with an out-of-range id raises
    SnError(SN_ERR_INDEX) after the call, the caller's flag still receives
    the bits, and in-range ids raise nothing."""
    d, k, n, vocab = 256, 20, 40, 50
    st, o, tok, _ = _small(d, k, n, vocab=vocab, seed=9)
    basis = sn.sn_basis_pack(dev(st["U"], "bf16"))
    E, P, X, Cin = (dev(st[x], "bf16") for x in ("E", "P", "X", "C"))
    bad_tok = tok.copy()
    bad_tok[5] = vocab + 1
    sn.set_check_ids(True)
    try:
        sn.sn_compress(basis, X, tok=ids(tok), E=E, P=P, seq_len=9)       # in range: no error
        sn.sn_decompress(basis, Cin, tok=ids(tok), E=E, P=P, seq_len=9)
        flag = torch.zeros(1, dtype=torch.int32, device="cuda")
        with pytest.raises(sn.SnError) as ei:
            sn.sn_compress(basis, X, tok=ids(bad_tok), E=E, P=P, seq_len=9, err_flag=flag)
        assert ei.value.status == sn.SN_ERR_INDEX
        assert int(flag.item()) == 1
        bad_pos = (np.arange(n) % 9).astype(np.int32)
        bad_pos[3] = 99
        with pytest.raises(sn.SnError) as ei:
            sn.sn_decompress(basis, Cin, P=P, pos=ids(bad_pos))
        assert ei.value.status == sn.SN_ERR_INDEX and "flag bits 2" in str(ei.value)
    finally:
        sn.set_check_ids(False)
    # checking off: the same call returns normally and only the flag reports
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    sn.sn_compress(basis, X, tok=ids(bad_tok), E=E, P=P, seq_len=9, err_flag=flag)
    torch.cuda.synchronize()
    assert int(flag.item()) == 1


def test_native_calls_and_python_form_agree(monkeypatch):
    """Each call through the native marshalling and through the Python form of
    the same function: bit-equal results, and what the native form leaves to
    Python (a wrong dtype, shape, stride, an odd object) raises there.  The
    native form takes every one of these calls itself, and leaves the operands of
    those it does not take as they were."""
    d, k, n = 256, 24, 70
    st, o, tok, pos = _small(d, k, n, dtype="bf16", seed=3)
    basis = sn.sn_basis_pack(dev(st["U"], "bf16"))
    X, C, E, P, G = (dev(st[x], "bf16") for x in ("X", "C", "E", "P", "G"))
    t, p = ids(tok), ids(pos)
    proj = sn.sn_embed_project(basis, E=E, P=P)
    CS = dev(synth.store(o["E"] @ o["U"], "bf16"), "bf16")
    side = torch.cuda.Stream()
    W0 = torch.randn(d, 264, device="cuda").bfloat16()
    M0, V0 = torch.rand(d, 264, device="cuda"), torch.rand(d, 264, device="cuda")

    def every():
        W, W1, W2 = W0.clone(), W0.clone(), W0[:, :256].clone()
        M, V, A = M0.clone(), V0.clone(), W0.clone()
        state = sn.sn_grassmann_state(basis)
        gcs = torch.zeros(E.shape[0], k, device="cuda")
        pad = torch.zeros(n, k + 3, device="cuda", dtype=torch.bfloat16)
        side.wait_stream(torch.cuda.current_stream())
        got = [sn.sn_compress(basis, X, tok=t, E=E, P=P, seq_len=9),
               sn.sn_compress(basis, X, tok=t, E=E, P=P, pos=p, out=pad[:, :k]), pad,
               sn.sn_compress(basis, X, P=P, pos=p), sn.sn_decompress(basis, C, tok=t, E=E),
               sn.sn_decompress(basis, C, tok=t, E=E, P=P, seq_len=9, stream=side),
               sn.sn_decompress(basis, C), sn.sn_grad_compress(basis, G),
               sn.sn_compress_projected(basis, X, proj, tok=t, seq_len=9),
               sn.sn_project_weights(basis, W), *sn.sn_project_weights_multi(basis, [W1, W2]),
               sn.sn_grassmann_accumulate(basis, G, state, want_cg=True), state.buf.clone(),
               sn.sn_embed_lowrank_forward(basis, CS, t, E=E, P=P, pos=p),
               sn.sn_embed_lowrank_backward(basis, G, t, gcs),
               sn.sn_adamw_step(A, W0, M, V, 3, 1e-3, weight_decay=0.1), M, V]
        torch.cuda.synchronize()
        return [g.clone() for g in got]

    calls, taken = sn._native(), {}

    class Recorder:
        def __getattr__(self, name):
            def call(*args):
                out = getattr(calls, name)(*args)
                taken.setdefault(name, []).append(out is not None)
                return out
            return call

    monkeypatch.setattr(sn, "_native", Recorder)
    native = every()
    assert set(taken) == {"compress", "decompress", "grad_compress", "compress_projected",
                          "project_weights", "project_weights_multi", "grassmann_accumulate",
                          "embed_lowrank_forward", "embed_lowrank_backward", "adamw_step"}
    assert all(all(t) for t in taken.values()), taken  # no ordinary call was left to Python
    monkeypatch.setattr(sn, "_native", lambda: None)
    python = every()
    for i, (a, b) in enumerate(zip(native, python)):
        assert a.dtype == b.dtype and a.shape == b.shape
        assert torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8)), i
    monkeypatch.undo()

    # what the native form leaves to Python it leaves untouched
    W, A, M, V = W0.clone(), W0.clone(), M0.clone(), V0.clone()
    gcs, state = torch.zeros(E.shape[0], k, device="cuda"), sn.sn_grassmann_state(basis)
    out, wide = torch.zeros(n, k, device="cuda", dtype=torch.bfloat16), torch.zeros_like(X)
    small = torch.empty(1, dtype=torch.uint8, device="cuda")
    held = [W, A, M, V, gcs, state.buf, out, wide]
    before = [h.clone() for h in held]
    for left in (calls.compress(basis, X.float(), t, E, P, None, 9, out, None, None),
                 calls.decompress(basis, C, t[:-1], E, P, None, 9, wide, None, None),
                 calls.compress_projected(basis, X, proj, t.long(), None, 9, out, None, None),
                 calls.project_weights(basis, W, small, None),
                 calls.project_weights_multi(basis, [W, W.float()], None, None),
                 calls.grassmann_accumulate(basis, G, state, True, True, out, small, None),
                 calls.embed_lowrank_forward(basis, CS, t, E[:-1], P, None, 9, wide, None, None, None),
                 calls.embed_lowrank_backward(basis, G, t, gcs, None, small, None),
                 calls.adamw_step(A, W0, M, V[:, :8], 3, 1e-3, 0.9, 0.999, 1e-8, 0.1, True, None,
                                  None)):
        assert left is None
    for i, (h, b) in enumerate(zip(held, before)):
        assert torch.equal(h.view(torch.uint8), b.view(torch.uint8)), i
    assert calls.grad_compress(basis, G[:1].expand(n, d), None, None) is None  # overlapping rows
    assert calls.grad_compress(basis, G.float(), None, None) is None
    assert calls.grad_compress(basis, G.t(), None, None) is None
    assert calls.grad_compress(basis, [1], None, None) is None
    assert calls.grad_compress(object(), G, None, None) is None
    for bad, status in ((lambda: sn.sn_grad_compress(basis, G.float()), 3),
                        (lambda: sn.sn_grad_compress(basis, G[:, :-1]), 2),
                        (lambda: sn.sn_grad_compress(basis, G[:1].expand(n, d)), 2),
                        (lambda: sn.sn_compress(basis, X, tok=t[:-1], E=E), 2),
                        (lambda: sn.sn_compress(basis, X, P=P, seq_len=0), 2),
                        (lambda: sn.sn_grad_compress(basis, G, out=G[:, :k]), 5)):
        with pytest.raises(sn.SnError) as e:
            bad()
        assert e.value.status == status

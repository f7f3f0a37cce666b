"""GPU parity of the attention backward pass (selection held constant): the HIP library through its C ABI against
the fp64 oracle on the same seeded bf16 inputs.

The GPU takes O and the log-sum-exp from its own forward (as a training step does), rebuilds the probabilities in
fp32, rounds P and dS to bf16 for the MFMA products, sums in fp32 and rounds the gradients to bf16.  A gradient
element is therefore a sum of terms each off by up to 2^-9 of itself, independently (standard deviation
2^-9/sqrt(3) of the root-sum-square T of its terms, which the oracle reports), plus the output rounding:
    |g_gpu - g_oracle| <= 2^-8 |g_oracle| + 2^-7 T + 1e-4          (2^-7 T is about seven standard deviations),
and the mean error must stay below a fifth of the mean bound.  Terms may cancel (rows that attend few keys with
large scores), so T, not |g|, is the unit.  delta = dO.O is a function of the O the caller hands over: the oracle is
given the same bf16 O (the oracle's own pins use the exact one).
"""
import ctypes

import numpy as np
import pytest
import torch

from paper_2604_08077_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_08077_amd import binding

    binding.load()  # raises if the HIP library was not built: there is no fallback
    return binding


def oshape(o, w):
    return o.Shape(w.T, w.H, w.W, w.ct, w.ch, w.cw, w.Hq, w.Hkv, w.D, w.text, w.lead)


def f64(t):
    return t.to(torch.float64).numpy()


def check_grad(name, got, want, terms):
    got, want, terms = (x.reshape(-1, x.shape[-1]) for x in (got, want, terms))
    err = np.abs(got - want)
    bound = 2.0 ** -8 * np.abs(want) + 2.0 ** -7 * terms + 1e-4
    print(f"[{name}] elements={err.size} max-abs={err.max():.3e} mean-abs={err.mean():.3e} "
          f"worst err/bound={np.max(err / bound):.3f} mean err/mean bound={err.mean() / bound.mean():.3f}", flush=True)
    assert np.isfinite(got).all()
    assert (err <= bound).all()
    assert err.mean() <= 0.2 * bound.mean()


def check_sums(name, dK, dV, dO, w):
    """Every row's probabilities sum to one and its dS to zero: sum over tokens of dV = sum over the group's rows of dO, of dK = 0.
    Every element of dV, dK carries its own bf16 rounding (relative 2^-9) and the noise of its rounded terms, which
    cancel in part (measured: about 7 x 2^-9 of the column's root-sum-square); over many tokens these add up like
    a random walk."""
    dVs, dKs = (x.to(torch.float64).sum(dim=0).cpu().numpy() for x in (dV, dK))  # [Hkv, D]
    dOs = dO.cuda().view(w.S, w.Hkv, w.Hq // w.Hkv, w.D).to(torch.float64).sum(dim=(0, 2)).cpu().numpy()
    tol_v = 16.0 * 2.0 ** -9 * torch.sqrt((dV.to(torch.float64) ** 2).sum(dim=0)).cpu().numpy() + 1e-3 * np.abs(dOs)
    tol_k = 16.0 * 2.0 ** -9 * torch.sqrt((dK.to(torch.float64) ** 2).sum(dim=0)).cpu().numpy()
    print(f"[{name}] sum dV - sum dO: max {np.abs(dVs - dOs).max():.3e} (tolerance {tol_v.min():.3e}..{tol_v.max():.3e}); "
          f"sum dK: max {np.abs(dKs).max():.3e} (tolerance {tol_k.min():.3e}..{tol_k.max():.3e})", flush=True)
    assert np.isfinite(dVs).all() and np.isfinite(dKs).all()
    assert (np.abs(dVs - dOs) <= tol_v).all()
    assert (np.abs(dKs) <= tol_k).all()


def workload(name):
    return synth.TEST_WORKLOADS.get(name) or synth.SAMPLED_WORKLOADS.get(name) or synth.WORKLOADS[name]


def run_case(B, oracle, name, p, dense=False, over={}):
    w = workload(name)
    sh, osh = B.Shape.of(w), oshape(oracle, w)
    Q, K, V = synth.generate(w)
    g = torch.Generator(device="cpu")
    g.manual_seed(synth.BASE_SEED + 31 * w.config_id)
    dO = torch.randn((w.S, w.Hq, w.D), generator=g, dtype=torch.float32).to(torch.bfloat16)
    kbar = oracle.cube_pool(osh, K)
    mask = oracle.cube_select(osh, Q, kbar, 1.0 if dense else p)[0]
    Qg, Kg, Vg, dOg = Q.cuda(), K.cuda(), V.cuda(), dO.cuda()
    mg = torch.from_numpy(mask.view(np.int32)).cuda()
    print(f"[{name}] forward p={p} dense={dense}", flush=True)
    if dense:
        O, lse = B.dense_attn(sh, Qg, Kg, Vg, return_lse=True)
    else:
        O, lse = B.sparse_attn(sh, Qg, Kg, Vg, mg, return_lse=True)
    torch.cuda.synchronize()
    Oc = f64(O.cpu()).reshape(-1, w.D)
    inputs = {"Q": Qg, "K": Kg, "V": Vg, "O": O, "dO": dOg}
    print(f"[{name}] backward {over}", flush=True)
    dQ, dK, dV = B.sparse_attn_bwd(sh, Qg, Kg, Vg, O, lse, dOg, sel_mask=None if dense else mg,
                                   **{out: inputs[i] for out, i in over.items()})
    torch.cuda.synchronize()
    T = {}
    rq, rk, rv, _ = oracle.bwd.sparse_attn_bwd(osh, f64(Q), f64(K), f64(V), mask, f64(dO).reshape(-1, w.D),
                                               O=Oc, scales=T)
    check_grad(f"{name} dV", f64(dV.cpu()), rv, T["dV"])
    check_grad(f"{name} dQ", f64(dQ.cpu()), rq, T["dQ"])
    check_grad(f"{name} dK", f64(dK.cpu()), rk, T["dK"])


@pytest.mark.parametrize("name,p", [("T_tiny", 0.8), ("T_mha64", 0.7), ("T_ragged", 0.9), ("T_text64", 0.8),
                                    ("T_lead64", 0.8), ("T_manycubes", 0.6), ("T_lead128", 0.9), ("C1", 0.9),
                                    ("M_bwd256", 0.8), ("T_cube2048", 0.9)])
def test_backward_matches_oracle(B, oracle, name, p):
    run_case(B, oracle, name, p)


# What the dK/dV kernel cuts by: one cube (no part to sum), cubes of 65 rows per KV head (a second 64-row word with one row),
# of 63 and 64 tokens, more than 64 words per cube (two lists) with four 256-key blocks, two cubes per part (with a text tail
# of one token, which fills the last range, and with a last range of a single cube), fourteen per part and a last range of four.
GATHER = [
    ("one_cube", (2, 4, 4), (2, 4, 4), 2, 1, 64, 1.0, 0),
    ("rows65", (3, 1, 26), (1, 1, 13), 5, 1, 128, 0.7, 0),
    ("tokens63", (4, 7, 9), (1, 7, 9), 3, 1, 128, 0.6, 0),
    ("tokens64", (5, 8, 8), (1, 8, 8), 2, 2, 64, 0.6, 1),
    ("two_lists", (8, 16, 16), (4, 16, 16), 7, 1, 64, 1.0, 0),
    ("parts", (65, 4, 4), (1, 4, 4), 1, 1, 128, 0.5, 1),
    ("parts_last_single", (65, 4, 4), (1, 4, 4), 1, 1, 128, 0.5, 0),
    ("parts_of_14", (60, 1, 4), (1, 1, 4), 8, 8, 64, 0.5, 0),
]


@pytest.mark.parametrize("name,grid,cube,hq,hkv,d,p,text", GATHER, ids=[c[0] for c in GATHER])
def test_backward_gathered_rows(B, oracle, monkeypatch, name, grid, cube, hq, hkv, d, p, text):
    w = synth.Workload(name, 40, *grid, *cube, hq, hkv, d, (p,), (1.0,) * hkv, text)
    monkeypatch.setitem(synth.TEST_WORKLOADS, name, w)
    run_case(B, oracle, name, p)
    run_case(B, oracle, name, 1.0, dense=True)


# Two wavefronts per 32 keys in the dK/dV kernel: cubes of up to 128 tokens and 6,000 rows of a KV head or more; cubes of 33, 97
# and 128 keys (one key, one of three and four wavefronts' worth of keys), and one row too few for it
SHARED = [
    ("keys33", (26, 3, 11), (1, 3, 11), 7, 64), ("keys97", (9, 1, 97), (1, 1, 97), 7, 128), ("keys128", (7, 8, 16), (1, 8, 16), 7, 128),
    ("rows5999", (1, 1, 857), (1, 1, 50), 7, 128),
]


@pytest.mark.parametrize("name,grid,cube,hq,d", SHARED, ids=[c[0] for c in SHARED])
def test_backward_shared_keys(B, oracle, monkeypatch, name, grid, cube, hq, d):
    monkeypatch.setitem(synth.TEST_WORKLOADS, name, synth.Workload(name, 43, *grid, *cube, hq, 1, d, (0.6,), (1.0,)))
    run_case(B, oracle, name, 0.6)


def dq_kernel(B, w):
    """Which dQ kernel a shape gets: wavefronts that share 32 rows, and whether every tile is worked as its first half."""
    cs = B.Shape.of(w)._c()
    return B.load().adaspark_internal_dq_waves(ctypes.byref(cs)), B.load().adaspark_internal_dq_half_tiles(ctypes.byref(cs))


# The dQ kernel with two wavefronts per 32 rows, on walks short enough for the oracle to take every row: cubes whose keys leave the second half
# of a tile empty, or with one key; row blocks of 128 and a remainder.
DQ = [
    ("keys31_rows124", (4, 1, 31), (1, 1, 31), 4, 1, 128, 0.7, 0),
    ("keys33_rows132", (4, 3, 11), (1, 3, 11), 4, 1, 128, 0.7, 5),
    ("keys97_rows291", (3, 1, 97), (1, 1, 97), 3, 1, 64, 0.7, 0),
]


@pytest.mark.parametrize("name,grid,cube,hq,hkv,d,p,text", DQ, ids=[c[0] for c in DQ])
def test_backward_shared_rows(B, oracle, monkeypatch, name, grid, cube, hq, hkv, d, p, text):
    w = synth.Workload(name, 42, *grid, *cube, hq, hkv, d, (p,), (1.0,) * hkv, text)
    assert dq_kernel(B, w) == (2, 0)
    monkeypatch.setitem(synth.TEST_WORKLOADS, name, w)
    run_case(B, oracle, name, p)
    run_case(B, oracle, name, 1.0, dense=True)


# Longer walks of the dQ kernels that only larger shapes get, against the oracle on a sample of rows.  Two wavefronts per 32 rows: more than 64
# cubes, text on both sides, clipped cubes, cubes of 256 and of 1,024 tokens with a text cube of one, row blocks with a remainder.  One, on
# whole tiles: last tiles of 1, 33 and 63 keys, clipped cubes and whole ones; on half tiles.  Both head dims.
LONG = [
    ("two_cubes82_text", (80, 3, 11), (1, 3, 11), 16, 16, 64, 9, 5, (2, 0)),
    ("two_clipped_text", (9, 10, 12), (4, 4, 8), 28, 4, 128, 33, 20, (2, 0)),
    ("two_cubes256", (6, 16, 16), (4, 8, 8), 28, 4, 128, 0, 0, (2, 0)),
    ("two_clipped256_text", (5, 13, 17), (4, 8, 8), 20, 4, 64, 33, 65, (2, 0)),
    ("two_cubes1024", (8, 16, 16), (4, 16, 16), 28, 7, 64, 1, 0, (2, 0)),
    ("one_last1_33_63", (18, 5, 13), (1, 5, 13), 64, 16, 64, 63, 33, (1, 0)),
    ("one_last33", (15, 1, 97), (1, 1, 97), 56, 8, 128, 0, 0, (1, 0)),
    ("one_clipped_text", (9, 10, 12), (4, 4, 8), 72, 18, 128, 40, 43, (1, 0)),
    ("one_cubes256", (6, 16, 16), (4, 8, 8), 56, 8, 64, 0, 0, (1, 0)),
    ("one_half_tiles", (13, 9, 12), (2, 4, 4), 64, 16, 128, 33, 20, (1, 1)),
]


@pytest.mark.parametrize("name,grid,cube,hq,hkv,d,text,lead,kernel", LONG, ids=[c[0] for c in LONG])
def test_backward_long_walks_sampled(B, oracle, name, grid, cube, hq, hkv, d, text, lead, kernel):
    """dQ of sampled rows, masked and dense; of dK and dV the identities of the full-size tests below (the dK/dV kernel reads what
    the dQ kernel found of the rows' sums)."""
    w = synth.Workload(name, 65, *grid, *cube, hq, hkv, d, (0.7,), (1.0,) * hkv, text, lead)
    assert dq_kernel(B, w) == kernel
    sh, osh = B.Shape.of(w), oshape(oracle, w)
    Q, K, V = synth.generate(w)
    g = torch.Generator(device="cpu")
    g.manual_seed(synth.BASE_SEED + 65)
    dO = torch.randn((w.S, w.Hq, w.D), generator=g, dtype=torch.float32).to(torch.bfloat16)
    Qg, Kg, Vg, dOg = Q.cuda(), K.cuda(), V.cuda(), dO.cuda()
    q, k, v, do = f64(Q), f64(K), f64(V), f64(dO).reshape(-1, w.D)
    tables = oracle.bwd.cube_tables(osh)
    G, c = w.Hq // w.Hkv, 1.0 / np.sqrt(w.D)
    rows = synth.sample_rows(w, 400)
    for dense in (False, True):
        mask = oracle.cube_select(osh, Q, oracle.cube_pool(osh, K), 1.0 if dense else 0.7)[0]
        mg = None if dense else torch.from_numpy(mask.view(np.int32)).cuda()
        print(f"[{name}] dense={dense}: {len(rows)} rows", flush=True)
        O, lse = B.dense_attn(sh, Qg, Kg, Vg, return_lse=True) if dense else B.sparse_attn(sh, Qg, Kg, Vg, mg, return_lse=True)
        dQ, dK, dV = B.sparse_attn_bwd(sh, Qg, Kg, Vg, O, lse, dOg, sel_mask=mg)
        torch.cuda.synchronize()
        o = f64(O.cpu()).reshape(-1, w.D)
        want, terms = [], []
        for r in rows:
            att, dq, _, _, _, ds, _ = oracle.bwd.row_backward(osh, q, k, v, mask[r], r, do[r], o[r], tables)
            want.append(dq)
            terms.append(c * np.sqrt((ds * ds) @ (k[att, (r % w.Hq) // G] ** 2)))
        check_grad(f"{name} dQ", f64(dQ.cpu()).reshape(-1, w.D)[rows], np.array(want), np.array(terms))
        check_sums(name, dK, dV, dO, w)


# The dQ kernel with eight wavefronts per 32 rows: walks of fewer steps than wavefronts and of many, cubes with one key in their last step,
# blocks of 32 rows across cubes, a block with one row, more than 64 cubes, text on both sides, clipped cubes
EIGHT = [
    ("rows353_keys1", (353, 1, 1), (1, 1, 1), 1, 1, 64, 0, 0),
    ("keys33", (12, 3, 11), (1, 3, 11), 2, 1, 128, 0, 0),
    ("keys65_text", (9, 5, 13), (1, 5, 13), 3, 1, 64, 70, 40),
    ("cubes70", (70, 2, 4), (1, 2, 4), 4, 2, 128, 9, 0),
    ("clipped", (9, 10, 12), (4, 4, 8), 3, 1, 128, 0, 30),
    ("blocks304", (38, 2, 4), (1, 2, 4), 8, 8, 64, 0, 0),
    ("blocks312", (39, 2, 4), (1, 2, 4), 8, 8, 64, 0, 0),
    ("keys33_blocks390", (130, 3, 11), (1, 3, 11), 3, 3, 128, 0, 0),
]


@pytest.mark.parametrize("name,grid,cube,hq,hkv,d,text,lead", EIGHT, ids=[c[0] for c in EIGHT])
def test_backward_eight_wavefronts_per_rows(B, oracle, monkeypatch, name, grid, cube, hq, hkv, d, text, lead):
    w = synth.Workload(name, 61, *grid, *cube, hq, hkv, d, (0.7,), (1.0,) * hkv, text, lead)
    assert dq_kernel(B, w) == (8, 0)
    monkeypatch.setitem(synth.TEST_WORKLOADS, name, w)
    run_case(B, oracle, name, 0.7)
    run_case(B, oracle, name, 1.0, dense=True)


# The dQ kernel with one wavefront per 32 rows on half tiles: 305 workgroups of 256 rows and more, many heads of short sequences; both head dims,
# clipped cubes with text around them, blocks over many cubes of three tokens, a block with a few rows.  And the last shape of the other side.
ONE = [
    ("heads154_text", (5, 5, 9), (2, 4, 4), 154, 154, 64, 33, 20, 1),
    ("heads306_cubes3", (1, 1, 130), (1, 1, 3), 306, 153, 128, 0, 0, 1),
    ("heads305_ragged", (3, 5, 7), (2, 2, 4), 305, 305, 128, 0, 0, 1),
    ("heads304_ragged", (3, 5, 7), (2, 2, 4), 304, 304, 128, 0, 0, 2),
]


@pytest.mark.parametrize("name,grid,cube,hq,hkv,d,text,lead,waves", ONE, ids=[c[0] for c in ONE])
def test_backward_one_wavefront_per_rows(B, oracle, monkeypatch, name, grid, cube, hq, hkv, d, text, lead, waves):
    w = synth.Workload(name, 52, *grid, *cube, hq, hkv, d, (0.7,), (1.0,) * hkv, text, lead)
    assert dq_kernel(B, w) == (waves, int(waves == 1))
    monkeypatch.setitem(synth.TEST_WORKLOADS, name, w)
    run_case(B, oracle, name, 0.7)
    run_case(B, oracle, name, 1.0, dense=True)


# Gradients written over the inputs they belong to: which output lies over which input.  dK and dV over Q or dO need as
# many KV heads as query heads.  "one_cube": keys with no parts to sum.
IN_PLACE = [
    ("T_ragged", {"dQ": "dO"}), ("T_ragged", {"dQ": "Q", "dK": "K", "dV": "V"}), ("M_bwd256", {"dQ": "dO"}),
    ("T_ragged", {"dQ": "O", "dK": "V", "dV": "K"}), ("T_mha64", {"dQ": "dO", "dK": "Q"}), ("T_mha64", {"dK": "Q", "dV": "dO"}),
    ("T_mha64", {"dQ": "Q", "dV": "O"}), ("one_cube", {"dQ": "dO"}), ("one_cube", {"dK": "Q", "dV": "dO"}),
]


@pytest.mark.parametrize("name,over", IN_PLACE, ids=[n + "_" + "_".join(o + "_" + i for o, i in ov.items()) for n, ov in IN_PLACE])
def test_backward_in_place(B, oracle, monkeypatch, name, over):
    w = synth.Workload(name, 44, 2, 8, 8, 2, 8, 8, 2, 2, 64, (0.8,), (1.0,) * 2)
    if name == "one_cube":
        monkeypatch.setitem(synth.TEST_WORKLOADS, name, w)
    run_case(B, oracle, name, 0.8, over=over)


@pytest.mark.parametrize("name", ["T_ragged", "T_text64"])
def test_a_row_that_is_not_finite_stays_in_its_kv_head(B, oracle, name):
    """dO of the last token's last query head is infinite, then not a number: what other KV heads get is bit for bit
    what they get with a finite one, whatever pads their tiles of rows."""
    w = workload(name)
    sh, osh = B.Shape.of(w), oshape(oracle, w)
    Q, K, V = synth.generate(w)
    g = torch.Generator(device="cpu")
    g.manual_seed(synth.BASE_SEED + 31 * w.config_id)
    dO = torch.randn((w.S, w.Hq, w.D), generator=g, dtype=torch.float32).to(torch.bfloat16)
    mask = oracle.cube_select(osh, Q, oracle.cube_pool(osh, K), 0.8)[0]
    Qg, Kg, Vg = Q.cuda(), K.cuda(), V.cuda()
    mg = torch.from_numpy(mask.view(np.int32)).cuda()
    O, lse = B.sparse_attn(sh, Qg, Kg, Vg, mg, return_lse=True)
    for sel in (mg, None):
        want = B.sparse_attn_bwd(sh, Qg, Kg, Vg, O, lse, dO.cuda(), sel_mask=sel)
        for bad in (float("inf"), float("nan")):
            worse = dO.clone()
            worse[-1, -1] = bad
            got = B.sparse_attn_bwd(sh, Qg, Kg, Vg, O, lse, worse.cuda(), sel_mask=sel)
            torch.cuda.synchronize()
            G = w.Hq // w.Hkv
            for nm, a, b, keep in zip(("dQ", "dK", "dV"), got, want, (w.Hq - G, w.Hkv - 1, w.Hkv - 1)):
                a, b = a[:, :keep].cpu(), b[:, :keep].cpu()
                print(f"[{name} dense={sel is None} {bad}] {nm}: not finite {int((~a.isfinite()).sum())}", flush=True)
                assert torch.equal(a, b)


@pytest.mark.parametrize("name,p", [("T_tiny", 0.8), ("T_ragged", 0.9), ("T_lead64", 0.8), ("M_bwd256", 0.8)])
def test_backward_matches_the_exact_gradient(B, oracle, name, p):
    """Against the oracle's own gradient: delta = dO.o from the exact fp64 forward, not from the bf16 O the GPU
    backward is handed.  What the forward's rounding of O does to the gradients enters through delta alone (dS_j =
    p_j (dO.v_j - delta)), so the bound of the other tests grows by the oracle's `dQ_delta` / `dK_delta`: the
    element's sensitivity to delta times the row's delta_error_bound (dV does not depend on delta).  The forward's
    O itself must be within that model too: |dO.O_gpu - dO.o| <= delta_error_bound, row by row."""
    w = workload(name)
    sh, osh = B.Shape.of(w), oshape(oracle, w)
    Q, K, V = synth.generate(w)
    g = torch.Generator(device="cpu")
    g.manual_seed(synth.BASE_SEED + 31 * w.config_id)
    dO = torch.randn((w.S, w.Hq, w.D), generator=g, dtype=torch.float32).to(torch.bfloat16)
    mask = oracle.cube_select(osh, Q, oracle.cube_pool(osh, K), p)[0]
    Qg, Kg, Vg, dOg = Q.cuda(), K.cuda(), V.cuda(), dO.cuda()
    mg = torch.from_numpy(mask.view(np.int32)).cuda()
    print(f"[{name}] forward + backward, exact-delta comparison", flush=True)
    O, lse = B.sparse_attn(sh, Qg, Kg, Vg, mg, return_lse=True)
    dQ, dK, dV = B.sparse_attn_bwd(sh, Qg, Kg, Vg, O, lse, dOg, sel_mask=mg)
    torch.cuda.synchronize()
    T = {}
    q, k, v, do = f64(Q), f64(K), f64(V), f64(dO).reshape(-1, w.D)
    rq, rk, rv, delta = oracle.bwd.sparse_attn_bwd(osh, q, k, v, mask, do, O=None, scales=T)
    # the forward's effect on delta, row by row, against the model the extra tolerance is built from
    tables = oracle.bwd.cube_tables(osh)
    d_gpu = (do * f64(O.cpu()).reshape(-1, w.D)).sum(axis=1)
    worst = 0.0
    for r in synth.sample_rows(w, 200):
        att, _, _, _, _, _, pr = oracle.bwd.row_backward(osh, q, k, v, mask[r], r, do[r], None, tables)
        n, a = divmod(int(r), w.Hq)
        gk = a // (w.Hq // w.Hkv)
        absdot = (np.abs(k[att, gk]) @ np.abs(q[n, a])).max() / np.sqrt(w.D)
        worst = max(worst, abs(d_gpu[r] - delta[r]) / oracle.bwd.delta_error_bound(do[r], pr @ v[att, gk], pr, v[att, gk], absdot))
    print(f"[{name}] |delta_gpu - delta_exact| / bound, worst of the sampled rows: {worst:.3f}", flush=True)
    assert worst <= 1.0
    for nm, got, want in (("dV", dV, rv), ("dQ", dQ, rq), ("dK", dK, rk)):
        got, want_, terms = (x.reshape(-1, w.D) for x in (f64(got.cpu()), want, T[nm]))
        extra = T[nm + "_delta"].reshape(-1, w.D) if nm != "dV" else 0.0
        err = np.abs(got - want_)
        bound = 2.0 ** -8 * np.abs(want_) + 2.0 ** -7 * terms + 1e-4 + extra
        print(f"[{name} {nm} vs exact] max-abs={err.max():.3e} worst err/bound={np.max(err / bound):.3f} "
              f"share of the bound that is the delta term: {np.mean(extra / bound):.2f}", flush=True)
        assert (err <= bound).all()


@pytest.mark.parametrize("name", ["T_ragged", "T_mha64"])
def test_dense_backward_matches_oracle(B, oracle, name):
    run_case(B, oracle, name, 1.0, dense=True)


def test_backward_with_nothing_selected(B, oracle):
    """p = 0: every row attends the causal part of its own cube only (and earlier text cubes, if any)."""
    run_case(B, oracle, "T_ragged", 0.0)
    run_case(B, oracle, "T_lead64", 0.0)


def test_backward_full_size_sampled(B, oracle):
    """65,536 tokens, p = 0.9, the launch configuration the benchmark times.  dQ: sampled rows recomputed by the
    oracle.  dK, dV: the last eight tokens of the last cube of one KV head (few rows attend them: the oracle takes
    them all), and two identities that hold at any size because every row's probabilities sum to one and its dS to
    zero: sum over tokens of dV = sum over the group's rows of dO, sum over tokens of dK = 0."""
    w = synth.WORKLOADS["C3"]
    p = 0.9
    sh, osh = B.Shape.of(w), oshape(oracle, w)
    Q, K, V = synth.generate(w)
    g = torch.Generator(device="cpu")
    g.manual_seed(synth.BASE_SEED + 31 * w.config_id)
    dO = torch.randn((w.S, w.Hq, w.D), generator=g, dtype=torch.float32).to(torch.bfloat16)
    Qg, Kg, Vg, dOg = Q.cuda(), K.cuda(), V.cuda(), dO.cuda()
    kbar = B.cube_pool(sh, Kg)
    mask_g, _, _, _ = B.cube_select(sh, Qg, kbar, p)
    print("[C3] forward", flush=True)
    O, lse = B.sparse_attn(sh, Qg, Kg, Vg, mask_g, return_lse=True)
    torch.cuda.synchronize()
    print("[C3] backward", flush=True)
    dQ, dK, dV = B.sparse_attn_bwd(sh, Qg, Kg, Vg, O, lse, dOg, sel_mask=mask_g)
    torch.cuda.synchronize()
    mask = mask_g.cpu().numpy().view(np.uint32)
    q, k, v, do = f64(Q), f64(K), f64(V), f64(dO).reshape(-1, w.D)
    o = f64(O.cpu()).reshape(-1, w.D)
    tables = oracle.bwd.cube_tables(osh)
    G, c = w.Hq // w.Hkv, 1.0 / np.sqrt(w.D)

    rows = synth.sample_rows(w, 24, seed=5)
    want, terms = [], []
    for r in rows:
        att, dq, _, _, _, ds, _ = oracle.bwd.row_backward(osh, q, k, v, mask[r], r, do[r], o[r], tables)
        want.append(dq)
        terms.append(c * np.sqrt((ds * ds) @ (k[att, (r % w.Hq) // G] ** 2)))
    got = f64(dQ.reshape(-1, w.D)[torch.as_tensor(rows).cuda()].cpu())
    check_grad("C3 dQ sampled rows", got, np.array(want), np.array(terms))

    # keys: the last eight tokens (in cube order) of the last cube, KV head 1; the rows that attend them are the
    # rows of those tokens themselves and of the later ones among them
    members = tables[2][-1]
    toks = members[-8:]
    gk = 1
    wk, wv = np.zeros((8, w.D)), np.zeros((8, w.D))
    tk, tv = np.zeros((8, w.D)), np.zeros((8, w.D))
    for x, n in enumerate(toks):
        for a in range(gk * G, (gk + 1) * G):
            r = n * w.Hq + a
            att, _, dk_t, dv_t, _, _, _ = oracle.bwd.row_backward(osh, q, k, v, mask[r], r, do[r], o[r], tables)
            for y in range(x + 1):                      # this row attends toks[0..x]
                pos = int(np.nonzero(att == toks[y])[0][0])
                wk[y] += dk_t[pos]
                wv[y] += dv_t[pos]
                tk[y] += dk_t[pos] ** 2
                tv[y] += dv_t[pos] ** 2
    idx = torch.as_tensor(toks).cuda()
    check_grad("C3 dK last tokens", f64(dK[idx, gk].cpu()), wk, np.sqrt(tk))
    check_grad("C3 dV last tokens", f64(dV[idx, gk].cpu()), wv, np.sqrt(tv))

    check_sums("C3", dK, dV, dO, w)


def test_backward_quarter_million_tokens(B, oracle):
    """262,144 tokens (1,024 cubes, the largest configuration): offsets and tables at full scale.  A few dQ rows
    against the oracle, and the identities sum(dV) = sum(dO) per KV head, sum(dK) = 0."""
    w = synth.WORKLOADS["C4"]
    p = 0.9
    sh, osh = B.Shape.of(w), oshape(oracle, w)
    Q, K, V = synth.generate(w)
    g = torch.Generator(device="cpu")
    g.manual_seed(synth.BASE_SEED + 31 * w.config_id)
    dO = torch.randn((w.S, w.Hq, w.D), generator=g, dtype=torch.float32).to(torch.bfloat16)
    Qg, Kg, Vg, dOg = Q.cuda(), K.cuda(), V.cuda(), dO.cuda()
    kbar = B.cube_pool(sh, Kg)
    mask_g, _, _, _ = B.cube_select(sh, Qg, kbar, p)
    print("[C4] forward", flush=True)
    O, lse = B.sparse_attn(sh, Qg, Kg, Vg, mask_g, return_lse=True)
    torch.cuda.synchronize()
    print("[C4] backward", flush=True)
    dQ, dK, dV = B.sparse_attn_bwd(sh, Qg, Kg, Vg, O, lse, dOg, sel_mask=mask_g)
    torch.cuda.synchronize()
    G, c = w.Hq // w.Hkv, 1.0 / np.sqrt(w.D)
    q, k, v = f64(Q), f64(K), f64(V)
    tables = oracle.bwd.cube_tables(osh)
    rows = np.array([0, w.Hq * 4097 + 3, w.Hq * (w.S // 2) + 11, w.Hq * (w.S - 300) + 27, w.S * w.Hq - 1])
    idx = torch.as_tensor(rows).cuda()
    mrows = mask_g[idx].cpu().numpy().view(np.uint32)
    do_rows, o_rows = f64(dO.reshape(-1, w.D)[rows]), f64(O.reshape(-1, w.D)[idx].cpu())
    want, terms = [], []
    for x, r in enumerate(rows):
        att, dq, _, _, _, ds, _ = oracle.bwd.row_backward(osh, q, k, v, mrows[x], r, do_rows[x], o_rows[x], tables)
        want.append(dq)
        terms.append(c * np.sqrt((ds * ds) @ (k[att, (r % w.Hq) // G] ** 2)))
    check_grad("C4 dQ sampled rows", f64(dQ.reshape(-1, w.D)[idx].cpu()), np.array(want), np.array(terms))
    check_sums("C4", dK, dV, dO, w)

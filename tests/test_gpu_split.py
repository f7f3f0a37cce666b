"""The attention kernel for short sequences at the sizes where its cutting can go wrong, against the fp64 oracle: row
blocks of 31 / 32 / 33 rows, cubes of 31 / 32 / 33 keys and of one, a walk shorter than the eight wavefronts that share it,
nothing selected, both causal modes, dense.  The entries choose it by shape; every test asserts which kernel its shape
gets.  And the dense walk kernel at head-dim 64, which short shapes no longer reach, on shapes of its side of the line."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2604_08077_amd import synth
from test_gpu_parity import B, MAX_ABS, MEAN_ABS, check_outputs, lse_bound, oshape, rows_of, stratified_rows  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [
    ("keys31", (3, 1, 31), (1, 1, 31), 1, 1, 64, 0),
    ("keys32", (4, 4, 8), (1, 4, 8), 2, 1, 128, 0),
    ("keys33", (5, 3, 11), (1, 3, 11), 1, 1, 128, 0),
    ("rows33", (2, 1, 22), (1, 1, 11), 3, 1, 64, 0),
    ("one_token_cubes", (2, 3, 7), (1, 1, 1), 4, 2, 64, 0),
    ("one_cube", (2, 4, 9), (2, 4, 9), 7, 1, 128, 0),
    ("text_tail", (3, 4, 8), (1, 4, 8), 6, 2, 128, 33),
]


def short(B, sh, causal):  # noqa: F811
    """1: the kernel for short sequences, 0: the walk."""
    cs = sh._c()
    return B.load().adaspark_internal_short_sequence(ctypes.byref(cs), int(causal))


@pytest.mark.parametrize("name,grid,cube,hq,hkv,d,text", SHAPES, ids=[s[0] for s in SHAPES])
def test_short_sequences(B, oracle, name, grid, cube, hq, hkv, d, text):  # noqa: F811
    w = synth.Workload(name, 41, *grid, *cube, hq, hkv, d, (0.6,), (1.0,) * hkv, text)
    sh, osh = B.Shape.of(w), oshape(oracle, w)
    Q, K, V = synth.generate(w)
    Qg, Kg, Vg = Q.cuda(), K.cuda(), V.cuda()
    kbar = oracle.cube_pool(osh, K)
    rows = np.arange(w.S * w.Hq)

    def check(what, got, want):
        err = np.abs(got.reshape(-1, d).float().cpu().numpy().astype(np.float64) - want)
        print(f"[{name} {what}] max-abs={err.max():.3e} mean-abs={err.mean():.3e}", flush=True)
        assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS

    for causal in (True, False):
        assert short(B, sh, causal) == 1
        for p in (0.0, 0.6):
            mask = oracle.cube_select(osh, Q, kbar, p, causal=causal)[0]
            print(f"[{name}] causal={causal} p={p}", flush=True)
            O, lse = B.sparse_attn(sh, Qg, Kg, Vg, torch.from_numpy(mask.view(np.int32)).cuda(), causal=causal, return_lse=True)
            torch.cuda.synchronize()
            check(f"causal={causal} p={p}", O, oracle.sparse_attn(osh, Q, K, V, mask, causal=causal)[0])
            if causal:
                want, absdot = oracle.bwd.lse_rows(osh, Q.double().numpy(), K.double().numpy(), mask, rows)
                assert (np.abs(lse.cpu().numpy().astype(np.float64) - want) <= lse_bound(absdot)).all()
        O = B.dense_attn(sh, Qg, Kg, Vg, causal=causal)
        torch.cuda.synchronize()
        check(f"causal={causal} dense", O, oracle.dense_attn(osh, Q, K, V, causal=causal))


WALK64 = [  # grid, cube, query heads, KV heads, text after and before
    ("cubes128", (64, 16, 16), (4, 4, 8), 4, 4, 0, 0),
    ("cubes256", (32, 16, 16), (4, 8, 8), 8, 2, 0, 0),
    ("clipped60_text", (16, 10, 15), (3, 4, 5), 48, 4, 70, 0),
    ("clipped60_text_around", (24, 10, 15), (3, 4, 5), 32, 4, 70, 45),
]


@pytest.mark.parametrize("name,grid,cube,hq,hkv,text,lead", WALK64, ids=[s[0] for s in WALK64])
def test_dense_walk_of_64(B, oracle, name, grid, cube, hq, hkv, text, lead):  # noqa: F811
    w = synth.Workload(name, 45, *grid, *cube, hq, hkv, 64, (0.6,), (1.0,) * hkv, text, lead)
    sh, osh = B.Shape.of(w), oshape(oracle, w)
    Q, K, V = synth.generate(w)
    rows = stratified_rows(oracle, osh, w, 400)
    for causal in (True, False):
        assert short(B, sh, causal) == 0
        print(f"[{name}] causal={causal}", flush=True)
        O = B.dense_attn(sh, Q.cuda(), K.cuda(), V.cuda(), causal=causal)
        torch.cuda.synchronize()
        check_outputs(f"{name} causal={causal}", rows_of(O, rows, w), oracle.dense_attn(osh, Q, K, V, rows=rows, causal=causal))


# The dense walk where no cube has more than 32 tokens, and more rows than the kernel for short sequences takes
@pytest.mark.parametrize("d", [64, 128])
def test_dense_walk_of_small_cubes(B, oracle, d):  # noqa: F811
    w = synth.Workload(f"cubes32_{d}", 63, 27, 12, 13, 2, 4, 4, 32, 8, d, (0.5,), (1.0,) * 8, 20, 0)
    sh, osh = B.Shape.of(w), oshape(oracle, w)
    Q, K, V = synth.generate(w)
    rows = stratified_rows(oracle, osh, w, 200)
    for causal in (True, False):
        O = B.dense_attn(sh, Q.cuda(), K.cuda(), V.cuda(), causal=causal)
        torch.cuda.synchronize()
        check_outputs(f"{w.name} causal={causal}", rows_of(O, rows, w), oracle.dense_attn(osh, Q, K, V, rows=rows, causal=causal))


# Few rows, which the masked walk takes in one round, where all KV heads select little, all select much, and one of two little:
# the kernel that the automatic choice has to take with room for the key-stationary one, and without.  (Grid, cube, query heads, KV
# heads, key scale of each, what is selected: Top-p or Top-K; kernel with room, kernel without.)
FEW = [
    ("cubes256_little", (56, 16, 16), (4, 8, 8), 6, 2, (1.0, 1.0), 0.5, "pairs", "masked"),
    ("cubes256_much", (56, 16, 16), (4, 8, 8), 6, 2, (1.0, 1.0), 0.9, "masked", "masked"),
    ("cubes256_one_little", (56, 16, 16), (4, 8, 8), 6, 2, (0.0, 4.0), 0.9, "masked", "masked"),
    ("cubes32_one", (15, 15, 16), (2, 4, 4), 28, 4, (1.0,) * 4, 1, "pairs", "split"),
    ("cubes32_little", (15, 15, 16), (2, 4, 4), 28, 4, (1.0,) * 4, 4, "pairs", "masked"),
    ("clipped256_third", (96, 9, 10), (4, 8, 8), 28, 4, (1.0,) * 4, 0.7, "masked", "masked"),  # (more rows: a head at a time)
    ("clipped256_none", (96, 9, 10), (4, 8, 8), 28, 4, (1.0,) * 4, 0.0, "pairs", "compact"),  # (room: not asked whether to compact)
    ("cubes32_two_little", (28, 12, 12), (2, 4, 4), 28, 4, (0.0, 0.0, 4.0, 4.0), 0.9, "masked", "masked"),  # (a little more than one round)
    ("cubes32_wide_much", (60, 16, 16), (2, 4, 4), 6, 2, (1.0, 1.0), 0.9, "masked", "masked"),
    ("cubes32_wide_few", (60, 16, 16), (2, 4, 4), 6, 2, (1.0, 1.0), 4, "pairs", "split"),
    ("cubes32_much", (15, 15, 16), (2, 4, 4), 28, 4, (1.0,) * 4, 0.8, "masked", "masked"),
]


@pytest.mark.parametrize("name,grid,cube,hq,hkv,scale,sel,room,no_room", FEW, ids=[s[0] for s in FEW])
def test_choice_for_few_rows(B, oracle, name, grid, cube, hq, hkv, scale, sel, room, no_room):  # noqa: F811
    w = synth.Workload(name, 50, *grid, *cube, hq, hkv, 128, (0.5,), scale)
    sh, osh = B.Shape.of(w), oshape(oracle, w)
    Q, K, V = synth.generate(w)
    Qg = Q.cuda()
    kbar = B.cube_pool(sh, K.cuda())
    mask, count = (B.cube_select(sh, Qg, kbar, sel) if isinstance(sel, float) else B.cube_select_topk(sh, Qg, kbar, sel))[:2]
    rows = stratified_rows(oracle, osh, w, 200)
    ref = oracle.sparse_attn(osh, Q, K, V, mask.cpu().numpy().view(np.uint32)[rows], rows=rows)[0]
    big = B.kv_pack(sh, K.cuda(), V.cuda(), workspace=B.alloc_workspace(sh, B.CALL_SPARSE_ATTN, pairs_capacity=int(count.sum())))
    small = B.kv_pack(sh, K.cuda(), V.cuda())
    forced = {"masked": B.sparse_attn_packed(sh, Qg, big, mask, kernel=B.SPARSE_MASKED).float(),
              "pairs": B.sparse_attn_packed(sh, Qg, big, mask, kernel=B.SPARSE_PAIRS).float()}
    for ws, expected in ((big, room), (small, no_room)):
        O = B.sparse_attn_packed(sh, Qg, ws, mask)
        torch.cuda.synchronize()
        check_outputs(f"{name} {expected}", rows_of(O, rows, w), ref)
        # kernels round at different places (2e-3 of the result), one kernel the same way each time but for a few rows
        off = {k: float((O.float() - x).norm() / x.norm()) for k, x in forced.items()}
        print(f"[{name}] expected {expected}: from the forced kernels' results {off}", flush=True)
        for k, x in off.items():
            assert (x < 1e-4) == (k == expected), (k, expected)


# Scratch for not quite the rows' own records, and nothing selected: with a little more than one round of the walk the compacting kernel has
# such a selection, as it has without scratch.
LITTLE_ROOM = [
    ("cubes32", (28, 12, 12), (2, 4, 4), 28, 4, 128),
    ("cubes256", (36, 16, 16), (4, 8, 8), 14, 2, 128),
    ("cubes256_64", (56, 16, 16), (4, 8, 8), 8, 2, 64),
]


@pytest.mark.parametrize("name,grid,cube,hq,hkv,d", LITTLE_ROOM, ids=[s[0] for s in LITTLE_ROOM])
def test_choice_with_too_little_scratch(B, name, grid, cube, hq, hkv, d):  # noqa: F811
    w = synth.Workload(name, 66, *grid, *cube, hq, hkv, d, (0.5,), (1.0,) * hkv)
    sh = B.Shape.of(w)
    Q, K, V = (x.cuda() for x in synth.generate(w))
    mask = B.cube_select(sh, Q, B.cube_pool(sh, K), 0.0)[0]
    n = B.pairs_workspace_bytes(sh, 0)
    O = {}
    for what, size, kernel in (("compact", n, B.SPARSE_COMPACT), ("masked", n, B.SPARSE_MASKED), ("little room", n - 4096, None),
                               ("none", B.workspace_bytes(sh, B.CALL_SPARSE_ATTN), None)):
        packed = B.kv_pack(sh, K, V, workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
        O[what] = B.sparse_attn_packed(sh, Q, packed, mask, kernel=kernel).float()
    torch.cuda.synchronize()
    off = {k: float((O["compact"] - x).norm() / x.norm()) for k, x in O.items()}
    print(f"[{name}] from the compacting kernel's results {off}", flush=True)
    assert off["masked"] > 1e-4 and off["none"] < 1e-4 and off["little room"] < 1e-4


# Some KV heads select next to nothing and go to the key-stationary kernel: the masked walk's workgroups are dealt out over the heads that
# remain, one, three (eight XCDs are no multiple of them) and five of six, and seven of eight.
@pytest.mark.parametrize("heads,flat,d", [(6, 1, 64), (6, 3, 64), (6, 5, 64), (8, 7, 64), (6, 3, 128), (6, 5, 128)])
def test_walk_of_the_heads_that_remain(B, heads, flat, d):  # noqa: F811
    w = synth.Workload(f"heads{heads}_flat{flat}", 62, 560 // heads, 16, 16, 4, 8, 8, heads, heads, d, (0.9,), (0.0,) * flat + (4.0,) * (heads - flat))
    sh = B.Shape.of(w)
    Q, K, V = (x.cuda() for x in synth.generate(w))
    mask, count = B.cube_select(sh, Q, B.cube_pool(sh, K), 0.9)[:2]
    packed = B.kv_pack(sh, K, V, workspace=B.alloc_workspace(sh, B.CALL_SPARSE_ATTN, pairs_capacity=int(count.sum())))
    want = B.sparse_attn_packed(sh, Q, packed, mask, kernel=B.SPARSE_MASKED).float()
    got = B.sparse_attn_packed(sh, Q, packed, mask, O=torch.full_like(Q, float("nan"))).float()
    torch.cuda.synchronize()
    off = [float((got[:, h] - want[:, h]).norm() / want[:, h].norm()) for h in range(heads)]
    print(f"[{w.name}] heads' results from the masked walk's: {off}", flush=True)
    # (the same kernel: bit for bit; the other one rounds elsewhere, 2e-3 of the result)
    assert all(x == 0.0 for x in off[:flat]) and all(0.0 < x < 1e-2 for x in off[flat:])

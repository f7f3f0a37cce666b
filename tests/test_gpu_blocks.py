"""The masked walk on shapes whose blocks of 256 rows lie across cubes, against the fp64 oracle: a KV head with 255, 256, 257
and 513 rows, blocks over many cubes of one token, over clipped cubes and over the borders of text and video, and last tiles
with 1, 31, 33 and 63 keys (the padding keys' probabilities are cleared in the short softmax step).  Tolerances are those of
the other attention tests.  And values that are not finite in cubes
behind a row's own, in all attention kernels whose blocks lie across cubes."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2604_08077_amd import synth
from test_gpu_parity import B, MAX_ABS, MEAN_ABS, lse_bound, oshape  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [  # grid, cube, query heads, KV heads, head_dim, text after and before
    ("rows255", (5, 3, 17), (2, 3, 5), 2, 2, 64, 0, 0),
    ("rows256", (4, 8, 8), (3, 3, 5), 1, 1, 128, 0, 0),
    ("rows257_one_token_cubes", (1, 1, 257), (1, 1, 1), 1, 1, 64, 0, 0),
    ("rows513", (9, 3, 19), (2, 2, 8), 2, 2, 128, 0, 0),
    ("heads_and_text", (5, 7, 9), (4, 4, 8), 6, 2, 128, 37, 29),
    ("last_tiles_1_63", (7, 5, 13), (4, 5, 13), 3, 1, 64, 63, 0),  # cubes of 260 and 195 tokens, text of 63
    ("last_tiles_33_31", (6, 1, 97), (1, 1, 97), 2, 1, 128, 31, 0),
    ("clipped_to_strips", (6, 9, 9), (4, 8, 8), 7, 1, 128, 0, 0),
]


@pytest.mark.parametrize("name,grid,cube,hq,hkv,d,text,lead", SHAPES, ids=[s[0] for s in SHAPES])
def test_blocks_across_cubes(B, oracle, name, grid, cube, hq, hkv, d, text, lead):  # noqa: F811
    w = synth.Workload(name, 47, *grid, *cube, hq, hkv, d, (0.6,), (1.0,) * hkv, text, lead)
    sh, osh = B.Shape.of(w), oshape(oracle, w)
    Q, K, V = synth.generate(w)
    kbar = oracle.cube_pool(osh, K)
    rows = np.arange(w.S * w.Hq)
    packed = B.kv_pack(sh, K.cuda(), V.cuda())
    for causal in (True, False):
        for p in (0.0, 0.6):
            mask = oracle.cube_select(osh, Q, kbar, p, causal=causal)[0]
            print(f"[{name}] causal={causal} p={p}", flush=True)
            lse = torch.empty(w.S * w.Hq, dtype=torch.float32, device="cuda")
            O = B.sparse_attn_packed(sh, Q.cuda(), packed, torch.from_numpy(mask.view(np.int32)).cuda(), causal=causal, lse=lse,
                                     kernel=B.SPARSE_MASKED)
            torch.cuda.synchronize()
            want = oracle.sparse_attn(osh, Q, K, V, mask, causal=causal)[0]
            err = np.abs(O.reshape(-1, d).float().cpu().numpy().astype(np.float64) - want)
            print(f"[{name}] max-abs={err.max():.3e} mean-abs={err.mean():.3e}", flush=True)
            assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS
            if causal:
                ref, absdot = oracle.bwd.lse_rows(osh, Q.double().numpy(), K.double().numpy(), mask, rows)
                assert (np.abs(lse.cpu().numpy().astype(np.float64) - ref) <= lse_bound(absdot)).all()


# No cube above 32 tokens, every tile worked as its first half: cubes of 32 and 31 with text, and of 33 on the other side.
HALF = [
    ("keys32_text", (6, 4, 12), (2, 4, 4), 6, 2, 64, 33, 31),
    ("keys32_128", (7, 5, 9), (2, 4, 4), 2, 1, 128, 1, 0),
    ("keys31_text", (9, 1, 31), (1, 1, 31), 4, 1, 128, 31, 5),
    ("keys33", (9, 3, 11), (1, 3, 11), 4, 1, 128, 0, 0),
]


@pytest.mark.parametrize("name,grid,cube,hq,hkv,d,text,lead", HALF, ids=[s[0] for s in HALF])
def test_half_tiles(B, oracle, name, grid, cube, hq, hkv, d, text, lead):  # noqa: F811
    test_blocks_across_cubes(B, oracle, name, grid, cube, hq, hkv, d, text, lead)


BEHIND = SHAPES + [  # the first two: the dense walk at both head-dims, and the dQ kernel with one wavefront per 32 rows; then with two; on half tiles
    ("clipped60_text", (16, 10, 15), (3, 4, 5), 48, 4, 64, 70, 45),
    ("clipped60", (18, 9, 15), (3, 4, 5), 36, 4, 128, 0, 0),
    ("clipped256_text", (5, 13, 17), (4, 8, 8), 20, 4, 64, 33, 65),
    ("clipped128_text", (9, 10, 12), (4, 4, 8), 28, 4, 128, 33, 20),
    ("cubes32_text", (13, 9, 12), (2, 4, 4), 64, 16, 128, 33, 20),
]


def test_every_dq_kernel_is_reached(B):  # noqa: F811
    """By the shapes of the test below."""
    kernels = set()
    for name, grid, cube, hq, hkv, d, text, lead in BEHIND:
        cs = B.Shape.of(synth.Workload(name, 49, *grid, *cube, hq, hkv, d, (0.6,), (1.0,) * hkv, text, lead))._c()
        kernels.add((d, B.load().adaspark_internal_dq_waves(ctypes.byref(cs)), B.load().adaspark_internal_dq_half_tiles(ctypes.byref(cs))))
    assert kernels >= {(64, 8, 0), (128, 8, 0), (64, 2, 0), (128, 2, 0), (64, 1, 0), (128, 1, 0), (128, 1, 1)}


def cube_of_tokens(w):
    """The cube of every token."""
    C = w.ct * w.ch * w.cw
    nt, nh, nw = -(-w.T // w.ct), -(-w.H // w.ch), -(-w.W // w.cw)
    t, h, x = np.indices((w.T, w.H, w.W)).reshape(3, -1)
    lead = -(-w.lead // C)
    return torch.from_numpy(np.concatenate([np.arange(w.lead) // C, lead + ((t // w.ct) * nh + h // w.ch) * nw + x // w.cw,
                                            lead + nt * nh * nw + np.arange(w.text) // C]))


@pytest.mark.parametrize("name,grid,cube,hq,hkv,d,text,lead", BEHIND, ids=[s[0] for s in BEHIND])
def test_what_is_not_finite_does_not_reach_rows_before_it(B, oracle, name, grid, cube, hq, hkv, d, text, lead):  # noqa: F811
    """K and V of a late cube hold infinities and NaN: what the rows of the cubes before it get is bit for bit what they get with
    finite ones, though their blocks walk that cube too."""
    w = synth.Workload(name, 49, *grid, *cube, hq, hkv, d, (0.6,), (1.0,) * hkv, text, lead)
    sh = B.Shape.of(w)
    Q, K, V = (x.cuda() for x in synth.generate(w))
    sel = B.cube_select(sh, Q, B.cube_pool(sh, K), 0.6)[0]
    g = torch.Generator(device="cpu")
    g.manual_seed(synth.BASE_SEED + 49)
    dO = torch.randn((w.S, w.Hq, w.D), generator=g, dtype=torch.float32).to(torch.bfloat16).cuda()
    cubes = cube_of_tokens(w)
    N = int(cubes.max()) + 1

    def forward(K, V):
        packed = B.kv_pack(sh, K, V)
        lse = [torch.empty(w.S * w.Hq, dtype=torch.float32, device="cuda") for _ in range(3)]
        O = [B.sparse_attn_packed(sh, Q, packed, sel, lse=lse[0], kernel=B.SPARSE_MASKED),
             B.sparse_attn_packed(sh, Q, packed, sel, lse=lse[1]), B.dense_attn_packed(sh, Q, packed, lse=lse[2])]
        return O, [x.view(w.S, w.Hq) for x in lse]

    want_O, want_lse = forward(K, V)
    grads = [(m, O, lse) for m, O, lse in zip((sel, None), want_O[1:], want_lse[1:])]
    want_dQ = [B.sparse_attn_bwd(sh, Q, K, V, O, lse.reshape(-1), dO, sel_mask=m)[0] for m, O, lse in grads]
    for c in sorted({N - 1, N // 2}):
        before, at = (cubes < c).cuda(), (cubes == c).cuda()
        for bad in (float("inf"), float("nan")):
            Kx, Vx = K.clone(), V.clone()
            Kx[at], Vx[at] = bad, bad
            print(f"[{name}] cube {c} of {N}: {bad}", flush=True)
            O, lse = forward(Kx, Vx)
            dQ = [B.sparse_attn_bwd(sh, Q, Kx, Vx, o, x.reshape(-1), dO, sel_mask=m)[0] for m, o, x in grads]
            torch.cuda.synchronize()
            for what, a, b in zip(("O masked", "O auto", "O dense", "lse masked", "lse auto", "lse dense", "dQ", "dQ dense"),
                                  O + lse + dQ, want_O + want_lse + want_dQ):
                wrong = int((a[before] != b[before]).sum())
                print(f"[{name}] {what}: {wrong} of {b[before].numel()}", flush=True)
                assert wrong == 0, what

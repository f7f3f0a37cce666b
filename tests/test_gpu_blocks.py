"""The masked walk on shapes whose blocks of 256 rows lie across cubes, against the fp64 oracle: a KV head with 255, 256, 257
and 513 rows, blocks over many cubes of one token, over clipped cubes and over the borders of text and video, and last tiles
with 1, 31, 33 and 63 keys (the padding keys' probabilities are cleared in the short softmax step).  Tolerances are those of
the other attention tests."""
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

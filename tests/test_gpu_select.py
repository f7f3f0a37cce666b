"""Cube selection where the kernel for up to 256 candidates changes its launch: one or two 16-row slabs per wavefront (few or
many rows), and in the second case launches of their own for the query cubes below 64, below 128 and the rest.  Sets against the
fp64 oracle, as in the parity tests."""
import numpy as np
import pytest
import torch

from paper_2604_08077_amd import synth
from test_gpu_parity import B, check_selection, oshape, to_u32  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [  # cubes, tokens of a cube, query heads, KV heads, head_dim
    ("few_64", 64, 5, 3, 1, 64),
    ("few_2", 2, 33, 2, 1, 128),  # up to 64 cubes: the wavefronts split the mean keys themselves
    ("few_16", 16, 7, 3, 1, 64),
    ("few_17", 17, 16, 2, 2, 128),
    ("few_64_128", 64, 3, 1, 1, 128),
    ("few_65", 65, 16, 1, 1, 128),
    ("few_129", 129, 17, 2, 2, 64),
    ("few_256", 256, 4, 4, 1, 128),
    ("many_64", 64, 64, 32, 8, 64),
    ("many_65", 65, 64, 32, 8, 64),
    ("many_128", 128, 64, 32, 8, 64),
    ("many_129", 129, 64, 32, 8, 64),
    ("many_205", 205, 33, 32, 16, 128),
]


@pytest.mark.parametrize("name,cubes,tokens,hq,hkv,d", SHAPES, ids=[s[0] for s in SHAPES])
def test_selection_launches(B, oracle, name, cubes, tokens, hq, hkv, d):  # noqa: F811
    w = synth.Workload(name, 43, cubes, 1, tokens, 1, 1, tokens, hq, hkv, d, (0.8,), (1.0,) * hkv)
    sh, osh = B.Shape.of(w), oshape(oracle, w)
    Q, K, _ = synth.generate(w)
    kbar = oracle.cube_pool(osh, K).astype(np.float32)
    print(f"[{name}] {w.S * hq} rows", flush=True)
    mask, count, _, _ = B.cube_select(sh, Q.cuda(), torch.from_numpy(kbar).cuda(), 0.8)
    torch.cuda.synchronize()
    ref_mask, ref_count, near = oracle.cube_select(osh, Q, kbar, 0.8)
    check_selection(name, to_u32(mask), count.cpu().numpy(), ref_mask, ref_count, near)


@pytest.mark.parametrize("cubes,hq,hkv,d", [(17, 2, 2, 128), (64, 3, 1, 64)])
def test_mean_keys_at_16_bytes(B, cubes, hq, hkv, d):  # noqa: F811
    """Mean keys 16 bytes behind a 32-byte border, which the entry takes: the sets are those of the aligned ones."""
    w = synth.Workload("at16", 44, cubes, 1, 5, 1, 1, 5, hq, hkv, d, (0.8,), (1.0,) * hkv)
    sh = B.Shape.of(w)
    Q, K, _ = (x.cuda() for x in synth.generate(w))
    kbar = B.cube_pool(sh, K)
    buf = torch.empty(kbar.numel() + 4, device="cuda")
    moved = buf[4:].view_as(kbar).copy_(kbar)
    assert kbar.data_ptr() % 32 == 0 and moved.data_ptr() % 32 == 16
    got, want = B.cube_select(sh, Q, moved, 0.8)[:2], B.cube_select(sh, Q, kbar, 0.8)[:2]
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])

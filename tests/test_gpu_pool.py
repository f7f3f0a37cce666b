"""Mean keys where the kernel cuts a token's row into parts, and the token index arithmetic where it divides in 32 bits: against float64."""
import pytest
import torch

from paper_2604_08077_amd import synth
from test_gpu_blocks import cube_of_tokens
from test_gpu_parity import B, KBAR_ABS, check_outputs, oshape  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [  # grid, cube, KV heads, head_dim, text after and before
    ("parts16", (4, 8, 8), (4, 8, 8), 4, 128, 0, 0),  # one cube
    ("parts2_of_40", (5, 7, 9), (2, 3, 4), 5, 128, 0, 0),  # 80 pieces of a row: 25 slots of 40, three threads an element
    ("whole_row_of_24", (5, 7, 9), (2, 3, 4), 3, 64, 11, 30),
    ("two_sweeps", (2, 3, 3), (1, 2, 2), 160, 128, 0, 0),  # 2,560 pieces
    ("cubes256", (256, 2, 2), (1, 2, 2), 4, 64, 0, 0),  # as many cubes as CUs: whole rows
    ("one_token", (3, 3, 3), (1, 1, 1), 1, 64, 2, 1),
    ("cubes_over_22_bits", (3, 5, 7), (4096, 32, 33), 2, 64, 0, 0),  # nominal size 4.3 M tokens
]


@pytest.mark.parametrize("name,grid,cube,hkv,d,text,lead", SHAPES, ids=[s[0] for s in SHAPES])
def test_mean_keys(B, name, grid, cube, hkv, d, text, lead):  # noqa: F811
    w = synth.Workload(name, 63, *grid, *cube, hkv, hkv, d, (0.5,), (1.0,) * hkv, text, lead)
    K = synth.generate(w)[1]
    got = B.cube_pool(B.Shape.of(w), K.cuda()).cpu().double()
    of = cube_of_tokens(w)
    want = torch.stack([K[of == c].double().mean(0) for c in range(int(of.max()) + 1)])
    print(f"[{name}] max-abs {float((got - want).abs().max()):.2e}", flush=True)
    assert float((got - want).abs().max()) <= KBAR_ABS


def test_attention_in_cubes_over_22_bits(B, oracle):  # noqa: F811
    w = synth.Workload("over_22_bits", 64, 3, 5, 7, 4096, 32, 33, 2, 1, 64, (0.5,), (1.0,))
    Q, K, V = synth.generate(w)
    O = B.dense_attn(B.Shape.of(w), Q.cuda(), K.cuda(), V.cuda())
    torch.cuda.synchronize()
    check_outputs("cubes over 22 bits", O.reshape(-1, w.D).float().cpu().numpy(), oracle.dense_attn(oshape(oracle, w), Q, K, V))

"""Mean keys where the kernel cuts a token's row into parts, where a row takes several sweeps of a workgroup, and the token index arithmetic
where it divides in 32 bits: against float64, and bit for bit in the order in which the sums are defined, whatever the parts."""
import numpy as np
import pytest
import torch

from paper_2604_08077_amd import synth
from test_gpu_blocks import cube_of_tokens
from test_gpu_parity import B, KBAR_ABS, check_outputs, oshape  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [  # grid, cube, KV heads, head_dim, text after and before
    ("parts8", (4, 8, 8), (4, 8, 8), 4, 128, 0, 0),  # one cube, 64 pieces of a row
    ("parts2_of_40", (5, 7, 9), (2, 3, 4), 5, 128, 0, 0),  # 80 pieces: 12 slots
    ("whole_row_of_24", (5, 7, 9), (2, 3, 4), 3, 64, 11, 30),
    ("parts32_of_80", (2, 3, 3), (1, 2, 2), 160, 128, 0, 0),  # 2,560 pieces: two parts lie across the borders of the row's sweeps
    ("parts_of_one_wavefront", (1, 2, 131), (1, 2, 131), 64, 128, 0, 0),  # 1,024 pieces in 128 parts
    ("sweeps3", (256, 1, 1), (1, 1, 1), 160, 128, 0, 0),  # as many cubes as CUs: whole rows, three sweeps
    ("piece320", (256, 1, 5), (1, 1, 5), 20, 128, 0, 0),  # more elements than threads, three slots
    ("cubes256", (256, 2, 2), (1, 2, 2), 4, 64, 0, 0),
    ("tokens2820", (1, 47, 60), (1, 47, 60), 3, 64, 0, 0),  # more tokens than are looked up at a time: 2,016 of 42 slots, and the rest
    ("one_token", (3, 3, 3), (1, 1, 1), 1, 64, 2, 1),
    ("cubes_over_22_bits", (3, 5, 7), (4096, 32, 33), 2, 64, 0, 0),  # nominal size 4.3 M tokens
]


def in_order(K, of):
    """The mean keys in float32, summed as they are defined: a row's 16-byte pieces in sweeps of up to 1,024, a sweep with as many slots as
    then fit 1,024 threads; a slot adds every slots-th token of the cube, the slots are added in their order."""
    rows = K.float().reshape(K.shape[0], -1).numpy()
    out = np.empty((int(of.max()) + 1, rows.shape[1]), np.float32)
    for c in range(len(out)):
        x = rows[(of == c).numpy()]
        for lo in range(0, x.shape[1], 8192):
            y = x[:, lo: lo + 8192]
            slots = 1024 // (y.shape[1] // 8)
            sums = np.zeros((slots, y.shape[1]), np.float32)
            for r in range(len(y)):
                sums[r % slots] += y[r]
            total = np.zeros(y.shape[1], np.float32)
            for s in sums:
                total += s
            out[c, lo: lo + 8192] = total / np.float32(len(y))
    return torch.from_numpy(out).view(len(out), *K.shape[1:])


@pytest.mark.parametrize("name,grid,cube,hkv,d,text,lead", SHAPES, ids=[s[0] for s in SHAPES])
def test_mean_keys(B, name, grid, cube, hkv, d, text, lead):  # noqa: F811
    w = synth.Workload(name, 63, *grid, *cube, hkv, hkv, d, (0.5,), (1.0,) * hkv, text, lead)
    K = synth.generate(w)[1]
    got = B.cube_pool(B.Shape.of(w), K.cuda()).cpu()
    of = cube_of_tokens(w)
    want = torch.stack([K[of == c].double().mean(0) for c in range(int(of.max()) + 1)])
    off, bits = float((got.double() - want).abs().max()), int((got != in_order(K, of)).sum())
    print(f"[{name}] max-abs {off:.2e}, {bits} elements not as defined", flush=True)
    assert off <= KBAR_ABS and bits == 0


def test_attention_in_cubes_over_22_bits(B, oracle):  # noqa: F811
    w = synth.Workload("over_22_bits", 64, 3, 5, 7, 4096, 32, 33, 2, 1, 64, (0.5,), (1.0,))
    Q, K, V = synth.generate(w)
    O = B.dense_attn(B.Shape.of(w), Q.cuda(), K.cuda(), V.cuda())
    torch.cuda.synchronize()
    check_outputs("cubes over 22 bits", O.reshape(-1, w.D).float().cpu().numpy(), oracle.dense_attn(oshape(oracle, w), Q, K, V))

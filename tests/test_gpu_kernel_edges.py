"""Edges of the kernels' tiles and of the rules that choose between them, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import gptaq_oracle as O
from paper_2504_02692_amd import synth
from tests import parity_util as PU

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


@pytest.mark.parametrize("bits,group,m,n,terms", [
    (4, 16, 65, 16, 3),        # one sub-block, one row more than a workgroup holds
    (4, 0, 64, 113, 3),        # one block, a last sub-block of one column, rows that take no vector stores
    (4, 32, 1, 160, 3),        # a block and a quarter, one row
    (4, 64, 129, 896, 3),      # seven of the eight blocks
    (4, 0, 63, 1041, 3),       # a second super-block of one sub-block and one column
    (4, 0, 63, 1041, 1), (4, 0, 63, 1041, 2), (4, 0, 63, 1041, 0),       # the ablations, without vector stores
    (4, 128, 70, 1280, 1), (4, 128, 70, 1280, 2), (4, 128, 70, 1280, 0)])
def test_column_loop_at_the_edges_of_its_blocks(bits, group, m, n, terms):
    """The super-block kernel: 16-column sub-blocks, 128-column blocks (one per wavefront), 64 rows per workgroup."""
    k = max(256, n + n // 2)
    Xb, Xtb = synth.make_activations(k, n, 31, "edge", 2, 20.0)
    H, A = O.accumulate(Xb, Xtb)
    U, P, _ = O.prepare(H, A, 0.01)
    U32, P32 = U.astype(np.float32), P.astype(np.float32)
    W = synth.make_weights(m, n, 31, f"edge{m}x{n}")
    got = PU.gpu_quantize(W, dev(U32), dev(P32) if terms & 2 else None, bits, group, False, 128, terms=terms)
    PU.check_against_oracle(W, U32.astype(np.float64), P32.astype(np.float64), got, bits, group, False,
                            label=f"edge W{bits} g{group} {m}x{n} terms {terms}", terms=terms)


# Sizes around the 16-column tiles and the 256-column outer blocks of the factorisation: a block of identity padding and one
# column, part of a tile, whole tiles, one column into the next block, three blocks with a ragged first one.
@pytest.mark.parametrize("n", [1, 15, 16, 17, 47, 240, 241, 255, 257, 273, 528, 767])
def test_factor_and_inverse_at_tile_edges(n):
    k = max(64, 4 * n)
    Xb, Xtb = synth.make_activations(k, n, 11, f"factor{n}", min(2, n - 1), 20.0)
    H, A = O.accumulate(Xb, Xtb)
    U, P, _ = O.prepare(H, A, 0.01)
    Hd, Ad = dev(np.triu(H)), dev(A)
    _, info = PU.gpu_prepare(Hd, Ad, 0.01)
    assert info.cpu().tolist() == [0, 0]
    # U: one rounding to fp32 of a result exact to ~1e-12, from an H rounded to fp32 (2^-24 each, condition number ~1e2);
    # P: products of bf16 hi + lo splits (2^-17 per operand)
    assert PU.rel_fro(Hd.cpu().numpy(), U) <= 1e-6
    if n > 1:
        assert PU.rel_fro(Ad.cpu().numpy(), P) <= 5e-5

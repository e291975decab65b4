"""Edges of the kernels' tiles and of the rules that choose between them, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import gptaq_oracle as O
from paper_2504_02692_amd import binding as B
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


def bf16_rne(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).bfloat16().float().numpy()


# Where the update of a column comes from: the rest of its sub-block's piece, another piece of the same block, another block of
# the super-block, the product after it.
@pytest.mark.parametrize("dst", [16, 32, 128, 1024])
def test_error_operand_carries_the_unrounded_product(dst):
    """-E = (W^ - v) / U_jj enters the products as bf16 hi + lo, lo the rounding of what hi leaves of (W^ - v) (1 / U_jj) before
    that product is rounded to fp32.  One column with an error meets one zero weight through a power of two, so the updated
    weight IS hi + lo, and the range of its group shows every bit of it."""
    m, n, bits, group, maxq = 4096, dst + 16, 4, 16, 15.0
    g = np.random.default_rng(dst)
    W = np.zeros((m, n), np.float32)
    W[:, 0] = g.uniform(0.1, 0.9, m)
    W[:, 1] = 1.0                                # the range of the first group
    U = np.diag(g.uniform(1.0, 2.0, n)).astype(np.float32)
    U[0, dst] = 0.5
    got = PU.gpu_quantize(W, dev(U), None, bits, group, False, 128, terms=1)
    sc, d = got["scales"][:, 0].astype(np.float64), got["codes"][:, 0] - got["zeros"][:, 0].astype(np.float64)
    v = W[:, 0].astype(np.float64)
    t = (sc * d - v).astype(np.float32).astype(np.float64)         # (fp64 holds the product and the sum exactly)
    prod = t * np.float64(np.float32(1) / U[0, 0])                 # exact: 48 bits
    hi = bf16_rne(prod.astype(np.float32)).astype(np.float64)
    lo = bf16_rne((prod - hi).astype(np.float32)).astype(np.float64)
    old = bf16_rne((prod.astype(np.float32) - hi).astype(np.float32)).astype(np.float64)
    w = 0.5 * (hi + lo)
    rows = w == w.astype(np.float32)             # where the updated weight is exact: lo is not all but zero
    assert rows.mean() > 0.9 and (lo != old)[rows].any()           # the inputs tell the two apart
    want = np.where(w == 0, 2.0 / maxq, np.abs(w) / maxq).astype(np.float32)
    assert np.array_equal(got["scales"][rows, dst // group], want[rows])


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


# Blocks whose buffers take turns (three of V, two of U's rows), ragged first blocks that end in either half, rows of dXXT that are not
# 16-byte aligned.  U against H itself: |U^T U (H + lambda I) - I|; the tolerances of test_factor_and_inverse_at_tile_edges.
@pytest.mark.parametrize("n,ld", [(1152, 1152), (1281, 1281), (1409, 1411), (1790, 1792), (2049, 2056)])
def test_factor_sweep_over_many_blocks(n, ld):
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((4 * n, n), device="cuda", generator=g).double()
    H = X.T.contiguous() @ X
    A = ((0.1 * torch.randn((4 * n, n), device="cuda", generator=g)).double().T.contiguous() @ X).float()
    Hd, Ad = torch.full((n, ld), 7.0, device="cuda"), torch.full((n, ld), 7.0, device="cuda")
    Hd[:, :n], Ad[:, :n] = H.float(), A
    ws = B.workspace(B.gptaq_prepare_workspace_bytes(n)).fill_(255)
    dead, info = torch.empty(n, dtype=torch.uint8, device="cuda"), torch.empty(2, dtype=torch.int32, device="cuda")
    assert B.load().gptaq_prepare(Hd.data_ptr(), Ad.data_ptr(), n, ld, 0.01, dead.data_ptr(), info.data_ptr(), ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream) == 0
    assert info.tolist() == [0, 0] and bool((Hd[:, n:] == 7).all()) and bool((Ad[:, n:] == 7).all())
    Hl = H.float().double().triu()
    Hl = (Hl + Hl.triu(1).T).cpu()
    Hl += 0.01 * Hl.diagonal().mean() * torch.eye(n, dtype=torch.float64)
    V = torch.linalg.cholesky(Hl.flip(0, 1)).flip(0, 1)              # H + lambda I = V V^T, V upper
    U = torch.linalg.inv(V)
    P = ((A.double().cpu() @ U.T.contiguous()).triu(1) @ U)
    assert PU.rel_fro(Hd[:, :n].cpu().numpy(), U.numpy()) <= 1e-6
    assert PU.rel_fro(Ad[:, :n].cpu().numpy(), P.numpy()) <= 5e-5


def test_two_factor_sweeps_beside_each_other():
    """Workgroups of a block wait for others of the same launch: two calls on two streams, each with its own buffers, both end, with the
    bits of a call alone."""
    n = 2304
    g = torch.Generator(device="cuda").manual_seed(5)
    X = torch.randn((2 * n, n), device="cuda", generator=g)
    H0, A0 = X.T.contiguous() @ X, (0.1 * torch.randn((2 * n, n), device="cuda", generator=g)).T.contiguous() @ X
    sets = [(H0.clone(), A0.clone(), B.workspace(B.gptaq_prepare_workspace_bytes(n)), torch.cuda.Stream()) for _ in range(2)]
    Ha, Aa = H0.clone(), A0.clone()
    B.gptaq_prepare(Ha, Aa, 0.01, sets[0][2])
    torch.cuda.synchronize()
    for _ in range(3):
        for H, A, ws, s in sets:
            with torch.cuda.stream(s):
                H.copy_(H0), A.copy_(A0)
                B.gptaq_prepare(H, A, 0.01, ws)
    torch.cuda.synchronize()
    for H, A, _, _ in sets:
        assert torch.equal(H, Ha) and torch.equal(A, Aa)


# The tile store of the bf16 product: inside the matrix, at its edges, rows farther apart than n, and so far apart that a tile is
# out of reach of 32-bit offsets; 128-tiles and (from 224 of them) 256-tiles.
@pytest.mark.parametrize("n,ld,tokens", [(8, 8, 40), (128, 128, 33), (136, 140, 64), (1032, 1032, 96), (3608, 3616, 64), (3840, 3840, 32),
                                         (136, 1 << 21, 50)])
@pytest.mark.parametrize("upper", [False, True])
def test_products_are_added_up_to_the_edge_and_no_further(n, ld, tokens, upper):
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((tokens, n), device="cuda", generator=g).bfloat16()
    Xt = (X.float() + 0.05 * torch.randn((tokens, n), device="cuda", generator=g)).bfloat16()
    start = [torch.randn((n, n), device="cuda", generator=g) for _ in range(2)]
    full = [torch.full((n, ld), -7.0, device="cuda") for _ in range(2)]
    H, A = full[0][:, :n], full[1][:, :n]
    H.copy_(start[0])
    A.copy_(start[1])
    ws = B.workspace(B.gptaq_accumulate_workspace_bytes(tokens, n))
    (B.gptaq_accumulate_upper if upper else B.gptaq_accumulate)(X, Xt, H, A, ws)
    torch.cuda.synchronize()
    Xd, Dd = X.double(), Xt.double() - X.double()
    # fp32 sums of `tokens` exact products and one rounding: 2^-24 each, far inside the accumulation's bar
    for got, ref, half in ((H, start[0].double() + Xd.T.contiguous() @ Xd, True), (A, start[1].double() + Dd.T.contiguous() @ Xd, upper)):
        got = got.double()
        if half:
            got, ref = got.triu(), ref.triu()
        assert float((got - ref).norm() / ref.norm()) <= 1e-5
    for f in full:
        assert bool((f[:, n:] == -7.0).all())


# The clip-range search inside the super-block kernel: every group size it takes, one candidate, fewer candidates than wavefronts,
# a full batch of ten per wavefront and one more, a last block cut short, a second super-block, rows that take no vector stores;
# and per-channel ranges, searched before the column loop.
@pytest.mark.parametrize("group,m,n,grid,steps", [(16, 65, 144, 100, 80), (32, 64, 160, 8, 1), (64, 130, 192, 10, 7), (128, 63, 1152, 100, 81),
                                                  (128, 1, 128, 100, 100), (0, 66, 130, 100, 80)])
def test_clip_search_in_the_column_loop(group, m, n, grid, steps):
    k = max(256, n + n // 2)
    Xb, Xtb = synth.make_activations(k, n, 37, "clip", 2, 20.0)
    H, A = O.accumulate(Xb, Xtb)
    U, P, _ = O.prepare(H, A, 0.01)
    U32, P32 = U.astype(np.float32), P.astype(np.float32)
    W = synth.make_weights(m, n, 37, f"clip{m}x{n}")
    got = PU.gpu_quantize(W, dev(U32), dev(P32), 4, group, False, 128, mse=(grid, steps))
    PU.check_against_oracle(W, U32.astype(np.float64), P32.astype(np.float64), got, 4, group, False,
                            label=f"clip g{group} {m}x{n} {steps}/{grid}", mse=(grid, steps))


# Group sizes that do not tile the super-block kernel's pieces are searched by the block-by-block kernel: one lane's columns, both of
# a lane's columns, several super-blocks (8 blocks of 64 columns).
@pytest.mark.parametrize("group,blocksize,m,n", [(8, 128, 70, 136), (96, 96, 66, 192), (8, 64, 33, 1160), (40, 120, 130, 240)])
def test_clip_search_in_the_block_kernel(group, blocksize, m, n):
    k = max(256, n + n // 2)
    Xb, Xtb = synth.make_activations(k, n, 41, "clipb", 2, 20.0)
    H, A = O.accumulate(Xb, Xtb)
    U, P, _ = O.prepare(H, A, 0.01)
    U32, P32 = U.astype(np.float32), P.astype(np.float32)
    W = synth.make_weights(m, n, 41, f"clipb{m}x{n}")
    got = PU.gpu_quantize(W, dev(U32), dev(P32), 4, group, False, blocksize, mse=(100, 80))
    PU.check_against_oracle(W, U32.astype(np.float64), P32.astype(np.float64), got, 4, group, False,
                            label=f"clip g{group} blocks of {blocksize} {m}x{n}", mse=(100, 80))


@pytest.mark.parametrize("m", [40, 1030])
@pytest.mark.parametrize("group", [32, 128])
def test_clip_search_beside_the_far_update(group, m):
    """Three super-blocks: from 1025 rows on the columns after the next one are updated on the helper stream."""
    n = 2304
    Xb, Xtb = synth.make_activations(3500, n, 43, "clip2", 2, 20.0)
    H, A = O.accumulate(Xb, Xtb)
    U, P, _ = O.prepare(H, A, 0.01)
    U32, P32 = U.astype(np.float32), P.astype(np.float32)
    W = synth.make_weights(m, n, 43, "clip2")
    got = PU.gpu_quantize(W, dev(U32), dev(P32), 4, group, False, 128, mse=(100, 80))
    PU.check_against_oracle(W, U32.astype(np.float64), P32.astype(np.float64), got, 4, group, False,
                            label=f"clip g{group} {m}x{n}", mse=(100, 80))


def test_clip_search_in_two_row_halves_equals_separate_calls():
    """From 10240 rows on a matrix goes through as two row halves on two streams, each with its own search."""
    m, n, half = 10500, 1152, 5376
    Xb, Xtb = synth.make_activations(1800, n, 44, "clip3", 2, 20.0)
    H, A = O.accumulate(Xb, Xtb)
    U, P, _ = O.prepare(H, A, 0.01)
    U32, P32 = dev(U.astype(np.float32)), dev(P.astype(np.float32))
    W = synth.make_weights(m, n, 44, "clip3")
    for group in (128, 0):
        one, a, b = (PU.gpu_quantize(w, U32, P32, 4, group, False, 128, mse=(100, 20)) for w in (W, W[:half], W[half:]))
        for key in ("codes", "scales", "zeros", "What"):
            assert np.array_equal(one[key], np.concatenate([a[key], b[key]])), (group, key)


# 96: the block-by-block kernel; the others: the super-block kernel.
@pytest.mark.parametrize("group", [32, 64, 96, 128])
def test_clip_search_does_not_lose_small_errors_behind_a_large_one(group):
    """Two candidates, scales 1 and s = 1 - 1/13000.  One weight is 0 under both and leaves 0.49^2; one is 3, exact under the first
    only, 9/13000^2 off under the second; all others are s: exact under the second, 1/13000^2 = 0.4 units in the last place of 0.49^2
    off under the first.  The second candidate is better by (group - 11) of those (10 units or more), but a single fp32 sum that meets
    the large square first drops every one of them.  In sums of four, added in pairs, at most three are next to the large one, and
    the roundings of the five to seven additions that follow cost half a unit each."""
    grid = 13000
    s = np.float32(1.0 - 1.0 / grid)
    m = group
    W = np.full((m, group), s, np.float32)
    for r in range(m):                           # the large square in every position
        W[r, r] = 0.49
        W[r, (r + 5) % group] = 3.0
    got = PU.gpu_quantize(W, dev(np.eye(group)), None, 2, group, False, 96 if group == 96 else 128, terms=0, mse=(grid, 2))
    assert np.array_equal(got["scales"], np.full((m, 1), s))


def test_clip_search_costs_what_its_candidates_cost():
    """The search is most of the time of a layer with 64 rows and 80 candidates (311 us of 1024 columns; 182 with 8, 345 with 100):
    eight candidates have to cost visibly less than 80, and 100 no more than a third above them."""
    m, n = 64, 1024
    U = dev(np.eye(n))
    W0 = dev(synth.make_weights(m, n, 5, "cost"))
    ws = B.workspace(B.gptaq_quantize_workspace_bytes(m, n))

    def best_ms(steps):
        times = []
        for _ in range(12):
            W = W0.clone()
            begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            begin.record()
            B.gptaq_quantize_layer(W, U, None, 4, 128, False, 128, ws, terms=1, mse_grid=100, mse_steps=steps)
            end.record()
            end.synchronize()
            times.append(begin.elapsed_time(end))
        return min(times)

    t8, t80, t100 = best_ms(8), best_ms(80), best_ms(100)
    print(f"clip search of 64 x 1024: {t8:.3f} ms with 8 candidates, {t80:.3f} with 80, {t100:.3f} with 100")
    assert t8 <= 0.8 * t80 and t100 <= 1.33 * t80


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1025, 2100])
def test_ranking_of_the_diagonal(n):
    """64 inputs per workgroup, 1024 compared at a time; many equal entries."""
    d = np.random.default_rng(n).integers(0, 40, n).astype(np.float32)
    perm = B.gptaq_act_order(dev(np.diag(d)))
    assert np.array_equal(perm.cpu().numpy(), O.act_order_permutation(np.diag(d)))


# Rows of 16-byte pieces (one, as many as the lanes keep, one more, a third round) and rows that are not; levels up to 16 bits.
@pytest.mark.parametrize("n", [8, 7, 2048, 2056, 2500, 4104])
@pytest.mark.parametrize("bits,clip", [(4, 0.9), (2, 1.0), (8, 0.3), (16, 0.9)])
def test_activation_quantiser_rows(n, bits, clip):
    Xb, _ = synth.make_activations(9, n, 13, "rows", 1, 20.0)
    Xb = Xb.copy()
    Xb[3] = 0                                    # an empty range
    Xb[4] = (Xb[4] & 0x807f) | (0x01 << 7)       # a range whose scale is a denormal number without a reciprocal
    Xb[5] = (Xb[5] & 0x807f) | (0xf0 << 7)       # a scale whose reciprocal is one
    X = PU.to_dev_bf16(Xb)
    got = B.gptaq_fake_quant_activations(X, bits, clip).contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
    ref, _, hints = O.fake_quant_activations(Xb, bits, clip, hint_bits=got, tau=PU.tau_for(bits))
    # (near-ties of x / scale in fp64; the library decides by the sign of an exact residual)
    assert hints <= max(2, PU.MAX_HINT_FRAC * got.size)
    assert np.array_equal(ref, got)


@pytest.mark.parametrize("m", [33, 1030])
def test_a_solve_can_be_captured(m):
    """gptaq_prepare (nine outer blocks) clears the flags of its workgroups in every replay.  gptaq_quantize_layer (three super-blocks) puts
    work on the helper stream from 1025 rows on; it joins the caller's stream in front of the end of the call, also in a capture.  Every replay is
    checked, with other work in between."""
    n = 2064
    g = torch.Generator(device="cuda").manual_seed(3)
    X = torch.randn((2 * n, n), device="cuda", generator=g)
    H0, A0 = X.T.contiguous() @ X, (0.1 * torch.randn((2 * n, n), device="cuda", generator=g)).T.contiguous() @ X
    W0 = 0.02 * torch.randn((m, n), device="cuda", generator=g)
    H, A, W = torch.empty_like(H0), torch.empty_like(A0), torch.empty_like(W0)
    dead, info = torch.empty(n, dtype=torch.uint8, device="cuda"), torch.empty(2, dtype=torch.int32, device="cuda")
    codes = torch.empty((m, n), dtype=torch.uint8, device="cuda")
    scales, zeros = torch.empty((m, n // 16), device="cuda"), torch.empty((m, n // 16), device="cuda")
    wp = B.workspace(B.gptaq_prepare_workspace_bytes(n))
    wq = B.workspace(B.gptaq_quantize_workspace_bytes(m, n))
    lib = B.load()

    def solve():
        H.copy_(H0), A.copy_(A0), W.copy_(W0)
        s = torch.cuda.current_stream().cuda_stream
        assert lib.gptaq_prepare(H.data_ptr(), A.data_ptr(), n, n, 0.01, dead.data_ptr(), info.data_ptr(), wp.data_ptr(), wp.numel(), s) == 0
        assert lib.gptaq_quantize_layer(W.data_ptr(), m, n, n, H.data_ptr(), A.data_ptr(), n, dead.data_ptr(), 4, 16, 0, 128,
                                        codes.data_ptr(), scales.data_ptr(), zeros.data_ptr(), wq.data_ptr(), wq.numel(), s) == 0

    out = (H, A, W, codes, scales, zeros, info)
    solve()
    torch.cuda.synchronize()
    eager = [t.clone() for t in out]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        solve()
    for i in range(3):
        for t in out:
            t.fill_(i)
        wp.fill_(255), wq.fill_(255)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(out, eager):
            assert torch.equal(a, b)
        solve()


# Sums taken in several parts of the tokens (few columns, many tokens): one tile and its edge, several tiles, k-tiles that do not divide
# over the parts, most and fewest parts; in a workspace of the operands alone they are taken in one part.  The diagonal of H, which
# act_order ranks by, has the bits of one part (8320 tokens: its loads' last round is a whole one).
@pytest.mark.parametrize("n,ld,tokens", [(8, 8, 8192), (136, 140, 8200), (264, 264, 8320), (392, 392, 10016), (1032, 1040, 16448), (1536, 1536, 32768)])
def test_sums_in_parts_are_the_sums(n, ld, tokens):
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((tokens, n), device="cuda", generator=g).bfloat16()
    Xt = (X.float() + 0.05 * torch.randn((tokens, n), device="cuda", generator=g)).bfloat16()
    start = torch.randn((n, n), device="cuda", generator=g)
    size = B.gptaq_accumulate_workspace_bytes(tokens, n)
    operands = 6 * -(-n // 128) * 128 * (-(-tokens // 64) * 64)
    assert size > operands
    out = {}
    for name, nb, call in (("full", size, B.gptaq_accumulate), ("upper", size, B.gptaq_accumulate_upper), ("one part", operands, B.gptaq_accumulate)):
        whole = [torch.full((n, ld), -7.0, device="cuda") for _ in range(2)]
        H, A = whole[0][:, :n], whole[1][:, :n]
        H.copy_(start)
        A.copy_(start)
        call(X, Xt, H, A, B.workspace(nb))
        torch.cuda.synchronize()
        assert ld == n or (whole[0][:, n:] == -7.0).all() and (whole[1][:, n:] == -7.0).all()
        out[name] = (H.triu(), A.triu() if name == "upper" else A.clone())
    assert torch.equal(out["full"][0], out["upper"][0]) and torch.equal(out["full"][1].triu(), out["upper"][1])
    assert torch.equal(out["full"][0].diagonal(), out["one part"][0].diagonal())
    assert n < 128 or not torch.equal(out["full"][1], out["one part"][1])          # (the parts were taken)
    Xd, Dd = X.double(), Xt.double() - X.double()
    refs = ((start.double() + Xd.T.contiguous() @ Xd).triu(), start.double() + Dd.T.contiguous() @ Xd)
    for name in ("full", "one part"):
        for got, ref in zip(out[name], refs):
            # fp32 sums of exact products: sqrt(tokens) 2^-24 = 1.1e-5 at most if every addition rounded the whole sum alike; 9e-7 seen
            assert float((got.double() - ref).norm() / ref.norm()) <= 3e-6


# The same with few tokens: the fewest of a size that are taken in parts, k-tiles that do not divide over them, a part of few k-tiles.
@pytest.mark.parametrize("n,ld,tokens", [(8, 8, 4160), (584, 592, 2080), (512, 520, 6000), (776, 776, 4100), (1280, 1280, 6000)])
def test_sums_in_parts_of_few_tokens(n, ld, tokens):
    test_sums_in_parts_are_the_sums(n, ld, tokens)


# The range of a whole row: candidates go through it eight at a time.  One, a few, a whole number of eights and a remainder; rows shorter than a
# wavefront and not a multiple of one; dead columns, which count as 0 whatever they hold.
@pytest.mark.parametrize("m,n,grid,steps,sym", [(3, 40, 100, 1, False), (65, 72, 100, 7, True), (130, 200, 100, 16, False), (31, 264, 60, 45, False), (200, 520, 100, 80, True)])
def test_row_range_search(m, n, grid, steps, sym):
    rng = np.random.default_rng(n)
    W = rng.standard_normal((m, n)).astype(np.float32)
    dead = np.zeros(n, np.uint8)
    dead[5::37] = 1
    alive = np.where(dead, np.float32(0), W)
    W[:, dead == 1] = 9.0
    got = PU.gpu_quantize(W, dev(np.eye(n)), None, 4, 0, sym, 128, dead=dev(dead).to(torch.uint8), terms=0, mse=(grid, steps))
    rows = torch.from_numpy(alive).double().numpy()
    lo, hi = np.minimum(rows.min(1), 0), np.maximum(rows.max(1), 0)
    if sym:
        hi = np.maximum(-lo, hi)
        lo = -hi
    base = (hi - lo) / 15
    zero = np.full(m, 8.0) if sym else np.rint(-lo / base.astype(np.float32))
    scale = np.stack([((1 - i / grid) * base).astype(np.float32) for i in range(steps)])            # (steps, m)
    q = np.clip(np.rint(rows[None] / scale[:, :, None].astype(np.float64)) + zero[None, :, None], 0, 15)
    err = (((q - zero[None, :, None]) * scale[:, :, None] - rows[None]) ** 2).sum(2)
    mine = got["scales"].reshape(m)
    at = np.abs(scale - mine[None]).argmin(0)
    assert np.array_equal(scale[at, np.arange(m)], mine) and np.array_equal(got["zeros"].reshape(m), zero)
    # an fp32 sum of n squares against the exact one: n 2^-24 at most of each of the two compared, and x / scale by a reciprocal may take an entry on a
    # boundary the other way, which changes nothing to first order
    assert (err[at, np.arange(m)] <= err.min(0) * (1 + 2 * n * 2.0 ** -24 + 1e-6)).all()


# Blocks of 32 x 64 with an eighth of the tokens to a wavefront: one block and its edges, an odd number of block rows, the most columns; k-tiles for a
# few wavefronts only, that do not divide over them, the most.  They need the operands' workspace and no more.
@pytest.mark.parametrize("n,ld,tokens", [(8, 8, 1), (40, 48, 64), (72, 72, 200), (136, 140, 1100), (264, 264, 330), (512, 512, 4096), (552, 560, 2048), (576, 576, 4090)])
def test_sums_of_narrow_inputs(n, ld, tokens):
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((tokens, n), device="cuda", generator=g).bfloat16()
    Xt = (X.float() + 0.05 * torch.randn((tokens, n), device="cuda", generator=g)).bfloat16()
    start = torch.randn((n, n), device="cuda", generator=g)
    size = B.gptaq_accumulate_workspace_bytes(tokens, n)
    assert size == 6 * -(-n // 128) * 128 * (-(-tokens // 64) * 64)
    Xd, Dd = X.double(), Xt.double() - X.double()
    refs = ((start.double() + Xd.T.contiguous() @ Xd).triu(), start.double() + Dd.T.contiguous() @ Xd)
    out = []
    for call in (B.gptaq_accumulate, B.gptaq_accumulate_upper):
        whole = [torch.full((n + 1, ld), -7.0, device="cuda") for _ in range(2)]
        H, A = whole[0][:n, :n], whole[1][:n, :n]
        H.copy_(start)
        A.copy_(start)
        call(X, Xt, H, A, B.workspace(size))
        assert all((w[n:] == -7.0).all() and (w[:, n:] == -7.0).all() for w in whole)
        out.append((H.triu(), A.clone()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1].triu(), out[1][1].triu())
    for got, ref in zip(out[0], refs):
        assert float((got.double() - ref).norm() / ref.norm()) <= 3e-6          # (as in test_sums_in_parts_are_the_sums)


@pytest.mark.parametrize("n", [40, 328, 576])
@pytest.mark.parametrize("upper", [False, True])
def test_staged_sums_of_narrow_inputs(n, upper):
    """Small chunks, the last one ragged, are the sums of one call, bit for bit, and so are those in the library's own workspace."""
    ws = B.workspace(B.gptaq_accumulate_workspace_bytes(32768, n))
    ws.fill_(0xff)                         # (what the calls do not write is not read as numbers)
    cuts = [0, 64, 192, 1216, 1301]
    X, Xt = synth.make_activations_device(cuts[-1], n, 1, "x", "cuda", noise=0.2)
    H, A, Hs, As, Hn, An = (torch.ones((n, n), device="cuda") for _ in range(6))
    (B.gptaq_accumulate_upper if upper else B.gptaq_accumulate)(X, Xt, H, A, B.workspace(B.gptaq_accumulate_workspace_bytes(cuts[-1], n)))
    pending = 0
    for t0, t1 in zip(cuts, cuts[1:]):
        pending = B.gptaq_accumulate_staged(X[t0:t1], Xt[t0:t1], Hs, As, ws, pending, flush=t1 == cuts[-1], upper=upper)
    assert pending == 0
    assert torch.equal(H.triu(), Hs.triu())
    assert torch.equal(A.triu(), As.triu()) and (upper or torch.equal(A, As))
    B.gptaq_accumulate_noalloc(X, Xt, Hn, An)
    assert torch.equal(H.triu(), Hn.triu()) and torch.equal(A.triu(), An.triu()) and (upper or torch.equal(A, An))


@pytest.mark.parametrize("n", [40, 328, 576])
def test_sums_of_narrow_inputs_that_are_not_finite(n):
    """An infinity in X, one in X~ and a NaN in X~: the entries that are not finite are those of the exact sums, and the others are what they should be."""
    tokens = 300
    X, Xt = synth.make_activations_device(tokens, n, 6, "x", "cuda", noise=0.2)
    X[70, 4], Xt[271, 21], Xt[3, n - 1] = float("inf"), float("-inf"), float("nan")
    Xd, Dd = X.double(), Xt.double() - X.double()
    refs = (Xd.T.contiguous() @ Xd, Dd.T.contiguous() @ Xd)
    ws = B.workspace(B.gptaq_accumulate_workspace_bytes(tokens, n))
    for upper in (False, True):
        H, A = torch.zeros((n, n), device="cuda"), torch.zeros((n, n), device="cuda")
        (B.gptaq_accumulate_upper if upper else B.gptaq_accumulate)(X, Xt, H, A, ws)
        for got, ref, tri in ((H, refs[0], True), (A, refs[1], upper)):
            keep = torch.ones_like(got, dtype=torch.bool).triu() if tri else torch.ones_like(got, dtype=torch.bool)
            assert torch.equal(got.isfinite() & keep, ref.isfinite() & keep)
            keep &= ref.isfinite()
            # (fp32 sums of 300 exact products: sqrt(300) 2^-24 if every addition rounded the whole sum alike)
            assert float((got[keep].double() - ref[keep]).norm() / ref[keep].norm()) <= 2.0 ** -24 * tokens ** 0.5


@pytest.mark.parametrize("n,tokens", [(264, 8192), (520, 16448), (1032, 32768)])
def test_sums_in_parts_round_the_total_once(n, tokens):
    """Whole numbers, whose sums are exact in fp32 in any order, on totals of 2^25 (steps of 2 and 4): what a call leaves is the exact
    total rounded once, in parts as in one part."""
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randint(-2, 3, (tokens, n), device="cuda", generator=g).bfloat16()
    D = torch.randint(-1, 2, (tokens, n), device="cuda", generator=g).bfloat16()
    start = (2.0 ** 25 * (0.5 + torch.rand((n, n), device="cuda", generator=g)))
    size = B.gptaq_accumulate_workspace_bytes(tokens, n)
    assert size > 6 * -(-n // 128) * 128 * (-(-tokens // 64) * 64)
    Xd, Dd = X.double(), D.double()
    refs = [(start.double() + S.T.contiguous() @ Xd).float() for S in (Xd, Dd)]
    for call in (B.gptaq_accumulate, B.gptaq_accumulate_upper):
        H, A = start.clone(), start.clone()
        call(X, X + D, H, A, B.workspace(size))
        torch.cuda.synchronize()
        assert torch.equal(H.triu(), refs[0].triu())
        assert torch.equal(A.triu(), refs[1].triu())
        assert call is B.gptaq_accumulate_upper or torch.equal(A, refs[1])


# Two row halves: the lines of the rule by rows and super-blocks, with and without vector stores; 3585 and 1300 rows are two chains, 744 one.
@pytest.mark.parametrize("m,n,group", [(8193, 2064, 0), (4097, 3201, 0), (3585, 5248, 128), (1300, 6784, 64), (760, 10250, 0), (744, 11264, 128), (4097, 5248, 128),
                                       (1025, 8208, 16), (1536, 10250, 0)])
def test_row_halves_equal_separate_calls(m, n, group):
    """Rows are independent: the result is bit for bit that of calls on 600 rows at a time, which are too few for halves."""
    g = torch.Generator(device="cuda").manual_seed(m)
    U = torch.randn((n, n), device="cuda", generator=g).mul_(n ** -0.5).triu_(1)
    U.diagonal().copy_(0.5 + torch.rand(n, device="cuda", generator=g))
    P = torch.randn((n, n), device="cuda", generator=g).mul_(0.1 * n ** -0.5).triu_(1)
    W0 = 0.02 * torch.randn((m, n), device="cuda", generator=g)

    def quantize(W):
        W = W.clone()
        out = B.gptaq_quantize_layer(W, U, P, 4, group, False, 128, B.workspace(B.gptaq_quantize_workspace_bytes(W.shape[0], n)))
        torch.cuda.synchronize()
        return (W, *out)

    whole = quantize(W0)
    parts = [quantize(W0[r:r + 600]) for r in range(0, m, 600)]
    for i, got in enumerate(whole):
        assert torch.equal(got, torch.cat([p[i].reshape(-1, got.shape[1]) for p in parts]))


# So few rows of so wide a matrix that only one half of whole tiles has rows, and the fewest of which both have.
@pytest.mark.parametrize("m,n", [(200, 42000), (256, 32768), (257, 32768)])
def test_few_rows_of_a_wide_matrix(m, n):
    """The result is bit for bit that of calls on 100 rows at a time, and nothing behind the last row is touched."""
    g = torch.Generator(device="cuda").manual_seed(m)
    U, P = torch.empty((n, n), device="cuda"), torch.empty((n, n), device="cuda")
    U.normal_(0, n ** -0.5, generator=g).triu_(1)
    U.diagonal().copy_(0.5 + torch.rand(n, device="cuda", generator=g))
    P.normal_(0, 0.1 * n ** -0.5, generator=g).triu_(1)
    W0 = 0.02 * torch.randn((m, n), device="cuda", generator=g)

    def quantize(W):
        out = [torch.full((W.shape[0] + 256, n), -7.0, device="cuda"), torch.full((W.shape[0] + 256, n), 99, dtype=torch.uint8, device="cuda"),
               *(torch.full((W.shape[0] + 256, 1), -7.0, device="cuda") for _ in range(2))]
        mine = [t[:W.shape[0]] for t in out]
        mine[0].copy_(W)
        B.gptaq_quantize_layer(mine[0], U, P, 4, 0, False, 128, B.workspace(B.gptaq_quantize_workspace_bytes(W.shape[0], n)), codes=mine[1],
                               scales=mine[2], zeros=mine[3])
        torch.cuda.synchronize()
        assert all((t[W.shape[0]:] == v).all() for t, v in zip(out, (-7.0, 99, -7.0, -7.0)))
        return mine

    whole = quantize(W0)
    parts = [quantize(W0[r:r + 100]) for r in range(0, m, 100)]
    for i, got in enumerate(whole):
        assert torch.equal(got, torch.cat([p[i] for p in parts]))


# Two chains (1025 to 4096 rows): the fewest super-blocks and the fewest rows; both sets of the -E / V buffers taken again; each term alone; the columns left
# where the second chain starts at once; and one row fewer, which is one chain.
@pytest.mark.parametrize("m,n,group,terms,far_updates", [(1025, 2064, 0, 3, 3), (1024, 3088, 16, 3, 3), (1025, 3088, 16, 3, 5), (2100, 4112, 0, 1, 7), (2100, 4112, 16, 2, 7),
                                                         (2100, 4112, 16, 3, 7), (2500, 9232, 0, 3, 17), (4096, 5120, 128, 3, 7), (1537, 9232, 16, 3, 17),
                                                         (4096, 6160, 16, 3, 11)])
def test_two_chains_equal_one(m, n, group, terms, far_updates):
    """The result is bit for bit that of calls on 700 rows at a time, which go through as one chain; columns of dead inputs are among them."""
    g = torch.Generator(device="cuda").manual_seed(m)
    U, P = (torch.randn((n, n), device="cuda", generator=g).mul_(f * n ** -0.5).triu_(1) for f in (1.0, 0.1))
    U.diagonal().copy_(0.5 + torch.rand(n, device="cuda", generator=g))
    W0 = 0.02 * torch.randn((m, n), device="cuda", generator=g)
    dead = torch.zeros(n, dtype=torch.uint8, device="cuda")
    dead[7::501] = 1
    W0[:, 7::501] = 5.0
    tag = B.PROFILE_TAGS.index("trailing_gemm")

    def quantize(W, launches):
        W = W.clone()
        B.gptaq_profile_enable(1 << tag)
        out = B.gptaq_quantize_layer(W, U, P, 4, group, False, 128, B.workspace(B.gptaq_quantize_workspace_bytes(W.shape[0], n)), dead=dead, terms=terms)
        assert B.gptaq_profile_read(tag)[0] == launches
        B.gptaq_profile_enable(0)
        torch.cuda.synchronize()
        return (W, *out)

    whole = quantize(W0, far_updates)
    parts = [quantize(W0[r:r + 700], (n - 1) // 1024) for r in range(0, m, 700)]
    for i, got in enumerate(whole):
        assert torch.equal(got, torch.cat([p[i].reshape(-1, got.shape[1]) for p in parts]))


# Row halves that make the super-block kernel's operands for themselves, against calls on 600 rows at a time, which are one chain.
@pytest.mark.parametrize("n,terms,steps", [(2064, 1, 0), (3200, 2, 0), (3072, 3, 5)])
def test_row_halves_with_operands_of_their_own(n, terms, steps):
    m, group = 10300, 64 if steps else 0
    g = torch.Generator(device="cuda").manual_seed(n)
    U, P = (torch.randn((n, n), device="cuda", generator=g).mul_(f * n ** -0.5).triu_(1) for f in (1.0, 0.1))
    U.diagonal().copy_(0.5 + torch.rand(n, device="cuda", generator=g))
    W0 = 0.02 * torch.randn((m, n), device="cuda", generator=g)

    def quantize(W):
        W = W.clone()
        out = B.gptaq_quantize_layer(W, U, P, 4, group, False, 128, B.workspace(B.gptaq_quantize_workspace_bytes(W.shape[0], n)), terms=terms,
                                     mse_grid=8 if steps else 0, mse_steps=steps)
        torch.cuda.synchronize()
        return (W, *out)

    whole = quantize(W0)
    parts = [quantize(W0[r:r + 600]) for r in range(0, m, 600)]
    for i, got in enumerate(whole):
        assert torch.equal(got, torch.cat([p[i].reshape(-1, got.shape[1]) for p in parts]))


def test_super_block_kernel_finds_its_operands_in_the_caches():
    """Behind the far updates of a large layer a super-block takes little longer than alone (1.17 times as long when this was written,
    1.66 with operands made for all super-blocks in front of the first)."""
    m, us = 8192, {}
    for n in (1024, 8192):
        U = torch.eye(n, device="cuda")
        W0 = 0.02 * torch.randn((m, n), device="cuda")
        ws = B.workspace(B.gptaq_quantize_workspace_bytes(m, n))
        times = []
        for _ in range(5):
            W = W0.clone()
            B.gptaq_profile_enable(1 << 4)
            B.gptaq_quantize_layer(W, U, None, 4, 128, False, 128, ws, terms=1)
            launches, ms = B.gptaq_profile_read(4)
            B.gptaq_profile_enable(0)
            assert launches == n // 1024
            times.append(1e3 * ms / launches)
        us[n] = min(times)
    assert us[8192] <= 1.4 * us[1024], us


def test_first_super_block_finds_its_operands_in_the_caches():
    """So does the first one: its operands are made behind the far updates'.  The eight launches of 8192 columns take 1.22 to 1.24 times as long
    as one alone, with the first one's operands driven out of the caches 1.30 to 1.31 times."""
    m, us = 8192, {}
    for n in (1024, 8192):
        U = torch.eye(n, device="cuda")
        W0 = 0.02 * torch.randn((m, n), device="cuda")
        ws = B.workspace(B.gptaq_quantize_workspace_bytes(m, n))
        times = []
        for _ in range(9):
            W = W0.clone()
            B.gptaq_profile_enable(1 << 4)
            B.gptaq_quantize_layer(W, U, None, 4, 128, False, 128, ws, terms=1)
            launches, ms = B.gptaq_profile_read(4)
            B.gptaq_profile_enable(0)
            assert launches == n // 1024
            times.append(1e3 * ms / launches)
        us[n] = min(times)
    assert us[8192] <= 1.28 * us[1024], us


# A launch of operands for each super-block and one for the far updates; a layer's first launch counts among them where it makes operands and
# nothing else that matters.
@pytest.mark.parametrize("n,group,terms,steps,launches", [(512, 128, 3, 0, 1), (2048, 128, 1, 0, 3), (2048, 0, 3, 0, 2), (512, 0, 3, 80, 0), (512, 0, 0, 0, 0), (512, 128, 0, 0, 0)])
def test_operands_are_timed_without_the_ranges(n, group, terms, steps, launches):
    m = 64
    W, ws = torch.randn((m, n), device="cuda"), B.workspace(B.gptaq_quantize_workspace_bytes(m, n))
    dead = torch.zeros(n, dtype=torch.uint8, device="cuda")
    B.gptaq_profile_enable(1 << B.PROFILE_TAGS.index("trailing_split"))
    B.gptaq_quantize_layer(W, torch.eye(n, device="cuda"), torch.zeros((n, n), device="cuda"), 4, group, False, 128, ws, dead=dead, terms=terms,
                           mse_grid=100 if steps else 0, mse_steps=steps)
    got = B.gptaq_profile_read(B.PROFILE_TAGS.index("trailing_split"))[0]
    B.gptaq_profile_enable(0)
    assert got == launches


@pytest.mark.parametrize("n,tokens", [(1928, 1), (1928, 2080), (2048, 96), (2496, 97), (3848, 64), (4104, 500)])
@pytest.mark.parametrize("kind", ["near", "far", "all", "rows"])
def test_sparse_remainder_of_the_difference(n, tokens, kind):
    """dXXT from remainders that few, some, all or the odd rows' entries have: the blocks of the sparse operand are of either form,
    alone and side by side.  (n = 1928: the fewest columns that take it; 3848: 256-tiles with a ragged edge.)"""
    g = torch.Generator(device="cuda")
    g.manual_seed(n + tokens)
    X = torch.randn((tokens, n), device="cuda", generator=g)
    e = torch.randn((tokens, n), device="cuda", generator=g)
    if kind in ("all", "rows"):            # |X| far below |dX|: hardly an entry of dX fits 8 bits
        small = torch.arange(n, device="cuda") % 2 if kind == "rows" else torch.ones(n, device="cuda")
        X, Xt = torch.where(small > 0, X * 2.0 ** -7, X).to(torch.bfloat16), e.to(torch.bfloat16)
    else:
        X, Xt = X.to(torch.bfloat16), (X + {"near": 0.05, "far": 0.2}[kind] * e).to(torch.bfloat16)
    H = torch.zeros((n, n), device="cuda")
    A, Au = torch.zeros_like(H), torch.zeros_like(H)
    ws = B.workspace(B.gptaq_accumulate_workspace_bytes(tokens, n))
    ws.fill_(0xff)                         # (what the call does not write is not read as numbers)
    B.gptaq_accumulate(X, Xt, H, A, ws)
    B.gptaq_accumulate_upper(X, Xt, torch.zeros_like(H), Au, ws)
    ref = (Xt.double() - X.double()).T @ X.double()
    assert torch.equal(A.triu(), Au.triu())
    # products are exact in fp32; the sum of a chain of tokens / 16 steps, three a k-tile, errs by about 2^-24 sqrt(steps) of itself
    # (the remainders themselves are 5e-4 of dXXT and more)
    bound = 2.0 ** -24 * max(4.0, (tokens / 8) ** 0.5)
    err = float((A.double() - ref).norm() / ref.norm())
    assert err <= bound, (err, bound)


def test_sparse_remainder_where_nothing_differs():
    X = torch.randn((300, 2056), device="cuda").to(torch.bfloat16)
    H = torch.zeros((2056, 2056), device="cuda")
    A = torch.zeros_like(H)
    B.gptaq_accumulate(X, X.clone(), H, A, B.workspace(B.gptaq_accumulate_workspace_bytes(300, 2056)))
    assert not bool(A.any()) and bool(H.any())


@pytest.mark.parametrize("n,tokens", [(3848, 1024), (4096, 2100)])
def test_quarters_of_the_last_tiles_have_the_bits_of_whole_ones(n, tokens):
    """The upper form of 16 tile rows has 16 tiles more than the chip has CUs and takes them as quarters; the full form has them whole."""
    X, Xt = synth.make_activations_device(tokens, n, 5, "x", "cuda")
    ws = B.workspace(B.gptaq_accumulate_workspace_bytes(tokens, n))
    Hf, Hu = torch.ones((n, n), device="cuda"), torch.ones((n, n), device="cuda")
    Af, Au = torch.ones_like(Hf), torch.ones_like(Hf)
    B.gptaq_accumulate(X, Xt, Hf, Af, ws)
    B.gptaq_accumulate_upper(X, Xt, Hu, Au, ws)
    assert torch.equal(Hf.triu(), Hu.triu()) and torch.equal(Af.triu(), Au.triu())
    ref = X.double().T @ X.double() + 1.0
    err = float((Hu.double() - ref).triu().norm() / ref.triu().norm())
    assert err <= 2.0 ** -24 * (tokens / 8) ** 0.5, err        # (a chain of tokens / 16 steps)


@pytest.mark.parametrize("n,tokens", [(1928, 96), (2496, 2080), (3848, 224), (4104, 512)])
@pytest.mark.parametrize("one_in", [9, 3])
def test_sparse_remainder_with_blocks_that_have_none_among_dense_ones(n, tokens, one_in):
    """One 32 x 32 block in nine, or in three, has no difference at all and the others no entry that fits 8 bits: with one in nine lo2 is
    taken for every block, with zeros in the place of those that have none; the first and the last k-tiles are among them."""
    g = torch.Generator(device="cuda").manual_seed(n)
    X = (2.0 ** -7 * torch.randn((tokens, n), device="cuda", generator=g)).to(torch.bfloat16)
    e = torch.randn((tokens, n), device="cuda", generator=g).to(torch.bfloat16)
    block = torch.arange(tokens, device="cuda")[:, None] // 32 + torch.arange(n, device="cuda")[None, :] // 32
    Xt = torch.where(block % one_in == 0, X, e)
    H = torch.zeros((n, n), device="cuda")
    A, Au = torch.zeros_like(H), torch.zeros_like(H)
    ws = B.workspace(B.gptaq_accumulate_workspace_bytes(tokens, n))
    ws.fill_(0xff)                         # (what the call does not write is not read as numbers)
    B.gptaq_accumulate(X, Xt, H, A, ws)
    ws.fill_(0xff)
    B.gptaq_accumulate_upper(X, Xt, torch.zeros_like(H), Au, ws)
    assert torch.equal(A.triu(), Au.triu())
    ref = (Xt.double() - X.double()).T @ X.double()
    # (bound: see test_sparse_remainder_of_the_difference)
    err = float((A.double() - ref).norm() / ref.norm())
    assert err <= 2.0 ** -24 * max(4.0, (tokens / 8) ** 0.5), err


def _accumulate_us(call, n, tokens, noise, repeats=5):
    X, Xt = synth.make_activations_device(tokens, n, 7, "x", "cuda", noise=noise)
    H = torch.zeros((n, n), device="cuda")
    A = torch.zeros_like(H)
    ws = B.workspace(B.gptaq_accumulate_workspace_bytes(tokens, n))
    times = []
    for _ in range(repeats + 2):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        call(X, Xt, H, A, ws)
        t1.record()
        torch.cuda.synchronize()
        times.append(1e3 * t0.elapsed_time(t1))
    return min(times[2:])


def test_dense_remainder_costs_what_its_products_cost():
    """Where every block of the remainder is dense, a tile of dXXT takes 2 units of products instead of 1.5 and 50 KB instead of 42 per
    k-tile, and H 1 and 32 either way: 1.2 times the time, as measured.  What finds its positions costs nothing beside that
    (taken from words of lo2 it was 1.5 times)."""
    assert _accumulate_us(B.gptaq_accumulate_upper, 4096, 32768, 0.5) <= 1.3 * _accumulate_us(B.gptaq_accumulate_upper, 4096, 32768, 0.001)


def test_reordered_inputs_cost_what_others_do():
    """gptaq_accumulate_upper_permuted fetches all of lo, 48 KB a k-tile of a tile of dXXT instead of 41, which is 1.17 times, and writes
    its operands to scattered rows, 5 % more (1.13 measured; with every block taken as a dense one it was 1.45 times)."""
    inv = torch.randperm(4096, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1)).int()
    permuted = lambda X, Xt, H, A, ws: B.gptaq_accumulate_upper_permuted(X, Xt, inv, H, A, ws)
    assert _accumulate_us(permuted, 4096, 32768, 0.05) <= 1.3 * _accumulate_us(B.gptaq_accumulate_upper, 4096, 32768, 0.05)


@pytest.mark.parametrize("n,tokens", [(1928, 96), (2496, 2080), (3848, 224)])
@pytest.mark.parametrize("kind", ["near", "far", "patches"])
def test_sparse_remainder_of_reordered_inputs(n, tokens, kind):
    """Rows of dense and of sparse blocks lie among each other; the sums are those of the other forms, bit for bit."""
    g = torch.Generator(device="cuda").manual_seed(n + 1)
    X = torch.randn((tokens, n), device="cuda", generator=g).to(torch.bfloat16)
    e = torch.randn((tokens, n), device="cuda", generator=g)
    Xt = (X.float() + {"near": 0.05, "far": 0.5, "patches": 0.5}[kind] * e).to(torch.bfloat16)
    if kind == "patches":
        block = torch.arange(tokens, device="cuda")[:, None] // 32 + torch.arange(n, device="cuda")[None, :] // 32
        Xt = torch.where(block % 3 == 0, Xt, X)
    inv = torch.randperm(n, device="cuda", generator=g).int()
    perm = torch.argsort(inv)
    ws = B.workspace(B.gptaq_accumulate_workspace_bytes(tokens, n))
    H, A, Hp, Ap = (torch.zeros((n, n), device="cuda") for _ in range(4))
    ws.fill_(0xff)
    B.gptaq_accumulate(X, Xt, H, A, ws)
    ws.fill_(0xff)
    B.gptaq_accumulate_upper_permuted(X, Xt, inv, Hp, Ap, ws)
    H = torch.triu(H) + torch.triu(H, 1).T
    assert torch.equal(Hp.triu(), H[perm][:, perm].triu()) and torch.equal(Ap.triu(), A[perm][:, perm].triu())


@pytest.mark.parametrize("n", [1928, 3848])
@pytest.mark.parametrize("upper", [False, True])
def test_staged_sums_with_the_sparse_remainder(n, upper):
    """Small chunks, the last one ragged, are the sums of one call, bit for bit; then another series in the same workspace, whose dense blocks are
    others."""
    ws = B.workspace(B.gptaq_accumulate_workspace_bytes(32768, n))
    call = B.gptaq_accumulate_upper if upper else B.gptaq_accumulate
    for seed, noise in ((1, 0.5), (2, 0.05)):
        cuts = [0, 128, 192, 384, 461]
        X, Xt = synth.make_activations_device(cuts[-1], n, seed, "x", "cuda", noise=noise)
        H, A, Hs, As = (torch.zeros((n, n), device="cuda") for _ in range(4))
        call(X, Xt, H, A, B.workspace(B.gptaq_accumulate_workspace_bytes(cuts[-1], n)))
        pending = 0
        for t0, t1 in zip(cuts, cuts[1:]):
            pending = B.gptaq_accumulate_staged(X[t0:t1], Xt[t0:t1], Hs, As, ws, pending, flush=t1 == cuts[-1], upper=upper)
        assert pending == 0
        assert torch.equal(H.triu(), Hs.triu())
        assert torch.equal(A.triu(), As.triu()) and (upper or torch.equal(A, As))


@pytest.mark.parametrize("n,tokens", [(1928, 700), (3848, 1500)])
def test_sums_in_the_library_s_own_workspace_with_the_sparse_remainder(n, tokens):
    X, Xt = synth.make_activations_device(tokens, n, 4, "x", "cuda", noise=0.1)
    H, A, Hn, An = (torch.zeros((n, n), device="cuda") for _ in range(4))
    B.gptaq_accumulate(X, Xt, H, A, B.workspace(32 << 20))
    B.gptaq_accumulate_noalloc(X, Xt, Hn, An)
    assert torch.equal(H.triu(), Hn.triu()) and torch.equal(A, An)


@pytest.mark.parametrize("n", [1928, 3848])
@pytest.mark.parametrize("noise", [0.05, 0.5])
def test_sparse_remainder_of_what_is_not_finite(n, noise):
    """An infinity in X, one in X~ and a NaN in X~: the entries that are not finite are those of the exact sums, in every form, and the others are
    what they should be.  (An entry is infinite or NaN as the products come: zeros of the remainder are not multiplied.)"""
    tokens = 200
    X, Xt = synth.make_activations_device(tokens, n, 6, "x", "cuda", noise=noise)
    X[70, 40], Xt[71, 130], Xt[3, 1500] = float("inf"), float("-inf"), float("nan")
    Xd, Dd = X.double(), Xt.double() - X.double()
    refs = (Xd.T.contiguous() @ Xd, Dd.T.contiguous() @ Xd)
    bound = 2.0 ** -24 * max(4.0, (tokens / 8) ** 0.5)
    ws = B.workspace(B.gptaq_accumulate_workspace_bytes(tokens, n))
    inv = torch.randperm(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(n)).int()
    perm = torch.argsort(inv)
    for form in ("full", "upper", "permuted"):
        H, A = torch.zeros((n, n), device="cuda"), torch.zeros((n, n), device="cuda")
        if form == "permuted":
            B.gptaq_accumulate_upper_permuted(X, Xt, inv, H, A, ws)
        else:
            (B.gptaq_accumulate if form == "full" else B.gptaq_accumulate_upper)(X, Xt, H, A, ws)
        for got, ref, tri in ((H, refs[0], True), (A, refs[1], form != "full")):
            if form == "permuted":
                ref = ref[perm][:, perm]
            keep = torch.ones_like(got, dtype=torch.bool).triu() if tri else torch.ones_like(got, dtype=torch.bool)
            assert torch.equal(got.isfinite() & keep, ref.isfinite() & keep)
            keep &= ref.isfinite()
            assert float((got[keep].double() - ref[keep]).norm() / ref[keep].norm()) <= bound


@pytest.mark.parametrize("n,tokens", [(3848, 1), (4096, 64), (3976, 200)])
def test_quarters_of_the_last_tiles_with_few_tokens(n, tokens):
    X, Xt = synth.make_activations_device(tokens, n, 5, "x", "cuda")
    ws = B.workspace(B.gptaq_accumulate_workspace_bytes(tokens, n))
    Hf, Hu, Af, Au = (torch.ones((n, n), device="cuda") for _ in range(4))
    B.gptaq_accumulate(X, Xt, Hf, Af, ws)
    B.gptaq_accumulate_upper(X, Xt, Hu, Au, ws)
    assert torch.equal(Hf.triu(), Hu.triu()) and torch.equal(Af.triu(), Au.triu())

"""Performance cases of the GPTAQ per-layer solve: the calls that a calibration program makes, layer after layer.

A case names one of the four kinds of work and its sizes:

  solve       the whole chain for one linear layer: sums over the calibration tokens, factors, column loop; with
              `act_bits` the activations are fake-quantised first, with `act_order` the columns are reordered, with
              `pack` the codes are packed
  accumulate  H and dXXT over `tokens` calibration tokens, handed over `chunk` tokens at a time
  prepare     U and P from H and dXXT
  quantize    the column loop of an m x n layer (or of several that share an input, stacked) on given U and P

Activations and weights follow paper_2504_02692_amd/synth.py (N(0,1) activations with a few outlier channels, weights
N(0, 0.02^2)).  The calls work in place; a pass starts from the same inputs every time, so run() first restores what
the last pass overwrote, as a program does that copies a layer's weights into its work buffer.
"""
import torch

from paper_2504_02692_amd import binding as B
from paper_2504_02692_amd import synth

DAMP = 0.01
BLOCKSIZE = 128


def _solve(name, m, n, tokens, bits, group, sym=False, act_order=False, act_bits=0, pack=False):
    return dict(name=name, kind="solve", m=m, n=n, tokens=tokens, bits=bits, group=group, sym=sym, act_order=act_order,
                act_bits=act_bits, pack=pack)


def _accumulate(name, n, tokens, chunk, form):
    return dict(name=name, kind="accumulate", n=n, tokens=tokens, chunk=chunk, form=form)


def _prepare(name, n):
    return dict(name=name, kind="prepare", n=n)


def _quantize(name, m, n, bits, group, sym=False, mse_steps=0):
    return dict(name=name, kind="quantize", m=m, n=n, bits=bits, group=group, sym=sym, mse_steps=mse_steps)


def listed():
    return [
        # a single small layer, 4-bit per-channel: launches and latency count (the first workload of the benchmark)
        _solve("solve_512", 512, 512, 4096, 4, 0),
        # the qkv layer of a ViT-L block on 128 images x 257 tokens, 4-bit per-channel symmetric, activations quantised,
        # columns reordered, codes packed: every neighbour of the solve takes part
        _solve("solve_vit_qkv_act_order", 3072, 1024, 32896, 4, 0, True, True, 4, True),
        # one calibration sample of 2048 tokens per call, as a forward hook hands it over
        _accumulate("accumulate_sample_4096", 4096, 2048, 2048, "upper"),
        # sixteen such samples through the staged calls
        _accumulate("accumulate_staged_4096", 4096, 32768, 2048, "staged_upper"),
        # every entry of dXXT (act_order in one pass), a width that fills no tile, a token count that fills no pass
        _accumulate("accumulate_full_2736", 2736, 32896, 32896, "full"),
        # the widest input of a Llama-2-7B block, samples concatenated to 32768 tokens a call
        _accumulate("accumulate_11008", 11008, 65536, 32768, "upper"),
        # factors of the attention and of the MLP-down input of that block
        _prepare("prepare_4096", 4096),
        _prepare("prepare_11008", 11008),
        # its layers: o_proj; gate and up stacked (they share an input); down_proj; W4 in groups of 128
        _quantize("quantize_4096x4096", 4096, 4096, 4, 128),
        _quantize("quantize_22016x4096", 22016, 4096, 4, 128),
        _quantize("quantize_4096x11008", 4096, 11008, 4, 128),
        # the clipping range of every group searched by squared error, the customary grid 100 with 80 steps
        _quantize("quantize_clip_4096x4096", 4096, 4096, 4, 128, False, 80),
    ]


def _log(rng, lo, hi, step):
    """A multiple of `step` between lo and hi, spread over the logarithm."""
    v = lo * (hi / lo) ** rng.random()
    return max(lo, min(hi, int(round(v / step)) * step))


# The drawn cases keep to 4 bits, and to symmetric grids per channel only.  An entry that lies on a rounding boundary may go
# either way in two correct implementations, and the compensation carries the step to the later columns of its row; with
# 2 or 3 bits one such step is as large as the weights' own deviation, and in a symmetric group the largest entry always lies
# on a boundary, so results of these could only be compared entry by entry against the near-tie rule of the tests.
def draw(rng):
    kind = rng.choice(("solve", "accumulate", "accumulate", "prepare", "quantize", "quantize"))
    if kind == "solve":
        group = rng.choice((0, 64, 128))
        n = _log(rng, 512, 2816, group if group else 8)
        order = rng.random() < 0.3
        return _solve("", _log(rng, 256, 4096, 1), n, _log(rng, 4096, 32896, 1), 4, group, group == 0 and rng.random() < 0.5,
                      order, rng.choice((0, 4)), rng.random() < 0.5)
    if kind == "accumulate":
        n = _log(rng, 512, 11008, 8)
        form = rng.choice(("upper", "upper", "full", "staged_upper"))
        most = min(65536, int(11008 * 11008 * 65536 / (n * n)) // (2 if form == "full" else 1))
        tokens = _log(rng, 256, most, 1)
        chunk = 2048 if form == "staged_upper" else min(tokens, rng.choice((2048, 32768, 32768)))
        return _accumulate("", n, tokens, chunk, form)
    if kind == "prepare":
        return _prepare("", _log(rng, 512, 11008, 8))
    group = rng.choice((0, 64, 128, 128))
    n = _log(rng, 512, 11008, group if group else 8)
    m = _log(rng, 256, min(22016, int(22016 * 4096 * 4096 / (n * n))), 1)
    clip = rng.random() < 0.25
    if clip:
        m, n = min(m, 4096), _log(rng, 512, 4096, group if group else 8)
    return _quantize("", m, n, 4, group, group == 0 and rng.random() < 0.5, 80 if clip else 0)


def _sums(n, tokens, seed):
    """H and dXXT of a layer input (upper triangles of the sums), as a calibration program has them."""
    X, Xt = synth.make_activations_device(tokens, n, seed, "x", "cuda")
    H = torch.zeros((n, n), device="cuda")
    A = torch.zeros_like(H)
    B.gptaq_accumulate_upper(X, Xt, H, A, B.workspace(B.gptaq_accumulate_workspace_bytes(tokens, n)))
    return H, A.triu_()


def _calibration_tokens(n):
    return max(4096, min(32768, 4 * n))


def prepare(case, seed):
    n, kind = case["n"], case["kind"]
    s = {"case": case}
    if kind in ("solve", "accumulate"):
        s["X"], s["Xt"] = synth.make_activations_device(case["tokens"], n, seed, "x", "cuda")
        s["H"], s["A"] = torch.empty((n, n), device="cuda"), torch.empty((n, n), device="cuda")
        per_call = 32768 if case.get("form") == "staged_upper" else case.get("chunk", 32768)
        s["ws_acc"] = B.workspace(B.gptaq_accumulate_workspace_bytes(min(per_call, case["tokens"])
                                                                     if case.get("form") != "staged_upper" else per_call, n))
    if kind == "prepare":
        s["H0"], s["A0"] = _sums(n, _calibration_tokens(n), seed)
        s["H"], s["A"] = torch.empty_like(s["H0"]), torch.empty_like(s["A0"])
    if kind in ("solve", "prepare"):
        s["ws_prep"] = B.workspace(B.gptaq_prepare_workspace_bytes(n))
        s["dead"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        s["info"] = torch.empty(2, dtype=torch.int32, device="cuda")
    if case.get("act_order"):
        s["ws_perm"] = B.workspace(B.gptaq_permute_hessian_workspace_bytes(n))
    if kind == "quantize":
        s["U"], s["P"] = _sums(n, _calibration_tokens(n), seed)
        s["dead"], _ = B.gptaq_prepare(s["U"], s["P"], DAMP, B.workspace(B.gptaq_prepare_workspace_bytes(n)))
    if kind in ("solve", "quantize"):
        m, g = case["m"], max(1, n // case["group"]) if case["group"] > 0 else 1
        s["W0"] = synth.make_weights_device(m, n, seed, "w", "cuda")
        s["W"] = torch.empty_like(s["W0"])
        s["codes"] = torch.empty((m, n), dtype=torch.uint8, device="cuda")
        s["scales"], s["zeros"] = torch.empty((m, g), device="cuda"), torch.empty((m, g), device="cuda")
        s["ws_q"] = B.workspace(B.gptaq_quantize_workspace_bytes(m, n))
    return s


def _run_accumulate(s, X):
    case, H, A = s["case"], s["H"], s["A"]
    H.zero_()
    A.zero_()
    tokens, form = case["tokens"], case.get("form", "full" if case.get("act_order") else "upper")
    chunk = case.get("chunk", 32768)
    if form == "staged_upper":
        pending = 0
        for t0 in range(0, tokens, chunk):
            t1 = min(tokens, t0 + chunk)
            pending = B.gptaq_accumulate_staged(X[t0:t1], s["Xt"][t0:t1], H, A, s["ws_acc"], pending, flush=t1 == tokens,
                                                upper=True)
    else:
        call = B.gptaq_accumulate if form == "full" else B.gptaq_accumulate_upper
        for t0 in range(0, tokens, chunk):
            call(X[t0:t0 + chunk], s["Xt"][t0:t0 + chunk], H, A, s["ws_acc"])
    return form


def _run_quantize(s, W, U, P):
    case = s["case"]
    return B.gptaq_quantize_layer(W, U, P, case["bits"], case["group"], case["sym"], BLOCKSIZE, s["ws_q"], dead=s["dead"],
                                  codes=s["codes"], scales=s["scales"], zeros=s["zeros"],
                                  mse_grid=100 if case.get("mse_steps") else 0, mse_steps=case.get("mse_steps", 0))


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "accumulate":
        # what lies below the diagonal of H (and, but for the full form, of dXXT) is unspecified: it is cleared
        form = _run_accumulate(s, s["X"])
        return s["H"].triu_(), s["A"] if form == "full" else s["A"].triu_()
    if kind == "prepare":
        s["H"].copy_(s["H0"])
        s["A"].copy_(s["A0"])
        B.gptaq_prepare(s["H"], s["A"], DAMP, s["ws_prep"], dead=s["dead"], info=s["info"])
        return s["H"], s["A"], s["dead"], s["info"]
    if kind == "quantize":
        s["W"].copy_(s["W0"])
        codes, scales, zeros = _run_quantize(s, s["W"], s["U"], s["P"])
        return s["W"], codes, scales, zeros
    X = B.gptaq_fake_quant_activations(s["X"], case["act_bits"]) if case["act_bits"] else s["X"]
    _run_accumulate(s, X)
    if case["act_order"]:
        perm = B.gptaq_act_order(s["H"])
        B.gptaq_permute_hessian(s["H"], s["A"], perm, s["ws_perm"])
        W = B.gptaq_permute_columns_f32(s["W0"], perm)
    else:
        W = s["W"].copy_(s["W0"])
    B.gptaq_prepare(s["H"], s["A"], DAMP, s["ws_prep"], dead=s["dead"], info=s["info"])
    codes, scales, zeros = _run_quantize(s, W, s["H"], s["A"])
    if case["act_order"]:
        W = B.gptaq_permute_columns_f32(W, perm, inverse=True)
        codes = B.gptaq_permute_columns_u8(codes, perm, inverse=True)
    out = [W, codes, scales, zeros]
    if not case["act_order"]:      # (reordered factors are of no use outside the solve)
        out += [s["H"], s["A"]]
    if case["pack"]:
        out.append(B.gptaq_pack_codes(codes, case["bits"]))
    return out


def _work_accumulate(n, tokens, full):
    # X and X~ once (bf16), the sums once; n(n+1) tokens flop for a triangle, 2 n^2 tokens for a whole matrix
    entries = n * (n + 1) / 2 + (n * n if full else n * (n + 1) / 2)
    return 4.0 * n * tokens + 4.0 * entries, 2.0 * entries * tokens


def _work_prepare(n):
    # two triangles in, U and P out; factorisation, triangular inverse and the two triangular products: n^3 / 3 each
    return 4.0 * n * (n + 1) + 8.0 * n * n, 4.0 / 3.0 * n ** 3


def _work_quantize(m, n, groups):
    # W in and out, a code per weight, the grids, the triangles of U and P; m n^2 flop for each of the two terms
    return 9.0 * m * n + 8.0 * m * groups + 4.0 * n * (n + 1), 2.0 * m * n * n


def work(case):
    n, kind = case["n"], case["kind"]
    parts = []
    if kind in ("solve", "accumulate"):
        parts.append(_work_accumulate(n, case["tokens"], case.get("form") == "full" or case.get("act_order", False)))
    if kind in ("solve", "prepare"):
        parts.append(_work_prepare(n))
    if kind in ("solve", "quantize"):
        parts.append(_work_quantize(case["m"], n, n // case["group"] if case["group"] > 0 else 1))
    if case.get("act_bits"):
        parts.append((4.0 * n * case["tokens"], 0.0))
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    # Measured: sums taken 1024 tokens at a time and blocks in fp64 against the calls' own sums (rel 2.5e-6, max 1.1e-4);
    # factors against fp64 (rel 9e-6, max 5e-4: P, from products of bf16 hi + lo splits); the column loop in the form that
    # works 128 columns at a time, with P off by 1e-5 and with U off by 6e-8 (rel 6.7e-3, 4e-4 of the codes: near-ties
    # that go the other way, each a step of the grid, at most 0.6 of the weights' deviation).  About four times that.
    if case["kind"] == "accumulate":
        return {"rel": 1e-5, "max": 4e-4}
    if case["kind"] == "prepare":
        return {"rel": 4e-5, "max": 2e-3}
    return {"rel": 0.025, "max": 0.95, "differ": 0.01 if case.get("pack") else 0.002}     # (packed: eight codes to a word)

"""GPU parity: the HIP path (through the C ABI) against the fp64 oracle on the
same seeded inputs, element by element.

Tolerances (gpu_util): tau |dtau| <= 1e-3 * max(1, |tau|); O, O2, dQ, dK, dV
max-abs <= 2e-2 for bf16 inputs and <= 1e-4 for fp32 inputs; block masks
bit-exact except blocks whose decisive score lies within 1e-4 * max(1, |tau|)
of the threshold (several masks are correct there); lookup tables bit-exact
against the mask.

Small shapes are checked on every row and column.  The workload shapes are
checked on whole heads where the oracle finishes in seconds, otherwise on
sampled query blocks (tau, O, O2, dQ, mask rows) and on the last key columns
(dK, dV), which depend only on the sampled rows under causal masking.
"""
import numpy as np
import pytest

import synth
from gpu_util import check_head, check_tables, list_entries, list_uses, log, oracle_head, run_gpu, \
    sorted_blocks, to_device

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_12082_amd  # noqa: F401  (fails loudly if the library is missing)


def _full_case(B, H, n, d, dtype, alpha, causal, bwd, c, seed, heads=None, label=""):
    inp = synth.attention_inputs(B, H, n, d, c=c, dtype=dtype, with_dout=bwd, seed=seed)
    scale = d ** -0.5
    log("case %s B%d H%d n%d d%d %s alpha=%g causal=%d bwd=%d c=%g" % (
        label, B, H, n, d, dtype, alpha, causal, bwd, c))
    gpu = run_gpu(inp, alpha, scale, causal, bwd, heads=heads)
    check_tables(gpu, causal, columns=bwd)
    errs = []
    for bh in (heads if heads is not None else range(B * H)):
        ref = oracle_head(inp, bh, alpha, scale, causal, bwd)
        errs.append(check_head(gpu, ref, bh, dtype, "%s bh=%d" % (label, bh)))
    log("  errors %s" % errs[0])
    return gpu, errs


def test_tiny_forward_fp32():
    """Tiny config: B1 H1 n256 d64 fp32, alpha 1.5, non-causal, forward."""
    gpu, errs = _full_case(1, 1, 256, 64, "f32", 1.5, False, False, 1.0, synth.SEED_BASE,
                           label="tiny")
    # the max pass always streams K; with the candidate cache collected in it,
    # the evaluations need no further K pass
    assert gpu["stats"][0].min() >= 1


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 257])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_small_shapes(dtype, n, causal, d):
    # alpha 1.6, 1.7, 1.75 run the general-alpha (exp2/log2) kernels.  For
    # alpha in (1.5, 2) u = z^(gamma-1) has an unbounded slope as z -> 0+, so
    # with fp32 inputs those kernels take x - tau in fp64 near the support
    # edge and refine tau in fp64 (tau + tau_lo); the 1e-4 bound holds there.
    for alpha, c in ((1.5, 2.0), (2.0, 1.0), (1.25, 3.0), (1.6, 2.0), (1.7, 2.0), (1.75, 2.0)):
        _full_case(1, 2, n, d, dtype, alpha, causal, True, c, 100 + n,
                   label="small-%s-a%g" % (dtype, alpha))


@pytest.mark.parametrize("alpha", [1.5, 1.7])
@pytest.mark.parametrize("causal", [False, True])
def test_f32_two_group_form(alpha, causal):
    """fp32 at a grid of 512 tiles of 256 rows (B2 H16 n4096 d128), which runs
    the two-group form of the solver, fwd+bwd on two whole heads: alpha 1.7
    takes the fp64 refinement of tau (tau + tau_lo) and x - tau in fp64 near
    the support edge in that form too."""
    _full_case(2, 16, 4096, 128, "f32", alpha, causal, True, 2.0, 300, heads=[0, 31],
               label="f32-g2-a%g" % alpha)


@pytest.mark.parametrize("c", [1.0, 4.0, 16.0])
def test_encoder_forward(c):
    """B8 H12 n1024 d64 bf16 forward, Q temperature c; 4 heads vs the oracle."""
    _full_case(8, 12, 1024, 64, "bf16", 1.5, False, False, c, synth.SEED_BASE,
               heads=[0, 37, 60, 95], label="encoder")


def test_decoder_step():
    """B4 H12 n4096 d64 bf16 causal, c=8, forward + backward; 2 whole heads."""
    _full_case(4, 12, 4096, 64, "bf16", 1.5, True, True, 8.0, synth.SEED_BASE,
               heads=[0, 29], label="decoder")


def _sampled_case(B, H, n, d, alpha, causal, c, block_rows, ncols, heads, label,
                  full_cols=False, col_blocks=None):
    inp = synth.attention_inputs(B, H, n, d, c=c, dtype="bf16", with_dout=True,
                                 seed=synth.SEED_BASE)
    scale = d ** -0.5
    log("case %s B%d H%d n%d d%d alpha=%g causal=%d c=%g" % (label, B, H, n, d, alpha, causal, c))
    gpu = run_gpu(inp, alpha, scale, causal, True, heads=heads)
    T = (n + 63) // 64
    rows = sorted(set(r for I in block_rows for r in range(I * 64, min(n, I * 64 + 64))))
    cols = list(range(n - ncols, n)) if ncols else None
    if col_blocks:
        cols = sorted(set(j for J in col_blocks for j in range(J * 64, min(n, J * 64 + 64))))
    out = []
    for bh in heads:
        ref = oracle_head(inp, bh, alpha, scale, causal, True, rows=rows, cols=cols,
                          block_rows=block_rows)
        out.append(check_head(gpu, ref, bh, "bf16", "%s bh=%d" % (label, bh), rows=rows,
                              cols=cols))
    log("  errors %s" % out[0])
    return gpu, inp


# The sparsity sweep (B1 H16 n8192 d128 bf16 non-causal, fwd+bwd): every
# (alpha, c) point that bench.py reports, one whole head each (every row and
# column of tau, O, O2, dQ, dK, dV and every block of the mask).
SWEEP_POINTS = ([(1.5, c) for c in (0.0625, 0.25, 1.0, 2.0, 4.0, 8.0, 16.0, 32.0)]
                + [(a, c) for a in (1.25, 2.0) for c in (1.0, 2.0, 4.0, 8.0, 16.0, 32.0)])


@pytest.mark.parametrize("alpha,c", SWEEP_POINTS)
def test_sweep_workload(alpha, c):
    bh = 3
    inp = synth.attention_inputs(1, 16, 8192, 128, c=c, dtype="bf16", with_dout=True,
                                 seed=synth.SEED_BASE)
    log("case sweep B1 H16 n8192 d128 alpha=%g c=%g (head %d)" % (alpha, c, bh))
    gpu = run_gpu(inp, alpha, 128 ** -0.5, False, True, heads=[bh])
    check_tables(gpu, False)
    ref = oracle_head(inp, bh, alpha, 128 ** -0.5, False, True)
    log("  errors %s" % check_head(gpu, ref, bh, "bf16", "sweep a=%g c=%g" % (alpha, c)))


@pytest.mark.parametrize("causal", [False, True])
def test_dkdv_sparse_key_block_pairs(causal):
    """bf16 d128 at a sparse mask (c = 32): dK and dV of the key blocks of
    several adjacent pairs, whose query-block lists differ; the d = 128 dK/dV
    kernel walks the union of each pair's lists."""
    n = 4096
    gpu, _ = _sampled_case(1, 2, n, 128, 1.5, causal, 32.0, block_rows=[0, 63], ncols=0,
                           heads=[0, 1], label="pairs", col_blocks=[0, 1, 20, 21, 62, 63])
    kc = gpu["k_count"][0]
    ki = gpu["k_index"][0]
    differ = [m for m in (0, 10, 31) if kc[2 * m] != kc[2 * m + 1]
              or not np.array_equal(ki[2 * m, :kc[2 * m]], ki[2 * m + 1, :kc[2 * m + 1]])]
    assert differ, "the chosen pairs should have different query-block lists"


@pytest.mark.parametrize("n", [16384, 32768, 65536])
def test_long_context(n):
    """B1 H8 d64 bf16 causal, c=16, fwd+bwd (every sequence length bench.py
    reports): first, middle and last query blocks; dK/dV on the last 64 keys
    (which depend only on the sampled last rows under causal masking), and at
    n = 16384 also on a key block in the middle (rows from there on)."""
    T = n // 64
    col_blocks = [T // 2, T - 1] if n <= 16384 else None
    gpu, inp = _sampled_case(1, 8, n, 64, 1.5, True, 16.0, block_rows=[0, T // 2, T - 1],
                             ncols=64, heads=[0, 7], label="long", col_blocks=col_blocks)
    check_tables({k: gpu[k][:1] for k in ("mask", "q_count", "q_index", "k_count", "k_index")},
                 True)
    # tau on 48 random rows of every head, and O on those rows of heads 0 and 7
    rng = np.random.default_rng(n)
    for bh in range(8):
        rows = np.sort(rng.choice(n, size=48, replace=False))
        ref = oracle_head(inp, bh, 1.5, 64 ** -0.5, True, False, rows=rows)
        tr, tg = ref["tau"][rows], gpu["tau"][bh][rows]
        rel = np.max(np.abs(tg - tr) / np.maximum(1.0, np.abs(tr)))
        assert rel <= 1e-3, ("long random rows", bh, rel)
        if bh in (0, 7):
            err = np.max(np.abs(gpu["o"][bh][rows] - ref["o"][rows]))
            assert err <= 2e-2, ("long random rows O", bh, err)
    log("  random rows: tau and O within bounds on all heads")


# ------------------------------------------------------------- invariants

def _device(inp):
    return to_device(inp["q"]), to_device(inp["k"]), to_device(inp["v"])


def test_invariants_and_determinism():
    import paper_2502_12082_amd as ea
    B, H, n, d = 1, 4, 1000, 128
    inp = synth.attention_inputs(B, H, n, d, c=2.0, dtype="bf16", with_dout=True, seed=77)
    q, k, v = _device(inp)
    do = to_device(inp["dout"])
    for causal in (False, True):
        log("invariants causal=%d" % causal)
        o, res = ea.forward(q, k, v, alpha=1.5, scale=d ** -0.5, causal=causal)
        dq, dk, dv = ea.backward(q, k, v, do, res)
        o_b, res_b = ea.forward(q, k, v, alpha=1.5, scale=d ** -0.5, causal=causal)
        dq_b, dk_b, dv_b = ea.backward(q, k, v, do, res_b)
        torch.cuda.synchronize()
        for a, b in ((o, o_b), (res.tau, res_b.tau), (res.o2, res_b.o2), (dq, dq_b),
                     (dk, dk_b), (dv, dv_b), (res.block_mask, res_b.block_mask)):
            assert torch.equal(a, b), "not bit-identical across runs"
        # sum_j dS_ij = 0  =>  sum_j dK_j = 0;  sum_j p_ij = 1  =>  sum_j dV_j = sum_i dO_i
        dk_sum = dk.double().sum(2).abs().max().item()
        assert dk_sum <= 1e-3 * max(1.0, dk.abs().max().item()) * 10, dk_sum
        dv_err = (dv.double().sum(2) - do.double().sum(2)).abs().max().item()
        assert dv_err <= 0.05 * max(1.0, do.double().sum(2).abs().max().item()), dv_err
        # V = 1  =>  O = sum_j p_ij = 1 + f(tau)
        ones = torch.ones_like(v)
        o1, _ = ea.forward(q, k, ones, alpha=1.5, scale=d ** -0.5, causal=causal,
                           need_bwd=False)
        assert (o1.float() - 1).abs().max().item() <= 8e-3


def test_nan_inputs_do_not_fault():
    """A NaN score gets probability 0 (the clamp of [x - tau]_+ maps NaN to 0),
    so NaN in Q or K leaves tau finite; NaN in V propagates to the rows that
    attend to that key.  Rows that never see the NaN stay finite."""
    import paper_2502_12082_amd as ea
    inp = synth.attention_inputs(1, 1, 128, 64, dtype="f32", seed=3)
    q, k, v = _device(inp)
    o_ref, _ = ea.forward(q, k, v)
    q2 = q.clone()
    q2[0, 0, 5, 0] = float("nan")
    o, res = ea.forward(q2, k, v)
    torch.cuda.synchronize()
    keep = [r for r in range(128) if r != 5]
    assert torch.isfinite(res.tau[0, keep]).all()
    assert (o[0, 0, keep] - o_ref[0, 0, keep]).abs().max().item() <= 1e-4
    v2 = v.clone()
    v2[0, 0, 9, :] = float("nan")
    o3, res3 = ea.forward(q, k, v2)
    torch.cuda.synchronize()
    assert torch.isfinite(res3.tau).all()
    assert torch.isnan(o3).any()


@pytest.mark.parametrize("dtype,d,n,alpha", [
    ("bf16", 64, 31, 1.5), ("bf16", 128, 256, 1.25), ("f32", 128, 511, 2.0), ("bf16", 64, 513, 1.5),
    ("f32", 64, 1024, 1.25), ("bf16", 128, 1000, 2.0), ("bf16", 64, 700, 1.6), ("bf16", 64, 300, 3.0)])
@pytest.mark.parametrize("causal", [False, True])
def test_short_sequence_solver(dtype, d, n, alpha, causal):
    """The solver for short sequences (scores in registers, lists in LDS): its
    three sizes at their edges and remainders.  c = 0.1 overflows its lists
    (the evaluations then run on the scores themselves)."""
    for c in ((4.0, 0.1) if alpha <= 2 else (1.0,)):
        inp = synth.attention_inputs(1, 2, n, d, c=c, dtype=dtype, with_dout=True, seed=n)
        bwd = alpha <= 2
        gpu = run_gpu(inp, alpha, d ** -0.5, causal, bwd, max_iter=12 if bwd else 40)
        check_tables(gpu, causal, columns=bwd)
        for bh in range(2):
            ref = oracle_head(inp, bh, alpha, d ** -0.5, causal, bwd)
            errs = check_head(gpu, ref, bh, dtype, "short n%d c%g bh=%d" % (n, c, bh))
        log("short %s d%d n%d alpha %g c %g causal %d: %s" % (dtype, d, n, alpha, c, causal, errs))


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("alpha", [1.25, 1.5, 2.0, 1.7])
@pytest.mark.parametrize("causal", [False, True])
def test_element_lists(dtype, d, alpha, causal):
    """Query blocks with element lists, without them, and both in one head:
    rows of a low query temperature (too many entries to list) in some blocks,
    and one key that every query attends to, whose dK and dV several groups of
    lanes share (more entries than one round of the dK/dV kernel takes).  The
    backward equals the oracle, and the one without lists: their thresholds no
    longer match once another forward has filled the residuals."""
    import paper_2502_12082_amd as ea
    n = 2500
    # (fp32: the rounding of larger scores alone would pass the bound of 1e-4)
    inp = synth.attention_inputs(1, 2, n, d, c=4.0 if dtype == "bf16" else 1.5, dtype=dtype,
                                 with_dout=True, seed=11)
    q, k = inp["q"].f32().copy(), inp["k"].f32().copy()
    k[:, 0, :, :8] *= 0.1
    k[:, 0, 100, :8] = 1.0                      # head 0: a key that all queries score highly
    q[:, 0, :, :8] += 32.0 if dtype == "bf16" else 12.0
    q[:, :, 640:768] = 0.0                      # two query blocks of equal scores (not listed)
    bits = synth.f32_to_bf16_bits if dtype == "bf16" else (lambda x: x)
    inp["q"], inp["k"] = synth.Tensor(bits(q), dtype), synth.Tensor(bits(k), dtype)
    scale = d ** -0.5
    gpu = run_gpu(inp, alpha, scale, causal, True)
    check_tables(gpu, causal)
    for bh in range(2):
        ref = oracle_head(inp, bh, alpha, scale, causal, True)
        # fp32: sums over all n queries of that key reach |dK| ~ 100, over all keys |dQ| ~ 50
        if dtype == "f32":  # in the 2-norm: the sums have 2500 terms where all scores are equal
            errs = {x: float(np.linalg.norm(gpu[x][bh] - ref[x]) / np.linalg.norm(ref[x]))
                    for x in ("tau", "o", "o2", "dq", "dk", "dv")}
            assert max(errs.values()) <= 2e-5, errs
        else:
            errs = check_head(gpu, ref, bh, dtype, "lists bh=%d" % bh)
    log("lists %s d%d alpha %g causal %d: %s" % (dtype, d, alpha, causal, errs))
    t = {x: to_device(inp[x]) for x in ("q", "k", "v", "dout")}
    o, res = ea.forward(t["q"], t["k"], t["v"], alpha=alpha, causal=causal)
    ws = ea.backward_workspace(res, res.tau.device)
    with_lists = ea.backward(t["q"], t["k"], t["v"], t["dout"], res, workspace=ws)
    T = (n + 63) // 64
    use, _ = list_uses(res.lists, 2 * T)
    used, heads = sorted_blocks(ws, 2 * n, 2 * T, 2)
    shared = [list_entries(res.lists, b) for b in range(T) if use[b]]
    shared = sum(int((key // 64 == 100 // 64).sum()) for _, key in shared)
    log("  uses %s, sorted %s of %d, entries of the shared key's block %d" % (
        np.bincount(use, minlength=8), (used & 2 > 0).sum(1), T, shared))
    assert (use > 0).any() and (used & 1).any()
    if alpha >= 1.5:  # the others are listed, and sorted
        assert heads.all() and ((used & 2 > 0).sum(1) == T - 2).all()
        assert shared > 2048  # more than one round of the dK/dV kernel
    lists, res.lists = res.lists, None
    without = ea.backward(t["q"], t["k"], t["v"], t["dout"], res)
    res.lists = lists
    ea.forward(t["q"], t["k"], t["v"], alpha=alpha, causal=causal, scale=2.0 * scale, res=res)
    stale, res.lists = res.lists.clone(), None  # lists of other thresholds
    ea.forward(t["q"], t["k"], t["v"], alpha=alpha, causal=causal, res=res)
    plain = ea.backward(t["q"], t["k"], t["v"], t["dout"], res)
    res.lists = stale
    assert (list_uses(stale, 2 * T)[0] > 0).any()
    with_stale = ea.backward(t["q"], t["k"], t["v"], t["dout"], res, workspace=ws)
    torch.cuda.synchronize()
    assert (sorted_blocks(ws, 2 * n, 2 * T, 2)[0] == 0).all()
    for a, b in zip(plain, with_stale):
        assert torch.equal(a, b), "lists of other thresholds were used"
    for a, b in zip(with_lists, without):
        # dV: one side rounds P to bf16, 2^-9 relative per term; the others, and
        # fp32, differ by the rounding of their sums of up to n terms
        rel = 4e-3 if dtype == "bf16" else 2e-5
        assert (a - b).norm().item() <= rel * b.norm().item()


@pytest.mark.parametrize("n,d,causal,c", [(2300, 64, True, 4.0), (2300, 64, False, 4.0),
                                          (2300, 128, True, 4.0), (1153, 64, True, 4.0)])
def test_dense_partly_listed(n, d, causal, c):
    """No-mask mode where part of a head's query blocks has element lists (two
    blocks of wide rows, which the sample does not meet, among sparse ones): the
    gradients are the masked path's (bf16 rounding of P: 2^-8 relative)."""
    import ctypes
    import paper_2502_12082_amd as ea
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k, v, do = (torch.randn(2, 2, n, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(4))
    q = q.float() * c
    q[:, :, 6 * 64:8 * 64] *= 0.02
    q = q.to(torch.bfloat16)
    _, res = ea.forward(q, k, v, alpha=1.5, causal=causal, lists=False)
    ref = ea.backward(q, k, v, do, res)
    _, tau, o2, lo = ea.forward_dense(q, k, v, alpha=1.5, causal=causal)
    got = ea.backward_dense(q, k, v, do, tau, o2, alpha=1.5, causal=causal, tau_lo=lo)
    for x, y in zip(got, ref):
        assert (x - y).norm() <= 2 ** -8 * y.norm()
    # the same call with buffers that can be looked at
    shape, params = ea.make_shape(q), ea.make_params(1.5, None, causal, head_dim=d)
    lists, ws = (torch.empty(size, dtype=torch.uint8, device=q.device) for size in (
        ea.entmax_attn_lists_bytes(shape, params), ea.entmax_attn_bwd_lists_workspace(shape, params)))
    p = lambda x: x.data_ptr()
    for x in got:
        x.fill_(float("nan"))
    ea._check(ea._lib.entmax_attn_bwd_dense_lists(
        ctypes.byref(shape), ctypes.byref(params), p(q), p(k), p(v), p(do), p(tau), None, p(o2), p(lists),
        lists.numel(), *map(p, got), p(ws), ws.numel(), torch.cuda.current_stream().cuda_stream), "dense")
    T = (n + 63) // 64
    used, heads = sorted_blocks(ws, 4 * n, 4 * T, 4)
    log("partly listed n%d d%d causal %d: %s of %d sorted" % (n, d, causal, (used & 2 > 0).sum(1), T))
    if n > 2000:
        assert heads.all() and ((used & 2 > 0).sum(1) < T).all()
    for x, y in zip(got, ref):
        assert (x - y).norm() <= 2 ** -8 * y.norm()


@pytest.mark.parametrize("B,H,n,d,causal", [(8, 12, 777, 64, False), (8, 12, 1000, 64, True),
                                            (16, 12, 300, 128, True), (16, 12, 511, 128, False)])
def test_cached_solver_short_sequences(B, H, n, d, causal):
    """Grids of many heads that the cached solver takes although they are
    short: 512 < n <= 1024 with more than 384 query blocks, and d = 128 from
    257 keys with more than 512."""
    _full_case(B, H, n, d, "bf16", 1.5, causal, True, 2.0, n, heads=[0, B * H - 1], label="many heads")


@pytest.mark.parametrize("n", [400, 1500])
def test_element_lists_non_finite(n):
    """Values that are not finite, where the query blocks have element lists:
    a V row reaches the rows that attend to its key and no others, a K row has
    probability 0 and reaches nothing, a Q row spoils its own row alone.  (Where
    a block is computed by products, 0 times a row that is not finite reaches
    all of its rows.)"""
    import paper_2502_12082_amd as ea
    inp = synth.attention_inputs(1, 2, n, 64, c=6.0, dtype="bf16", with_dout=True, seed=n)
    q, k, v, do = (to_device(inp[x]) for x in ("q", "k", "v", "dout"))
    T = (n + 63) // 64
    o, res = ea.forward(q, k, v, alpha=1.5)
    use, _ = list_uses(res.lists, 2 * T)
    assert (use & 3 == 3).all()
    j = 70
    attends = torch.zeros(n, dtype=torch.bool)
    for b in range(T):
        row, key = list_entries(res.lists, b)
        attends[b * 64 + row[key == j]] = True
    assert 0 < attends.sum() < n
    for bad in (float("nan"), float("inf")):
        v2 = v.clone()
        v2[0, 0, j] = bad
        o2, r2 = ea.forward(q, k, v2, alpha=1.5)
        grads = ea.backward(q, k, v2, do, r2)
        torch.cuda.synchronize()
        fin = torch.isfinite(o2[0, 0].float()).all(-1).cpu()
        assert torch.equal(fin, ~attends) and torch.equal(o2[0, 0, fin.cuda()], o[0, 0, fin.cuda()])
        assert torch.isfinite(o2[0, 1].float()).all()
        assert torch.equal(torch.isfinite(grads[0][0, 0]).all(-1).cpu(), ~attends)
        assert all(torch.isfinite(x[0, 1]).all() for x in grads)
    k2, q2 = k.clone(), q.clone()
    k2[0, 0, j] = float("nan")
    q2[0, 0, 5] = float("nan")
    for qq, kk, skip in ((q, k2, None), (q2, k, 5)):
        o2, r2 = ea.forward(qq, kk, v, alpha=1.5)
        grads = ea.backward(qq, kk, v, do, r2)
        torch.cuda.synchronize()
        rows = [i for i in range(n) if i != skip]
        assert torch.isfinite(r2.tau[0, rows]).all() and torch.isfinite(o2[0, 0, rows].float()).all()
        assert torch.isfinite(grads[0][0, 0, rows]).all()
        assert all(torch.isfinite(x[0, 1]).all() for x in grads)


@pytest.mark.parametrize("d,n", [(128, 128), (128, 100), (64, 70), (64, 512)])
@pytest.mark.parametrize("alpha", [1.25, 1.5, 2.0])
def test_short_fp32_scores_are_the_recomputed_ones(d, n, alpha):
    """fp32 on the short-sequence solver: the probabilities that it lists and
    those that the forward recomputes from tau come from the same scores, bit
    for bit (at alpha = 2 u jumps from 0 to 1 at the support's edge, and one
    stage may read the lists where another recomputes).  With V's first d rows
    the unit matrix O is P itself, exactly."""
    import paper_2502_12082_amd as ea
    g = torch.Generator(device="cuda").manual_seed(1)
    q, k = (torch.randn(1, 8, n, d, generator=g, device="cuda") for _ in range(2))
    v = torch.zeros_like(q)
    m = min(n, d)
    v[:, :, range(m), range(m)] = 1.0
    shape, params = ea.make_shape(q), ea.make_params(alpha, head_dim=d)
    res = ea.Residuals(shape, params, q.device)
    assert res.lists is not None
    p_listed, _ = ea.forward(q, k, v, alpha=alpha, res=res)
    tau = res.tau.clone()
    res.lists = None
    p, _ = ea.forward(q, k, v, alpha=alpha, res=res)
    assert torch.equal(tau, res.tau)
    assert (p > 0).any() and torch.equal(p_listed, p)


@pytest.mark.parametrize("alpha", [2.5, 3.0])
@pytest.mark.parametrize("n", [300, 1000])
def test_short_sequence_bracket_above_two(alpha, n):
    """alpha > 2 (f is not convex, and the iteration may halve the bracket at
    every step): the short-sequence solver's bracket is as narrow as that of
    the longer ones, which takes 8 equal scores into account.  With all keys
    the same row, tau = x - n^(1 - alpha), the upper end, and the bracket is
    8^(1 - alpha) wide at most: k updates after its midpoint leave at most
    2^-(k+2) of it, and the rounding of x and tau."""
    import paper_2502_12082_amd as ea
    g = torch.Generator(device="cuda").manual_seed(n)
    q = torch.randn(1, 2, n, 64, generator=g, device="cuda").bfloat16()
    k = torch.randn(1, 2, 1, 64, generator=g, device="cuda").bfloat16().expand(1, 2, n, 64).contiguous()
    x = (alpha - 1) * 0.125 * (q.double() @ k[:, :, 0].double()[..., None])[..., 0]
    tau = x.reshape(2, n) - float(n) ** (1 - alpha)
    for it in (0, 4, 12):
        _, res = ea.forward(q, k, k, alpha=alpha, max_iter=it, need_bwd=False)
        err = (res.tau.double() - tau).abs().max().item()
        log("alpha %g n %d, %d updates: dtau %.2e" % (alpha, n, it, err))
        assert err <= 8.0 ** (1 - alpha) / 2 ** (it + 2) + 1e-6 * max(5.0, x.abs().max().item())


@pytest.mark.parametrize("dtype,n", [("bf16", 1500), ("f32", 300)])
def test_backward_leaves_the_lists_alone(dtype, n):
    """The backward only reads the residuals' element lists: they are the same
    bytes afterwards, and two backwards of one forward, on two streams and of
    different output gradients, are each what they are alone.  A workspace
    without room to sort the lists gives the backward without them."""
    import paper_2502_12082_amd as ea
    inp = synth.attention_inputs(2, 3, n, 64, c=4.0, dtype=dtype, with_dout=True, seed=6)
    q, k, v, do = (to_device(inp[x]) for x in ("q", "k", "v", "dout"))
    do2 = (2.0 * do.flip(2)).contiguous()
    _, res = ea.forward(q, k, v, alpha=1.5)
    before = res.lists.clone()
    ref, ref2 = ea.backward(q, k, v, do, res), ea.backward(q, k, v, do2, res)
    torch.cuda.synchronize()
    assert torch.equal(res.lists, before)
    streams = [torch.cuda.Stream() for _ in range(2)]
    for _ in range(3):
        got = []
        for st, d in zip(streams, (do, do2)):
            with torch.cuda.stream(st):
                got.append(ea.backward(q, k, v, d, res))
        torch.cuda.synchronize()
        for a, b in zip(ref + ref2, got[0] + got[1]):
            assert torch.equal(a, b)
    small = torch.empty(res.sizes.ws_bwd, dtype=torch.uint8, device=q.device)
    got = ea.backward(q, k, v, do, res, workspace=small)
    lists, res.lists = res.lists, None
    plain = ea.backward(q, k, v, do, res)
    res.lists = lists
    torch.cuda.synchronize()
    assert not all(torch.equal(a, b) for a, b in zip(ref, plain))  # the lists were in use above
    for a, b in zip(plain, got):
        assert torch.equal(a, b)

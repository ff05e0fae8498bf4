"""Parity at the sizes where a launch rule changes kernel: the permutation's
chunk counts, the rank contraction's tile sizes, the expert GEMM's row counts,
the CKA projection's probe tiles, and the pre-combined path with and without
pair_row.  Oracle and tolerances as in the other GPU tests: integers bit for
bit, rel-L2 2e-2 (bf16) and 1e-5 (fp32), CKA entries within 1e-4."""
import numpy as np
import pytest
import torch

from gpu_harness import (TOL, check_all, check_dB_rows, f64, make_case, oracle_bwd, oracle_fwd,
                         run_gpu, say)
from oracle import ace_oracle as O
from oracle import consolidation_oracle as C
from paper_2609_06072_amd import workloads as W
from test_gpu_moe import case_and_weights, oracle_y, run_moe
from test_gpu_parity import _perm_check, _perm_compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2609_06072_amd import ace  # noqa: F401  (fails loudly if libace.so is missing)


@pytest.mark.parametrize("T,k", [(1, 8), (32, 8), (33, 8), (64, 8), (96, 8), (128, 8), (129, 8),
                                 (103, 5), (8, 32), (25, 32), (33, 32)])
def test_permute_chunk_counts(T, k):
    """One launch for up to four chunks of 256 pairs, two from five; with ids
    out of range, repeated ids and experts outside every group."""
    from paper_2609_06072_amd import ace
    say(f"permute T={T} k={k}")
    rng = np.random.default_rng(T * 100 + k)
    E, G = 40, 7
    ids = rng.integers(0, E, size=(T, k)).astype(np.int32)   # repeats within a token
    ids[rng.random((T, k)) < 0.05] = E + 3
    ids[rng.random((T, k)) < 0.05] = -1
    e2g = rng.integers(0, G + 1, size=E).astype(np.int32)    # G: outside [0, G)
    for mode in (0, 1, 2):
        _perm_check(ids, E, e2g, G, mode)
    g, e = ace.ace_group_expert_permute(torch.from_numpy(ids).cuda(), E, torch.from_numpy(e2g).cuda(), G)
    _perm_compare(g, ids, E, e2g, G, 0)
    _perm_compare(e, ids, E, e2g, G, 2)


# (tokens, E, k, group size, r): tiles of 16 rows (up to 256 of them); one
# 64-row tile per block (bf16, up to 256); 32-row tiles (fp32, ranks up to 64);
# 64-row tiles shared out over the XCDs, fp32 keys of mixed ranks among them
CONTRACT = [
    ("bf16", 40, 8, 2, ("consecutive", 4), 5),
    ("bf16", 1984, 8, 2, ("consecutive", 4), 8),     # the last size of 16-row tiles
    ("bf16", 1985, 8, 2, ("consecutive", 4), 8),
    ("bf16", 2500, 8, 2, ("consecutive", 4), 16),
    ("bf16", 2500, 8, 2, ("consecutive", 4), 24),
    ("bf16", 2500, 8, 2, ("consecutive", 4), 40),
    ("f32", 40, 8, 2, ("consecutive", 4), 40),
    ("f32", 2500, 8, 2, ("consecutive", 4), 3),
    ("f32", 2500, 16, 2, ("uneven", 0), 8),
    ("f32", 2500, 16, 2, ("uneven", 0), 16),
    ("f32", 8200, 16, 2, ("uneven", 0), 16),
    ("f32", 2500, 8, 2, ("consecutive", 4), 40),
]


@pytest.mark.parametrize("dtype,T,E,k,groups,r_e", CONTRACT)
@pytest.mark.parametrize("path", ["grouped", "down_expertwise"])
def test_contraction_tiles(dtype, T, E, k, groups, r_e, path):
    base = W.CONFIGS["olmoe_bf16"]
    cfg = base.scaled(dtype=dtype, T=T, E=E, k=k, groups=groups, r_e=r_e, d_model=136, d_ffn=72)
    say(f"contraction {dtype} T={T} E={E} r={r_e} {groups} {path}")
    c = make_case(cfg, path, seed=3, with_w=path == "grouped")
    out = run_gpu(c, reuse_h=True)
    tol = TOL[dtype]
    check_all("y", f64(out["y"]), oracle_fwd(c), tol)
    dx, dA, dB = oracle_bwd(c)
    check_all("dx", f64(out["dx"]), dx, tol)
    check_all("dA", f64(out["dA"]), dA, tol)
    check_dB_rows("dB", f64(out["dB"]), dB, c.ranks, c.d_out, tol)


# fp32 beyond the small batches: (tokens, k, d_model, group size, r) of the
# register kernel (64-row tiles at ranks to 32 and to 64, 32-row tiles to 128)
# and, one step away, of the 32- and 16-row tiles
REG = [(6200, 2, 136, 2, 8), (6200, 2, 136, 4, 12), (8300, 2, 136, 4, 12), (2500, 2, 1032, 4, 25),
       (2500, 2, 1020, 4, 25), (2500, 2, 264, 4, 40)]


@pytest.mark.parametrize("T,k,d_model,size,r_e", REG)
@pytest.mark.parametrize("path", ["grouped", "expertwise"])
def test_contraction_registers_f32(T, k, d_model, size, r_e, path):
    cfg = W.CONFIGS["olmoe_bf16"].scaled(dtype="f32", T=T, E=8, k=k, groups=("consecutive", size), r_e=r_e,
                                         d_model=d_model, d_ffn=72)
    say(f"f32 contraction T={T} d={d_model} r={r_e}x{size} {path}")
    c = make_case(cfg, path, seed=4)
    out = run_gpu(c, reuse_h=True)
    tol = TOL["f32"]
    check_all("y", f64(out["y"]), oracle_fwd(c), tol)
    dx, dA, dB = oracle_bwd(c)
    check_all("dx", f64(out["dx"]), dx, tol)
    check_all("dA", f64(out["dA"]), dA, tol)
    check_dB_rows("dB", f64(out["dB"]), dB, c.ranks, c.d_out, tol)


def test_contraction_error_by_rank_f32():
    """Every fp32 contraction sums in four chains or more, at every rank: the
    error of a long one against 64 bits (rounding grows with the square root
    of a chain's length) is at ranks above 64 and above 128 no larger than at
    rank 40.  B_q = I, so that y is h; two chains would show 1.4 times."""
    from paper_2609_06072_amd import ace
    T, K, n = 4200, 8192, 512
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x = torch.randn(T, K, generator=g, device="cuda")
    A = torch.randn(256, K, generator=g, device="cuda")
    ids = torch.zeros(T, 1, dtype=torch.int32, device="cuda")
    rt = ace.ace_group_permute(ids, 1, None, 0, ace.ACE_ROWS_EXPERT)
    ref = x[:n].double() @ A[:40].double().t()
    err = {}
    for r in (40, 100, 160, 256):
        say(f"f32 contraction error rank {r}")
        y = torch.zeros(T, r, device="cuda")
        ace.ace_expertwise_lora_fwd(x, A[:r].contiguous(), torch.eye(r, device="cuda").flatten(), 1, r, float(r), rt, y)
        err[r] = float((y[:n, :40].double() - ref).norm() / ref.norm())
    say(str(err))
    for r in (100, 160, 256):
        assert err[r] <= 1.1 * err[40], err


def test_contraction_second_grid_row_f32():
    """More than 2^21 tiles of 16 rows: the rows of the grid's second row."""
    from paper_2609_06072_amd import ace
    T, r, d = (1 << 25) + 1000, 130, 4
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("h does not fit the free memory")
    say("f32 contraction of 2^25 rows")
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    x = torch.randn(T, d, generator=g, device="cuda")
    A, B = torch.randn(r, d, generator=g, device="cuda"), torch.randn(d, r, generator=g, device="cuda")
    ids = torch.zeros(T, 1, dtype=torch.int32, device="cuda")
    rt = ace.ace_group_permute(ids, 1, None, 0, ace.ACE_ROWS_EXPERT)
    y = torch.zeros(T, d, device="cuda")
    ace.ace_expertwise_lora_fwd(x, A, B.flatten(), 1, r, 2.0 * r, rt, y)
    for rows in (slice(0, 500), slice((1 << 25) - 500, T)):
        want = 2.0 * (x[rows].double() @ A.double().t()) @ B.double().t()
        check_all("y", f64(y[rows]), f64(want), TOL["f32"])
    del x, y, rt
    torch.cuda.empty_cache()


# rows per expert on average (T k / E): the streaming kernel's tiles of 16, 32
# and 64 rows, the medium tiles, the large ones; d_in of one, two, three and a
# ragged number of 64-index stages, an odd number of column tiles
@pytest.mark.parametrize("dtype,T", [("bf16", 9), ("bf16", 32), ("bf16", 33), ("bf16", 80), ("bf16", 81),
                                     ("bf16", 112), ("bf16", 113), ("bf16", 128), ("bf16", 129), ("bf16", 256), ("bf16", 257), ("bf16", 767), ("bf16", 768),
                                     ("bf16", 1100), ("f32", 32), ("f32", 33), ("f32", 640), ("f32", 641),
                                     ("f32", 2048), ("f32", 2049)])
@pytest.mark.parametrize("d_model,d_ffn,r_e", [(64, 128, 8), (192, 328, 24), (256, 520, 5)])
def test_expert_rows(dtype, T, d_model, d_ffn, r_e):
    cfg = W.CONFIGS["mixtral_bf16"].scaled(dtype=dtype, T=T, k=1, E=4, d_model=d_model, d_ffn=d_ffn,
                                           r_e=r_e, groups=("consecutive", 4))
    for path in ("grouped", "down_expertwise"):
        say(f"expert rows {dtype} T={T} {d_model}x{d_ffn} r={r_e} {path}")
        c, Wt = case_and_weights(cfg, path, seed=12)
        check_all("y", f64(run_moe(c, Wt)), oracle_y(c, Wt), TOL[dtype])


# where the medium tiles leave few CUs idle (224 of one per expert) they take
# over from 48 rows per expert, where they fill them (384) from 24
@pytest.mark.parametrize("E,T", [(56, 20), (56, 21), (56, 48), (56, 49), (96, 20), (96, 24), (96, 25)])
def test_expert_rows_many_experts(E, T):
    cfg = W.CONFIGS["mixtral_bf16"].scaled(T=T * E, k=1, E=E, d_model=72, d_ffn=1000, r_e=4, groups=("consecutive", 4))
    say(f"expert rows of {E} experts, {T} each")
    c, Wt = case_and_weights(cfg, "grouped", seed=15)
    check_all("y", f64(run_moe(c, Wt)), oracle_y(c, Wt), TOL["bf16"])


# 5420 to 6500 rows fill the 256 CUs with one round of 128 x 256 tiles
@pytest.mark.parametrize("T", [5410, 5420, 6500, 6600])
@pytest.mark.parametrize("path", ["grouped", "down_expertwise"])
def test_expert_rows_many_f32(T, path):
    """fp32: streaming kernel or medium tiles, with ragged columns and d_in."""
    d_in, d_out = 204, 1276
    dims = dict(d_model=d_in, d_ffn=d_out) if path == "grouped" else dict(d_model=d_out, d_ffn=d_in)
    cfg = W.CONFIGS["mixtral_bf16"].scaled(dtype="f32", T=T, k=1, E=2, r_e=5, groups=("consecutive", 2), **dims)
    say(f"expert rows f32 T={T} {path}")
    c, Wt = case_and_weights(cfg, path, seed=14)
    check_all("y", f64(run_moe(c, Wt)), oracle_y(c, Wt), TOL["f32"])


# x of 4 GiB, and of 2^32 elements, with many and with few rows per expert
# (large tiles whose offsets count 16-byte chunks), of 64 GiB (streaming)
@pytest.mark.parametrize("gib,E,d_in", [(4, 2, 8192), (4, 2, 8136), (8, 2, 8192), (8, 256, 131072), (8, 256, 131000),
                                        (64, 2, 65536)])
@pytest.mark.parametrize("mode", ["shared", "per_pair"])
def test_expert_rows_big_x(gib, E, d_in, mode):
    """Rows on both sides of the last one that a 32-bit offset reaches; only
    the rows that are checked are set."""
    from paper_2609_06072_amd import ace
    bound = (gib << 30) // (2 * d_in)   # first row at or past gib GiB
    T, d_out = bound + 200, 24
    if torch.cuda.mem_get_info()[0] < (gib + 4) << 30:
        pytest.skip("x does not fit the free memory")
    say(f"expert rows, x of {gib} GiB, E={E} d_in={d_in} {mode}")
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    x = torch.empty(T, d_in, dtype=torch.bfloat16, device="cuda")
    Wt = torch.randn(E, d_out, d_in, generator=g, device="cuda").bfloat16()
    ids = (torch.arange(T, device="cuda", dtype=torch.int32) % E)[:, None].contiguous()
    rt = ace.ace_group_permute(ids, E, None, 0, ace.ACE_ROWS_EXPERT)
    rows = torch.tensor([0, 1, 199, bound // 2 - 1, bound // 2 + 1, bound - 2, bound - 1, bound, bound + 1, bound + 57,
                         T - 1], device="cuda")
    x[rows] = torch.randn(len(rows), d_in, generator=g, device="cuda").bfloat16()
    y = torch.zeros(T, d_out, dtype=torch.bfloat16, device="cuda")
    ace.ace_moe_lora_fwd(x, Wt, rt, y,
                         input_mode=ace.ACE_INPUT_SHARED if mode == "shared" else ace.ACE_INPUT_PER_PAIR)
    want = (Wt[ids[rows, 0].long()].double() * x[rows].double()[:, None]).sum(-1)
    check_all("y", f64(y[rows]), f64(want), TOL["bf16"])
    del x, y
    torch.cuda.empty_cache()


def test_expert_rows_empty_and_dropped():
    """Large tiles with an expert of no rows, one of a single row and dropped
    pairs: their y rows stay as they were."""
    cfg = W.CONFIGS["mixtral_bf16"].scaled(T=1500, k=1, E=4, d_model=136, d_ffn=264, r_e=4,
                                           groups=("consecutive", 2))
    c, Wt = case_and_weights(cfg, "grouped", seed=13)
    ids = np.where(np.arange(cfg.T) % 3 == 0, 0, 3).astype(np.int32)[:, None]
    ids[7] = 1
    ids[::50] = -1
    c.rt.topk_ids[:] = ids
    y0 = torch.full((cfg.P, c.d_out), 7.0, dtype=c.x.dtype, device="cuda")
    y = f64(run_moe(c, Wt, y=y0))
    keep = ids[:, 0] >= 0
    assert np.all(y[~keep] == 7.0)
    check_all("y", y[keep], oracle_y(c, Wt)[keep], TOL["bf16"])


@pytest.mark.parametrize("dtype,T", [("bf16", 9), ("bf16", 128), ("bf16", 400), ("bf16", 1100), ("f32", 20),
                                     ("f32", 400), ("f32", 2600)])
def test_expert_rows_infinite(dtype, T):
    """An infinity in the last 16-byte chunk of a W row or of x, with d_in
    that ends inside a stage: the chunks past d_in add nothing, so its products
    stay infinite (no NaN) and the rest of y finite."""
    from paper_2609_06072_amd import ace
    say(f"infinite operands {dtype} T={T}")
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    E, d_in, d_out = 4, 200 if dtype == "bf16" else 204, 264
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    x = torch.rand(T, d_in, generator=g, device="cuda").to(t) + 0.5
    Wt = torch.rand(E, d_out, d_in, generator=g, device="cuda").to(t) + 0.5
    ids = (torch.arange(T, device="cuda", dtype=torch.int32) % E)[:, None].contiguous()
    rt = ace.ace_group_permute(ids, E, None, 0, ace.ACE_ROWS_EXPERT)
    Wt[:, 131, d_in - 1] = float("inf")
    x[5, d_in - 2] = float("-inf")
    y = torch.zeros(T, d_out, dtype=t, device="cuda")
    ace.ace_moe_lora_fwd(x, Wt, rt, y)
    # (row 5, column 131 adds inf and -inf)
    want = (Wt.double()[ids[:, 0].long()] * x.double()[:, None]).sum(-1)
    inf = want.isinf()
    assert inf.sum() == T - 1 + d_out - 1
    assert torch.equal(y.double()[inf], want[inf])
    fin = want.isfinite()
    assert y[fin].isfinite().all()
    check_all("y", f64(torch.where(fin, y, 0)), f64(torch.where(fin, want, 0)), TOL[dtype])


@pytest.mark.parametrize("N", [8192, 9001, 16384, 16388, 20480, 24001, 28000, 32701])
@pytest.mark.parametrize("d_in", [64, 136])
def test_cka_probe_tiles(N, d_in):
    """Probe tiles of 32 to 128 rows in steps of 16 (one round of 256 blocks
    each) and rows too long for the mean pass's registers (above 16384)."""
    from paper_2609_06072_amd import ace
    cfg = W.CONFIGS["olmoe_bf16"].scaled(d_model=d_in, d_ffn=24, E=5, r_e=4, groups=("consecutive", 3))
    pa = W.make_probe_adapters(cfg, "gate", N=N, seed=2, device="cuda")
    say(f"cka N={N} d_in={d_in}")
    S = f64(ace.ace_pairwise_cka(pa.X, pa.A, pa.B, pa.E, pa.r))
    ref = C.cka_matrix(f64(pa.X), f64(pa.A), f64(pa.B), pa.E, pa.r)
    assert np.max(np.abs(S - ref)) <= 1e-4


@pytest.mark.parametrize("reuse_h", [False, True])
@pytest.mark.parametrize("pair_row", [True, False])
@pytest.mark.parametrize("path,r_e", [("combined", 5), ("combined", 16), ("combined_expertwise", 8)])
def test_combined_row_sums(path, r_e, pair_row, reuse_h, monkeypatch):
    """bf16 rows summed in the contraction; a routing without pair_row (which
    these calls don't ask for) takes the pass of its own."""
    from paper_2609_06072_amd import ace
    cfg = W.CONFIGS["olmoe_bf16"].scaled(T=333, k=6, E=16, d_model=136, d_ffn=72, r_e=r_e)
    c = make_case(cfg, path, seed=5, with_w=True)
    if not pair_row:
        permute = ace.ace_group_permute

        def without(*a, **kw):
            rt = permute(*a, **kw)
            rt.c.pair_row = None
            return rt
        monkeypatch.setattr(ace, "ace_group_permute", without)
    say(f"{path} r={r_e} pair_row={pair_row} reuse_h={reuse_h}")
    out = run_gpu(c, reuse_h=reuse_h)
    tol = TOL["bf16"]
    check_all("y", f64(out["y"]), oracle_fwd(c), tol)
    dx, dA, dB = oracle_bwd(c)
    check_all("dx", f64(out["dx"]), dx, tol)
    check_all("dA", f64(out["dA"]), dA, tol)
    check_dB_rows("dB", f64(out["dB"]), dB, c.ranks, c.d_out, tol)


@pytest.mark.parametrize("path", ["combined", "combined_expertwise", "grouped"])
@pytest.mark.parametrize("E,r_e", [(60, 5), (15, 5), (6, 6), (12, 12)])
def test_row_sums_ragged_rank_total(path, E, r_e):
    """Dense rows of a total rank that is no multiple of 8 (300, 75, 36): a
    rank chunk that starts at a multiple of 8 is 16-byte aligned in some
    tokens' rows only (144: in all of them)."""
    cfg = W.CONFIGS["olmoe_bf16"].scaled(T=333, k=3, E=E, d_model=136, d_ffn=72, r_e=r_e,
                                         groups=("consecutive", 4))
    c = make_case(cfg, path, seed=10, with_w=True)
    say(f"{path} total rank {sum(c.ranks)}")
    out = run_gpu(c, reuse_h=True)
    tol = TOL["bf16"]
    check_all("y", f64(out["y"]), oracle_fwd(c), tol)
    dx, dA, dB = oracle_bwd(c)
    check_all("dx", f64(out["dx"]), dx, tol)
    check_all("dA", f64(out["dA"]), dA, tol)
    check_dB_rows("dB", f64(out["dB"]), dB, c.ranks, c.d_out, tol)


@pytest.mark.parametrize("path", ["combined", "combined_pairs"])
@pytest.mark.parametrize("fwd_pair_row,bwd_pair_row", [(True, False), (False, True)])
def test_combined_h_place(path, fwd_pair_row, bwd_pair_row):
    """Where the backward finds the forward's h (bf16) depends on the type and
    the row mode, not on whether either call's routing has pair_row."""
    from paper_2609_06072_amd import ace
    cfg = W.CONFIGS["olmoe_bf16"].scaled(T=333, k=6, E=16, d_model=136, d_ffn=72, r_e=8)
    c = make_case(cfg, path, seed=9, with_w=True)
    say(f"{path} pair_row fwd={fwd_pair_row} bwd={bwd_pair_row}")
    rt = ace.ace_group_permute(torch.from_numpy(c.rt.topk_ids).cuda(), cfg.E,
                               torch.from_numpy(c.rt.expert_to_group).cuda(), c.rt.G, c.mode)
    pair_row = rt.c.pair_row
    need = ace.ace_workspace_bytes(ace.ACE_OP_FWD, cfg.T, cfg.k, c.d_in, c.d_out, c.n_keys, max(c.ranks))
    ws = torch.full((need,), 0xff, dtype=torch.uint8, device="cuda")   # NaN where nothing is stored
    y = torch.zeros(cfg.T, c.d_out, dtype=c.x.dtype, device="cuda")
    rt.c.pair_row = pair_row if fwd_pair_row else None
    ace.ace_grouped_lora_fwd(c.x, c.A, c.B, c.ranks, cfg.alpha, rt, y, c.pair_w, c.input_mode, ws)
    dx, dA = torch.zeros_like(c.x), torch.empty(sum(c.ranks), c.d_in, device="cuda")
    dB = torch.empty(sum(c.ranks) * c.d_out, device="cuda")
    rt.c.pair_row = pair_row if bwd_pair_row else None
    ace.ace_grouped_lora_bwd(c.x, c.A, c.B, c.ranks, cfg.alpha, rt, c.dy, dx, dA, dB, c.pair_w, c.input_mode,
                             h_fwd=ws)
    tol = TOL["bf16"]
    check_all("y", f64(y), oracle_fwd(c), tol)
    rx, rA, rB = oracle_bwd(c)
    check_all("dx", f64(dx), rx, tol)
    check_all("dA", f64(dA), rA, tol)
    check_dB_rows("dB", f64(dB), rB, c.ranks, c.d_out, tol)


@pytest.mark.parametrize("reuse_h", [False, True])
@pytest.mark.parametrize("with_w", [False, True])
@pytest.mark.parametrize("dtype,T", [("bf16", 57), ("bf16", 900), ("f32", 57), ("f32", 900)])
def test_combined_single_pair_rows(dtype, T, with_w, reuse_h):
    """Pre-combined output over group-keyed rows of single pairs: a token has
    several rows of a group, whose h add up in its dense row while dB keeps
    each row's own."""
    cfg = W.CONFIGS["olmoe_bf16"].scaled(dtype=dtype, T=T, k=6, E=16, d_model=136, d_ffn=72, r_e=8)
    c = make_case(cfg, "combined_pairs", seed=8, with_w=with_w)
    say(f"combined pairs {dtype} T={T} w={with_w} reuse_h={reuse_h}")
    out = run_gpu(c, reuse_h=reuse_h)
    tol = TOL[dtype]
    check_all("y", f64(out["y"]), oracle_fwd(c), tol)
    dx, dA, dB = oracle_bwd(c)
    check_all("dx", f64(out["dx"]), dx, tol)
    check_all("dA", f64(out["dA"]), dA, tol)
    check_dB_rows("dB", f64(out["dB"]), dB, c.ranks, c.d_out, tol)


def test_rank_lists_by_value():
    """A rank list changed in place between calls is read anew."""
    cfg = W.CONFIGS["olmoe_bf16"].scaled(T=50, E=4, k=2, groups=("consecutive", 2), d_model=64, d_ffn=64)
    c = make_case(cfg, "grouped", seed=6)
    for ranks in ([16, 16], [8, 24], [24, 8]):
        c.ranks[:] = ranks
        check_all(f"y {ranks}", f64(run_gpu(c, bwd=False)["y"]), oracle_fwd(c), TOL["bf16"])

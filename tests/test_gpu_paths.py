"""The bf16 transpose kernel, and the block calls with a workspace against
the same calls without one.

With a workspace the forward runs from W^T and dW from X^T and dY^T (both
operands contiguous along k); without one they read W, X and dY as given
(transposing LDS reads), and so does a call with one where its model has the
copies cost more than they give: every dW of the small cases here, so the
copies have cases of their own.  Both layouts sum each element's products in the
same order, so the paths give the same bits, except that with a workspace
chunk products with too few output tiles to fill the chip are split over k,
which sums in a different order: there the paths agree to fp32 rounding,
and a bf16 output differs by at most a couple of units in the last place
where the two fp32 values straddle a rounding boundary.  fc1's dW and db are
token sums of the bf16 dh_pre, which may sit one unit apart between the
paths, so they get a looser bound.  Where no product splits (the wide 8 x 1
layer) the paths agree bit for bit.  Both paths are checked against the
oracle elsewhere."""
import pytest
import torch

import paper_2301_08658_amd as atp
import synth_inputs as S
from helpers import assert_paths_agree, make_block_inputs, run_block_bwd, run_block_fwd

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def bits(t):
    return t.contiguous().view(torch.int16 if t.element_size() == 2 else torch.int32)


@pytest.mark.parametrize("rows,cols,pad_s,pad_d", [
    (1, 8, 0, 0), (7, 16, 8, 0), (64, 64, 0, 8), (65, 72, 0, 0), (300, 200, 16, 24),
    (513, 1032, 8, 8), (4096, 2560, 0, 0), (2, 4104, 0, 8),
    # multiples of 8 (the register-block kernel), with partial 64 x 256 tiles
    (8, 8, 0, 0), (72, 264, 8, 8), (4104, 520, 0, 8), (136, 2056, 16, 0)])
def test_transpose_matches_torch(rows, cols, pad_s, pad_d):
    print(f"transpose {rows}x{cols} pads {pad_s},{pad_d}", flush=True)
    src_full = S.randint_bf16((rows, cols + pad_s), 7, 901).to(DEV)
    src = src_full[:, :cols]
    ldd = ((rows + 7) // 8) * 8 + pad_d
    dst_full = torch.full((cols, ldd), -1.0, dtype=torch.bfloat16, device=DEV)
    atp.atp_transpose_bf16(src, dst_full[:, :rows])
    torch.cuda.synchronize()
    assert torch.equal(bits(dst_full[:, :rows]), bits(src.t().contiguous()))
    if ldd > rows:   # the padding columns are left alone
        assert torch.all(dst_full[:, rows:] == -1.0)


def test_transpose_empty_and_errors():
    z = torch.empty((0, 8), dtype=torch.bfloat16, device=DEV)
    atp.atp_transpose_bf16(z, torch.empty((8, 0), dtype=torch.bfloat16, device=DEV))
    a = torch.zeros((16, 16), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(atp.AtpError):
        atp.atp_transpose_bf16(a, a)            # in place is not supported


CASES = [  # (mode, mesh, coord, T, h, chunks)
    ("col", (2, 2), (1, 0), 256, 512, 2),
    ("col", (2, 4), (1, 3), 512, 1024, 4),
    ("row", (4, 2), (3, 1), 512, 1024, 4),
    ("col", (1, 1), (0, 0), 128, 256, 1),
    ("col", (8, 1), (7, 0), 256, 2048, 2),
    ("col", (2, 2), (0, 1), 200, 512, 2),     # tokens % 8 == 0, not a tile multiple
    ("row", (2, 2), (1, 1), 132, 512, 2),     # tokens % 8 != 0: dW falls back to TN
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}{c[1][0]}x{c[1][1]}_T{c[3]}")
def test_block_forward_workspace_equals_direct(case):
    mode, mesh, coord, T, h, chunks = case
    inp = make_block_inputs(mode, mesh, coord, T, h, 0.02, seed=21, on_device=True)
    print(f"fwd {case}", flush=True)
    a = run_block_fwd(inp, chunks)
    b = run_block_fwd(inp, chunks, workspace=True)
    torch.cuda.synchronize()
    for k in ("qkv", "o", "h", "pre", "z"):
        assert_paths_agree(a[k], b[k], k)
    for i, (x, y) in enumerate(zip(a["own"], b["own"])):
        if x is not None:
            assert_paths_agree(x, y, f"partial {i}")


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}{c[1][0]}x{c[1][1]}_T{c[3]}")
def test_block_backward_workspace_equals_direct(case):
    mode, mesh, coord, T, h, chunks = case
    inp = make_block_inputs(mode, mesh, coord, T, h, 0.02, seed=22, on_device=True, bwd=True)
    print(f"bwd {case}", flush=True)
    a = run_block_bwd(inp, chunks)
    b = run_block_bwd(inp, chunks, workspace=True)
    torch.cuda.synchronize()
    _check_bwd_paths(a, b)


def _check_bwd_paths(a, b):
    for k in ("dh_pre", "dx_qkv", "dx_fc1", "d_attn"):
        assert_paths_agree(a[k], b[k], k)
    for i in range(4):
        rel = 2e-3 if i == 2 else 1e-4
        assert_paths_agree(a["dw"][i], b["dw"][i], f"dw {i}", rel)
        assert_paths_agree(a["db"][i], b["db"][i], f"db {i}", rel)


def _names(fn):
    atp.atp_profile_enable(1)
    try:
        fn()
        torch.cuda.synchronize()
        return {r["name"]: r["launches"] for r in atp.atp_profile_collect(256)}
    finally:
        atp.atp_profile_enable(0)


# sizes at which all four dW run from copies: long token ranges of few columns,
# whose last 64-row block of column partials holds 8 rows
COPY_CASES = [("col", (4, 2), (1, 0), 8200, 512, 2), ("row", (1, 8), (0, 5), 8200, 512, 1)]


@pytest.mark.parametrize("layout", [atp.ATP_W_KN, atp.ATP_W_NK], ids=["kn", "nk"])
@pytest.mark.parametrize("case", COPY_CASES, ids=lambda c: f"{c[0]}{c[1][0]}x{c[1][1]}")
def test_weight_gradients_from_copies_equal_direct(case, layout):
    """dW and db from X^T (one copy of x for QKV and fc1) and dY^T against the
    call that reads X and dY as given: the profile shows which ran."""
    mode, mesh, coord, T, h, chunks = case
    print(f"dW copies {case} layout {layout}", flush=True)
    inp = make_block_inputs(mode, mesh, coord, T, h, 0.02, seed=24, on_device=True, bwd=True,
                            layout=layout)
    res = []
    a = _names(lambda: res.append(run_block_bwd(inp, chunks)))
    b = _names(lambda: res.append(run_block_bwd(inp, chunks, workspace=True)))
    assert any(n.startswith("gemm_tn") for n in a) and "transpose" not in a, a
    assert not any(n.startswith("gemm_tn") for n in b), b
    # X^T of x, attention block and H, dY^T of four linears, and with weights
    # stored [n][k] their four [k][n] copies
    assert b["transpose"] == (7 if layout == atp.ATP_W_KN else 11), b
    _check_bwd_paths(*res)
    for i in (0, 1, 3):     # fc1's dY is a reduced product, which may be split
        assert torch.equal(bits(res[0]["dw"][i]), bits(res[1]["dw"][i])), f"dw {i}"
        assert torch.equal(bits(res[0]["db"][i]), bits(res[1]["db"][i])), f"db {i}"


def test_benchmark_workload_workspace_equals_direct():
    """No chunk product of the wide 8 x 1 layer splits: bit for bit."""
    w = S.WORKLOADS["wide_h20480_col_8x1"]
    inp = make_block_inputs(w["mode"], w["mesh"], (0, 0), w["tokens"], w["h"], w["sigma_w"],
                            seed=23, on_device=True, bwd=True)
    print("bench workload fwd+bwd, both paths", flush=True)
    fa = run_block_fwd(inp, w["chunks"])
    fb = run_block_fwd(inp, w["chunks"], workspace=True)
    ba = run_block_bwd(inp, w["chunks"])
    bb = run_block_bwd(inp, w["chunks"], workspace=True)
    torch.cuda.synchronize()
    for k in ("qkv", "o", "h", "pre", "z"):
        assert torch.equal(bits(fa[k]), bits(fb[k])), k
    for k in ("dh_pre", "dx_qkv", "dx_fc1", "d_attn"):
        assert torch.equal(bits(ba[k]), bits(bb[k])), k
    for i in range(4):
        assert torch.equal(bits(ba["dw"][i]), bits(bb["dw"][i])), f"dw {i}"
        assert torch.equal(bits(ba["db"][i]), bits(bb["db"][i])), f"db {i}"


def test_largest_leading_dimension_runs_from_copies():
    """Leading dimensions of 4M elements are accepted, and more than a product's
    32-bit offsets span: with a workspace W and X of that pitch are read only
    by the copies (forward W^T, backward X^T), with the same results."""
    print("leading dimension 4M", flush=True)
    T, h = 8, 64
    inp = make_block_inputs("col", (1, 1), (0, 0), T, h, 0.02, seed=47, bwd=True)

    def wide(t):
        w = torch.empty((t.shape[0], 1 << 22), dtype=t.dtype, device=t.device)[:, :t.shape[1]]
        return w.copy_(t)
    ref, rbwd = run_block_fwd(inp, 1, workspace=True), run_block_bwd(inp, 1, workspace=True)
    torch.cuda.synchronize()
    out = run_block_fwd(dict(inp, w=[wide(inp["w"][0])] + inp["w"][1:]), 1, workspace=True)
    bwd = run_block_bwd(dict(inp, x=wide(inp["x"])), 1, workspace=True)
    torch.cuda.synchronize()
    for k in ("qkv", "o", "h", "pre", "z"):
        assert torch.equal(out[k], ref[k]), k
    for i in range(4):
        assert torch.equal(bwd["dw"][i], rbwd["dw"][i]) and torch.equal(bwd["db"][i],
                                                                        rbwd["db"][i]), i

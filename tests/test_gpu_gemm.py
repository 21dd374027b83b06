"""GPU parity of the shard-linear GEMMs (Sec. 3.2 forward, Sec. 4.2
backward) against the fp64 oracle.  Integer-valued inputs make every fp32
sum exact, so those cases must match bit for bit; random inputs are held to
the stated tolerance.  Shapes are ragged on purpose (not multiples of the
256 x 256 x 64 tile) and span several tiles."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2301_08658_amd as atp
import synth_inputs as S
from helpers import DEV, assert_close, to64

pytestmark = pytest.mark.gpu


def _sync():
    torch.cuda.synchronize()


@pytest.mark.parametrize("T,K,N,chunks", [(300, 200, 264, 1), (512, 320, 520, 4),
                                          (96, 64, 8, 3), (8, 8, 8, 1)])
def test_fwd_nn_integer_bit_exact(T, K, N, chunks):
    m = atp.mesh(1, 1)
    x = S.randint_bf16((T, K), 1, 1).to(DEV)
    w = S.randint_bf16((K, N), 1, 2).to(DEV)
    y = torch.full((T, N), float("nan"), device=DEV)
    atp.atp_shard_linear_fwd(m, atp.ATP_ROW_FIRST, T, K, N, chunks, x, w, None,
                             atp.ATP_EPI_NONE, y)
    _sync()
    ref = O.matmul(x.cpu(), w.cpu())
    np.testing.assert_array_equal(to64(y), ref)


@pytest.mark.parametrize("T,K,N,chunks", [(300, 200, 264, 3), (640, 72, 296, 2)])
def test_bwd_nt_tn_colsum_integer_bit_exact(T, K, N, chunks):
    m = atp.mesh(1, 1)
    x = S.randint_bf16((T, K), 2, 1).to(DEV)
    w = S.randint_bf16((K, N), 2, 2).to(DEV)
    dy = S.randint_bf16((T, N), 2, 3).to(DEV)
    dx = torch.full((T, K), float("nan"), device=DEV)
    dw = torch.full((K, N), float("nan"), device=DEV)
    db = torch.full((N,), float("nan"), device=DEV)
    atp.atp_shard_linear_bwd(m, atp.ATP_ROW_FIRST, T, K, N, chunks, x, w, dy, dx, dw, db)
    _sync()
    rdx, rdw, rdb = O.linear_bwd(x.cpu(), w.cpu(), dy.cpu())
    np.testing.assert_array_equal(to64(dx), rdx)
    np.testing.assert_array_equal(to64(dw), rdw)
    np.testing.assert_array_equal(to64(db), rdb)


@pytest.mark.parametrize("T,K,N,chunks", [(1, 8, 8, 1), (7, 16, 24, 1), (64, 40, 8, 2),
                                          (257, 168, 40, 1), (700, 488, 1000, 2),
                                          (512, 160, 2056, 4), (1024, 1288, 72, 8)])
def test_dx_nt_ragged_integer_bit_exact(T, K, N, chunks):
    """dX = dY W^T on the small tiles (64 x 64 to 128 x 128):
    outputs of one row, sub-tile and multi-tile sizes with ragged edges, and
    contractions shorter than one K step or ending in a partial one."""
    m = atp.mesh(1, 1)
    x = S.randint_bf16((T, K), 6, 1).to(DEV)
    w = S.randint_bf16((K, N), 6, 2).to(DEV)
    dy = S.randint_bf16((T, N), 6, 3).to(DEV)
    dx = torch.full((T, K), float("nan"), device=DEV)
    dw = torch.full((K, N), float("nan"), device=DEV)
    atp.atp_shard_linear_bwd(m, atp.ATP_ROW_FIRST, T, K, N, chunks, x, w, dy, dx, dw, None)
    _sync()
    rdx, rdw, _ = O.linear_bwd(x.cpu(), w.cpu(), dy.cpu())
    np.testing.assert_array_equal(to64(dx), rdx)
    np.testing.assert_array_equal(to64(dw), rdw)


@pytest.mark.parametrize("epi", [atp.ATP_EPI_NONE, atp.ATP_EPI_BIAS, atp.ATP_EPI_BIAS_GELU])
@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
def test_fwd_epilogues_group_of_one(epi, out_dtype):
    T, K, N = 264, 136, 392
    m = atp.mesh(1, 1)
    x = S.randn_bf16((T, K), 1.0, 3, 1).to(DEV)
    w = S.randn_bf16((K, N), 0.1, 3, 2).to(DEV)
    b = S.randn_bf16((N,), 0.5, 3, 3).to(DEV)
    y = torch.full((T, N), float("nan"), device=DEV, dtype=out_dtype)
    pre = torch.full((T, N), float("nan"), device=DEV, dtype=torch.bfloat16) \
        if epi == atp.ATP_EPI_BIAS_GELU else None
    atp.atp_shard_linear_fwd(m, atp.ATP_COL_FIRST, T, K, N, 2, x, w, b, epi, y, preact=pre)
    _sync()
    oepi = {atp.ATP_EPI_NONE: O.EPI_NONE, atp.ATP_EPI_BIAS: O.EPI_BIAS,
            atp.ATP_EPI_BIAS_GELU: O.EPI_BIAS_GELU}[epi]
    ref, rpre = O.linear_fwd_reduced(x.cpu(), w.cpu(), 0, [], b.cpu(), oepi)
    assert_close(y, ref, "y")
    if pre is not None:
        assert_close(pre, rpre, "preact")


@pytest.mark.parametrize("mesh,mode", [((2, 2), 0), ((2, 4), 1), ((4, 2), 0)])
def test_partial_block_every_coordinate(mesh, mode):
    """The device's Partial(SUM) block for every coordinate, cut from global
    X and W by the shard geometry, against the oracle's spec-derived block."""
    d1, d2 = mesh
    T, K, N = 136, 256, 512
    X = S.randn_bf16((T, K), 1.0, 4, 1)
    W = S.randn_bf16((K, N), 0.05, 4, 2)
    for i1 in range(d1):
        for i2 in range(d2):
            m = atp.mesh(d1, d2, i1, i2)
            g = atp.atp_shard_geometry(m, mode, K, N)
            x_loc = X[:, g.k_off:g.k_off + g.k_loc].contiguous().to(DEV)
            w_loc = W[g.k_off:g.k_off + g.k_loc, g.n_off:g.n_off + g.n_loc].contiguous().to(DEV)
            y = torch.empty((T, g.n_loc), device=DEV)
            atp.atp_shard_linear_fwd(m, mode, T, K, N, 2, x_loc, w_loc, None, 0, y)
            _sync()
            ref = O.local_partial(X, W, mesh, (i1, i2), mode)
            assert_close(y, ref, f"partial {(i1, i2)}")


def test_fwd_leading_dimensions_and_empty():
    """Strided views (ld > cols) and zero tokens."""
    T, K, N = 130, 64, 136
    m = atp.mesh(1, 1)
    xb = S.randint_bf16((T, K + 24), 5, 1).to(DEV)
    wb = S.randint_bf16((K, N + 40), 5, 2).to(DEV)
    yb = torch.full((T, N + 8), -7.0, device=DEV)
    x, w, y = xb[:, :K], wb[:, :N], yb[:, :N]
    atp.atp_shard_linear_fwd(m, 0, T, K, N, 2, x, w, None, 0, y)
    _sync()
    np.testing.assert_array_equal(to64(y), O.matmul(x.cpu(), w.cpu()))
    assert torch.all(yb[:, N:] == -7.0)
    y0 = torch.empty((0, N), device=DEV)
    atp.atp_shard_linear_fwd(m, 0, 0, K, N, 4, x[:0], w, None, 0, y0)
    _sync()


@pytest.mark.parametrize("tile,M,N,K", [
    ("64", 8, 8, 8), ("64", 520, 1160, 72), ("64x128", 1000, 1032, 136), ("128", 520, 6152, 200),
    ("128", 1000, 2056, 1608), ("256x128", 1000, 6152, 136), ("256x128", 776, 6152, 1000),
    ("256", 2048, 8000, 328), ("256", 1400, 7160, 1000), ("256", 520, 13608, 40),
    ("", 4872, 1544, 40), ("", 520, 10904, 328), ("", 520, 13088, 1608)])
def test_every_tile_and_layout_integer_bit_exact(tile, M, N, K):
    """Each tile configuration that serves the three layouts (NN forward, NT
    dX, TN dW; no suffix: 256 x 160) at sizes with partial tiles on both sides and a partial last K step
    (one shorter than the copy ring), against the 64-bit product: integer
    inputs keep every fp32 sum exact.  The profile names the tile that ran."""
    m = atp.mesh(1, 1)
    draw = lambda r, c, t: S.randint_bf16((r, c), 8, t).to(DEV)  # noqa: E731
    nan = lambda r, c: torch.full((r, c), float("nan"), device=DEV)  # noqa: E731
    print(f"tile {tile} {M}x{N}x{K}", flush=True)
    got, names = {}, []
    atp.atp_profile_enable(1)
    try:
        x, w = draw(M, K, 1), draw(K, N, 2)
        y = nan(M, N)
        atp.atp_shard_linear_fwd(m, 0, M, K, N, 1, x, w, None, atp.ATP_EPI_NONE, y)
        got["nn"] = (y, x, w)
        dy, wt = draw(M, K, 3), draw(N, K, 4)          # dX [M, N] = dY [M, K] W^T [K, N]
        dx = nan(M, N)
        atp.atp_shard_linear_bwd(m, 0, M, N, K, 1, draw(M, N, 5), wt, dy, dx, nan(N, K))
        got["nt"] = (dx, dy, wt.t())
        xs, dys = draw(K, M, 6), draw(K, N, 7)         # dW [M, N] = X^T [M, K] dY [K, N]
        dw = nan(M, N)
        atp.atp_shard_linear_bwd(m, 0, K, M, N, 1, xs, draw(M, N, 8), dys, nan(K, M), dw)
        got["tn"] = (dw, xs.t(), dys)
        torch.cuda.synchronize()
        names = [r["name"] for r in atp.atp_profile_collect(64)]
    finally:
        atp.atp_profile_enable(0)
    for lay, (out, a, b) in got.items():
        assert any(n.startswith(f"gemm_{lay}{tile}_") for n in names), (lay, names)
        ref = torch.matmul(a.double(), b.double())
        assert torch.equal(out.double(), ref), lay


@pytest.mark.parametrize("tile,M,N,K", [
    ("320", 1310, 10800, 72), ("320", 1537, 9240, 40), ("320", 1537, 9240, 1000),
    ("256", 533, 13608, 360), ("", 4867, 1544, 72)])
def test_large_k_contiguous_tiles_ragged_integer_bit_exact(tile, M, N, K):
    """256 x 320 (K steps of 32), 256 x 256 and 256 x 160 of a product with both
    operands along k (dX): rows that are no multiple of 8, partial last row and
    column tiles, a contraction of one or two K steps and a partial last one,
    against the 64-bit product of integer inputs."""
    m = atp.mesh(1, 1)
    print(f"NT tile {tile or 160} {M}x{N}x{K}", flush=True)
    dy, w = S.randint_bf16((M, K), 11, 1).to(DEV), S.randint_bf16((N, K), 11, 2).to(DEV)
    x, dw = S.randint_bf16((M, N), 11, 3).to(DEV), torch.empty((N, K), device=DEV)
    dx = torch.full((M, N), float("nan"), device=DEV)
    atp.atp_profile_enable(1)
    try:
        atp.atp_shard_linear_bwd(m, 0, M, N, K, 1, x, w, dy, dx, dw)
        _sync()
        names = [r["name"] for r in atp.atp_profile_collect(8)]
    finally:
        atp.atp_profile_enable(0)
    assert f"gemm_nt{tile}_e0_f32" in names, names
    assert torch.equal(dx.double(), torch.matmul(dy.double(), w.double().t()))


@pytest.mark.parametrize("epi", [atp.ATP_EPI_NONE, atp.ATP_EPI_BIAS, atp.ATP_EPI_BIAS_GELU])
def test_tiles_of_calls_with_and_without_events_same_bits(epi):
    """A forward runs on 256 x 160 tiles where nothing is beside it and on others
    where the caller passes chunk events, with the same bits; so do the fused
    peer sum there and the product with its reduction."""
    T, K, N = 520, 328, 10904
    print(f"alone and with events epi={epi}", flush=True)
    x, w = S.randn_bf16((T, K), 1.0, 12, 1).to(DEV), S.randn_bf16((K, N), 0.05, 12, 2).to(DEV)
    b = S.randn_bf16((N,), 0.5, 12, 3).to(DEV) if epi != atp.ATP_EPI_NONE else None
    out, pre, names = [], [], []
    for ev in (None, [atp.HipEvent()]):
        y = torch.full((T, N), float("nan"), device=DEV, dtype=torch.bfloat16)
        q = torch.empty_like(y) if epi == atp.ATP_EPI_BIAS_GELU else None
        atp.atp_profile_enable(1)
        try:
            atp.atp_shard_linear_fwd(atp.mesh(1, 1), 0, T, K, N, 1, x, w, b, epi, y, preact=q,
                                     chunk_done=ev)
            _sync()
            names.append([r["name"] for r in atp.atp_profile_collect(8)][0])
        finally:
            atp.atp_profile_enable(0)
        out.append(y)
        pre.append(q)
    assert names[0].startswith("gemm_nn_e") and not names[1].startswith("gemm_nn_e"), names
    assert torch.equal(*out) and (pre[0] is None or torch.equal(*pre))
    # a group of two: the fused peer sum on 256 x 160 against product, then reduction
    m = atp.mesh(2, 1, 1, 0)
    g = atp.atp_shard_geometry(m, atp.ATP_ROW_FIRST, 2 * K, N)
    assert (g.k_loc, g.n_loc, g.red_size, g.red_index) == (K, N, 2, 1)
    peer, own = S.randn_f32((T, N), 1.0, 12, 4).to(DEV), torch.empty((T, N), device=DEV)
    atp.atp_shard_linear_fwd(m, atp.ATP_ROW_FIRST, T, 2 * K, N, 1, x, w, None, atp.ATP_EPI_NONE, own)
    want, fused = torch.empty_like(out[0]), torch.empty_like(out[0])
    pw, pf = ((torch.empty_like(want), torch.empty_like(want))
              if epi == atp.ATP_EPI_BIAS_GELU else (None, None))
    atp.atp_chunked_partial_reduce(2, T, N, 1, [peer, own], b, epi, want, preact_out=pw)
    atp.atp_shard_linear_fwd_fused(m, atp.ATP_ROW_FIRST, T, 2 * K, N, x, w, [peer, None], b, epi,
                                   fused, pf)
    _sync()
    assert torch.equal(want, fused) and (pw is None or torch.equal(pw, pf))


@pytest.mark.parametrize("T,N", [(1, 8), (4099, 40), (130, 72), (2100, 4096), (2100, 4104),
                                 (1024, 8192), (5000, 8200), (3, 16392), (1030, 16392)])
def test_bias_gradient_rounds_and_widths_integer_bit_exact(T, N):
    """db alone (the column sum) over one and several rounds of row blocks,
    in blocks of 16, 32 and 64 columns (up to 4096 columns; up to 8192 and,
    from 1000 rows on, past 16384; the others), with partial 8-row groups, row
    blocks and column blocks."""
    print(f"column sum {T}x{N}", flush=True)
    dy = S.randint_bf16((T, N), 9, 1).to(DEV)
    x, w = S.randint_bf16((T, 8), 9, 2).to(DEV), S.randint_bf16((8, N), 9, 3).to(DEV)
    db = torch.full((N,), float("nan"), device=DEV)
    atp.atp_shard_linear_bwd(atp.mesh(1, 1), 0, T, 8, N, 1, x, w, dy,
                             torch.empty((T, 8), device=DEV), torch.empty((8, N), device=DEV), db)
    _sync()
    assert torch.equal(db.double(), dy.double().sum(0))


@pytest.mark.parametrize("marked", [(), (1,), (0, 2), (0, 1, 2, 3)])
def test_chunks_run_together_up_to_the_next_event(marked):
    """Chunks with no event between them run as one launch: the products, the
    reduction and every event's rows are those of single chunks."""
    T, K, N, chunks = 264, 96, 136, 4
    m = atp.mesh(1, 1)
    print(f"events at {marked}", flush=True)
    ev = [atp.HipEvent() if c in marked else None for c in range(chunks)]
    x, w = S.randint_bf16((T, K), 10, 1).to(DEV), S.randint_bf16((K, N), 10, 2).to(DEV)
    dy = S.randint_bf16((T, N), 10, 3).to(DEV)
    y, dx = torch.full((T, N), float("nan"), device=DEV), torch.full((T, K), float("nan"), device=DEV)
    dw, z = torch.empty((K, N), device=DEV), torch.full((T, N), float("nan"), device=DEV)
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    atp.atp_shard_linear_fwd(m, 0, T, K, N, chunks, x, w, None, atp.ATP_EPI_NONE, y, chunk_done=ev)
    # the reduction on another stream waits for the same events, then for all
    if marked and marked[-1] != chunks - 1 or not marked:
        torch.cuda.synchronize()
    atp.atp_chunked_partial_reduce(2, T, N, chunks, [y, y], None, atp.ATP_EPI_NONE, z,
                                   stream=other, chunk_ready=ev)
    atp.atp_shard_linear_bwd(m, 0, T, K, N, chunks, x, w, dy, dx, dw, None, dx_chunk_done=ev)
    for e in ev:
        if e is not None:
            e.synchronize()
    _sync()
    ref = torch.matmul(x.double(), w.double())
    assert torch.equal(y.double(), ref) and torch.equal(z.double(), 2 * ref)
    assert torch.equal(dx.double(), torch.matmul(dy.double(), w.double().t()))

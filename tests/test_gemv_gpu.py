"""Parity of the HIP GEMV (through the C ABI) against the float64 oracle on MI355X.

Tolerance (stated by the benchmark spec): max relative error <= 2e-3 with fp32 accumulation and
fp16 output, the denominator floored at 1% of the rms of the reference vector.
Packed buffers are compared bit for bit in tests/test_pack_bitexact.py (no GPU needed).
"""
from __future__ import annotations

import numpy as np
import pytest

import gqsa_inputs as gi
import oracle
import paper_2412_17560_amd as gq

pytestmark = pytest.mark.gpu

TOL = 2e-3


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    return torch


def run_gemv(torch, h, x_np, panels=False):
    x = torch.from_numpy(np.ascontiguousarray(x_np)).cuda()
    n = gq.gqsa_info(h)["N"]
    y = torch.full((x.shape[0], n), float("nan"), dtype=torch.float16, device="cuda")
    gq.gqsa_gemv(h, x, y, panels=panels)
    torch.cuda.synchronize()
    return y.cpu().numpy()


def check(torch, h, c, x_np, tol=TOL, panels=False):
    y = run_gemv(torch, h, x_np, panels)
    ref = oracle.gemv(c, x_np, threads=8)
    assert np.isfinite(y).all()
    for b in range(x_np.shape[0]):
        err = oracle.rel_error(y[b], ref[b])
        assert err <= tol, f"batch row {b}: rel err {err:.3e}"
    # rows without stored groups are exactly +0
    empty = np.diff(c.rowIndex) == 0
    if empty.any():
        assert (y.view(np.uint16)[:, empty] == 0).all()
    return y, ref


def test_tiny_config(torch_cuda):
    W, x = gi.tiny_config()
    h = gq.gqsa_pack(W, 16, 4, 0.5)
    c = oracle.pack(W, 16, 4, sparsity=0.5)
    check(torch_cuda, h, c, x)


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("sparsity", [0.0, 0.3, 0.5, 0.7, 1.0])
def test_balanced_ragged_shapes(torch_cuda, bits, sparsity):
    # 301 rows x 61 group-columns: nothing aligns with 64-group blocks or 256-group tiles
    N, K = 301, 976
    W = gi.dense_weight(N, K, seed=100 + bits)
    h = gq.gqsa_pack(W, 16, bits, sparsity)
    c = oracle.pack(W, 16, bits, sparsity=sparsity)
    check(torch_cuda, h, c, gi.activations(1, K, seed=5))


@pytest.mark.parametrize("part", [(1, 1), (2, 1), (3, 1), (7, 1), (1, 16), (2, 16), (3, 5), (33, 2),
                                  (13, 16), (200, 1), (256, 16)])
def test_partition_sweep_imbalanced(torch_cuda, part):
    """Rows shared by 2 and by many wavefronts, inside one workgroup and across workgroups,
    empty rows, dense rows: the carry fix-up through LDS and through device memory."""
    N, K = 257, 2048
    W = gi.dense_weight(N, K, seed=31)
    keep = gi.imbalanced_keep_counts(N, K // 16, seed=31)
    c = oracle.pack(W, 16, 4, keep_per_row=keep)
    h = gq.gqsa_pack_rows(W, keep, 16, 4)
    gq.gqsa_set_partition(h, *part)
    check(torch_cuda, h, c, gi.activations(1, K, seed=6))


@pytest.mark.parametrize("part", [(8, 4), (5, 7), (16, 2), (3, 16)])
@pytest.mark.parametrize("batch", [1, 2])
def test_rows_spanning_two_and_more_workgroups(torch_cuda, part, batch):
    """Long rows over few blocks per wavefront: a row's workers sit in one, two or three
    workgroups, several of them on either side of a workgroup boundary (partial sums through LDS
    on each side, then one meeting point; three or more workgroups through the arrival counter)."""
    N, K = 9, 5120                       # 320 group-columns per row
    W = gi.dense_weight(N, K, seed=77)
    keep = np.array([320, 200, 0, 320, 37, 320, 1, 320, 255], dtype=np.int32)
    c = oracle.pack(W, 16, 4, keep_per_row=keep)
    h = gq.gqsa_pack_rows(W, keep, 16, 4)
    gq.gqsa_set_partition(h, *part)
    check(torch_cuda, h, c, gi.activations(batch, K, seed=8))


@pytest.mark.parametrize("part", [(1, 0, 1), (1, 0, 4), (2, 0, 3), (4, 0, 4), (3, 0, 16), (16, 0, 8), (4, 64, 4),
                                  (1000, 3, 16)])
@pytest.mark.parametrize("batch", [1, 3])
def test_rows_kept_inside_workgroup_spans(torch_cuda, part, batch):
    """The aligned form of the stream: null groups before the span boundaries, workers whose whole
    run is null, rows longer than a span (shared by workgroups as in the plain form), empty rows."""
    N, K = 301, 2048
    W = gi.dense_weight(N, K, seed=78)
    keep = gi.imbalanced_keep_counts(N, K // 16, seed=78)
    keep[[0, 5, 6, 7, 300]] = 0
    keep[100] = K // 16
    c = oracle.pack(W, 16, 4, keep_per_row=keep)
    h = gq.gqsa_pack_rows(W, keep, 16, 4)
    gq.gqsa_set_partition_aligned(h, *part)
    assert gq.gqsa_info(h)["span_tiles"] == part[0]
    check(torch_cuda, h, c, gi.activations(batch, K, seed=9))


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("shape", [(3, 60, 0, 4), (3, 44, 0, 1), (4, 32, 0, 4), (4, 64, 0, 16), (5, 36, 0, 3), (5, 64, 40, 8), (3, 32, 0, 4),
                                   (6, 60, 0, 8), (8, 44, 0, 4), (8, 64, 0, 16)])
def test_rows_kept_inside_workers_tiles(torch_cuda, shape, bits):
    """Tiles of a chosen shape (3, 4, 5, 6, 8 blocks; 32..64 lanes in use), one per worker, whole rows in
    them -- and, with 3 x 32, rows longer than a tile, shared by workers as in the other forms;
    ragged rows, empty rows, workers whose tile is null; every kernel for 1, 2, 4, 8 activation
    rows (3 and 7 rows run in the kernels for 4 and 8)."""
    N, K = 301, 2048
    W = gi.dense_weight(N, K, seed=78)
    keep = gi.imbalanced_keep_counts(N, K // 16, seed=78)
    keep[[0, 5, 6, 7, 300]] = 0
    keep[100] = K // 16
    c = oracle.pack(W, 16, bits, keep_per_row=keep)
    h = gq.gqsa_pack_rows(W, keep, 16, bits)
    u, lanes, wgs, wpw = shape
    if u > 5 and bits == 8:
        pytest.skip("tiles of 6 and 8 blocks exist for 4-bit codes only")
    gq.gqsa_set_partition_rows(h, u, lanes, 1, wgs, wpw)
    assert gq.gqsa_info(h)["needs_fixup"] == (1 if u * lanes < 128 else 0)
    for batch in (1, 2, 3, 4, 7, 8, 16):
        check(torch_cuda, h, c, gi.activations(batch, K, seed=9 + batch))


def test_rows_of_a_batch_are_the_single_row_results_with_chosen_tile_shapes(torch_cuda):
    """Tiles of 3 x 60 (179 groups per row): every batch size gives, row for row, the bits of the
    one-row call; q/k/v-like matrices of that shape share a launch and give the bits of separate
    calls; a matrix of another tile shape in the same call goes out in a launch of its own."""
    torch = torch_cuda
    K = 4096
    hs, cs = [], []
    for i, (N, keep_n) in enumerate(((512, 179), (128, 179), (130, 179), (256, 77))):
        W = gi.dense_weight(N, K, seed=300 + i)
        keep = np.full(N, keep_n, dtype=np.int32)
        hs.append(gq.gqsa_pack_rows(W, keep, 16, 4))
        cs.append(oracle.pack(W, 16, 4, keep_per_row=keep))
    assert [gq.gqsa_partition(h)[3:5] for h in hs] == [(3, 60), (3, 60), (3, 60), (3, 52)]
    x16 = gi.activations(16, K, seed=31)
    y16 = run_gemv(torch, hs[0], x16)
    for batch in (1, 2, 3, 4, 5, 7, 8, 11):
        y = run_gemv(torch, hs[0], x16[:batch])
        assert np.array_equal(y.view(np.uint16), y16[:batch].view(np.uint16)), batch
    for batch in (1, 4):
        x = torch.from_numpy(x16[:batch]).cuda()
        for group in (hs[:3], hs):
            ys = gq.gqsa_gemv_multi(group, x)
            torch.cuda.synchronize()
            for h, c, y in zip(group, cs, ys):
                got = y.cpu().numpy()
                assert np.array_equal(got.view(np.uint16), run_gemv(torch, h, x16[:batch]).view(np.uint16))
                ref = oracle.gemv(c, x16[:batch])
                for b in range(batch):
                    assert oracle.rel_error(got[b], ref[b]) <= TOL


@pytest.mark.parametrize("keep_n,expect,aligned", [(179, (1024, 4, 1, 3, 60, 1), (820, 4, 4)), (77, (512, 4, 1, 3, 52, 1), (316, 4, 4)),
                                                   (100, (512, 4, 1, 4, 52, 1), (412, 4, 4)), (205, (1024, 4, 1, 4, 52, 1), (456, 4, 8))])
def test_default_keeps_rows_inside_workers_full_size(torch_cuda, keep_n, expect, aligned):
    """4096x4096 with rows that do not divide the tiles of 4 x 64 (S = 30 %, 70 %, 61 %, 20 %): the default
    takes a tile shape that whole rows fill and no worker shares a row; every output checked, also
    of the form that keeps the rows inside the workgroups' spans and of the plain form with as
    many workers (rows shared by wavefronts and by workgroups)."""
    N, K = 4096, 4096
    W = gi.dense_weight_chunked(N, K, seed=41)
    keep = np.full(N, keep_n, dtype=np.int32)
    c = oracle.pack(W, 16, 4, keep_per_row=keep)
    h = gq.gqsa_pack_rows(W, keep, 16, 4)
    assert gq.gqsa_partition(h) == expect
    info = gq.gqsa_info(h)
    assert info["needs_fixup"] == 0
    assert gq.gqsa_export_device_blob(h) == oracle.device_blob_for(c, info)
    x = gi.activations(1, K, seed=10)
    check(torch_cuda, h, c, x)
    gq.gqsa_free(h)
    h1 = gq.gqsa_pack_rows(W, keep, 16, 4)
    gq.gqsa_set_partition_aligned(h1, aligned[2], aligned[0], aligned[1])
    assert gq.gqsa_partition(h1) == aligned + (4, 64, 0) and gq.gqsa_info(h1)["needs_fixup"] == 1
    check(torch_cuda, h1, c, x)
    gq.gqsa_free(h1)
    h2 = gq.gqsa_pack_rows(W, keep, 16, 4)     # the plain form with the same workers: rows shared by workgroups
    gq.gqsa_set_partition(h2, aligned[0], 4)
    check(torch_cuda, h2, c, x)


def adversarial_keeps(N, kg):
    one_row = np.zeros(N, dtype=np.int32); one_row[N // 2] = kg
    alternating = np.where(np.arange(N) % 2 == 0, 0, kg).astype(np.int32)
    singles = np.ones(N, dtype=np.int32)                      # many rows inside one lane
    singles_gaps = np.where(np.arange(N) % 3 == 0, 0, 1).astype(np.int32)
    ends_empty = np.full(N, kg // 2, dtype=np.int32); ends_empty[:3] = 0; ends_empty[-3:] = 0
    ramp = (np.arange(N) % (kg + 1)).astype(np.int32)
    exact64 = np.full(N, 64, dtype=np.int32)                  # rows end exactly on block boundaries
    return {"one_row": one_row, "alternating": alternating, "singles": singles,
            "singles_gaps": singles_gaps, "ends_empty": ends_empty, "ramp": ramp, "exact64": exact64}


@pytest.mark.parametrize("name", ["one_row", "alternating", "singles", "singles_gaps", "ends_empty",
                                  "ramp", "exact64"])
@pytest.mark.parametrize("part", [None, (5, 1), (2, 3)])
def test_adversarial_row_structures(torch_cuda, name, part):
    N, K = 96, 2048
    keep = adversarial_keeps(N, K // 16)[name]
    W = gi.dense_weight(N, K, seed=41)
    c = oracle.pack(W, 16, 4, keep_per_row=keep)
    h = gq.gqsa_pack_rows(W, keep, 16, 4)
    if part:
        gq.gqsa_set_partition(h, *part)
    check(torch_cuda, h, c, gi.activations(2, K, seed=7))


def test_single_row_matrix(torch_cuda):
    W = gi.dense_weight(1, 4096, seed=43)
    for s in (0.0, 0.5):
        c = oracle.pack(W, 16, 4, sparsity=s)
        h = gq.gqsa_pack(W, 16, 4, s)
        check(torch_cuda, h, c, gi.activations(1, 4096, seed=8))


@pytest.mark.parametrize("bits", [4, 8])
def test_unit_vectors_are_bit_exact(torch_cuda, bits):
    """x = e_k: y is column k of W^ and (q - z) s is exact in fp32, so the fp16 output must
    equal the correctly rounded oracle value bit for bit (pins gather + dequantisation)."""
    N, K = 128, 512
    W = gi.dense_weight(N, K, seed=47)
    c = oracle.pack(W, 16, bits, sparsity=0.5)
    h = gq.gqsa_pack(W, 16, bits, 0.5)
    ks = [0, 1, 15, 16, 17, 255, 256, 300, 511]
    x = np.concatenate([gi.unit_vector(K, k) for k in ks])
    y = run_gemv(torch_cuda, h, x)
    ref = oracle.gemv(c, x).astype(np.float16)
    assert np.array_equal(y.view(np.uint16), ref.view(np.uint16))


def test_ones_vector_row_sums(torch_cuda):
    N, K = 128, 512
    W = gi.dense_weight(N, K, seed=53)
    c = oracle.pack(W, 16, 4, sparsity=0.3)
    h = gq.gqsa_pack(W, 16, 4, 0.3)
    check(torch_cuda, h, c, gi.ones_vector(K))


def test_free_scale_and_zero_parameters(torch_cuda):
    """Sec. 3.4 trains s and z after the codes are frozen: the kernel must take any fp16 s, z."""
    N, K = 64, 1024
    W = gi.dense_weight(N, K, seed=59)
    c = oracle.pack(W, 16, 4, sparsity=0.5)
    rng = np.random.default_rng(2)
    c.scales = (c.scales.view(np.float16) * np.float16(0.83)).view(np.uint16)
    c.zeros = (c.zeros.view(np.float16) + rng.standard_normal(c.nnzg).astype(np.float16) * np.float16(3)).view(np.uint16)
    h = gq.gqsa_import(c.rowIndex, c.groups, c.values, c.scales, c.zeros, N, K, 16, 4)
    check(torch_cuda, h, c, gi.activations(1, K, seed=9))


@pytest.mark.parametrize("bits", [4, 8])
def test_small_batches(torch_cuda, bits):
    N, K = 512, 2048
    W = gi.dense_weight(N, K, seed=61)
    c = oracle.pack(W, 16, bits, sparsity=0.5)
    h = gq.gqsa_pack(W, 16, bits, 0.5)
    x = gi.activations(16, K, seed=10)
    y16, _ = check(torch_cuda, h, c, x)
    for b in range(1, 16):
        yb, _ = check(torch_cuda, h, c, x[:b])
        assert np.array_equal(yb.view(np.uint16), y16[:b].view(np.uint16))


@pytest.mark.parametrize("part", [None, (37, 3)])
def test_three_and_seven_rows_in_the_kernels_for_four_and_eight(torch_cuda, part):
    """3 rows run in the kernel for 4 and 7 in the kernel for 8 (also as the tail of 11 and 15):
    the rows that are not there must neither be read past the end of x nor reach y.  y sits in
    the middle of a larger buffer of a marker value; rows shared by wavefronts and workgroups,
    rows without groups (their zero fill), several matrices per launch."""
    torch = torch_cuda
    N, K = 300, 2048
    W = gi.dense_weight(N, K, seed=62)
    keep = gi.imbalanced_keep_counts(N, K // 16, seed=62)
    keep[[0, 7, 299]] = 0
    c = oracle.pack(W, 16, 4, keep_per_row=keep)
    h = gq.gqsa_pack_rows(W, keep, 16, 4)
    h2 = gq.gqsa_pack_rows(W, keep, 16, 4)
    if part:
        gq.gqsa_set_partition(h, *part)
        gq.gqsa_set_partition(h2, *part)
    x16 = gi.activations(16, K, seed=11)
    y16 = run_gemv(torch, h, x16)
    marker = np.float16(-777.0)
    for b in (3, 7, 11, 15):
        xt = torch.from_numpy(x16[:b].copy()).cuda()              # exactly b rows: nothing behind them is ours
        big = torch.full((b + 4, N), float(marker), dtype=torch.float16, device="cuda")
        big2 = torch.full((b + 4, N), float(marker), dtype=torch.float16, device="cuda")
        gq.gqsa_gemv(h, xt, big[2:2 + b])
        torch.cuda.synchronize()
        out = big.cpu().numpy()
        assert np.array_equal(out[2:2 + b].view(np.uint16), y16[:b].view(np.uint16))
        assert (out[:2] == marker).all() and (out[2 + b:] == marker).all()
        big.fill_(float(marker))
        gq.gqsa_gemv_multi([h, h2], xt, [big[2:2 + b], big2[2:2 + b]])
        torch.cuda.synchronize()
        for o in (big.cpu().numpy(), big2.cpu().numpy()):
            assert np.array_equal(o[2:2 + b].view(np.uint16), y16[:b].view(np.uint16))
            assert (o[:2] == marker).all() and (o[2 + b:] == marker).all()
    err = max(oracle.rel_error(y16[i], oracle.gemv(c, x16, threads=8)[i]) for i in range(16))
    assert err <= TOL


@pytest.mark.parametrize("part", [None, (37, 3)])
def test_run_to_run_determinism(torch_cuda, part):
    """Same input -> same bits, also when calls with other inputs run in between (a stale
    carry record or counter from an earlier call would show up here)."""
    N, K = 1000, 11008
    W = gi.dense_weight(N, K, seed=67)
    h = gq.gqsa_pack(W, 16, 4, 0.5)
    if part:
        gq.gqsa_set_partition(h, *part)     # rows shared across workgroups
    assert gq.gqsa_info(h)["needs_fixup"] == 1
    c = oracle.pack(W, 16, 4, sparsity=0.5)
    xa = gi.activations(1, K, seed=11)
    xb = gi.activations(1, K, seed=12)
    ya, _ = check(torch_cuda, h, c, xa)
    yb, _ = check(torch_cuda, h, c, xb)
    for _ in range(10):
        assert np.array_equal(run_gemv(torch_cuda, h, xa).view(np.uint16), ya.view(np.uint16))
        assert np.array_equal(run_gemv(torch_cuda, h, xb).view(np.uint16), yb.view(np.uint16))


def test_y_is_fully_overwritten_and_nothing_else(torch_cuda):
    torch = torch_cuda
    N, K = 300, 1024
    W = gi.dense_weight(N, K, seed=71)
    h = gq.gqsa_pack(W, 16, 4, 0.5)
    x = torch.from_numpy(gi.activations(1, K, seed=12)).cuda()
    buf = torch.full((N + 64,), 7.0, dtype=torch.float16, device="cuda")
    y = buf[32:32 + N].view(1, N)
    gq.gqsa_gemv(h, x, y)
    torch.cuda.synchronize()
    out = buf.cpu().numpy()
    assert (out[:32] == 7.0).all() and (out[32 + N:] == 7.0).all()
    c = oracle.pack(W, 16, 4, sparsity=0.5)
    assert oracle.rel_error(out[32:32 + N], oracle.gemv(c, x.cpu().numpy())[0]) <= TOL


def test_gemv_error_paths_on_device(torch_cuda):
    torch = torch_cuda
    W = gi.dense_weight(16, 64, seed=1)
    h = gq.gqsa_pack(W, 16, 4, 0.5)
    x = torch.zeros((17, 64), dtype=torch.float16, device="cuda")
    with pytest.raises(gq.GqsaError) as e:
        gq.gqsa_gemv(h, x)
    assert e.value.status == 3
    xm = torch.zeros((1, 64 + 4), dtype=torch.float16, device="cuda")[:, 4:]
    with pytest.raises(gq.GqsaError) as e:
        gq.gqsa_gemv(h, xm)           # 8 bytes past a 16-byte boundary
    assert e.value.status == 8
    xt = torch.zeros((64, 2), dtype=torch.float16, device="cuda").t()
    with pytest.raises(ValueError):
        gq.gqsa_gemv(h, xt)           # not contiguous: refused by the binding
    gq.gqsa_upload(h)
    with pytest.raises(gq.GqsaError) as e:
        gq.gqsa_set_partition(h, 8, 16)   # not after upload
    assert e.value.status == 3
    assert gq.gqsa_info(h)["on_device"] == 1


# ----------------------------------------------------------------------------- several matrices, one launch

@pytest.mark.parametrize("part", [None, "mixed", (3, 4), (1, 16), (40, 2), (512, 4), (1024, 4)])
@pytest.mark.parametrize("batch", [1, 3, 8])
def test_gemv_multi_equals_separate_calls(torch_cuda, part, batch):
    """q/k/v-style: matrices of different N sharing x; the fused launch must give the bits of the
    separate calls (and both must match the oracle).  Partitions: the defaults (wavefronts per
    workgroup differ with the size: separate launches behind the call), different worker counts
    with the same workgroup size (one launch, each matrix its own share of the grid), equal ones;
    with (512, 4) and (1024, 4) the launches of several rows take the workers 8 and 16 to a workgroup."""
    torch = torch_cuda
    K = 2048
    shapes = [(300, 0.5, None), (64, 0.0, None), (257, None, "imbalanced"), (128, 1.0, None)]
    hs, cs = [], []
    for i, (N, sp, kind) in enumerate(shapes):
        W = gi.dense_weight(N, K, seed=200 + i)
        if kind:
            keep = gi.imbalanced_keep_counts(N, K // 16, seed=200 + i)
            h = gq.gqsa_pack_rows(W, keep, 16, 4)
            c = oracle.pack(W, 16, 4, keep_per_row=keep)
        else:
            h = gq.gqsa_pack(W, 16, 4, sp)
            c = oracle.pack(W, 16, 4, sparsity=sp)
        if part == "mixed":
            gq.gqsa_set_partition(h, (5, 1, 9, 2)[i], 4)
        elif part:
            gq.gqsa_set_partition(h, *part)
        hs.append(h)
        cs.append(c)
    x_np = gi.activations(batch, K, seed=77)
    x = torch.from_numpy(x_np).cuda()
    ys = [torch.full((batch, c.N), float("nan"), dtype=torch.float16, device="cuda") for c in cs]
    gq.gqsa_gemv_multi(hs, x, ys)
    torch.cuda.synchronize()
    for h, c, y in zip(hs, cs, ys):
        single = run_gemv(torch, h, x_np)
        got = y.cpu().numpy()
        assert np.array_equal(got.view(np.uint16), single.view(np.uint16))
        ref = oracle.gemv(c, x_np)
        for b in range(batch):
            assert oracle.rel_error(got[b], ref[b]) <= TOL
    # two matrices only, and the fused call again (workspaces are reusable)
    ys2 = gq.gqsa_gemv_multi(hs[:2], x)
    torch.cuda.synchronize()
    for y2, y in zip(ys2, ys[:2]):
        assert torch.equal(y2, y)


@pytest.mark.parametrize("bits,G,sizes,K", [(4, 16, (512, 512), 11008), (4, 16, (512, 512, 512), 11008), (8, 16, (512, 200), 12288),
                                            (8, 64, (700, 700), 11008), (8, 64, (512, 512, 512, 512), 12288)])
def test_gemv_multi_equals_separate_calls_rows_over_many_workers(torch_cuda, bits, G, sizes, K):
    """Unpruned rows that follow one another without gaps, each spread over three or four workers: how the workers
    are grouped decides where its pieces meet and so, now and then, the last bit.  A launch for several
    matrices has more workers than each alone and must group them as the separate launches do."""
    torch = torch_cuda
    gen = torch.Generator(device="cuda").manual_seed(K + G)
    hs = [gq.gqsa_pack_device(torch.randn((N, K), generator=gen, device="cuda"), G, bits, 0.0) for N in sizes]
    assert any(gq.gqsa_partition(h)[2] == 0 for h in hs)          # (rows without gaps)
    x = torch.randn((16, K), generator=gen, device="cuda").to(torch.float16)
    for batch in (1, 2, 3, 4, 7, 8, 16):
        together = gq.gqsa_gemv_multi(hs, x[:batch].contiguous())
        for h, y in zip(hs, together):
            alone = gq.gqsa_gemv(h, x[:batch].contiguous())
            assert torch.equal(y.view(torch.int16), alone.view(torch.int16)), batch


@pytest.mark.parametrize("n_mats,workgroups,waves,span", [(4, 272, 4, 1), (2, 272, 3, 1), (4, 400, 4, 3), (2, 1080, 1, 1)])
def test_gemv_multi_equals_separate_calls_rows_longer_than_spans(torch_cuda, n_mats, workgroups, waves, span):
    """The same with spans that are shorter than the rows, the workers' own (waves of 3: no whole number of them in a larger
    workgroup) or the workgroups'.  The two halves of a row nearly cancel, so that the order of the sum shows."""
    torch = torch_cuda
    N, K = 290, 11008
    hs = []
    for i in range(n_mats):
        W = gi.dense_weight(N, K, seed=210 + i)
        W[:, :K // 2] += 1.0
        W[:, K // 2:] -= 1.0
        h = gq.gqsa_pack(W, 16, 4, 0.0)
        if span == 1:
            gq.gqsa_set_partition_rows(h, 4, 64, 1, workgroups, waves)
        else:
            gq.gqsa_set_partition_aligned(h, span, workgroups, waves)
        assert gq.gqsa_info(h)["needs_fixup"]
        hs.append(h)
    x = torch.from_numpy((1.0 + 0.1 * gi.activations(16, K, seed=78).astype(np.float32)).astype(np.float16)).cuda()
    for batch in (1, 2, 3, 4, 8, 16):
        together = gq.gqsa_gemv_multi(hs, x[:batch].contiguous())
        for h, y in zip(hs, together):
            alone = gq.gqsa_gemv(h, x[:batch].contiguous())
            assert torch.equal(y.view(torch.int16), alone.view(torch.int16)), batch


def test_gemv_multi_error_paths(torch_cuda):
    torch = torch_cuda
    W = gi.dense_weight(32, 256, seed=1)
    W2 = gi.dense_weight(32, 512, seed=2)
    h1, h1b, h2 = gq.gqsa_pack(W, 16, 4, 0.5), gq.gqsa_pack(W, 16, 8, 0.5), gq.gqsa_pack(W2, 16, 4, 0.5)
    x = torch.zeros((1, 256), dtype=torch.float16, device="cuda")
    y = [torch.zeros((1, 32), dtype=torch.float16, device="cuda") for _ in range(5)]
    for hs, status in (([h1, h1], 2), ([h1, h1b], 2), ([h1] * 5, 3)):
        with pytest.raises(gq.GqsaError) as e:
            gq.gqsa_gemv_multi(hs, x, y[:len(hs)])
        assert e.value.status == status
    with pytest.raises(ValueError):
        gq.gqsa_gemv_multi([h1, h2], x, y[:2])      # K differs: refused by the binding
    h3 = gq.gqsa_pack(gi.dense_weight(32, 256, seed=3), 16, 4, 0.5)
    gq.gqsa_set_partition(h3, 2, 8)
    gq.gqsa_gemv_multi([h1, h3], x, y[:2])          # partitions may differ
    torch.cuda.synchronize()


@pytest.mark.parametrize("bits", [4, 8])
def test_largest_and_smallest_reduction_lengths(torch_cuda, bits):
    """K = 32768 is the most gqsa_gemv takes (x, its halves and group sums fill 96 KB of LDS; a
    batch of 2 goes out as two launches), K = 16 with one row the least; one more group-column
    than the limit packs but is refused by gqsa_gemv."""
    torch = torch_cuda
    N, K = 48, 32768
    W = gi.dense_weight(N, K, seed=200 + bits)
    keep = gi.imbalanced_keep_counts(N, K // 16, seed=200 + bits)
    h = gq.gqsa_pack_rows(W, keep, 16, bits)
    c = oracle.pack(W, 16, bits, keep_per_row=keep)
    check(torch, h, c, gi.activations(2, K, seed=13))
    W1 = gi.dense_weight(1, 16, seed=300 + bits)
    h1 = gq.gqsa_pack(W1, 16, bits, 0.0)
    check(torch, h1, oracle.pack(W1, 16, bits, sparsity=0.0), gi.activations(3, 16, seed=14))
    Wb = np.zeros((2, 32768 + 16), dtype=np.float32)
    hb = gq.gqsa_pack(Wb, 16, bits, 0.5)
    x = torch.zeros((1, 32768 + 16), dtype=torch.float16, device="cuda")
    y = torch.zeros((1, 2), dtype=torch.float16, device="cuda")
    with pytest.raises(gq.GqsaError) as e:
        gq.gqsa_gemv(hb, x, y)
    assert e.value.status == 3


# ----------------------------------------------------------------------------- other group sizes

@pytest.mark.parametrize("bits,G", [(4, 8), (8, 8), (4, 32), (4, 64), (4, 128), (8, 32), (8, 64)])
@pytest.mark.parametrize("part", [None, (5, 3), (2, 16)])
def test_other_group_sizes(torch_cuda, bits, G, part):
    """G = 32, 64, 128: several 16-element chunks per stored group, code planes, smaller
    tiles; rows of very different lengths, shared rows, empty rows; batch 1 and 3."""
    N, K = 150, 2048
    W = gi.dense_weight(N, K, seed=91)
    keep = gi.imbalanced_keep_counts(N, K // G, seed=91)
    h = gq.gqsa_pack_rows(W, keep, G, bits)
    c = oracle.pack(W, G, bits, keep_per_row=keep)
    if part is not None:
        gq.gqsa_set_partition(h, *part)
    check(torch_cuda, h, c, gi.activations(1, K, seed=9))
    check(torch_cuda, h, c, gi.activations(3, K, seed=10))


@pytest.mark.parametrize("bits,G", [(4, 8), (8, 8), (4, 32), (4, 64), (4, 128), (8, 32), (8, 64)])
@pytest.mark.parametrize("K,part", [(128, None), (4096, None), (4096, (3, 4)), (4224, None), (8320, None)])
def test_other_group_sizes_small_batches(torch_cuda, bits, G, K, part):
    """The kernels for several activation rows, on both sides of the steps of K at which fewer rows fit a
    launch (4096, 8192), one tile to a worker and several: every batch against the oracle, every row of it
    the single-row result to the last bit (each row is summed by the same operations in the same
    order), nothing written outside y."""
    torch = torch_cuda
    N = 101
    W = gi.dense_weight(N, K, seed=92)
    keep = gi.imbalanced_keep_counts(N, K // G, seed=92)
    keep[[0, 50, 100]] = 0, K // G, 0
    h = gq.gqsa_pack_rows(W, keep, G, bits)
    c = oracle.pack(W, G, bits, keep_per_row=keep)
    if part is not None:
        gq.gqsa_set_partition(h, *part)
    x16 = gi.activations(16, K, seed=12)
    rows = np.concatenate([run_gemv(torch, h, x16[b:b + 1]) for b in range(16)])
    for batch in (2, 3, 4, 5, 7, 8, 11, 16):
        y, _ = check(torch, h, c, x16[:batch])
        assert np.array_equal(y.view(np.uint16), rows[:batch].view(np.uint16)), batch
    buf = torch.full((8, N), 7.0, dtype=torch.float16, device="cuda")
    gq.gqsa_gemv(h, torch.from_numpy(x16[:7].copy()).cuda(), buf[:7])
    torch.cuda.synchronize()
    assert (buf[7] == 7.0).all()


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("own_tiles", [True, False])
@pytest.mark.parametrize("K", [16, 256, 4096, 4176, 8192, 8208])
def test_small_batches_of_unpruned_matrices(torch_cuda, bits, own_tiles, K):
    """Unpruned matrices in the format's own tiles have kernels of their own for several rows: every batch against the
    oracle, each row the single-row bits, on both sides of the share of stored groups (63 in 64) that
    decides, and in one launch with a pruned matrix; and the same with the partitions that such matrices have
    by default, whose tiles often have a chosen shape and no such form."""
    torch = torch_cuda
    N, columns = 72, K // 16
    W = gi.dense_weight(N, K, seed=93)
    x16 = gi.activations(16, K, seed=13)
    full = np.full(N, columns)
    edge, below = full.copy(), full.copy()
    dropped = N * columns // 64                          # the most that may be missing
    for keep, missing in ((edge, dropped), (below, dropped + 1)):
        keep -= missing // N
        keep[:missing % N] -= 1
        assert keep.sum() == N * columns - missing
    pruned = np.full(N, columns // 2)
    hs = [gq.gqsa_pack_rows(W, keep, 16, bits) for keep in (full, edge, below, pruned)]
    cs = [oracle.pack(W, 16, bits, keep_per_row=keep) for keep in (full, edge, below, pruned)]
    if own_tiles:
        for h in hs[:3]:
            gq.gqsa_set_partition(h, 5, 4)
            assert gq.gqsa_partition(h)[3:5] == (4, 64)
    gq.gqsa_set_partition(hs[3], 3, 2)          # (several tiles to a worker)
    for h, c in zip(hs, cs):
        rows = np.concatenate([run_gemv(torch, h, x16[b:b + 1]) for b in range(16)])
        for batch in (2, 3, 4, 7, 8, 13):
            y, _ = check(torch, h, c, x16[:batch])
            assert np.array_equal(y.view(np.uint16), rows[:batch].view(np.uint16)), batch
    x = torch.from_numpy(x16[:4].copy()).cuda()
    for group in ((0, 2), (0, 1), (0, 1, 2, 3)):
        ys = [torch.full((4, N), float("nan"), dtype=torch.float16, device="cuda") for _ in group]
        gq.gqsa_gemv_multi([hs[i] for i in group], x, ys)
        torch.cuda.synchronize()
        for i, y in zip(group, ys):
            assert np.array_equal(y.cpu().numpy().view(np.uint16), run_gemv(torch, hs[i], x16[:4]).view(np.uint16))


@pytest.mark.parametrize("K", [32, 1024, 4096, 4128, 8224, 16416, 32768])
def test_one_row_of_unpruned_groups_of_32(torch_cuda, K):
    """4-bit groups of 32 have a form for one row of (nearly) unpruned matrices: on both sides of the share of stored groups (31 in
    32) that decides, against the oracle, and in one launch with a matrix that takes the other form."""
    torch = torch_cuda
    N, columns = 72, K // 32
    W = gi.dense_weight(N, K, seed=98)
    x = gi.activations(1, K, seed=21)
    hs = []
    for missing in (0, N * columns // 32, N * columns // 32 + 1, N * columns // 2):
        keep = np.full(N, columns) - missing // N
        keep[:missing % N] -= 1
        h = gq.gqsa_pack_rows(W, keep, 32, 4)
        gq.gqsa_set_partition(h, 5, 4)
        check(torch, h, oracle.pack(W, 32, 4, keep_per_row=keep), x)
        hs.append(h)
    for group in (hs[:2], hs[1:3], hs):
        for h, y in zip(group, gq.gqsa_gemv_multi(group, torch.from_numpy(x.copy()).cuda())):
            assert np.array_equal(y.cpu().numpy().view(np.uint16), run_gemv(torch, h, x).view(np.uint16))


@pytest.mark.parametrize("bits,G,sparsity", [(4, 16, 0.5), (4, 16, 0.0), (8, 16, 0.3), (4, 8, 0.5), (4, 32, 0.5), (8, 64, 0.3), (4, 128, 0.5)])
@pytest.mark.parametrize("K", [4224, 8192, 8320, 11008, 12288, 12416, 16384, 16512])
def test_several_rows_that_fill_lds(torch_cuda, bits, G, sparsity, K):
    """Four copies of x fit LDS up to K = 12288 in a form of their own, four up to 16384, eight up to 8192 and two
    beyond 16384 without room to spare: every batch against the oracle, each row the single-row bits, at the
    ends of those ranges and on either side of them."""
    torch = torch_cuda
    W = gi.dense_weight(200, K, seed=95)
    x16 = gi.activations(8, K, seed=14)
    h = gq.gqsa_pack(W, G, bits, sparsity)
    c = oracle.pack(W, G, bits, sparsity)
    rows = np.concatenate([run_gemv(torch, h, x16[b:b + 1]) for b in range(8)])
    for batch in (2, 3, 4, 5, 7, 8):
        y, _ = check(torch, h, c, x16[:batch])
        assert np.array_equal(y.view(np.uint16), rows[:batch].view(np.uint16)), batch


@pytest.mark.parametrize("bits,G,N,K,sparsity", [(4, 16, 1000, 5120, 0.0), (4, 16, 512, 11008, 0.0), (4, 16, 700, 8320, 0.3), (4, 32, 2500, 8704, 0.5),
                                                 (8, 16, 2500, 8192, 0.7), (8, 64, 1000, 5120, 0.0), (8, 8, 500, 8320, 0.3), (4, 32, 2500, 11008, 0.7)])
def test_several_rows_more_workgroups_than_fit_at_once(torch_cuda, bits, G, N, K, sparsity):
    """Default partitions of between one and two workgroups per compute unit, which launches of several rows take together into
    one round: every batch against the oracle, and each row the single-row bits unless rows are spread over
    workers without regard to the grouping."""
    torch = torch_cuda
    W = gi.dense_weight(N, K, seed=96)
    x16 = gi.activations(8, K, seed=15)
    h = gq.gqsa_pack(W, G, bits, sparsity)
    c = oracle.pack(W, G, bits, sparsity)
    part = gq.gqsa_partition(h)
    assert 256 < part[0] < 512
    rows = np.concatenate([run_gemv(torch, h, x16[b:b + 1]) for b in range(8)])
    for batch in (2, 3, 4, 7, 8):
        y, _ = check(torch, h, c, x16[:batch])
        if part[2] > 0:
            assert np.array_equal(y.view(np.uint16), rows[:batch].view(np.uint16)), batch


@pytest.mark.parametrize("bits,G,K,workgroups", [(4, 32, 8192, 256), (4, 32, 8192, 257), (4, 128, 4224, 257), (4, 16, 8192, 257), (8, 32, 8192, 257),
                                                 (4, 16, 11264, 513), (4, 16, 11280, 512), (4, 16, 11280, 513), (4, 16, 16384, 513), (8, 16, 11280, 513)])
def test_three_rows_of_many_workgroups(torch_cuda, bits, G, K, workgroups):
    """Three rows go out in one launch or in two by the format, K and the number of workgroups: on both sides of
    each line the oracle's values, the single-row bits and nothing written beyond the third row."""
    torch = torch_cuda
    N = 16 * workgroups - 5
    W = gi.dense_weight(64, K, seed=97)
    kept = gi.imbalanced_keep_counts(64, 6, seed=97)           # (few groups a row: the number of workgroups is what counts)
    c = oracle.pack(W, G, bits, keep_per_row=kept)
    times = -(-N // 64)
    rows = np.concatenate([[0], np.cumsum(np.tile(np.diff(c.rowIndex), times)[:N])]).astype(np.int32)
    h = gq.gqsa_import(rows, *(np.tile(a, times)[:rows[-1] * (len(a) // c.nnzg)] for a in (c.groups, c.values, c.scales, c.zeros)), N, K, G, bits)
    info = gq.gqsa_info(h)
    gq.gqsa_set_partition_rows(h, info["tile_blocks"], 64, 1, workgroups, 16)
    x = gi.activations(3, K, seed=18)
    ref = oracle.gemv(c, x, threads=4)
    single = np.concatenate([run_gemv(torch, h, x[b:b + 1]) for b in range(3)])
    buf = torch.full((4, N), 7.0, dtype=torch.float16, device="cuda")
    gq.gqsa_gemv(h, torch.from_numpy(x.copy()).cuda(), buf[:3])
    torch.cuda.synchronize()
    y = buf[:3].cpu().numpy()
    assert (buf[3] == 7.0).all()
    assert np.array_equal(y.view(np.uint16), single.view(np.uint16))
    for b in range(3):
        assert oracle.rel_error(y[b], np.tile(ref[b], times)[:N]) <= TOL


@pytest.mark.parametrize("G", [8, 32, 64, 128])
def test_other_group_sizes_full_size_and_sparsities(torch_cuda, G):
    """4096x4096 W4 at G = 32, 64, 128, S = 0 and 50 %, default partition."""
    W = gi.dense_weight(4096, 4096, seed=gi.config_seed(3, 0))
    for sparsity in (0.0, 0.5):
        h = gq.gqsa_pack(W, G, 4, sparsity)
        c = oracle.pack(W, G, 4, sparsity=sparsity)
        info = gq.gqsa_info(h)
        assert gq.gqsa_export_device_blob(h) == oracle.device_blob_for(c, info)
        check(torch_cuda, h, c, gi.activations(1, 4096, seed=11))


def test_gemv_multi_with_larger_groups(torch_cuda):
    """Two G = 32 matrices of different N in one launch: the oracle's values and the bits of the
    separate calls."""
    torch = torch_cuda
    K = 1024
    x_np = gi.activations(1, K, seed=12)
    x = torch.from_numpy(x_np).cuda()
    hs, cs = [], []
    for i, N in enumerate((96, 200)):
        W = gi.dense_weight(N, K, seed=100 + i)
        hs.append(gq.gqsa_pack(W, 32, 4, 0.5))
        cs.append(oracle.pack(W, 32, 4, sparsity=0.5))
    for h in hs:
        gq.gqsa_set_partition(h, 3, 4)
    ys = gq.gqsa_gemv_multi(hs, x)
    torch.cuda.synchronize()
    for h, y, c in zip(hs, ys, cs):
        assert oracle.rel_error(y.cpu().numpy()[0], oracle.gemv(c, x_np, threads=4)[0]) <= TOL
        assert np.array_equal(y.cpu().numpy().view(np.uint16), run_gemv(torch, h, x_np).view(np.uint16))


def test_hessian_pruned_and_reloaded_matrices_multiply(torch_cuda, tmp_path):
    """A matrix pruned by the Hessian metric (Eq. 4) against the oracle, and the same matrix after
    a trip through a file: identical output bits."""
    N, K = 300, 4096
    W = gi.dense_weight(N, K, seed=61)
    d = np.exp(np.random.default_rng(62).standard_normal(K)).astype(np.float32)
    h = gq.gqsa_pack_hessian(W, d, 16, 4, 0.5)
    c = oracle.pack(W, 16, 4, sparsity=0.5, hinv_diag=d)
    x_np = gi.activations(2, K, seed=63)
    check(torch_cuda, h, c, x_np)
    path = str(tmp_path / "layer.gqsa")
    gq.gqsa_save(h, path)
    h2 = gq.gqsa_load(path)
    y1, y2 = run_gemv(torch_cuda, h, x_np), run_gemv(torch_cuda, h2, x_np)
    assert np.array_equal(y1.view(np.uint16), y2.view(np.uint16))


# ----------------------------------------------------------------------------- full sizes

@pytest.mark.parametrize("idx", [0, 4, 6])
def test_llama7b_layer_shapes_full_size(torch_cuda, idx):
    """q_proj 4096x4096, gate_proj 11008x4096, down_proj 4096x11008 at W4S50 G=16, batch 1,
    default partition (the launch configuration the benchmark times); every output checked."""
    name, N, K = gi.LLAMA7B_LAYER[idx]
    W = gi.dense_weight(N, K, seed=gi.config_seed(2, idx))
    h = gq.gqsa_pack(W, 16, 4, 0.5)
    c = oracle.pack(W, 16, 4, sparsity=0.5)
    info = gq.gqsa_info(h)
    assert gq.gqsa_export_device_blob(h) == oracle.device_blob_for(c, info)
    check(torch_cuda, h, c, gi.activations(1, K, seed=gi.config_seed(2, idx)))


@pytest.mark.parametrize("sparsity", [0.0, 0.3, 0.5, 0.7])
@pytest.mark.parametrize("idx", [0, 1, 2, 3])
def test_llama3_8b_sparsity_sweep_full_size(torch_cuda, idx, sparsity):
    """Every shape of the LLaMA-3-8B-like set at every sparsity of the sweep, at full size, with the
    default partition (the launch configuration the benchmark times): the device image bit for
    bit and every output against the oracle."""
    name, N, K = gi.LLAMA3_8B_SHAPES[idx]
    W = gi.dense_weight(N, K, seed=gi.config_seed(3, idx))
    h = gq.gqsa_pack(W, 16, 4, sparsity)
    c = oracle.pack(W, 16, 4, sparsity=sparsity)
    info = gq.gqsa_info(h)
    assert gq.gqsa_partition(h) == gq.gqsa_default_partition(c.rowIndex, K)
    assert gq.gqsa_export_device_blob(h) == oracle.device_blob_for(c, info)
    check(torch_cuda, h, c, gi.activations(1, K, seed=gi.config_seed(3, idx)))
    gq.gqsa_free(h)


@pytest.mark.parametrize("idx", [0, 1])
def test_imbalanced_stress_full_size(torch_cuda, idx):
    name, N, K = gi.IMBALANCED_SHAPES[idx]
    seed = gi.config_seed(4, idx)
    W = gi.dense_weight(N, K, seed=seed)
    keep = gi.imbalanced_keep_counts(N, K // 16, seed=seed)
    h = gq.gqsa_pack_rows(W, keep, 16, 4)
    c = oracle.pack(W, 16, 4, keep_per_row=keep)
    assert gq.gqsa_info(h)["needs_fixup"] == 1
    check(torch_cuda, h, c, gi.activations(1, K, seed=seed))


def test_vocabulary_sized_matrix(torch_cuda):
    """128256x4096 (the output projection of a LLaMA-3-8B-like model), W4S50: 16.4 M stored groups,
    64 128 tiles, four (eight rows) per wavefront in 4008 workgroups -- the largest deal the default makes.
    Every output checked."""
    N, K = 128256, 4096
    W = gi.dense_weight_chunked(N, K, seed=51)
    h = gq.gqsa_pack(W, 16, 4, 0.5)
    c = oracle.pack(W, 16, 4, sparsity=0.5)
    del W
    info = gq.gqsa_info(h)
    assert info["nnz_groups"] == N * 128
    assert gq.gqsa_partition(h) == (4008, 4, 4, 4, 64, 1)
    check(torch_cuda, h, c, gi.activations(1, K, seed=52))
    gq.gqsa_free(h)


@pytest.mark.parametrize("integer_zeros", [True, False])
@pytest.mark.parametrize("bits,G", [(4, 16), (4, 32), (4, 64), (4, 128), (8, 16), (8, 32), (8, 64)])
def test_panel_kernel_more_than_four_panels_per_compute_unit(torch_cuda, bits, G, integer_zeros):
    """Two matrices of 601 + 512 and of 1024 + 1024 panels in one launch (just beyond four for each of 256 workgroups, and
    the most there are of eight); 601 + 1447 and 601 + 1448, which a matrix of more than 1024 panels or more than 2048 in
    all keep apart; 1113 panels of one matrix.  Dense rows (a quad's records do not fit their staging
    area at once) and ragged ones; every row against the oracle, and the bits of separate calls."""
    torch = torch_cuda
    K = 4 * 32 * 16 + G if G <= 32 else 2048 + G       # (the last slice is a short one)
    rng = np.random.default_rng(bits * 1000 + G)

    def packed(panels, seed, dense):
        n = 16 * panels - 5
        W = np.tile(gi.dense_weight(96, K, seed=seed), (n // 96 + 1, 1))[:n]
        keep = np.full(n, K // G) if dense else gi.imbalanced_keep_counts(n, K // G, seed=seed)
        c = oracle.pack(W, G, bits, keep_per_row=keep)
        if not integer_zeros:
            c.zeros = (c.zeros.view(np.float16) + rng.standard_normal(c.nnzg).astype(np.float16)).view(np.uint16)
        h = gq.gqsa_import(c.rowIndex, c.groups, c.values, c.scales, c.zeros, n, K, G, bits)
        gq.gqsa_build_panels(h)
        assert gq.gqsa_info(h)["panel_integer_zeros"] == int(integer_zeros)
        return h, c

    a, b, c, d, e, f, g = (packed(601, 1, True), packed(512, 2, False), packed(1447, 3, False), packed(1448, 4, False),
                           packed(1113, 5, False), packed(1024, 6, True), packed(1024, 7, False))
    x_np = gi.activations(16, K, seed=31)
    for batch in (16, 5):
        x = torch.from_numpy(x_np[:batch].copy()).cuda()

        def run(group):
            ys = [torch.full((batch, p[1].N), float("nan"), dtype=torch.float16, device="cuda") for p in group]
            gq.gqsa_gemv_multi([p[0] for p in group], x, ys)
            torch.cuda.synchronize()
            return [y.cpu().numpy() for y in ys]

        for group in ((a, b), (f, g), (a, c), (a, d), (e,)):
            for (h, packing), y in zip(group, run(group)):
                ref = oracle.gemv(packing, x_np[:batch], threads=8)
                for row in range(batch):
                    assert oracle.rel_error(y[row], ref[row]) <= TOL
                if len(group) > 1:
                    alone = run(((h, packing),))[0]
                    assert np.array_equal(y.view(np.uint16), alone.view(np.uint16))


@pytest.mark.parametrize("integer_zeros", [True, False])
@pytest.mark.parametrize("bits,G", [(4, 16), (4, 32), (4, 64), (4, 128), (8, 16), (8, 32), (8, 64)])
@pytest.mark.parametrize("panels", [769, 2561])
def test_panel_kernel_staging_area_used_again(torch_cuda, bits, G, integer_zeros, panels):
    """Dense rows, four panels to a workgroup or six (two quads) and two units and more to the first wavefront: its
    staging area is filled again for panels 2 and 3, for the next quad and for the next unit.  The rows
    repeat a pattern of 80, whose products the oracle has."""
    torch = torch_cuda
    period, N, K = 80, 16 * panels, (4096 if bits == 4 else 2048) + G
    rng = np.random.default_rng(bits * 1000 + G)
    c = oracle.pack(gi.dense_weight(period, K, seed=97), G, bits, sparsity=0.0)
    if not integer_zeros:
        c.zeros = (c.zeros.view(np.float16) + rng.standard_normal(c.nnzg).astype(np.float16)).view(np.uint16)
    columns, times = K // G, -(-N // period)
    h = gq.gqsa_import(np.arange(N + 1, dtype=np.int32) * columns,
                       *(np.tile(a, times)[:N * columns * (len(a) // (period * columns))] for a in (c.groups, c.values, c.scales, c.zeros)),
                       N, K, G, bits)
    gq.gqsa_build_panels(h)
    assert gq.gqsa_info(h)["panel_integer_zeros"] == int(integer_zeros)
    x = gi.activations(16, K, seed=17)
    ref = oracle.gemv(c, x, threads=8)
    for rows in (16, 8):                # (with G = 16 the form for up to 8 rows stages on its own)
        y = run_gemv(torch, h, x[:rows], panels=True)
        for b in range(rows):
            assert oracle.rel_error(y[b][:period], ref[b]) <= TOL
            assert np.array_equal(y[b].view(np.uint16), np.tile(y[b][:period], times)[:N].view(np.uint16))


@pytest.mark.parametrize("bits,G", [(4, 16), (8, 16), (4, 64), (8, 32)])
@pytest.mark.parametrize("integer_zeros", [True, False])
@pytest.mark.parametrize("panels", [(37,), (300, 301), (611, 690), (1100,)])
def test_panel_kernel_panels_of_very_different_lengths(torch_cuda, bits, G, integer_zeros, panels):
    """A workgroup's panels (one, two or three, six, two to three) take none, one, two or three loads for their records in a unit: the slots
    of the staging area go by the longest, an empty panel's load counts all the same.  One unit for some wavefronts and two for
    others, the last slice short; 16, 9 and up to 8 rows; the rows repeat a pattern whose products the oracle has."""
    rng = np.random.default_rng(bits * 100 + G)
    units = {4: 16, 8: 8}[bits] * 16
    K = 20 * units + G if G == 16 else 20 * units
    columns = K // G
    # (panels of 16 rows: dense, empty, a single group in one row, half, ragged)
    keep = np.concatenate([np.full(16, columns), np.zeros(16), np.eye(1, 16, 5)[0], np.full(16, columns // 2),
                           gi.imbalanced_keep_counts(16, columns, seed=3)]).astype(np.int64)
    c = oracle.pack(gi.dense_weight(80, K, seed=61), G, bits, keep_per_row=keep)
    if not integer_zeros:
        c.zeros = (c.zeros.view(np.float16) + rng.standard_normal(c.nnzg).astype(np.float16)).view(np.uint16)
    x = gi.activations(16, K, seed=62)
    ref = oracle.gemv(c, x, threads=8)

    def repeated_rows(n):
        times = -(-n // 80)
        lengths = np.tile(np.diff(c.rowIndex), times)[:n]
        row_index = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
        arrays = (np.tile(a, times)[:int(row_index[-1]) * (len(a) // c.nnzg)] for a in (c.groups, c.values, c.scales, c.zeros))
        h = gq.gqsa_import(row_index, *arrays, n, K, G, bits)
        gq.gqsa_build_panels(h)
        return h

    handles = [repeated_rows(16 * p - 3) for p in panels]
    for rows in (16, 9, 8, 5):
        xd = torch_cuda.from_numpy(x[:rows].copy()).cuda()
        ys = [torch_cuda.full((rows, 16 * p - 3), float("nan"), dtype=torch_cuda.float16, device="cuda") for p in panels]
        for _ in range(2):
            if len(panels) > 1:
                gq.gqsa_gemv_multi(handles, xd, ys)
            else:
                gq.gqsa_gemv(handles[0], xd, ys[0])
        torch_cuda.cuda.synchronize()
        for y, p in zip(ys, panels):
            y, n = y.cpu().numpy(), 16 * p - 3
            for b in range(rows):
                assert oracle.rel_error(y[b][:80], ref[b]) <= TOL
                assert np.array_equal(y[b].view(np.uint16), np.tile(y[b][:80], -(-n // 80))[:n].view(np.uint16))


@pytest.mark.parametrize("bits,G,K,first", [(4, 16, 4096, (5, 5)), (8, 16, 4096, (5, 5)), (4, 16, 8320, (5, 3)), (8, 16, 8320, (5, 3)), (8, 32, 4096, (5, 3)),
                                            (8, 64, 1024, (5, 3)), (4, 32, 4096, (3, 3)), (8, 64, 8320, (3, 3))])
def test_batch_from_which_the_second_image_is_used(torch_cuda, bits, G, K, first):
    """first = the smallest batch that a matrix with 13 in 25 of its groups stored, and one with a group more, is
    multiplied from the second image; in one call each takes the image it takes alone."""
    torch = torch_cuda
    N, columns = 1200, K // G          # (the kernels' sums differ in about one fp16 value of a thousand: 27600 values tell them apart)
    total = N * columns * 13 // 25
    hs, plain = [], []
    for more in (0, 1):
        keep = np.full(N, total // N)
        keep[:total % N + more] += 1
        assert keep.sum() == total + more
        W = gi.dense_weight(N, K, seed=131 + more)
        h, p = gq.gqsa_pack_rows(W, keep, G, bits), gq.gqsa_pack_rows(W, keep, G, bits)
        gq.gqsa_build_panels(h)
        hs.append(h)
        plain.append(p)
    x_np = gi.activations(8, K, seed=19)
    differ = 0
    for batch in (1, 2, 3, 4, 5, 8):
        x = torch.from_numpy(x_np[:batch].copy()).cuda()
        together = gq.gqsa_gemv_multi(hs, x)
        for h, p, y, f in zip(hs, plain, together, first):
            alone = run_gemv(torch, h, x_np[:batch])
            of_panels, of_blocks = run_gemv(torch, h, x_np[:batch], panels=True), run_gemv(torch, p, x_np[:batch])
            expected = of_panels if batch >= f else of_blocks
            assert np.array_equal(alone.view(np.uint16), expected.view(np.uint16)), batch
            assert np.array_equal(y.cpu().numpy().view(np.uint16), alone.view(np.uint16)), batch
            differ += int(not np.array_equal(of_panels.view(np.uint16), of_blocks.view(np.uint16)))
    assert differ > 0          # (the two kernels add in different orders: the bits tell them apart)


@pytest.mark.parametrize("bits,G", [(4, 16), (8, 16), (4, 32), (4, 64), (4, 128), (8, 32), (8, 64)])
@pytest.mark.parametrize("batch", [1, 2, 5, 8, 9, 13, 16])
def test_panel_kernel_ragged(torch_cuda, bits, G, batch):
    """1..16 activation rows on the matrix cores, from the panel image: 301 rows (the last panel
    has 13), 61 group-columns (the second slice has 29), imbalanced rows, empty rows."""
    N, K = 301, 61 * G
    W = gi.dense_weight(N, K, seed=90 + bits)
    keep = gi.imbalanced_keep_counts(N, K // G, seed=90 + bits)
    keep[[0, 5, 6, 300]] = 0
    keep[17] = K // G
    c = oracle.pack(W, G, bits, keep_per_row=keep)
    h = gq.gqsa_pack_rows(W, keep, G, bits)
    gq.gqsa_build_panels(h)
    check(torch_cuda, h, c, gi.activations(batch, K, seed=11 + batch), panels=True)


def replay_times(torch, calls):
    """The shortest of 15 replays, in turn, of a graph of 20 launches for each of (handle, batch), from the second image."""
    graphs = []
    for h, batch in calls:
        N, K = gq.gqsa_info(h)["N"], gq.gqsa_info(h)["K"]
        x = torch.from_numpy(gi.activations(batch, K, seed=6)).cuda()
        y = torch.empty((batch, N), dtype=torch.float16, device="cuda")
        gq.gqsa_gemv(h, x, y, panels=True)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                gq.gqsa_gemv(h, x, y, panels=True)
        graphs.append((graph, x, y))
    times = [float("inf")] * len(graphs)
    for _ in range(15):
        for i, (graph, *_) in enumerate(graphs):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            graph.replay()
            end.record()
            end.synchronize()
            times[i] = min(times[i], start.elapsed_time(end))
    return times


@pytest.mark.parametrize("G", [64, 128])
def test_panel_kernel_few_rows_of_large_groups_cost_less_than_sixteen(torch_cuda, G):
    """3 rows of 4096x11008 take 0.76 to 0.79 of the time of 16 where the copies of the last row are one request each,
    0.96 in the form that loads every row's activations and turns them in LDS whatever the rows."""
    h = gq.gqsa_pack(gi.dense_weight(4096, 11008, seed=5), G, 4, 0.5)
    gq.gqsa_build_panels(h)
    three, sixteen = replay_times(torch_cuda, ((h, 3), (h, 16)))
    assert three < 0.88 * sixteen


def repeated(period, times, N, K, G, bits, sparsity, integer_zeros, seed):
    """A matrix of N rows that repeat a pattern of `period`, with its second image, and the pattern."""
    rng = np.random.default_rng(bits * 1000 + G)
    c = oracle.pack(gi.dense_weight(period, K, seed=seed), G, bits, sparsity=sparsity)
    if not integer_zeros:
        c.zeros = (c.zeros.view(np.float16) + rng.standard_normal(c.nnzg).astype(np.float16)).view(np.uint16)
    per_row = c.nnzg // period
    h = gq.gqsa_import(np.arange(N + 1, dtype=np.int32) * per_row,
                       *(np.tile(a, times)[:N * per_row * (len(a) // (period * per_row))] for a in (c.groups, c.values, c.scales, c.zeros)),
                       N, K, G, bits)
    gq.gqsa_build_panels(h)
    return h, c


@pytest.mark.parametrize("integer_zeros", [True, False])
@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("sparsity,loads", [(0.5, 2), (0.9, 1)])
@pytest.mark.parametrize("panels,batches", [((640, 700), (16, 9, 8)), ((1024, 1020), (16, 8)), ((2600,), (8,)), ((3900,), (5,))])
def test_panel_kernel_slots_of_the_staging_area_taken_over(torch_cuda, bits, integer_zeros, sparsity, loads, panels, batches):
    """Five to eight panels to a workgroup (of 16 wavefronts, several matrices; of 8, one matrix), every panel's records of a unit two loads -- four slots,
    which the fifth to eighth panel take over -- or one, eight slots.  More units than wavefronts, the last one short."""
    wavefronts = 16 if len(panels) > 1 else 8
    columns = {4: 16, 8: 8}[bits]                       # of a unit
    period, K = 80, 16 * ((wavefronts + 3) * columns + 1)
    x = gi.activations(16, K, seed=71)
    made = [repeated(period, -(-(16 * p - 3) // period), 16 * p - 3, K, 16, bits, sparsity, integer_zeros, seed=72) for p in panels]
    c = made[0][1]
    row = np.repeat(np.arange(period), np.diff(c.rowIndex))
    held = np.bincount(row // 16 * (wavefronts + 4) + c.groups // columns, minlength=period // 16 * (wavefronts + 4))
    held = held.reshape(-1, wavefronts + 4)[:, :-1] * {4: 12, 8: 24}[bits]      # bytes of a panel's records in a full unit
    longest = held.max(axis=0)                          # of a workgroup's panels, which have all of the pattern
    assert longest.max() <= 1024 * loads and (loads == 1 or longest.min() > 1024 * (loads - 1))        # (one load also where there is nothing)
    ref = oracle.gemv(c, x, threads=8)
    for batch in batches:
        xd = torch_cuda.from_numpy(x[:batch].copy()).cuda()
        ys = [torch_cuda.full((batch, 16 * p - 3), float("nan"), dtype=torch_cuda.float16, device="cuda") for p in panels]
        gq.gqsa_gemv_multi([h for h, _ in made], xd, ys)
        torch_cuda.cuda.synchronize()
        for y in ys:
            y = y.cpu().numpy()
            for b in range(batch):
                assert oracle.rel_error(y[b][:period], ref[b]) <= TOL
                assert np.array_equal(y[b].view(np.uint16), np.tile(y[b][:period], -(-y.shape[1] // period))[:y.shape[1]].view(np.uint16))


@pytest.mark.parametrize("integer_zeros", [True, False])
@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("panels", [769, 1537, 2561])
def test_panel_kernel_up_to_eight_rows_of_which_three_panels_fit(torch_cuda, bits, integer_zeros, panels):
    """10 and 20 % pruned, up to 8 rows: three loads a panel, so that the staging area has two slots.  Four panels to a
    workgroup of 16 or of 8 wavefronts, six, and fewer."""
    period, K = 80, (4096 if bits == 4 else 2048) + 16
    N = 16 * panels - 3
    times = -(-N // period)
    x = gi.activations(8, K, seed=18)
    for sparsity in (0.1, 0.2):
        h, c = repeated(period, times, N, K, 16, bits, sparsity, integer_zeros, seed=99)
        ref = oracle.gemv(c, x, threads=8)
        for rows in (5, 8):
            y = run_gemv(torch_cuda, h, x[:rows], panels=True)
            for b in range(rows):
                assert oracle.rel_error(y[b][:period], ref[b]) <= TOL
                assert np.array_equal(y[b].view(np.uint16), np.tile(y[b][:period], times)[:N].view(np.uint16))


def test_panel_kernel_a_tenth_fewer_groups_take_no_longer(torch_cuda):
    """32000x2048, trained zeros, 8 rows: with 10 % pruned three of a workgroup's four panels would fit the staging area; staged
    three and one they took 1.07 to 1.09 times as long as the unpruned ones (panel by panel, in two slots: no longer)."""
    N, K, period = 32000, 2048, 80
    full, pruned = (repeated(period, N // period, N, K, 16, 4, s, False, seed=98)[0] for s in (0.0, 0.1))
    all_groups, fewer = replay_times(torch_cuda, ((full, 8), (pruned, 8)))
    assert fewer < 1.04 * all_groups


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("integer_zeros", [True, False])
def test_panel_kernel_up_to_eight_rows(torch_cuda, bits, integer_zeros):
    """At most 8 activation rows (two columns a product): odd and even counts of columns around a pair, a unit (16 or 8
    columns) and a slice (32), one panel and several, pruned rows next to full ones, and 9 rows beside them."""
    rng = np.random.default_rng(17)
    for N, columns in ((3, 1), (16, 2), (17, 7), (40, 8), (100, 9), (33, 16), (5000, 17), (20, 31), (4500, 33), (70, 127)):
        K = 16 * columns
        W = gi.dense_weight(N, K, seed=columns)
        keep = rng.integers(0, columns + 1, N).astype(np.int32)
        keep[::5] = columns
        keep[N // 2] = 0
        c = oracle.pack(W, 16, bits, keep_per_row=keep)
        if not integer_zeros:
            c.zeros = (c.zeros.view(np.float16) + rng.standard_normal(c.nnzg).astype(np.float16)).view(np.uint16)
        h = gq.gqsa_import(c.rowIndex, c.groups, c.values, c.scales, c.zeros, N, K, 16, bits)
        gq.gqsa_build_panels(h)
        x = gi.activations(9, K, seed=columns + 1)
        y8, _ = check(torch_cuda, h, c, x[:8], panels=True)
        check(torch_cuda, h, c, x, panels=True)
        for batch in (1, 5, 7):
            y, _ = check(torch_cuda, h, c, x[:batch], panels=True)
            assert np.array_equal(y.view(np.uint16), y8[:batch].view(np.uint16)), (N, columns, batch)


@pytest.mark.parametrize("integer_zeros", [True, False])
@pytest.mark.parametrize("bits,G", [(4, 16), (4, 32), (4, 64), (4, 128), (8, 16), (8, 32), (8, 64)])
def test_panel_kernel_rows_have_the_same_bits_in_other_batches(torch_cuda, bits, G, integer_zeros):
    """A row has the same bits in every batch of up to 8 rows and in every batch of 9 to 16, and with G > 16 in all of them, whichever
    way the activations are loaded (one matrix of at most 256 panels: another way from 9, 11 or 12 rows on; more panels: one way)."""
    for N, K in ((70, 35 * G), (4112, 16 * G)):
        c = oracle.pack(gi.dense_weight(N, K, seed=51), G, bits, sparsity=0.4)
        if not integer_zeros:
            c.zeros = (c.zeros.view(np.float16) + np.float16(0.375)).view(np.uint16)
        h = gq.gqsa_import(c.rowIndex, c.groups, c.values, c.scales, c.zeros, N, K, G, bits)
        gq.gqsa_build_panels(h)
        x = gi.activations(16, K, seed=52)
        y = {batch: check(torch_cuda, h, c, x[:batch], panels=True)[0].view(np.uint16) for batch in (1, 3, 8, 9, 10, 11, 12, 13, 16)}
        for batch, rows in y.items():
            same = y[8] if batch <= 8 and G == 16 else y[16]
            assert np.array_equal(rows, same[:batch]), (N, batch)


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("batch", [8, 16])
def test_panel_kernel_infinite_activations_stay_in_their_column(torch_cuda, bits, batch):
    """An infinite or undefined activation reaches the rows that store a group of its column, and no others: rows of even
    columns, rows of odd ones, rows of all; the two columns of a pair share a product, absent groups read a neighbour's."""
    N, columns = 48, 37
    K = 16 * columns
    W = gi.dense_weight(N, K, seed=3)
    for r in range(N):
        W.reshape(N, columns, 16)[r, (1 - r % 3) % 2::2] *= 1e-3 if r % 3 < 2 else 1.0    # r % 3: even columns, odd columns, all of them
    keep = np.array([(columns + 1) // 2 if r % 3 == 0 else columns // 2 if r % 3 == 1 else columns for r in range(N)], np.int32)
    c = oracle.pack(W, 16, bits, keep_per_row=keep)
    stored = np.zeros((N, columns), bool)
    for r in range(N):
        stored[r, c.groups[c.rowIndex[r]:c.rowIndex[r + 1]]] = True
    h = gq.gqsa_pack_rows(W, keep, 16, bits)
    gq.gqsa_build_panels(h)
    x = gi.activations(batch, K, seed=4)
    plain, _ = check(torch_cuda, h, c, x, panels=True)
    for row, column, value in ((0, 4, np.inf), (2, 5, -np.inf), (batch - 1, 36, np.nan)):
        bad = x.copy()
        bad[row, 16 * column + 3] = value
        y = run_gemv(torch_cuda, h, bad, panels=True)
        others = np.arange(batch) != row
        assert np.array_equal(y[others].view(np.uint16), plain[others].view(np.uint16))
        reached = stored[:, column]
        assert not np.isfinite(y[row, reached]).any()
        assert np.isfinite(y[row, ~reached]).all()
        bad[row, 16 * column + 3] = 0
        zero = run_gemv(torch_cuda, h, bad, panels=True)
        assert np.array_equal(y[row, ~reached].view(np.uint16), zero[row, ~reached].view(np.uint16))


@pytest.mark.parametrize("bits", [4, 8])
def test_panel_kernel_unit_vectors_are_bit_exact(torch_cuda, bits):
    """x = e_k in 16 activation rows: y[b] is column k_b of W^, and (q - z) s is exact in fp32, so
    every output is fp16((q - z) s) to the bit -- operand layout of the products, decode, scale
    and zero with no tolerance.  8 of them at a time as well: two columns a product, every place in a
    column and columns on both sides of a pair."""
    N, K = 100, 1024
    W = gi.dense_weight(N, K, seed=95)
    c = oracle.pack(W, 16, bits, sparsity=0.5)
    h = gq.gqsa_pack(W, 16, bits, 0.5)
    gq.gqsa_build_panels(h)
    ks = [0, 1, 15, 16, 17, 255, 256, 511, 512, 513, 777, 1000, 1008, 1022, 1023, 300]
    Wd = oracle.densify(c)
    for group in (ks, ks[:8], ks[8:], *(range(k, k + 8) for k in (0, 8, 16, 24, 992, 1000, 1008, 1016))):
        x = np.zeros((len(group), K), dtype=np.float16)
        for b, k in enumerate(group):
            x[b, k] = 1.0
        y = run_gemv(torch_cuda, h, x)        # from 5 rows on gqsa_gemv itself takes the panel image
        ref = Wd[:, list(group)].T.astype(np.float32).astype(np.float16)
        assert np.array_equal(y.view(np.uint16), ref.view(np.uint16))


def test_panel_kernel_only_from_five_rows(torch_cuda):
    """Below 5 activation rows a handle with a panel image runs the wavefront kernel in gqsa_gemv:
    same bits as a handle without one.  From 5 on it is gqsa_gemv_panels, whose results differ in
    rounding only."""
    N, K = 512, 2048
    W = gi.dense_weight(N, K, seed=96)
    c = oracle.pack(W, 16, 4, sparsity=0.3)
    h1 = gq.gqsa_pack(W, 16, 4, 0.3)
    h2 = gq.gqsa_pack(W, 16, 4, 0.3)
    gq.gqsa_build_panels(h2)
    assert gq.gqsa_info(h2)["panel_bytes"] > 0
    for batch in (1, 3, 4):
        x = gi.activations(batch, K, seed=12)
        assert np.array_equal(run_gemv(torch_cuda, h1, x).view(np.uint16), run_gemv(torch_cuda, h2, x).view(np.uint16))
    x = gi.activations(5, K, seed=13)
    y, _ = check(torch_cuda, h2, c, x)
    assert np.array_equal(y.view(np.uint16), run_gemv(torch_cuda, h2, x, panels=True).view(np.uint16))
    with pytest.raises(gq.GqsaError):
        gq.gqsa_build_panels(h1)         # not after the upload
    with pytest.raises(gq.GqsaError) as e:
        run_gemv(torch_cuda, h1, x, panels=True)     # no such image
    assert e.value.status == 3
    # K above 8192: from 3 rows on
    N, K = 48, 8208
    W = gi.dense_weight(N, K, seed=99)
    c = oracle.pack(W, 16, 4, sparsity=0.5)
    h1 = gq.gqsa_pack(W, 16, 4, 0.5)
    h2 = gq.gqsa_pack(W, 16, 4, 0.5)
    gq.gqsa_build_panels(h2)
    x = gi.activations(3, K, seed=18)
    assert np.array_equal(run_gemv(torch_cuda, h1, x[:2]).view(np.uint16), run_gemv(torch_cuda, h2, x[:2]).view(np.uint16))
    y, _ = check(torch_cuda, h2, c, x)
    assert np.array_equal(y.view(np.uint16), run_gemv(torch_cuda, h2, x, panels=True).view(np.uint16))


@pytest.mark.parametrize("bits,G", [(4, 16), (8, 16), (4, 32)])
def test_panel_kernel_several_matrices_share_a_launch(torch_cuda, bits, G):
    """q/k/v-like: three matrices of different N (4200 rows: 263 panels, more than one per
    workgroup; 130 and 70 rows: ragged last panels) and different sparsity on the same
    activations, 16 and 7 rows.  One launch gives the bits of three separate calls and stays
    within the bound against the oracle; a fourth matrix whose zeros are not integers (the other
    form of Eq. 3) makes the call fall back to one launch per matrix, same bits again."""
    torch = torch_cuda
    K = 24 * G
    shapes = [(4200, 0.5), (130, 0.3), (70, 0.0)]
    hs, cs = [], []
    for i, (N, sp) in enumerate(shapes):
        W = gi.dense_weight(N, K, seed=120 + i)
        cs.append(oracle.pack(W, G, bits, sparsity=sp))
        h = gq.gqsa_pack(W, G, bits, sp)
        gq.gqsa_build_panels(h)
        hs.append(h)
    c4 = oracle.pack(gi.dense_weight(50, K, seed=124), G, bits, sparsity=0.5)
    c4.zeros = (c4.zeros.view(np.float16) + np.float16(0.25)).view(np.uint16)
    h4 = gq.gqsa_import(c4.rowIndex, c4.groups, c4.values, c4.scales, c4.zeros, 50, K, G, bits)
    gq.gqsa_build_panels(h4)
    assert gq.gqsa_info(h4)["panel_integer_zeros"] == 0
    for batch in (16, 7):
        x = gi.activations(batch, K, seed=17 + batch)
        xt = torch.from_numpy(x).cuda()
        single = [check(torch, h, c, x, panels=True)[0] for h, c in zip(hs + [h4], cs + [c4])]
        for group in (hs, hs + [h4], [h4] + hs[:2]):
            ys = [torch.full((batch, gq.gqsa_info(h)["N"]), float("nan"), dtype=torch.float16, device="cuda") for h in group]
            gq.gqsa_gemv_multi(group, xt, ys)
            torch.cuda.synchronize()
            for h, yy in zip(group, ys):
                want = single[(hs + [h4]).index(h)]
                assert np.array_equal(yy.cpu().numpy().view(np.uint16), want.view(np.uint16))


@pytest.mark.parametrize("bits,G,sparsity", [(4, 16, 0.5), (8, 16, 0.3), (4, 64, 0.5), (4, 16, 0.0)])
def test_panel_kernel_more_workgroups_than_compute_units(torch_cuda, bits, G, sparsity):
    """More than 1024 panels (17 603 rows: 1101 panels, the last with 3 rows): 512 workgroups of
    8 wavefronts, two to a compute unit, each wavefront with several units of the panels."""
    N, K = 17603, 40 * G
    W = gi.dense_weight_chunked(N, K, seed=130)
    c = oracle.pack(W, G, bits, sparsity=sparsity)
    h = gq.gqsa_pack(W, G, bits, sparsity)
    gq.gqsa_build_panels(h)
    x = gi.activations(13, K, seed=19)
    y, _ = check(torch_cuda, h, c, x, panels=True)
    if (bits, G, sparsity) == (4, 16, 0.5):
        # two such matrices in one gqsa_gemv_multi call: too many panels for one launch, so one each
        torch = torch_cuda
        h2 = gq.gqsa_pack(W, G, bits, sparsity)
        gq.gqsa_build_panels(h2)
        ys = [torch.full((13, N), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2)]
        gq.gqsa_gemv_multi([h, h2], torch.from_numpy(x).cuda(), ys)
        torch.cuda.synchronize()
        for yy in ys:
            assert np.array_equal(yy.cpu().numpy().view(np.uint16), y.view(np.uint16))


def test_panel_kernel_seeded_shapes(torch_cuda):
    """Forty seeded draws of (code width, group size, N, K, per-row keep counts, activation rows):
    row counts that leave the last panel ragged or give a workgroup one to four panels, K from one
    group-column to several slices with a short last one, rows from empty to full."""
    rng = np.random.default_rng(2024)
    formats = [(4, 16), (8, 16), (4, 32), (4, 64), (4, 128), (8, 32), (8, 64)]
    for case in range(40):
        bits, G = formats[case % len(formats)]
        N = int(rng.choice([1, 15, 16, 17, 100, 257, 1000, 4100, 4200, 8300]))
        cols = int(rng.choice([1, 2, 15, 16, 17, 31, 32, 33, 47, 64, 70]))
        if N > 1000:
            cols = min(cols, 33)
        K = cols * G
        batch = int(rng.integers(1, 17))
        style = case % 4
        if style == 0:
            keep = rng.integers(0, cols + 1, size=N)
        elif style == 1:
            keep = np.full(N, cols)
        elif style == 2:
            keep = np.where(rng.random(N) < 0.5, 0, rng.integers(0, cols + 1, size=N))
        else:
            keep = np.full(N, (cols + 1) // 2)
        keep = keep.astype(np.int32)
        W = gi.dense_weight(N, K, seed=500 + case)
        c = oracle.pack(W, G, bits, keep_per_row=keep)
        h = gq.gqsa_pack_rows(W, keep, G, bits)
        gq.gqsa_build_panels(h)
        try:
            check(torch_cuda, h, c, gi.activations(batch, K, seed=600 + case), panels=True)
        except AssertionError as e:
            raise AssertionError(f"case {case}: bits={bits} G={G} N={N} K={K} batch={batch} style={style}: {e}")
        gq.gqsa_free(h)


@pytest.mark.parametrize("bits,G,sparsity", [(4, 16, 0.0), (4, 16, 0.2), (8, 16, 0.0), (4, 64, 0.1), (8, 64, 0.0)])
def test_panel_kernel_dense_panels(torch_cuda, bits, G, sparsity):
    """Four panels per workgroup (769 panels on 256 workgroups) that are dense or nearly so: a
    wavefront's staging area in LDS then holds two panels' records at a time, not four (and the
    fullest records a unit can have, 16 rows x all its columns).  The last panel has 5 rows."""
    N, K = 16 * 768 + 5, 32 * G
    W = gi.dense_weight_chunked(N, K, seed=98)
    c = oracle.pack(W, G, bits, sparsity=sparsity)
    h = gq.gqsa_pack(W, G, bits, sparsity)
    gq.gqsa_build_panels(h)
    x = gi.activations(16, K, seed=16)
    check(torch_cuda, h, c, x, panels=True)
    check(torch_cuda, h, c, x[:8], panels=True)


@pytest.mark.parametrize("bits,G", [(4, 16), (8, 16), (4, 64), (8, 32)])
@pytest.mark.parametrize("zeros", ["fractional", "large", "extreme_integers"])
def test_panel_kernel_any_zero(torch_cuda, bits, G, zeros):
    """The matrix-core kernel subtracts the zero from the codes only when every stored zero is an
    integer of at most 1024 in magnitude (then exactly); trained zeros (Sec. 3.4) may be any fp16
    number and take the other form of Eq. 3, s (sum q x - z sum x).  Fractional zeros, zeros
    beyond 1024, and integer zeros at +-1024 with the codes at both ends of their range."""
    N, K = 77, 40 * G
    W = gi.dense_weight(N, K, seed=97)
    c = oracle.pack(W, G, bits, sparsity=0.4)
    rng = np.random.default_rng(3)
    z = c.zeros.view(np.float16).astype(np.float32)
    if zeros == "fractional":
        z = z + rng.standard_normal(c.nnzg).astype(np.float32) * 3
    elif zeros == "large":
        z[::7] = 1025.0
        z[3::11] = -2048.0
    else:
        z[::2] = 1024.0
        z[1::2] = -1024.0
        c.values[: c.values.size // 2] = 0xFF
        c.values[c.values.size // 2:] = 0x00
    c.zeros = z.astype(np.float16).view(np.uint16)
    h = gq.gqsa_import(c.rowIndex, c.groups, c.values, c.scales, c.zeros, N, K, G, bits)
    gq.gqsa_build_panels(h)
    assert gq.gqsa_info(h)["panel_integer_zeros"] == (1 if zeros == "extreme_integers" else 0)
    x = gi.activations(16, K, seed=15)
    check(torch_cuda, h, c, x, panels=True)
    check(torch_cuda, h, c, x[:8], panels=True)


@pytest.mark.parametrize("bits,shape_idx", [(4, 0), (8, 1)])
def test_panel_kernel_full_size(torch_cuda, bits, shape_idx):
    """4096x4096 (W4) and 14336x4096 (W8) at S = 50 %, 16 activation rows; every output checked.
    Also several matrices in one call."""
    name, N, K = gi.SMALL_BATCH_SHAPES[shape_idx]
    W = gi.dense_weight_chunked(N, K, seed=gi.config_seed(5, shape_idx))
    c = oracle.pack(W, 16, bits, sparsity=0.5)
    h = gq.gqsa_pack(W, 16, bits, 0.5)
    gq.gqsa_build_panels(h)
    x = gi.activations(16, K, seed=14)
    y, ref = check(torch_cuda, h, c, x)
    if shape_idx == 0:
        h2 = gq.gqsa_pack(W, 16, bits, 0.5)
        gq.gqsa_build_panels(h2)
        xt = torch_cuda.from_numpy(x).cuda()
        ys = [torch_cuda.full((16, N), float("nan"), dtype=torch_cuda.float16, device="cuda") for _ in range(2)]
        gq.gqsa_gemv_multi([h, h2], xt, ys)
        torch_cuda.cuda.synchronize()
        for yy in ys:
            assert np.array_equal(yy.cpu().numpy().view(np.uint16), y.view(np.uint16))


def test_graph_replays_match_eager(torch_cuda):
    """The calls captured in a HIP graph (as the benchmark and a decoder would issue them) and
    replayed several times, with eager work and synchronisation between the replays: every replay
    gives the bits of the eager calls.  Rows shared by wavefronts and by workgroups (the fix-up
    leaves its counters and meeting points ready for the next launch by itself), several
    matrices per launch, tiles of a chosen shape, and the matrix-core kernel."""
    torch = torch_cuda
    N, K = 257, 2048
    W = gi.dense_weight(N, K, seed=61)
    keep = gi.imbalanced_keep_counts(N, K // 16, seed=61)
    ha = gq.gqsa_pack_rows(W, keep, 16, 4)
    gq.gqsa_set_partition(ha, 37, 3)                         # chains across workgroups
    hb = gq.gqsa_pack_rows(W, keep, 16, 4)
    gq.gqsa_set_partition_aligned(hb, 4, 0, 4)               # rows kept inside the workgroups' spans
    hf = gq.gqsa_pack_rows(W, keep, 16, 4)
    gq.gqsa_set_partition_rows(hf, 5, 60, 1, 0, 4)            # tiles of a chosen shape, whole rows per worker
    hc = gq.gqsa_pack_rows(W, keep, 16, 4)
    gq.gqsa_set_partition(hc, 5, 4)
    hp = gq.gqsa_pack_rows(W, keep, 16, 8)
    gq.gqsa_build_panels(hp)
    hq = [gq.gqsa_pack_rows(W, keep, 16, 4) for _ in range(3)]   # three matrices in one launch of the matrix-core kernel
    for h in hq:
        gq.gqsa_build_panels(h)
    x7 = torch.from_numpy(gi.activations(7, K, seed=65)).cuda()
    x1 = torch.from_numpy(gi.activations(1, K, seed=62)).cuda()
    x3 = torch.from_numpy(gi.activations(3, K, seed=63)).cuda()
    x16 = torch.from_numpy(gi.activations(16, K, seed=64)).cuda()

    def outputs():
        return [torch.full((1, N), float("nan"), dtype=torch.float16, device="cuda"),
                torch.full((3, N), float("nan"), dtype=torch.float16, device="cuda"),
                torch.full((1, N), float("nan"), dtype=torch.float16, device="cuda"),
                torch.full((1, N), float("nan"), dtype=torch.float16, device="cuda"),
                torch.full((16, N), float("nan"), dtype=torch.float16, device="cuda"),
                torch.full((7, N), float("nan"), dtype=torch.float16, device="cuda"),
                torch.full((7, N), float("nan"), dtype=torch.float16, device="cuda"),
                torch.full((7, N), float("nan"), dtype=torch.float16, device="cuda"),
                torch.full((7, N), float("nan"), dtype=torch.float16, device="cuda"),
                torch.full((1, N), float("nan"), dtype=torch.float16, device="cuda"),
                torch.full((3, N), float("nan"), dtype=torch.float16, device="cuda")]

    def issue(ys):
        gq.gqsa_gemv(ha, x1, ys[0])
        gq.gqsa_gemv(ha, x3, ys[1])
        gq.gqsa_gemv_multi([hb, hc], x1, [ys[2], ys[3]])
        gq.gqsa_gemv(hp, x16, ys[4])
        gq.gqsa_gemv_multi(hq, x7, ys[5:8])
        gq.gqsa_gemv(hb, x7, ys[8])                         # 7 rows in the kernel for 8
        gq.gqsa_gemv(hf, x1, ys[9])
        gq.gqsa_gemv(hf, x3, ys[10])

    eager = outputs()
    issue(eager)
    torch.cuda.synchronize()
    want = [y.cpu().numpy().view(np.uint16).copy() for y in eager]
    assert all(np.isfinite(y.cpu().numpy()).all() for y in eager)

    ys = outputs()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        issue(ys)                                           # (uploads and first-use set-up happen outside the capture)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        issue(ys)
    torch.cuda.synchronize()
    for replay in range(4):
        for y in ys:
            y.fill_(float("nan"))                          # eager work between the replays
        issue(outputs())                                    # and the same kernels, eagerly, on the handles' workspaces
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for y, w in zip(ys, want):
            assert np.array_equal(y.cpu().numpy().view(np.uint16), w), f"replay {replay}"


def test_llama7b_qkv_and_gate_up_fused_full_size(torch_cuda):
    """The fused launches the benchmark times: q/k/v (3 x 4096x4096) and gate/up (2 x 11008x4096)."""
    torch = torch_cuda
    x_np = gi.activations(1, 4096, seed=gi.config_seed(2, 0))
    x = torch.from_numpy(x_np).cuda()
    for idxs in ((0, 1, 2), (4, 5)):
        hs, cs = [], []
        for idx in idxs:
            name, N, K = gi.LLAMA7B_LAYER[idx]
            W = gi.dense_weight(N, K, seed=gi.config_seed(2, idx))
            hs.append(gq.gqsa_pack(W, 16, 4, 0.5))
            cs.append(oracle.pack(W, 16, 4, sparsity=0.5))
        ys = gq.gqsa_gemv_multi(hs, x)
        torch.cuda.synchronize()
        for y, c in zip(ys, cs):
            assert oracle.rel_error(y.cpu().numpy()[0], oracle.gemv(c, x_np, threads=8)[0]) <= TOL


def test_w8_full_size(torch_cuda):
    W = gi.dense_weight(4096, 4096, seed=gi.config_seed(5, 0))
    h = gq.gqsa_pack(W, 16, 8, 0.5)
    c = oracle.pack(W, 16, 8, sparsity=0.5)
    check(torch_cuda, h, c, gi.activations(2, 4096, seed=gi.config_seed(5, 0)))


@pytest.mark.parametrize("bits", [4, 8])
def test_small_batch_4096x4096_wavefront_kernel_full_size(torch_cuda, bits):
    """4096x4096 S50 with 1, 2, 4, 8 and 16 activation rows on the wavefront kernel (a handle
    without the second image), default partition: every output of every row against the oracle,
    every row identical whatever the batch size it was part of."""
    torch = torch_cuda
    N, K = 4096, 4096
    seed = gi.config_seed(5, 0)
    W = gi.dense_weight(N, K, seed=seed)
    h = gq.gqsa_pack(W, 16, bits, 0.5)
    c = oracle.pack(W, 16, bits, sparsity=0.5)
    assert gq.gqsa_info(h)["panel_bytes"] == 0
    x_np = gi.activations(16, K, seed=seed)
    ref = oracle.gemv(c, x_np, threads=8)
    y16 = run_gemv(torch, h, x_np)
    for batch in (1, 2, 3, 4, 8, 16):
        y = run_gemv(torch, h, x_np[:batch])
        for b in range(batch):
            assert oracle.rel_error(y[b], ref[b]) <= TOL, (batch, b)
        assert np.array_equal(y.view(np.uint16), y16[:batch].view(np.uint16)), batch


@pytest.mark.parametrize("bits", [4, 8])
def test_small_batch_full_size(torch_cuda, bits):
    """14336x4096 S50 with 1, 2, 4, 8 and 16 activation rows (16 = two launches of 8): every
    output of every row against the oracle, and row 0 identical whatever the batch size."""
    torch = torch_cuda
    N, K = 14336, 4096
    seed = gi.config_seed(5, 1)
    W = gi.dense_weight(N, K, seed=seed)
    h = gq.gqsa_pack(W, 16, bits, 0.5)
    c = oracle.pack(W, 16, bits, sparsity=0.5)
    x_np = gi.activations(16, K, seed=seed)
    ref = oracle.gemv(c, x_np, threads=8)
    first = None
    for batch in (1, 2, 4, 8, 16):
        y = run_gemv(torch, h, x_np[:batch])
        for b in range(batch):
            assert oracle.rel_error(y[b], ref[b]) <= TOL, (batch, b)
        if first is None:
            first = y[0].copy()
        assert np.array_equal(y[0].view(np.uint16), first.view(np.uint16)), batch


# ----------------------------------------------------------------------------- side-by-side kernels

def test_dense_f16_gemv_baseline(torch_cuda):
    torch = torch_cuda
    N, K = 1000, 4096
    W = gi.dense_weight(N, K, seed=73).astype(np.float16)
    x = gi.activations(2, K, seed=13)
    y = gq.gqsa_dense_f16_gemv(torch.from_numpy(W).cuda(), torch.from_numpy(x).cuda())
    torch.cuda.synchronize()
    ref = x.astype(np.float64) @ W.astype(np.float64).T
    for b in range(2):
        assert oracle.rel_error(y[b].cpu().numpy(), ref[b]) <= TOL


def test_stream_read_kernel_runs(torch_cuda):
    torch = torch_cuda
    buf = torch.arange(1 << 20, dtype=torch.int32, device="cuda")
    sink = torch.zeros(gq.gqsa_stream_read_workgroups(), dtype=torch.int32, device="cuda")
    gq.gqsa_stream_read(buf, sink)
    torch.cuda.synchronize()
    x = 0
    for v in sink.cpu().numpy().view(np.uint32):
        x ^= int(v)
    ref = int(np.bitwise_xor.reduce(np.arange(1 << 20, dtype=np.uint32)))
    assert x == ref


def test_copy_kernel(torch_cuda):
    torch = torch_cuda
    src = torch.arange(1 << 18, dtype=torch.int32, device="cuda")
    dst = torch.zeros_like(src)
    gq.gqsa_copy(dst, src)
    torch.cuda.synchronize()
    assert torch.equal(dst, src)

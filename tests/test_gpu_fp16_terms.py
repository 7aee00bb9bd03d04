"""Operands in terms (gemm_terms.h) beyond what test_gpu_term_tiles.py holds: scales of the fp16 terms' rows,
whose first K-slice says nothing about the rest of them, in every tile of the steps, and of the columns of
the weight gradients, whose sums may consist of the smallest values of a column alone; the wide tiles of
the adjoint and the projection."""
import numpy as np
import pytest
import torch

from oracle import mgrit_gru_oracle as orc
from synthetic_inputs import random_small

pytestmark = pytest.mark.gpu
T, CF = 6, 3


# batch sizes and widths of the five tiles of each direction (two launch rows per batch row), K tails, and of
# the tiles for one workgroup per CU: the adjoint's 128 x 256 and 64 x 128 and the forward 64 x 64 with split
# K, with gates of whole K-slices (416 = 13 x 32, 448 = 7 x 64) and without.  Per case the forward tile, the
# adjoint's of relaxation and of the residual (None: one that another case is for).
NARROW, MID, BIG = "2, 1, 1, 1, 3, true, 2, 1, 2", "2, 2, 1, 1, 3, true, 1, 1, 2", "2, 2, 2, 1, 3, true, 1, 1, 2"
A_MID, A_WIDE = "2, 2, 1, 1, 1, true, 2, 1, 2", "2, 2, 1, 2, 1, true, 1, 1, 2"
A_BIG8, A_BIG = "4, 2, 1, 2, 1, true, 1, 1, 2", "2, 2, 2, 2, 1, true, 1, 1, 2"
HUGE, WIDE_KS, MID_KS = "2, 4, 2, 2, 1, true, 1, 1, 1", "2, 2, 1, 2, 1, true, 2, 1, 1", "2, 2, 1, 1, 3, true, 2, 1, 1"
TILES = [(2050, 136, NARROW, A_MID, A_MID), (6145, 136, MID, A_WIDE, A_WIDE), (12225, 136, BIG, A_BIG8, A_BIG),
         (1350, 264, NARROW, A_MID, A_MID), (4100, 264, MID, A_WIDE, A_WIDE), (6100, 392, None, HUGE, HUGE),
         (6100, 416, None, HUGE, HUGE), (1000, 392, MID_KS, None, None), (1000, 448, MID_KS, None, None),
         (1801, 392, None, WIDE_KS, WIDE_KS), (1801, 448, None, WIDE_KS, WIDE_KS)]


def kernels(step, *tiles):
    """Name parts of the kernels of the modes relaxation (0) and residual (1) on these tiles."""
    return [f"{step}_step_kernel_bf16<mg::TileCfgB<{c}, 3, 32, true, false>, {m}" for m, c in enumerate(tiles) if c]


@pytest.mark.parametrize("B,H,phi,adj,adj_resid", TILES, ids=[f"{c[0]}-{c[1]}" for c in TILES])
def test_rows_that_differ_from_their_first_slice(B, H, phi, adj, adj_resid):
    """Row 0: nothing but zeros; 1: zeros in the first 72 columns (both K-split groups' slice); 2: the
    rest 2^14 times the first slice, which overflows in its scale, so that its tile's rows are read
    through; 3: a first slice 2^14 times the rest; 4: all of it 2^-40.  The bar is that of the other
    parity tests, 1e-5 of a row's largest value; an fp16 term that overflowed or a row scaled by
    another one's exponent would be off by a power of two.  (No state is beyond one: gates of states of
    2^14 saturate on sums that fp32 itself rounds to 1e-3.)"""
    import gpu_harness as gh
    print("fp16 terms, rows", B, H, flush=True)
    d = random_small(11, T, B, 8, H, scale=0.5 / np.sqrt(H))

    def mark(a):
        a[0] = 0
        a[1, :72] = 0
        a[2, :72] *= 2.0 ** -14
        a[3, 32:] *= 2.0 ** -14
        a[4] *= 2.0 ** -40

    mark(d["h0"])
    mark(d["dL_dhT"])
    r = [0, 1, 2, 3, 4, 5, B - 1]
    P, z = (d["W"], d["U"], d["b_i"], d["b_h"]), np.zeros((T + 1, len(r), H))
    h_ref, _ = orc.mgrit_forward(*P, d["x"][:, r], d["h0"][r], z, CF, 2, 1)
    run = gh.GpuRun(d, cf=CF, levels=2)
    box = []
    gh.expect_kernels(lambda: box.append(run.forward_iterates(1)),
                      *kernels("phi", phi, phi))
    h = box[0][0][-1]
    for i, b in enumerate(r):
        for t in range(T + 1):
            assert gh.rel_err(h[t, b], h_ref[t, i]) <= 1e-5 or not h_ref[t, i].any(), ("h", b, t)
    box = []
    gh.expect_kernels(lambda: box.append(run.backward_iterates(h, 1)),
                      *kernels("adj", adj, adj_resid))
    w = box[0][0][-1]
    want = orc.mgrit_backward(*P, d["x"][:, r], h[:, r], d["dL_dhT"][r], z, CF, 2, 1)[0]
    for i, b in enumerate(r):
        for t in range(T + 1):
            if want[t, i].any():
                assert gh.rel_err(w[t, b], want[t, i]) <= 1e-5, ("w", b, t)
            else:
                assert not np.asarray(w[t, b]).any(), ("w", b, t)


@pytest.mark.parametrize("B,H,phi,adj,adj_resid", TILES, ids=[f"{c[0]}-{c[1]}" for c in TILES])
def test_rows_beside_one_that_is_not_finite(B, H, phi, adj, adj_resid):
    """An infinity in a batch row of the first tile: the tiles that hold it are read through, then contracted
    in fp32 operand by operand, and the other rows come out as if it were not there."""
    import gpu_harness as gh
    print("fp16 terms, beside an infinity", B, H, flush=True)
    d, bad, r = random_small(15, T, B, 8, H, scale=0.5 / np.sqrt(H)), 2, [0, 1, 3, 31, 33, 62, B - 1]
    P, z = (d["W"], d["U"], d["b_i"], d["b_h"]), np.zeros((T + 1, len(r), H))
    h_ref, _ = orc.mgrit_forward(*P, d["x"][:, r], d["h0"][r], z, CF, 2, 1)
    want = orc.mgrit_backward(*P, d["x"][:, r], h_ref.astype(np.float32), d["dL_dhT"][r], z, CF, 2, 1)[0]
    run = gh.GpuRun(d, cf=CF, levels=2)
    h_fin = run.forward_iterates(1)[0][-1]
    run.t["h0"][bad, 7] = float("inf")
    box = []
    gh.expect_kernels(lambda: box.append(run.forward_iterates(1)), *kernels("phi", phi, phi))
    h = box[0][0][-1]
    assert not np.isfinite(h[:, bad]).all()
    for i, b in enumerate(r):
        assert gh.rel_err(h[:, b], h_ref[:, i]) <= 1e-5, ("h", b)
    run.t["dL_dhT"][bad, 7] = float("inf")
    box = []
    gh.expect_kernels(lambda: box.append(run.backward_iterates(h_fin, 1)), *kernels("adj", adj, adj_resid))
    w = box[0][0][-1]
    assert not np.isfinite(w[:, bad]).all()
    for i, b in enumerate(r):
        assert gh.rel_err(w[:, b], want[:, i]) <= 1e-5, ("w", b)


@pytest.mark.parametrize("D", [72, 200])
def test_columns_that_differ_from_their_last_slice(D):
    """Weight gradients: the columns of both operands are scaled, by scales that move along the rows.  Inputs
    that become zeros (3), smaller by 2^14 (5) and larger by 2^14 (6) in the last steps; an adjoint column
    (7, of all three gates) that starts at zero.  128-column tiles (D 72), both widths (D 200)."""
    import gpu_harness as gh
    print("fp16 terms, columns", D, flush=True)
    steps, B, H = 64, 67, 136
    d = random_small(12, steps, B, D, H, scale=0.3 / np.sqrt(H))
    d["x"][-2:, :, 3] = 0
    d["x"][-2:, :, 5] *= 2.0 ** -14
    d["x"][:-2, :, 6] *= 2.0 ** -14
    d["dL_dhT"][:, 7] = 0
    P = (d["W"], d["U"], d["b_i"], d["b_h"])
    h = orc.serial_scan(*P, d["x"], d["h0"]).astype(np.float32)
    want = orc.serial_bptt(*P, d["x"], h, d["dL_dhT"])
    run = gh.GpuRun(d)
    box = []
    gh.expect_kernels(lambda: box.append(run.serial_backward(h)), "grad_gemm_x3_kernel")
    for name, g, r in zip(("w", "dW", "dU", "db_i", "db_h"), box[0], want):
        assert gh.rel_err(g, r) <= 1e-5, name
    for n in (3, 5, 6):
        assert gh.rel_err(box[0][1][:, n], want[1][:, n]) <= 1e-5, ("dW", n)
    for m in (7, H + 7, 2 * H + 7):
        assert gh.rel_err(box[0][2][m], want[2][m]) <= 1e-5, ("dU", m)


def graded(kind, d):
    """Inputs whose weight gradients, or single columns of them, are sums of numbers far below others of the
    same column of an operand.  (The adjoint decays backwards, by 2^-0.3 to 2^-1 a step; with one batch row
    a row split holds 128 steps.)  Returns the columns of dW to look at."""
    T, B, D = d["x"].shape
    if kind.startswith("ends"):              # no inputs in the last steps (end-padded sequences)
        d["x"][T - int(kind[4:]):] = 0
    elif kind.startswith("event"):           # one input that is there in one step only
        d["x"][:, :, 3] = 0
        d["x"][T - int(kind[5:]), :, 3] = 1
    elif kind == "decaying":                 # inputs that fade while the adjoint grows
        d["x"] *= 2.0 ** -np.maximum(0, np.arange(T) - T + 100)[:, None, None]
    elif kind == "impulse":                  # states that fade: one input step, no biases
        d["x"][:] = 0
        d["x"][T - 100] = 1
        d["h0"][:] = d["b_i"][:] = d["b_h"][:] = 0
    elif kind == "sample":                   # an input of a batch row that the loss hardly depends on
        d["dL_dhT"][5] *= 2.0 ** -40
        d["x"][:, :, 3] = 0
        d["x"][:, 5, 3] = 1
    elif kind == "masked":                   # a batch row with large inputs that the loss does not depend on
        d["x"][:, 5] *= 2.0 ** 24
        d["dL_dhT"][5] = 0
    elif kind == "small":                    # the loss depends on the batch row with the smallest inputs only
        d["x"][:, 5] *= 2.0 ** -40
        d["dL_dhT"][:5] = d["dL_dhT"][6:] = 0
    d.update({k: np.ascontiguousarray(v, dtype=np.float32) for k, v in d.items()})


@pytest.mark.parametrize("prop", [orc.IMPLICIT, orc.CLASSIC])
@pytest.mark.parametrize("kind,T,B", [("ends32", 1024, 1), ("ends64", 1024, 1), ("ends96", 1024, 1),
                                      ("ends16", 256, 4), ("event50", 1024, 1), ("event20", 512, 2),
                                      ("event100", 1024, 1), ("decaying", 1024, 1), ("impulse", 1024, 1),
                                      ("sample", 65, 33), ("masked", 64, 33), ("small", 64, 33)])
@pytest.mark.parametrize("D", [72, 200])
def test_gradients_of_graded_sums(D, kind, T, B, prop):
    """Every column of dW and dU to 1e-5 of its own largest value, however small beside the others: a
    32-bit sum gives that, whatever the largest value is that the same column of an operand holds at
    another step or in another batch row.  (65 x 33 rows: the last slice is a row long.)"""
    import gpu_harness as gh
    print("graded sums", D, kind, T, B, prop, flush=True)
    H = 136
    d = random_small(14, T, B, D, H, scale=0.3 / np.sqrt(H))
    graded(kind, d)
    P = (d["W"], d["U"], d["b_i"], d["b_h"])
    h = orc.serial_scan(*P, d["x"], d["h0"], prop).astype(np.float32)
    want = orc.serial_bptt(*P, d["x"], h, d["dL_dhT"], prop)
    run = gh.GpuRun(d, propagator=prop)
    box = []
    gh.expect_kernels(lambda: box.append(run.serial_backward(h)), "grad_gemm_x3_kernel")
    worst = {}
    for name, g, r in (("dW", box[0][1], want[1]), ("dU", box[0][2], want[2])):
        for n in range(r.shape[1]):
            top = np.max(np.abs(r[:, n]))
            if top > 2.0 ** -90:
                worst[name] = max(worst.get(name, (0, 0)), (gh.rel_err(g[:, n], r[:, n]), n))
    print(worst, flush=True)
    assert worst and all(e <= 1e-5 for e, _ in worst.values()), worst


@pytest.mark.parametrize("value", [None, 3.4e38])
def test_wide_projection(value):
    """128 x 256 tiles on three bf16 terms, packed weights: rows, columns (600) and K (136) with tails; one
    input beyond the terms, whose tiles are contracted again in fp32."""
    import gpu_harness as gh
    print("wide projection", value, flush=True)
    B, D, H = 1363, 136, 200
    d = random_small(13, T, B, D, H, scale=0.5 / np.sqrt(H))
    if value:
        d["x"][2, 5, 11] = value
    run = gh.GpuRun(d, cf=CF, levels=2)
    gh.expect_kernels(lambda: run.forward_iterates(1), "projection_kernel_wide")
    got = run.ws[:T * B * 3 * H * 4].view(torch.float32).view(T * B, 3 * H).cpu().numpy()
    want = orc.input_projection(d["W"], d["b_i"], d["x"]).reshape(T * B, 3 * H)
    top = np.max(np.abs(want), axis=1, keepdims=True)
    assert np.all(np.abs(got.astype(np.float64) - want) <= 1e-5 * top)

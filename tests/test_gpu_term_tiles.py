"""The step kernels with fp32 operands as two fp16 terms (gemm_terms.h), tile by tile: each tile of the
dispatch with row, column and K tails, and a row that holds a value near the largest there is (rows
beside one that is not finite: test_gpu_fp16_terms.py).  Every case checks by the names of the launched
kernels that the tile it names has run.  Batch rows are independent, so the oracle (fp64) follows some of
them only.  Bar: 1e-5 of the largest value."""
import numpy as np
import pytest
import torch

import paper_2203_04738_amd as mg
from oracle import lstm_oracle as lo
from oracle import mgrit_gru_oracle as orc
from paper_2203_04738_amd.binding import MgritGruCfg
from synthetic_inputs import random_lstm, random_small, round_to_bf16

pytestmark = pytest.mark.gpu

# tiles: the head of the configuration (waves, blocks, gates) and, where two share it, the K split
NARROW, MID, BIG = "TileCfgB<2, 1, 1, 1, 3, true, 2", "TileCfgB<2, 2, 1, 1, 3, true, 1", "TileCfgB<2, 2, 2, 1, 3, true, 1"
A_MID, A_WIDE = "TileCfgB<2, 2, 1, 1, 1, true, 2", "TileCfgB<2, 2, 1, 2, 1, true, 1"
A_BIG8, A_BIG = "TileCfgB<4, 2, 1, 2, 1, true, 1", "TileCfgB<2, 2, 2, 2, 1, true, 1"
# B (2 B rows per level-0 launch: T = 6, cf = 3), H, forward tile, adjoint tile of relaxation and of
# the residual.  136 and 264 columns: column and K tails everywhere; B: a few rows in the last tile
CASES = [(2050, 136, NARROW, A_MID, A_MID), (6145, 136, MID, A_WIDE, A_WIDE),
         (12225, 136, BIG, A_BIG8, A_BIG), (1350, 264, NARROW, A_MID, A_MID),
         (4100, 264, MID, A_WIDE, A_WIDE)]
T, CF = 6, 3
BIG_VALUE = 3.4e38                  # finite; its row is scaled by 2^-121


@pytest.fixture(scope="module")
def gh():
    import gpu_harness
    return gpu_harness


def _rows(B):
    """Batch rows the oracle follows: the first tile's, one in the middle, the last tile's."""
    return [0, 1, 2, 31, 33, 63, B // 2, B - 2, B - 1]


def _problem(B, H, seed=1):
    d = random_small(seed, T, B, 8, H, scale=0.5 / np.sqrt(H))
    d["U"] *= 2
    return d


def _oracle(d, r):
    """States after one cycle and the adjoint after one, rows r."""
    P, z = (d["W"], d["U"], d["b_i"], d["b_h"]), np.zeros((T + 1, len(r), d["U"].shape[1]))
    h, _ = orc.mgrit_forward(*P, d["x"][:, r], d["h0"][r], z, CF, 2, 1)
    return P, z, h


def _close(got, want, what):
    """Every batch row against its own largest value, elements beyond 1e30 one by one."""
    got = np.asarray(got, dtype=np.float64)
    assert np.all(np.isfinite(got)), what
    huge = np.abs(want) > 1e30
    assert np.all(np.abs(got - want)[huge] <= 1e-5 * np.abs(want)[huge]), what
    rest = np.where(huge, 0.0, want)
    scale = np.max(np.abs(rest), axis=(0, 2), keepdims=True)
    assert np.all(np.where(huge, 0.0, np.abs(got - want)) <= 1e-5 * scale), what


@pytest.mark.parametrize("value", [None, BIG_VALUE])
@pytest.mark.parametrize("B,H,phi,adj,adj_resid", CASES, ids=[f"{c[0]}-{c[1]}" for c in CASES])
def test_gru_tiles(gh, B, H, phi, adj, adj_resid, value):
    """One batch row in the first tile starts at a value that only its row's scale brings into fp16, and all
    rows of its tiles come out as in fp32."""
    print("term tiles", B, H, value, flush=True)
    d, r, bad, col = _problem(B, H), _rows(B), 2, 7
    if value:
        d["h0"][bad, col] = value
    P, z, h_ref = _oracle(d, r)
    run = gh.GpuRun(d, cf=CF, levels=2)
    box = []
    gh.expect_kernels(lambda: box.append(run.forward_iterates(1)),          # relaxation, residual
                      *(f"phi_step_kernel_bf16<mg::{phi}, 1, 2, 3, 32, true, false>, {m}" for m in (0, 1)))
    h = box[0][0][-1]
    _close(h[:, r], h_ref, "h")

    # the adjoint along finite states
    if value:
        d = _problem(B, H)
        P, z, h_ref = _oracle(d, r)
        run = gh.GpuRun(d, cf=CF, levels=2)
        h = run.forward_iterates(1)[0][-1]
        d["dL_dhT"][bad, col] = value
        run.t["dL_dhT"].copy_(torch.from_numpy(d["dL_dhT"]))
    box = []
    gh.expect_kernels(lambda: box.append(run.backward_iterates(h, 1)),
                      f"adj_step_kernel_bf16<mg::{adj}, 1, 2, 3, 32, true, false>, 0",
                      f"adj_step_kernel_bf16<mg::{adj_resid}, 1, 2, 3, 32, true, false>, 1")
    w = box[0][0][-1]
    want = orc.mgrit_backward(*P, d["x"][:, r], h[:, r], d["dL_dhT"][r], z, CF, 2, 1)[0]
    # (linear: the row with the huge terminal value is huge altogether)
    for i in range(len(r)):
        assert gh.rel_err(w[:, r[i]], want[:, i]) <= 1e-5, ("w", r[i])


@pytest.mark.parametrize("form,tol", [("bf16", 2e-2), ("bf16s2", 1e-4)])
@pytest.mark.parametrize("B,H,adj", [(250, 264, "1, 1, 1, 1, 1, true, 4, 1, 2, 1, 64"),
                                     (250, 520, "1, 2, 1, 1, 1, true, 4, 1, 2, 1, 64"),
                                     (457, 520, "1, 4, 1, 1, 1, true, 2, 1, 2, 1, 64"),
                                     (4111, 40, "2, 2, 1, 1, 1, true, 1, 1, 2, 1, 64"),
                                     (829, 520, "2, 2, 1, 1, 1, true, 2, 1, 2, 1, 64"),
                                     (921, 520, "2, 2, 1, 2, 1, true, 2, 1, 2, 1, 64"),
                                     (1665, 520, "2, 4, 1, 2, 1, true, 1, 1, 2, 1, 128"),
                                     (8215, 104, "4, 2, 1, 2, 1, true, 1, 1, 2, 1, 64"),
                                     (8215, 200, "2, 4, 2, 2, 1, true, 1, 1, 2, 1, 64")])
def test_adjoint_tiles_on_bf16_weights(gh, B, H, adj, form, tol):
    """Every tile of the rule with row, column and K tails, relaxation and residual; the bars of the two
    forms are those of the oracle parity tests."""
    print("bf16 adjoint tiles", B, H, form, flush=True)
    d, r = _problem(B, H), _rows(B)
    for k in ("x", "W", "U"):
        d[k] = round_to_bf16(d[k])
    P, z, _ = _oracle(d, r)
    run = gh.GpuRun(d, cf=CF, levels=2, dtype=form)
    h = run.forward_iterates(1)[0][-1]
    box = []
    two = "true" if form == "bf16s2" else "false"
    gh.expect_kernels(lambda: box.append(run.backward_iterates(h, 1)),
                      *(f"adj_step_kernel_bf16<mg::TileCfgB<{adj}, {two}, false>, {m}" for m in (0, 1)))
    want = orc.mgrit_backward(*P, d["x"][:, r], h[:, r], d["dL_dhT"][r], z, CF, 2, 1)[0]
    for i in range(len(r)):
        assert gh.rel_err(box[0][0][-1][:, r[i]], want[:, i]) <= tol, ("w", r[i])


@pytest.mark.parametrize("value", [None, BIG_VALUE])
def test_projection_and_input_gradients(gh, value):
    """Projection (its only user of D as the contracted width) and input gradients, D and 3 H with
    tails; an input row beyond three bf16 terms, contracted again in fp32, and an adjoint row near the largest
    values there are."""
    B, D, H, bad, col = 520, 136, 200, 5, 11
    print("term tiles projection, dx", value, flush=True)
    rng = np.random.default_rng(8)
    d = random_small(9, T, B, D, H, scale=0.5 / np.sqrt(H))
    P = (d["W"], d["U"], d["b_i"], d["b_h"])
    dL = np.zeros((T + 1, B, H), np.float32)
    dL[1:] = rng.standard_normal((T, B, H))
    run = gh.GpuRun(d, cf=CF, levels=2)
    h = run.forward_iterates(1)[0][-1]
    if value:
        dL[T, bad, col] = value
    box = []
    gh.expect_kernels(lambda: box.append(run.backward_steps_iterates(h, dL, 1)),
                      "input_grad_kernel_bf16<mg::TileCfgB<4, 2, 1, 2, 1, true, 1, 1, 2, 3")
    its, _, out = box[0]
    dx = orc.input_gradients(*P, d["x"], h, its[-1])
    for b in range(B):
        assert gh.rel_err(out[4][:, b], dx[:, b]) <= 1e-5, b
    # projection: the first bytes of the workspace
    if value:
        d["x"][2, bad, col] = value
        run.t["x"].copy_(torch.from_numpy(d["x"]))
    gh.expect_kernels(lambda: run.forward_iterates(1),
                      "projection_kernel_bf16<mg::TileCfgB<2, 2, 2, 2, 1, true, 1, 1, 2, 3")
    got = run.ws[:T * B * 3 * H * 4].view(torch.float32).view(T * B, 3 * H).cpu().numpy()
    want = orc.input_projection(d["W"], d["b_i"], d["x"]).reshape(T * B, 3 * H)
    for i in range(T * B):
        assert gh.rel_err(got[i], want[i]) <= 1e-5, i


@pytest.mark.parametrize("value", [None, BIG_VALUE])
@pytest.mark.parametrize("B,H", [(2050, 136), (1030, 264)])
def test_lstm_tiles(gh, B, H, value):
    print("term tiles lstm", B, H, value, flush=True)
    d = random_lstm(3, T, B, 8, H, scale=0.5 / np.sqrt(H))
    r = _rows(B)
    if value:
        d["u0"][2, 7] = value       # the h half of the state
    t = {k: torch.from_numpy(v).to("cuda:0") for k, v in d.items()}
    cfg = MgritGruCfg(T, B, 8, H, cf=CF, levels=2, iters=1)
    ws = torch.empty(mg.mgrit_lstm_workspace_bytes(cfg), dtype=torch.uint8, device="cuda:0")
    u = torch.zeros(T + 1, B, 2 * H, device="cuda:0")

    def solve():
        u.zero_()
        mg.mgrit_lstm_forward(cfg, t["W"], t["U"], t["b_i"], t["b_h"], t["x"], t["u0"], u, None, ws)

    # relaxation, residual, coarse right-hand side
    gh.expect_kernels(solve, *("lstm_step_kernel_x3<mg::TileCfgB<2, 2, 1, 1, 4, true, 1, 1, 2, 3, 32, "
                               f"true, false>, {m}" for m in (0, 1, 2)))
    want, _ = lo.mgrit_lstm_forward(d["W"], d["U"], d["b_i"], d["b_h"], d["x"][:, r], d["u0"][r],
                                    np.zeros((T + 1, len(r), 2 * H)), CF, 2, 1)
    _close(u.cpu().numpy()[:, r], want, "u")


def test_an_infinity_stays_in_its_row(gh):
    """An infinite element: what depends on it is not finite, the other rows of its tile are those
    of the oracle."""
    B, H, _, _, _ = CASES[0]
    d, r, bad = _problem(B, H), _rows(B), 2
    _, _, h_ref = _oracle(d, r)
    d["h0"][bad, 7] = float("inf")
    run = gh.GpuRun(d, cf=CF, levels=2)
    h = run.forward_iterates(1)[0][-1]
    assert not np.isfinite(h[1:, bad, 7]).any()
    keep = [i for i in range(len(r)) if r[i] != bad]
    _close(h[:, [r[i] for i in keep]], h_ref[:, keep], "h")

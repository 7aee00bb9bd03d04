"""Serial solves with a row block per XCD (kernels_scan_xcd.hip) against the oracles: one and two row
quads per block, one and two blocks per XCD, one and two column tiles, ragged rows, columns and K, rings
that wrap several times; and the launch behind them, which takes over what no XCD has taken.
Bar: 1e-5 of the largest value (fp32 sums of at most 1024 terms over 11 steps)."""
import numpy as np
import pytest
import torch

import paper_2203_04738_amd as mg
from oracle import demo_ode_oracle as oo
from oracle import lstm_oracle as lo
from oracle import mgrit_gru_oracle as orc
from paper_2203_04738_amd.binding import MgritGruCfg
from synthetic_inputs import random_lstm, random_ode, random_small

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
T = 11
# B, H -> column tiles, row quads per block (both as the kernel's template arguments say)
SHAPES = [(3, 136, 1, 1), (60, 200, 1, 1), (41, 260, 1, 2), (32, 512, 1, 1), (30, 1000, 2, 1),
          (64, 520, 2, 2)]


@pytest.fixture(scope="module")
def gh():
    import gpu_harness
    return gpu_harness


def _rel(a, b):
    a = a.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(a))
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


def _gru(B, H, steps):
    d = random_small(B * 1000 + H, steps, B, 8, H, scale=0.7 / np.sqrt(H))
    t = {k: torch.from_numpy(v).to(DEV) for k, v in d.items()}
    cfg = MgritGruCfg(steps, B, 8, H)
    ws = torch.empty(mg.mgrit_gru_workspace_bytes(cfg), dtype=torch.uint8, device=DEV)
    g = [torch.empty(3 * H, 8, device=DEV), torch.empty(3 * H, H, device=DEV),
         torch.empty(3 * H, device=DEV), torch.empty(3 * H, device=DEV)]
    h, w = (torch.full((steps + 1, B, H), 7.0, device=DEV) for _ in range(2))
    return d, t, cfg, ws, (t["W"], t["U"], t["b_i"], t["b_h"], t["x"]), h, w, g


@pytest.mark.parametrize("B,H,ct,rb", SHAPES)
def test_against_the_oracles(gh, B, H, ct, rb):
    print("xcd case", B, H, flush=True)
    d, t, cfg, ws, p, h, w, g = _gru(B, H, T)
    P = (d["W"], d["U"], d["b_i"], d["b_h"])

    def kernel(kind):
        return f"xcd_scan_kernel<{kind}, {ct}, "

    gh.expect_kernels(lambda: mg.gru_serial_scan(cfg, *p, t["h0"], h, ws), kernel(0))
    want = orc.serial_scan(*P, d["x"], d["h0"])
    assert _rel(h, want) <= 1e-5
    # (two quads of 32 columns: the adjoint goes another way)
    gh.expect_kernels(lambda: mg.gru_serial_scan_backward(cfg, *p, h, t["dL_dhT"], w, *g, ws),
                      kernel(1) if ct * rb < 4 else "adj_")
    for got, ref in zip((w, *g), orc.serial_bptt(*P, d["x"], want, d["dL_dhT"])):
        assert _rel(got, ref) <= 1e-5
    d = random_lstm(1, T, B, 8, H, scale=0.7 / np.sqrt(H))
    t = {k: torch.from_numpy(v).to(DEV) for k, v in d.items()}
    lws = torch.empty(mg.mgrit_lstm_workspace_bytes(cfg), dtype=torch.uint8, device=DEV)
    u = torch.full((T + 1, B, 2 * H), 7.0, device=DEV)
    gh.expect_kernels(lambda: mg.lstm_serial_scan(cfg, t["W"], t["U"], t["b_i"], t["b_h"], t["x"],
                                                  t["u0"], u, lws),
                      kernel(2) if ct == 1 else "scan_kernel<2, ")
    assert _rel(u, lo.lstm_serial_scan(d["W"], d["U"], d["b_i"], d["b_h"], d["x"], d["u0"])) <= 1e-5
    d = random_ode(2, T, B, 8, H)
    t = {k: torch.from_numpy(v).to(DEV) for k, v in d.items()}
    gh.expect_kernels(lambda: mg.ode_serial_scan(cfg, 0.25, t["A"], t["Bw"], t["b"], t["d"], t["h0"], h,
                                                 lws), kernel(3))
    assert _rel(h, oo.ode_serial_scan(d["A"], d["Bw"], d["b"], d["d"], d["h0"], 0.25)) <= 1e-5


@pytest.mark.parametrize("B,H", [(60, 200), (32, 512), (30, 1000)])
def test_any_part_may_be_taken_over(B, H, monkeypatch):
    # limits around the time the workgroups need to arrive: some XCDs take their rows, some do not
    def solve():
        d, t, cfg, ws, p, h, w, g = _gru(B, H, 40)
        mg.gru_serial_scan(cfg, *p, t["h0"], h, ws)
        mg.gru_serial_scan_backward(cfg, *p, h, t["dL_dhT"], w, *g, ws)
        return h, w, *g

    print("xcd case takeover", B, H, flush=True)
    want = solve()
    for ticks in (0, 30, 100, 200, 300, 400, 600, 1000):
        monkeypatch.setenv("MGRIT_SCAN_WAIT_TICKS", str(ticks))
        assert all(torch.equal(a, b) for a, b in zip(solve(), want)), ticks

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
from paper_2203_04738_amd.binding import MGRIT_BF16, MGRIT_F32, MgritGruCfg
from synthetic_inputs import random_lstm, random_ode, random_small, round_to_bf16

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
T = 11
# B, H -> column tiles, row quads per block, as the kernel's template arguments say
SHAPES = [(3, 136, 1, 1), (60, 200, 1, 1), (41, 260, 1, 2), (32, 512, 1, 1), (30, 1000, 2, 1),
          (64, 520, 2, 2), (90, 512, 1, 3), (125, 388, 1, 4), (255, 132, 1, 3), (70, 1024, 2, 3),
          (101, 516, 2, 4)]


@pytest.fixture(scope="module")
def gh():
    import gpu_harness
    return gpu_harness


def _rel(a, b):
    a = a.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(a))
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


def _gru(B, H, steps, half=False):
    d = random_small(B * 1000 + H, steps, B, 8, H, scale=0.7 / np.sqrt(H))
    t = {}
    for k, v in d.items():
        if half and k in ("x", "W", "U"):
            d[k] = round_to_bf16(v)
        t[k] = torch.from_numpy(d[k]).to(DEV)
        if half and k in ("x", "W", "U"):
            t[k] = t[k].to(torch.bfloat16)
    cfg = MgritGruCfg(steps, B, 8, H, dtype=MGRIT_BF16 if half else MGRIT_F32)
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
        inner = "2, 2, 4" if ct == 2 and kind == 1 else "1, 2, 8" if ct == 2 else \
            f"1, 1, {4 if H <= 256 else 8}"
        return f"xcd_scan_kernel<{kind}, {ct}, {inner}, {rb}, "

    gh.expect_kernels(lambda: mg.gru_serial_scan(cfg, *p, t["h0"], h, ws), kernel(0))
    want = orc.serial_scan(*P, d["x"], d["h0"])
    assert _rel(h, want) <= 1e-5
    gh.expect_kernels(lambda: mg.gru_serial_scan_backward(cfg, *p, h, t["dL_dhT"], w, *g, ws),
                      "adj_" + kernel(1))
    for got, ref in zip((w, *g), orc.serial_bptt(*P, d["x"], want, d["dL_dhT"])):
        assert _rel(got, ref) <= 1e-5
    d = random_lstm(1, T, B, 8, H, scale=0.7 / np.sqrt(H))
    t = {k: torch.from_numpy(v).to(DEV) for k, v in d.items()}
    lws = torch.empty(mg.mgrit_lstm_workspace_bytes(cfg), dtype=torch.uint8, device=DEV)
    u = torch.full((T + 1, B, 2 * H), 7.0, device=DEV)
    gh.expect_kernels(lambda: mg.lstm_serial_scan(cfg, t["W"], t["U"], t["b_i"], t["b_h"], t["x"],
                                                  t["u0"], u, lws),
                      kernel(2) if ct == 1 else "scan_kernel<2, " if B <= 64 else "lstm_step_kernel")
    assert _rel(u, lo.lstm_serial_scan(d["W"], d["U"], d["b_i"], d["b_h"], d["x"], d["u0"])) <= 1e-5
    d = random_ode(2, T, B, 8, H)
    t = {k: torch.from_numpy(v).to(DEV) for k, v in d.items()}
    gh.expect_kernels(lambda: mg.ode_serial_scan(cfg, 0.25, t["A"], t["Bw"], t["b"], t["d"], t["h0"], h,
                                                 lws), kernel(3))
    assert _rel(h, oo.ode_serial_scan(d["A"], d["Bw"], d["b"], d["d"], d["h0"], 0.25)) <= 1e-5


@pytest.mark.parametrize("B,H,ct", [(3, 72, 1), (60, 200, 1), (41, 264, 1), (8, 520, 2), (2, 1024, 2),
                                    (64, 1000, 2), (100, 264, 1), (99, 1024, 2)])
def test_state_in_terms_on_bf16_weights(gh, B, H, ct):
    # exact products of the fp32 state with the weights, fp32 sums: the fp32 bar
    print("xcd case terms", B, H, flush=True)
    d, t, cfg, ws, p, h, *_ = _gru(B, H, T, half=True)
    P = (d["W"], d["U"], d["b_i"], d["b_h"])

    def solve():
        gh.expect_kernels(lambda: mg.gru_serial_scan(cfg, *p, t["h0"], h, ws), f"xcd_scan_kernel<0, {ct}, ")
        return h

    assert _rel(solve(), orc.serial_scan(*P, d["x"], d["h0"])) <= 1e-5
    if B > 2:                       # row 1: a NaN with every bit set; row 2: infinite
        clean = h.clone()
        t["h0"].view(torch.int32)[1, 3] = -1
        t["h0"][2, 5] = float("inf")
        solve()
        keep = [b for b in range(B) if b not in (1, 2)]
        assert torch.equal(h[:, keep], clean[:, keep])
        assert torch.isnan(h[1:, 1]).all() and not torch.isfinite(h[1:, 2, 5]).any()
    # large states: no term overflows
    d["h0"] = (np.random.default_rng(1).uniform(1, 3, (B, H)) * 2.0 ** 120).astype(np.float32)
    t["h0"].copy_(torch.from_numpy(d["h0"]))
    with np.errstate(over="ignore"):
        want = orc.serial_scan(*P, d["x"], d["h0"])
    assert _rel(solve(), want) <= 1e-5


@pytest.mark.parametrize("B,H", [(60, 200), (32, 512), (30, 1000), (100, 512), (100, 1000)])
def test_any_part_may_be_taken_over(B, H, monkeypatch):
    # limits around the time the workgroups need to arrive (who solves what is chance here; the cases of
    # test_some_xcds_solve_and_the_takeover_the_rest choose it)
    def solve():
        out = []
        for half in (False, True):
            d, t, cfg, ws, p, h, w, g = _gru(B, H, 40, half)
            mg.gru_serial_scan(cfg, *p, t["h0"], h, ws)
            mg.gru_serial_scan_backward(cfg, *p, h, t["dL_dhT"], w, *g, ws)
            out += [h, w, *g]
        return out

    print("xcd case takeover", B, H, flush=True)
    want = solve()
    for ticks in (0, 30, 100, 200, 300, 400, 600, 1000):
        monkeypatch.setenv("MGRIT_SCAN_WAIT_TICKS", str(ticks))
        assert all(torch.equal(a, b) for a, b in zip(solve(), want)), ticks


@pytest.mark.parametrize("B,H", [(3, 72), (8, 520), (60, 512), (99, 1024)])
def test_infinite_bf16_weights(gh, B, H):
    # an infinite weight saturates a gate; it makes no NaN where the state it meets is not zero, though
    # most states have terms that are (r, z and n gate, first and last K slice, first and last column)
    print("xcd case infinite weights", B, H, flush=True)
    d, t, cfg, ws, p, h, *_ = _gru(B, H, T, half=True)
    d["h0"] = np.where(np.arange(H) % 2, 0.5, -0.75).astype(np.float32) + 0 * d["h0"]
    # (columns of states that stay away from zero, whose sign is beyond doubt)
    away = np.abs(orc.serial_scan(d["W"], d["U"], d["b_i"], d["b_h"], d["x"], d["h0"])).min((0, 1))
    low, mid, high = (np.argmax(away[i:i + H // 3]) + i for i in (0, H // 3, H - H // 3))
    for row, k, sign in ((1, low, 1), (H + 5, high, -1), (3 * H - 2, mid, 1), (H - 1, high, 1)):
        d["U"][row, k] = sign * np.inf
    t["U"].copy_(torch.from_numpy(d["U"]))
    t["h0"].copy_(torch.from_numpy(d["h0"]))
    with np.errstate(over="ignore"):
        want = orc.serial_scan(d["W"], d["U"], d["b_i"], d["b_h"], d["x"], d["h0"])
    assert np.isfinite(want).all() and np.abs(want[:, :, [low, mid, high]]).min() > 1e-4
    mg.gru_serial_scan(cfg, *p, t["h0"], h, ws)
    assert _rel(h, want) <= 1e-5


def _groups(ws, cfg, width, gates):
    """Groups of row blocks that XCDs have taken, from the control words a scan has left at the head of the
    gradient partials (behind projection, coefficients, U^T and W^T)."""
    def up(n):
        return -(-n // 256) * 256

    T_, B, D, H = cfg.T, cfg.B, cfg.D, width
    at = up(T_ * B * 3 * H * 4) + up((T_ + 1) * B * H * 20) + up(3 * H * H * 4) + up(3 * H * D * 4)
    ctl = ws[at:at + 64].view(torch.int32).cpu().numpy().astype(np.int64)
    nibbles = [(int(ctl[4]) >> 4 * x) & 15 for x in range(8)]
    assert sum(0 < v < 15 for v in nibbles) <= sum(ctl[8:] > 0)     # (words of such a solve: tickets per XCD)
    return sum(0 < v < 15 for v in nibbles)


@pytest.mark.parametrize("xcds", [0x01, 0x5a, 0x7f])
@pytest.mark.parametrize("B,H,need", [(60, 200, 8), (41, 260, 6), (32, 512, 8), (30, 1000, 8), (100, 512, 7),
                                      (255, 132, 8), (100, 200, 7), (100, 1000, 7)])
def test_some_xcds_solve_and_the_takeover_the_rest(B, H, need, xcds, monkeypatch):
    # all kinds, above 64 rows the takeover's grid is larger than the chip; `need` XCDs solve alone
    def solve():
        out, taken = [], []
        for half in ((False, True) if H % 8 == 0 else (False,)):
            d, t, cfg, ws, p, h, w, g = _gru(B, H, 24, half)
            mg.gru_serial_scan(cfg, *p, t["h0"], h, ws)
            taken.append(_groups(ws, cfg, H, 3))
            mg.gru_serial_scan_backward(cfg, *p, h, t["dL_dhT"], w, *g, ws)
            out += [h, w, *g]
        cfg = MgritGruCfg(24, B, 8, H)
        lws = torch.empty(mg.mgrit_lstm_workspace_bytes(cfg), dtype=torch.uint8, device=DEV)
        if H <= 512:
            t = {k: torch.from_numpy(v).to(DEV) for k, v in
                 random_lstm(1, 24, B, 8, H, scale=0.7 / np.sqrt(H)).items()}
            u = torch.full((25, B, 2 * H), 7.0, device=DEV)
            mg.lstm_serial_scan(cfg, t["W"], t["U"], t["b_i"], t["b_h"], t["x"], t["u0"], u, lws)
            taken.append(_groups(lws, cfg, 2 * H, 4))
            out.append(u)
        t = {k: torch.from_numpy(v).to(DEV) for k, v in random_ode(2, 24, B, 8, H).items()}
        o = torch.full((25, B, H), 7.0, device=DEV)
        mg.ode_serial_scan(cfg, 0.25, t["A"], t["Bw"], t["b"], t["d"], t["h0"], o, lws)
        taken.append(_groups(lws, cfg, H, 1))
        return out + [o], taken

    print("xcd case shared", B, H, hex(xcds), flush=True)
    monkeypatch.setenv("MGRIT_SCAN_WAIT_TICKS", "2000000")     # (20 ms: whoever may start does)
    want, taken = solve()
    assert all(torch.isfinite(a).all() for a in want) and set(taken) == {need}
    monkeypatch.setenv("MGRIT_SCAN_XCDS", str(xcds))
    got, taken = solve()
    assert set(taken) == {min(need, bin(xcds).count("1"))}
    assert all(torch.equal(a, b) for a, b in zip(got, want))

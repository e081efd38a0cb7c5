"""GPU parity: the HIP path through the C ABI against the float64 oracle on the same seeded
inputs.  Floating point bar: relative L2 error <= 1e-5 per output tensor (fp32 arithmetic);
mode bookkeeping is covered bit-exactly in test_host_logic.py."""
import numpy as np
import pytest
import torch

from oracle import fno_oracle as O
from paper_2204_01205_amd import binding as B
from paper_2204_01205_amd import synth

pytestmark = pytest.mark.gpu
TOL = 1e-5


def rel(a, b):
    a = np.asarray(a)
    b = np.asarray(b)
    return float(np.linalg.norm((a - b).ravel()) / max(np.linalg.norm(b.ravel()), 1e-300))


def dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    return t.cpu().numpy()


class Layer:
    """Seeded inputs of one layer, on both sides."""

    def __init__(self, batch, c_in, c_out, grid, modes, rule=0, seed=0, activation=B.FNO_ACT_GELU):
        self.spec = O.LayerSpec(tuple(grid), tuple(modes), rule)
        self.counts = tuple(len(k) for k in O.mode_lists(self.spec))
        self.batch, self.c_in, self.c_out = batch, c_in, c_out
        self.act = activation
        self.x = synth.normal_field(seed, synth.T_X, batch, c_in, grid)
        self.R = synth.spectral_weights(seed, c_in, c_out, self.counts)
        self.W = synth.linear_weights(seed, c_out, c_in)
        self.b = synth.bias(seed, c_out)
        self.desc = B.make_desc(batch, c_in, c_out, grid, modes, rule, activation)

    def act_name(self):
        return "gelu" if self.act == B.FNO_ACT_GELU else "identity"


def gpu_spectral_fwd(L, x=None):
    x = dev(L.x if x is None else x)
    y = torch.empty((L.batch, L.c_out) + L.spec.grid, device="cuda")
    xh = torch.empty((L.batch, L.c_in) + L.counts, dtype=torch.complex64, device="cuda")
    ws = B.alloc_workspace(L.desc, B.FNO_OP_SPECTRAL_CONV_FWD)
    B.fno_spectral_conv_fwd(L.desc, x, dev(L.R), y, xh, ws)
    torch.cuda.synchronize()
    return host(y), host(xh)


def gpu_block_fwd(L):
    out = torch.empty((L.batch, L.c_out) + L.spec.grid, device="cuda")
    z = torch.empty_like(out)
    xh = torch.empty((L.batch, L.c_in) + L.counts, dtype=torch.complex64, device="cuda")
    ws = B.alloc_workspace(L.desc, B.FNO_OP_BLOCK_FWD)
    B.fno_block_fwd(L.desc, dev(L.x), dev(L.R), dev(L.W), dev(L.b), out, z, xh, ws)
    torch.cuda.synchronize()
    return host(out), host(z), host(xh)


SMALL = [
    # batch, cin, cout, grid, modes, rule
    (1, 8, 8, (16, 16, 16, 8), (4, 4, 4, 3), 0),       # the small workload
    (2, 3, 3, (6, 5, 12, 6), (2, 2, 3, 4), 0),         # no large power of two on x,y: folded axis products; Nyquist kept
    (1, 2, 3, (4, 6, 8, 7), (1, 2, 2, 4), 1),          # symmetric rule, odd Nt, Cin != Cout
    (1, 4, 4, (32, 24, 64, 16), (6, 5, 12, 8), 0),     # several tiles, ragged column tails
    (5, 2, 2, (8, 8, 8, 4), (2, 2, 2, 3), 0),          # batch above the mix kernel's register tile
    (1, 2, 2, (8, 8, 8, 8), (4, 4, 4, 5), 0),          # every mode kept (L = N, mt = Nt/2+1)
    (1, 2, 2, (8, 4, 8, 8), (1, 1, 1, 1), 0),          # a single t mode
    (1, 1, 1, (1, 1, 1, 1), (0, 0, 0, 1), 1),          # one-point grid
    (1, 3, 2, (10, 3, 20, 5), (2, 1, 4, 2), 1),        # symmetric rule, Cin != Cout, every stage folded
    (1, 3, 3, (2, 3, 32, 16), (1, 1, 4, 5), 0),        # folded inverse, 6 columns, padded channels
    (2, 2, 3, (3, 2, 32, 16), (1, 1, 6, 9), 0),        # same, 17 columns, Cin != Cout
    (1, 20, 20, (2, 2, 32, 32), (1, 1, 8, 9), 0),      # column kernel (Nt = 32), width 20
    (1, 24, 24, (2, 2, 32, 16), (1, 1, 4, 4), 0),      # folded inverse, width 24: one row of a pair at a time
    (1, 8, 8, (2, 3, 128, 32), (1, 1, 16, 9), 0),      # column kernel (Nt = 32): four steps per column; the convolution on the per-tile kernel
    (2, 3, 5, (3, 2, 64, 32), (1, 1, 6, 5), 0),        # folded inverse, padded channel tiles, Cin != Cout
    (1, 4, 4, (2, 2, 32, 32), (1, 1, 16, 17), 0),      # per-tile kernel, every z and t mode kept
    (1, 20, 20, (2, 3, 128, 16), (1, 1, 16, 9), 0),    # column kernel (Nt = 16): width 20 in two passes, two steps; the convolution per tile
    (2, 20, 20, (2, 2, 64, 16), (1, 1, 12, 8), 0),     # same, one step, 24 kept z frequencies and 8 t bins
    (1, 8, 8, (2, 3, 64, 16), (1, 1, 8, 5), 0),        # block per tile, convolution folded, width 8
    (2, 3, 5, (3, 2, 128, 16), (1, 1, 10, 7), 0),      # folded inverse, padded channel tiles, Cin != Cout
    (1, 6, 6, (2, 2, 64, 16), (1, 1, 5, 4), 0),        # block per tile with padded channel tiles, convolution folded
    (1, 2, 2, (2, 2, 16, 64), (1, 1, 4, 9), 0),        # 64-point t axis (forward: the in-register 64-point real transform)
    (1, 2, 2, (2, 2, 256, 16), (1, 1, 20, 5), 0),      # 256-point z axis: one plane fills the forward block, 16 residue classes
    (2, 2, 2, (2, 2, 8, 32), (1, 1, 4, 17), 0),        # 8-point z axis under 32 t points: the forward tile's row stride (17) exceeds N + 1
    (1, 8, 8, (3, 2, 32, 30), (1, 1, 4, 8), 0),        # per-tile kernel, t axis padded 30 -> 32
    (2, 3, 3, (2, 3, 32, 12), (1, 1, 6, 4), 0),        # folded both ways, runs of three steps, padded channel tiles
    (1, 20, 20, (2, 2, 64, 30), (1, 1, 12, 8), 0),     # per-tile kernel, width 20, the z and t lengths of the paper's samples
    (1, 3, 3, (4, 3, 21, 6), (1, 1, 5, 3), 0),         # odd z length: folded both ways
    (2, 5, 4, (2, 2, 37, 16), (1, 1, 9, 8), 0),        # same, prime z length, a ragged second tile of pairs, Cin != Cout
    (1, 2, 2, (3, 3, 35, 4), (1, 1, 6, 2), 1),         # same, two tiles of pairs, symmetric rule
    (1, 2, 2, (2, 2, 135, 8), (1, 1, 30, 3), 0),       # same, two row tiles of frequencies, five tiles of pairs
    (1, 4, 4, (3, 5, 6, 7), (1, 2, 2, 3), 0),          # width 4 with 630 points (not a multiple of 64): the wide
                                                       # backward pointwise kernel (erff / expf), where case 3 of the
                                                       # same width takes the other one (rational erf)
]


@pytest.mark.parametrize("case", SMALL)
def test_spectral_conv_fwd_matches_oracle(case):
    L = Layer(*case)
    y, xh = gpu_spectral_fwd(L)
    yo, xho = O.spectral_conv_fwd(L.x, L.R, L.spec, return_xhat=True)
    assert rel(xh, xho) <= TOL
    assert rel(y, yo) <= TOL


@pytest.mark.parametrize("case", SMALL)
def test_spectral_conv_bwd_matches_oracle(case):
    L = Layer(*case)
    gy = synth.normal_field(1, synth.T_GOUT, L.batch, L.c_out, L.spec.grid)
    gxo, gRo = O.spectral_conv_bwd(L.x, L.R, gy, L.spec)
    ws = B.alloc_workspace(L.desc, B.FNO_OP_SPECTRAL_CONV_BWD)
    gx = torch.empty((L.batch, L.c_in) + L.spec.grid, device="cuda")
    gR = torch.empty((L.c_in, L.c_out) + L.counts, dtype=torch.complex64, device="cuda")
    B.fno_spectral_conv_bwd(L.desc, dev(L.x), None, dev(L.R), dev(gy), gx, gR, ws)
    torch.cuda.synchronize()
    assert rel(host(gx), gxo) <= TOL
    assert rel(host(gR), gRo) <= TOL
    # with the saved spectrum instead of x, and with only one of the two outputs requested
    _, xh = gpu_spectral_fwd(L)
    gR2 = torch.empty_like(gR)
    B.fno_spectral_conv_bwd(L.desc, None, dev(xh), dev(L.R), dev(gy), None, gR2, ws)
    gx2 = torch.empty_like(gx)
    B.fno_spectral_conv_bwd(L.desc, None, None, dev(L.R), dev(gy), gx2, None, ws)
    torch.cuda.synchronize()
    assert rel(host(gR2), gRo) <= TOL
    assert rel(host(gx2), gxo) <= TOL


BLOCKS = [c for c in SMALL if c[1] == c[2]]


@pytest.mark.parametrize("case", BLOCKS)
@pytest.mark.parametrize("activation", [B.FNO_ACT_GELU, B.FNO_ACT_IDENTITY])
def test_block_fwd_and_bwd_match_oracle(case, activation):
    L = Layer(*case, activation=activation)
    out, z, xh = gpu_block_fwd(L)
    oo, zo, xho = O.block_fwd(L.x, L.R, L.W, L.b, L.spec, L.act_name())
    assert rel(out, oo) <= TOL and rel(z, zo) <= TOL and rel(xh, xho) <= TOL

    target = synth.normal_field(2, synth.T_TARGET, L.batch, L.c_out, L.spec.grid)
    gout = synth.normal_field(3, synth.T_GOUT, L.batch, L.c_out, L.spec.grid)
    ws = B.alloc_workspace(L.desc, B.FNO_OP_BLOCK_BWD)
    for mse in (False, True):
        desc = B.make_desc(L.batch, L.c_in, L.c_out, L.spec.grid, L.spec.modes, L.spec.rule,
                           activation, B.FNO_FLAG_MSE_TARGET if mse else 0)
        g_in = target if mse else gout
        # the oracle differentiates its own forward; the GPU gets the z it saved itself
        g_ref = O.mse_grad(oo, target) if mse else gout
        ref = O.block_bwd(L.x, L.R, L.W, L.b, g_ref, L.spec, L.act_name())
        gx = torch.empty((L.batch, L.c_in) + L.spec.grid, device="cuda")
        gR = torch.empty((L.c_in, L.c_out) + L.counts, dtype=torch.complex64, device="cuda")
        gW = torch.empty((L.c_out, L.c_in), device="cuda")
        gb = torch.empty((L.c_out,), device="cuda")
        B.fno_block_bwd(desc, dev(L.x), dev(L.R), dev(L.W), dev(z), dev(xh) if mse else None,
                        dev(g_in), gx, gR, gW, gb, ws)
        torch.cuda.synchronize()
        assert rel(host(gx), ref["gx"]) <= TOL
        assert rel(host(gR), ref["gR"]) <= TOL
        assert rel(host(gW), ref["gW"]) <= TOL
        # gb is a sum of terms of either sign: where they cancel, the error is bounded by the
        # size of the summands (root-sum-square), elsewhere by the sum itself
        gb_scale = np.abs(ref["gb"]) + np.sqrt(np.sum(ref["gz"] ** 2, axis=(0, 2, 3, 4, 5)))
        assert np.max(np.abs(host(gb) - ref["gb"]) / np.maximum(gb_scale, 1e-300)) <= TOL
        assert rel(host(gb), ref["gb"]) <= TOL          # and the criterion of every other tensor, as a vector
        # identical bits on a second run (fixed reduction order)
        gW2 = torch.empty_like(gW)
        gb2 = torch.empty_like(gb)
        gx2 = torch.empty_like(gx)
        B.fno_block_bwd(desc, dev(L.x), dev(L.R), dev(L.W), dev(z), dev(xh) if mse else None,
                        dev(g_in), gx2, None, gW2, gb2, ws)
        torch.cuda.synchronize()
        assert torch.equal(gW, gW2) and torch.equal(gb, gb2) and torch.equal(gx, gx2)


def test_forward_activation_over_its_whole_range():
    # W = 1, R = 0: the pre-activation is x, and the output differs from float64 by the tail's fit (5.1e-8) and the roundings of
    # its exponent (|z| T(|z|) times one unit of log2 T: at most 2.5e-7, near |z| = 4) and of the result
    grid, modes, c = (16, 16, 16, 16), (2, 2, 2, 2), 4
    n = c * 16 ** 4
    x = torch.linspace(-45.0, 45.0, n, dtype=torch.float64).float()
    x[:8] = torch.tensor([0.0, -0.0, 1e20, -1e20, 1e-30, -1e-30, 13.7, -13.7])
    x = x.view(1, c, *grid).cuda()
    desc = B.make_desc(1, c, c, grid, modes, 0, B.FNO_ACT_GELU)
    R = torch.zeros(c, c, 4, 4, 4, 2, dtype=torch.complex64, device="cuda")
    out = torch.empty_like(x)
    B.fno_block_fwd(desc, x, R, torch.eye(c, device="cuda"), torch.zeros(c, device="cuda"), out, None, None,
                    B.alloc_workspace(desc, B.FNO_OP_BLOCK_FWD))
    z = x.double().cpu()
    want = 0.5 * z * torch.erfc(-z / 2 ** 0.5)
    over = (out.cpu().double() - want).abs() - (3.5e-7 + 6.0e-8 * want.abs())
    assert float(over.max()) <= 0.0


@pytest.mark.parametrize("hidden", [8, 2048])
def test_forward_activation_of_huge_values(hidden):
    """W1 = W2 = 1, one hidden unit in use (2048: the kernel whose weights do not fit LDS, with erff): a negative value of any
    size gives zero, a positive one itself, minus infinity what infinity times zero gives, NaN stays.  (As parts of 16 bits
    infinity itself has none: NaN as well.)"""
    big = [16.2, 1e3, 1e20, 1e26, 1e30, 3e38]
    x = torch.tensor([-v for v in big] + big + [-float("inf"), float("nan"), -float("nan")], device="cuda").view(1, 1, -1)
    n = x.shape[2]
    W1, W2, u = torch.zeros(hidden, 1, device="cuda"), torch.zeros(1, hidden, device="cuda"), torch.empty(1, 1, n, device="cuda")
    W1[0, 0] = W2[0, 0] = 1.0
    B.fno_pointwise_mlp2(1, 1, hidden, 1, n, x, W1, torch.zeros(hidden, device="cuda"), W2, torch.zeros(1, device="cuda"), u)
    u = u.view(-1).cpu()
    assert float(u[:6].abs().max()) <= 1e-30
    assert torch.equal(u[6:12], torch.tensor(big))
    assert bool(torch.isnan(u[12:]).all())


@pytest.mark.parametrize("c", [7, 17, 25])
def test_activation_slope_over_its_whole_range(c):
    # W = 1, R = 0 and a cotangent of ones: gx is the activation's slope as the kernel for any width forms it (one to four
    # waves to a point).  Off by the tail's and the density's exponential (an exponent off by a unit in its last place and
    # one more of the result: 2 x 2^-24 of a tail up to 1/2, 4 x 2^-24 of |z| phi(z) up to 0.25) and three roundings of
    # values up to 1.13: 2^-24 (1 + 1 + 3.4) at most
    grid, modes = (16, 16, 16, 5), (2, 2, 2, 2)
    n = c * 16 ** 3 * 5
    z = torch.linspace(-16.0, 16.0, n, dtype=torch.float64).float()
    z[:8] = torch.tensor([0.0, -0.0, 1e18, -1e18, 1e-30, -1e-30, 40.0, -40.0])
    z = z.view(1, c, *grid).cuda()
    desc = B.make_desc(1, c, c, grid, modes, 0, B.FNO_ACT_GELU)
    R = torch.zeros(c, c, 4, 4, 4, 2, dtype=torch.complex64, device="cuda")
    W, gx = torch.eye(c, device="cuda"), torch.empty_like(z)
    B.fno_block_bwd(desc, torch.zeros_like(z), R, W, z, torch.zeros_like(R[:1]), torch.ones_like(z), gx, torch.empty_like(R),
                    torch.empty_like(W), torch.empty(c, device="cuda"), B.alloc_workspace(desc, B.FNO_OP_BLOCK_BWD))
    zd = z.double().cpu()
    want = 0.5 * torch.erfc(-zd / 2 ** 0.5) + zd * torch.exp(-0.5 * zd * zd) / (2 * np.pi) ** 0.5
    assert float((gx.cpu().double() - want).abs().max()) <= 5.4 * 2.0 ** -24


@pytest.mark.parametrize("mse", [False, True])
@pytest.mark.parametrize("c", [4, 20])
def test_activation_and_slope_of_units_that_are_off(c, mse):
    """W = 1, R = 0, widths and points of the matrix-core kernel: gx is the slope, with a target of zeros 2 / n times value times
    slope.  The tail T is fitted to 3.5e-8 of max(|z|, 1) T and to 1.7e-3 of T; the exponential it shares with the
    density is off by three roundings of z^2 / 2 and its own unit, and eight more roundings are counted."""
    grid, modes, eps = (16, 16, 16, 5), (2, 2, 2, 2), 2.0 ** -24
    n = c * 16 ** 3 * 5
    z = torch.linspace(-8.0 if mse else -12.5, 16.0, n, dtype=torch.float64).float()
    if not mse:
        z[:4] = torch.tensor([-40.0, -1e18, -1e-30, 1e18])
    z = z.view(1, c, *grid).cuda()
    desc = B.make_desc(1, c, c, grid, modes, 0, B.FNO_ACT_GELU, B.FNO_FLAG_MSE_TARGET if mse else 0)
    R = torch.zeros(c, c, 4, 4, 4, 2, dtype=torch.complex64, device="cuda")
    W, gx = torch.eye(c, device="cuda"), torch.empty_like(z)
    B.fno_block_bwd(desc, torch.zeros_like(z), R, W, z, torch.zeros_like(R[:1]), torch.zeros_like(z) if mse else torch.ones_like(z),
                    gx, torch.empty_like(R), torch.empty_like(W), torch.empty(c, device="cuda"),
                    B.alloc_workspace(desc, B.FNO_OP_BLOCK_BWD))
    z = z.double().cpu()
    a = z.abs()
    tail, dens = 0.5 * torch.erfc(a / 2 ** 0.5), torch.exp(-0.5 * z * z) / (2 * np.pi) ** 0.5
    cdf = torch.where(z < 0, tail, 1 - tail)
    value, slope = z * cdf, cdf + z * dens
    rounds = (1.5 * a * a).clamp(max=1e4) + 8
    on = torch.where(z < 0, 0.0, 2 * eps)
    tail_off = torch.minimum(3.6e-8 / a.clamp(min=1), 1.75e-3 * tail) + eps * rounds * tail
    slope_off = tail_off + eps * rounds * a * dens + on
    value_off = a * (tail_off + on)
    if mse:
        want = value * slope * (2.0 / n)
        bound = (2.0 / n) * (value.abs() * slope_off + slope.abs() * value_off + value_off * slope_off + 4 * eps * (value * slope).abs())
    else:
        want, bound = slope, slope_off
    worst = float(((gx.cpu().double() - want).abs() / bound.clamp(min=1e-45)).max())
    assert worst <= 1.0


def test_accumulate_flag_adds_parameter_gradients_of_successive_calls():
    """FNO_FLAG_ACCUMULATE_GRADS: gR, gW, gb of a second call are added to those of the first (the
    gradient of a broadcast weight is a sum, Sec. 2.1), gx is overwritten; compared with the sum of
    the oracle's gradients for the two cotangents."""
    L = Layer(2, 4, 4, (8, 6, 16, 8), (2, 2, 4, 4), 0)
    _, z, xh = gpu_block_fwd(L)
    g1 = synth.normal_field(3, synth.T_GOUT, L.batch, L.c_out, L.spec.grid)
    g2 = synth.normal_field(4, synth.T_GOUT, L.batch, L.c_out, L.spec.grid)
    r1 = O.block_bwd(L.x, L.R, L.W, L.b, g1, L.spec, "gelu")
    r2 = O.block_bwd(L.x, L.R, L.W, L.b, g2, L.spec, "gelu")
    ws = B.alloc_workspace(L.desc, B.FNO_OP_BLOCK_BWD)
    gx = torch.empty((L.batch, L.c_in) + L.spec.grid, device="cuda")
    gR = torch.empty((L.c_in, L.c_out) + L.counts, dtype=torch.complex64, device="cuda")
    gW = torch.empty((L.c_out, L.c_in), device="cuda")
    gb = torch.empty((L.c_out,), device="cuda")
    acc = B.make_desc(L.batch, L.c_in, L.c_out, L.spec.grid, L.spec.modes, L.spec.rule, B.FNO_ACT_GELU,
                      B.FNO_FLAG_ACCUMULATE_GRADS)
    B.fno_block_bwd(L.desc, dev(L.x), dev(L.R), dev(L.W), dev(z), dev(xh), dev(g1), gx, gR, gW, gb, ws)
    B.fno_block_bwd(acc, dev(L.x), dev(L.R), dev(L.W), dev(z), dev(xh), dev(g2), gx, gR, gW, gb, ws)
    torch.cuda.synchronize()
    assert rel(host(gx), r2["gx"]) <= TOL
    for name, got in (("gR", gR), ("gW", gW), ("gb", gb)):
        assert rel(host(got), r1[name] + r2[name]) <= TOL, name
    # the spectral convolution's own adjoint: gR accumulates, gx does not
    ws2 = B.alloc_workspace(L.desc, B.FNO_OP_SPECTRAL_CONV_BWD)
    gx1o, gR1o = O.spectral_conv_bwd(L.x, L.R, g1, L.spec)
    gx2o, gR2o = O.spectral_conv_bwd(L.x, L.R, g2, L.spec)
    B.fno_spectral_conv_bwd(L.desc, dev(L.x), None, dev(L.R), dev(g1), gx, gR, ws2)
    B.fno_spectral_conv_bwd(acc, dev(L.x), None, dev(L.R), dev(g2), gx, gR, ws2)
    torch.cuda.synchronize()
    assert rel(host(gx), gx2o) <= TOL
    assert rel(host(gR), gR1o + gR2o) <= TOL


def test_planned_tables_give_the_same_bits_as_rebuilt_ones():
    """fno_plan_tables + FNO_FLAG_TABLES_READY: the calls skip their table kernels and return the
    same bits, forward and backward, also after other calls used the workspace in between."""
    L = Layer(2, 4, 4, (8, 6, 16, 8), (2, 2, 4, 4), 0)
    out0, z0, xh0 = gpu_block_fwd(L)
    flags = B.FNO_FLAG_TABLES_READY
    ready = B.make_desc(L.batch, L.c_in, L.c_out, L.spec.grid, L.spec.modes, L.spec.rule, B.FNO_ACT_GELU, flags)
    ws = B.alloc_workspace(ready, B.FNO_OP_BLOCK_BWD)
    ws.fill_(0xFF)                                   # nothing usable in it before the plan
    B.fno_plan_tables(ready, B.FNO_OP_BLOCK_BWD, ws)
    out = torch.empty((L.batch, L.c_out) + L.spec.grid, device="cuda")
    z = torch.empty_like(out)
    xh = torch.empty((L.batch, L.c_in) + L.counts, dtype=torch.complex64, device="cuda")
    gout = synth.normal_field(3, synth.T_GOUT, L.batch, L.c_out, L.spec.grid)
    gx, gR = torch.empty_like(out), torch.empty((L.c_in, L.c_out) + L.counts, dtype=torch.complex64, device="cuda")
    gW, gb = torch.empty((L.c_out, L.c_in), device="cuda"), torch.empty((L.c_out,), device="cuda")
    ref = {}
    for name, desc in (("rebuilt", L.desc), ("planned", ready), ("planned again", ready)):
        B.fno_block_fwd(desc, dev(L.x), dev(L.R), dev(L.W), dev(L.b), out, z, xh, ws)
        B.fno_block_bwd(desc, dev(L.x), dev(L.R), dev(L.W), z, xh, dev(gout), gx, gR, gW, gb, ws)
        torch.cuda.synchronize()
        got = [t.clone() for t in (out, z, torch.view_as_real(xh), gx, torch.view_as_real(gR), gW, gb)]
        if not ref:
            ref = got
            assert np.array_equal(host(out), out0) and np.array_equal(host(z), z0)
        else:
            assert all(torch.equal(a, b) for a, b in zip(got, ref)), name


@pytest.mark.parametrize("case", [(1, 8, 8, (2, 3, 128, 32), (1, 1, 16, 9), 0),      # column kernel
                                  (1, 20, 20, (2, 3, 128, 16), (1, 1, 16, 9), 0),   # column kernel, Nt = 16
                                  (2, 3, 3, (6, 5, 12, 6), (2, 2, 3, 4), 0),        # folded products
                                  (1, 20, 20, (2, 2, 64, 30), (1, 1, 12, 8), 0),    # per-tile kernel
                                  (1, 8, 8, (16, 16, 16, 8), (4, 4, 4, 3), 0)])     # generic kernel, FFT on x and y
def test_block_forward_and_backward_replay_identically_from_a_hip_graph(case):
    """The calls only enqueue kernels on the caller's stream (no allocation, no memset, no
    synchronisation), so a caller may capture them in a HIP graph: three replays, with eager work and
    synchronisations in between, each give the bits of the eager call."""
    L = Layer(*case)
    dx, dR, dW, db = dev(L.x), dev(L.R), dev(L.W), dev(L.b)
    gout = dev(synth.normal_field(3, synth.T_GOUT, L.batch, L.c_out, L.spec.grid))
    ws = B.alloc_workspace(L.desc, B.FNO_OP_BLOCK_BWD)
    out = torch.empty((L.batch, L.c_out) + L.spec.grid, device="cuda")
    z = torch.empty_like(out)
    xh = torch.empty((L.batch, L.c_in) + L.counts, dtype=torch.complex64, device="cuda")
    gx = torch.empty_like(out)
    gR = torch.empty((L.c_in, L.c_out) + L.counts, dtype=torch.complex64, device="cuda")
    gW, gb = torch.empty((L.c_out, L.c_in), device="cuda"), torch.empty((L.c_out,), device="cuda")
    outs = (out, z, gx, gW, gb)

    def step():
        B.fno_block_fwd(L.desc, dx, dR, dW, db, out, z, xh, ws)
        B.fno_block_bwd(L.desc, dx, dR, dW, z, xh, gout, gx, gR, gW, gb, ws)

    step()
    torch.cuda.synchronize()
    eager = [t.clone() for t in outs] + [torch.view_as_real(xh).clone(), torch.view_as_real(gR).clone()]
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        step()
    for _ in range(3):
        for t in outs:
            t.fill_(float("nan"))                    # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = list(outs) + [torch.view_as_real(xh), torch.view_as_real(gR)]
        assert all(torch.equal(a, b) for a, b in zip(got, eager))


def test_spectral_branch_alone_is_not_masked_by_the_linear_term():
    """The spectral term is much smaller than W x + b; zero W and b isolate it inside the block."""
    L = Layer(1, 4, 4, (16, 16, 32, 8), (4, 4, 8, 4))
    L.W[:] = 0
    L.b[:] = 0
    L.act = B.FNO_ACT_IDENTITY
    L.desc = B.make_desc(1, 4, 4, L.spec.grid, L.spec.modes, 0, B.FNO_ACT_IDENTITY)
    out, z, _ = gpu_block_fwd(L)
    yo = O.spectral_conv_fwd(L.x, L.R, L.spec)
    assert rel(out, yo) <= TOL and np.array_equal(out, z)


def test_one_hot_frequency_is_exactly_truncated():
    """A plane wave outside the kept set gives a spectral output at rounding level only."""
    grid, modes = (16, 16, 16, 8), (4, 4, 4, 3)
    L = Layer(1, 1, 1, grid, modes)
    L.R[:] = 1.0
    n = np.meshgrid(*[np.arange(g) for g in grid], indexing="ij")
    for k4, kept in [((3, -4, 2, 2), True), ((5, 0, 0, 0), False), ((4, 0, 0, 1), False), ((-4, 0, 0, 1), True), ((0, 0, 5, 1), False), ((1, 1, 1, 3), False),
                     ((-4, -4, -4, 0), True)]:
        th = 2 * np.pi * sum(k4[a] * n[a] / grid[a] for a in range(4))
        x = np.cos(th)[None, None].astype(np.float32)
        y, _ = gpu_spectral_fwd(L, x)
        yo = O.spectral_conv_fwd(x, L.R, L.spec)
        if kept:
            assert rel(y, yo) <= TOL and np.max(np.abs(yo)) > 0.1
        else:
            assert np.max(np.abs(yo)) < 1e-7 and np.max(np.abs(y)) < 2e-6   # float32 rounding of the input leaks a little


def test_cfg2_block_forward_full_size_elementwise():
    c = synth.CONFIGS["cfg2"]
    L = Layer(c["batch"], c["width"], c["width"], c["grid"], c["modes"])
    out, z, xh = gpu_block_fwd(L)
    ys, _ = gpu_spectral_fwd(L)
    # oracle one batch entry at a time (the layer does not couple batch entries)
    for b in range(L.batch):
        oo, zo, xho = O.block_fwd(L.x[b:b + 1], L.R, L.W, L.b, L.spec)
        assert rel(out[b:b + 1], oo) <= TOL
        assert rel(xh[b:b + 1], xho) <= TOL
        yso = zo - O.channel_affine(L.x[b:b + 1], L.W, L.b)
        assert rel(ys[b:b + 1], yso) <= TOL


def test_pointwise_lift_and_projection_and_small_network():
    """Lift 5->20, four blocks, projection 20->128->1 on a reduced grid of the cfg3 structure."""
    grid, modes = (16, 16, 8, 8), (4, 4, 2, 3)
    spec = O.LayerSpec(grid, modes, 0)
    counts = tuple(len(k) for k in O.mode_lists(spec))
    npts = int(np.prod(grid))
    a = np.concatenate([synth.smooth_gaussian_field(0, grid, 3.0)[None], synth.coordinate_channels(grid)])[None]
    lw, lb = synth.linear_weights(0, 20, 5, synth.T_LIFT), synth.bias(0, 20, synth.T_LIFT)
    blocks = [(synth.spectral_weights(10 + k, 20, 20, counts), synth.linear_weights(10 + k, 20, 20),
               synth.bias(10 + k, 20)) for k in range(4)]
    w1, b1 = synth.linear_weights(1, 128, 20, synth.T_PROJ), synth.bias(1, 128, synth.T_PROJ)
    w2, b2 = synth.linear_weights(2, 1, 128, synth.T_PROJ), synth.bias(2, 1, synth.T_PROJ)
    want = O.fno_forward(a, lw, lb, blocks, (w1, b1, w2, b2), spec)

    desc = B.make_desc(1, 20, 20, grid, modes)
    ws = B.alloc_workspace(desc, B.FNO_OP_BLOCK_FWD)
    v = torch.empty((1, 20) + grid, device="cuda")
    B.fno_pointwise_linear(1, 5, 20, npts, dev(a.astype(np.float32)), dev(lw), dev(lb), v)
    torch.cuda.synchronize()
    assert rel(host(v), O.pointwise_linear(a, lw, lb)) <= TOL
    for (r, w, b) in blocks:
        nxt = torch.empty_like(v)
        B.fno_block_fwd(desc, v, dev(r), dev(w), dev(b), nxt, None, None, ws)
        v = nxt
    u = torch.empty((1, 1) + grid, device="cuda")
    B.fno_pointwise_mlp2(1, 20, 128, 1, npts, v, dev(w1), dev(b1), dev(w2), dev(b2), u)
    torch.cuda.synchronize()
    assert rel(host(u), want) <= TOL


@pytest.mark.parametrize("npts,ci,co", [(630, 5, 20), (632, 5, 20), (1024, 20, 1), (1026, 20, 1), (256, 3, 32)])
def test_pointwise_linear_point_counts_and_widths(npts, ci, co):
    """Point counts that are and are not multiples of 4 (16-byte and scalar kernels), all width classes."""
    rng = np.random.default_rng(npts + co)
    x = rng.standard_normal((2, ci, npts)).astype(np.float32)
    w = synth.linear_weights(3, co, ci, synth.T_LIFT)
    b = synth.bias(3, co, synth.T_LIFT)
    y = torch.empty((2, co, npts), device="cuda")
    B.fno_pointwise_linear(2, ci, co, npts, dev(x), dev(w), dev(b), y)
    torch.cuda.synchronize()
    want = O.pointwise_linear(x.reshape(2, ci, npts, 1, 1, 1), w, b).reshape(2, co, npts)
    assert rel(host(y), want) <= TOL


def test_block_against_the_stored_oracle_fixture():
    """The HIP path reproduces tests/golden/block_small.txt, values the float64 oracle wrote once.

    The inputs are regenerated here from the fixture's seed (float64 draws rounded to float32 for
    the GPU, which moves the results by a few 1e-8 relative to their scale); the expected values
    are read from the text file and never recomputed.
    """
    import os
    here = os.path.dirname(os.path.abspath(__file__))
    want = {}
    for line in open(os.path.join(here, "golden", "block_small.txt")):
        if line.startswith("#") or not line.strip():
            continue
        name, val = line.rstrip("\n").split("\t")
        want[name] = float(val)
    grid, modes = (6, 4, 8, 6), (2, 1, 2, 3)
    spec = O.LayerSpec(grid, modes, 0)
    rng = np.random.default_rng([2204, 1205])
    lx, ly, lz, lt = [len(k) for k in O.mode_lists(spec)]
    x = rng.standard_normal((2, 3) + grid)
    r = (rng.standard_normal((3, 3, lx, ly, lz, lt)) + 1j * rng.standard_normal((3, 3, lx, ly, lz, lt))) / 3.0
    w = rng.standard_normal((3, 3)) / np.sqrt(3.0)
    b = 0.1 * rng.standard_normal(3)
    target = rng.standard_normal(x.shape)

    desc = B.make_desc(2, 3, 3, grid, modes, 0, B.FNO_ACT_GELU, B.FNO_FLAG_MSE_TARGET)
    ws = B.alloc_workspace(desc, B.FNO_OP_BLOCK_BWD)
    dx, dr = dev(x.astype(np.float32)), dev(r.astype(np.complex64))
    dw, db, dt = dev(w.astype(np.float32)), dev(b.astype(np.float32)), dev(target.astype(np.float32))
    out = torch.empty((2, 3) + grid, device="cuda")
    z = torch.empty_like(out)
    xh = torch.empty((2, 3, lx, ly, lz, lt), dtype=torch.complex64, device="cuda")
    B.fno_block_fwd(desc, dx, dr, dw, db, out, z, xh, ws)
    gx = torch.empty_like(out)
    gR = torch.empty_like(dr)
    gW = torch.empty_like(dw)
    gb = torch.empty_like(db)
    B.fno_block_bwd(desc, dx, dr, dw, z, xh, dt, gx, gR, gW, gb, ws)
    torch.cuda.synchronize()
    out, z, xh, gx, gR, gW, gb = [host(t) for t in (out, z, xh, gx, gR, gW, gb)]

    # each value against the scale of the tensor it belongs to (single entries can be near zero)
    def close(got, name, scale):
        assert abs(float(got) - want[name]) <= TOL * scale, (name, float(got), want[name])

    for p in [(0, 0, 0, 0, 0, 0), (1, 2, 5, 3, 7, 5), (0, 1, 2, 1, 3, 4), (1, 0, 4, 2, 6, 1)]:
        close(out[p], "out" + str(p), np.abs(out).max())
        close(z[p], "z" + str(p), np.abs(z).max())
        close(gx[p], "gx" + str(p), np.abs(gx).max())
    close(xh[1, 2, 3, 1, 2, 1].real, "xhat_re", np.abs(xh).max())
    close(xh[1, 2, 3, 1, 2, 1].imag, "xhat_im", np.abs(xh).max())
    close(gR[2, 1, 1, 0, 3, 2].real, "gR_re", np.abs(gR).max())
    close(gR[2, 1, 1, 0, 3, 2].imag, "gR_im", np.abs(gR).max())
    close(gR[0, 2, 3, 1, 1, 0].real, "gR_kt0_re", np.abs(gR).max())
    for o in range(3):
        close(gb[o], f"gb[{o}]", np.abs(gb).max())
        for i in range(3):
            close(gW[o, i], f"gW[{o}][{i}]", np.abs(gW).max())


@pytest.mark.parametrize("shape", [
    # batch, c_in, c_out, spatial grid, nt
    (2, 2, 20, (6, 5, 4), 30),        # the paper's two input channels, nt not a multiple of 4
    (1, 3, 8, (4, 4, 8), 16),         # whole float4 rows
    (1, 1, 24, (3, 2, 5), 7),         # odd nt, one input channel, width above 20
    (1, 2, 20, (60, 60, 64), 30),     # a training sample of the paper (Sec. 4), full size
])
def test_time_lift_matches_oracle(shape):
    batch, c_in, c_out, grid, nt = shape
    rng = np.random.default_rng([7, batch, c_in, c_out, nt])
    a = rng.standard_normal((batch, c_in) + grid + (1,)).astype(np.float32)
    wt = rng.standard_normal(nt).astype(np.float32)
    bt = rng.standard_normal(nt).astype(np.float32)
    wc = (rng.standard_normal((c_out, c_in)) / np.sqrt(c_in)).astype(np.float32)
    bc = (0.1 * rng.standard_normal(c_out)).astype(np.float32)
    nspace = int(np.prod(grid))
    out = torch.empty((batch, c_out) + grid + (nt,), device="cuda")
    B.fno_time_lift(batch, c_in, c_out, nspace, nt, dev(a), dev(wt), dev(bt), dev(wc), dev(bc), out)
    torch.cuda.synchronize()
    assert rel(host(out), O.time_lift(a, wt, bt, wc, bc)) <= TOL
    # without the biases
    B.fno_time_lift(batch, c_in, c_out, nspace, nt, dev(a), dev(wt), None, dev(wc), None, out)
    torch.cuda.synchronize()
    assert rel(host(out), O.time_lift(a, wt, np.zeros(nt), wc, np.zeros(c_out))) <= TOL


@pytest.mark.parametrize("shape", [
    # batch, c_in, c_out, spatial grid, nt
    (2, 2, 20, (6, 5, 4), 30),        # the paper's two input channels, one chunk per batch entry
    (1, 3, 8, (4, 4, 8), 16),         # three input channels on the four-channel register tile
    (3, 1, 24, (3, 2, 5), 7),         # odd nt, one input channel, pairs that do not fill the last block
    (1, 5, 4, (7, 9, 11), 4),         # five input channels, a ragged tail of positions
    (1, 2, 20, (60, 60, 64), 30),     # a training sample of the paper (Sec. 4), full size: 450 chunks
])
def test_time_lift_adjoint_matches_oracle(shape):
    batch, c_in, c_out, grid, nt = shape
    rng = np.random.default_rng([23, batch, c_in, c_out, nt])
    a = rng.standard_normal((batch, c_in) + grid + (1,)).astype(np.float32)
    wt = rng.standard_normal(nt).astype(np.float32)
    bt = rng.standard_normal(nt).astype(np.float32)
    wc = (rng.standard_normal((c_out, c_in)) / np.sqrt(c_in)).astype(np.float32)
    g = rng.standard_normal((batch, c_out) + grid + (nt,)).astype(np.float32)
    nspace = int(np.prod(grid))
    ws = torch.empty(B.fno_time_lift_bwd_workspace_bytes(c_in, c_out, nt) // 4 + 2, dtype=torch.float32,
                     device="cuda")
    gwt, gbt = torch.empty(nt, device="cuda"), torch.empty(nt, device="cuda")
    gwc, gbc = torch.empty((c_out, c_in), device="cuda"), torch.empty(c_out, device="cuda")
    B.fno_time_lift_bwd(batch, c_in, c_out, nspace, nt, dev(a), dev(wt), dev(bt), dev(wc), dev(g),
                        gwt, gbt, gwc, gbc, ws)
    torch.cuda.synchronize()
    want = O.time_lift_bwd(a, wt, bt, wc, g)
    for name, got in (("gWt", gwt), ("gbt", gbt), ("gWc", gwc), ("gbc", gbc)):
        assert rel(host(got), want[name]) <= TOL, name
    # same bits on a second run; without the time bias; a subset of the outputs
    gwt2, gwc2 = torch.empty_like(gwt), torch.empty_like(gwc)
    B.fno_time_lift_bwd(batch, c_in, c_out, nspace, nt, dev(a), dev(wt), dev(bt), dev(wc), dev(g),
                        gwt2, None, gwc2, None, ws)
    torch.cuda.synchronize()
    assert torch.equal(gwt, gwt2) and torch.equal(gwc, gwc2)
    B.fno_time_lift_bwd(batch, c_in, c_out, nspace, nt, dev(a), dev(wt), None, dev(wc), dev(g),
                        None, None, gwc2, None, ws)
    torch.cuda.synchronize()
    assert rel(host(gwc2), O.time_lift_bwd(a, wt, np.zeros(nt), wc, g)["gWc"]) <= TOL


@pytest.mark.parametrize("n", [7, 100003, 60 * 60 * 64 * 30])
def test_relative_l2_loss_and_gradient_match_oracle(n):
    rng = np.random.default_rng([11, n])
    target = rng.standard_normal(n).astype(np.float32)
    pred = (target + 0.3 * rng.standard_normal(n)).astype(np.float32)
    ws = torch.empty(B.fno_rel_l2_workspace_bytes() // 4, dtype=torch.float32, device="cuda")
    loss = torch.empty(1, device="cuda")
    grad = torch.empty(n, device="cuda")
    B.fno_rel_l2_loss(n, dev(pred), dev(target), loss, grad, ws)
    torch.cuda.synchronize()
    want = O.rel_l2_loss(pred, target)
    assert abs(float(loss.cpu()) - want) <= TOL * want
    assert rel(host(grad), O.rel_l2_grad(pred, target)) <= TOL
    # same bits on a second run; loss alone; a perfect prediction has loss 0 and a zero gradient
    loss2 = torch.empty(1, device="cuda")
    B.fno_rel_l2_loss(n, dev(pred), dev(target), loss2, None, ws)
    B.fno_rel_l2_loss(n, dev(target), dev(target), loss, grad, ws)
    torch.cuda.synchronize()
    assert abs(float(loss2.cpu()) - want) <= TOL * want
    assert float(loss.cpu()) == 0.0 and not bool(grad.any())


def test_adam_steps_match_oracle_for_real_and_complex_parameters():
    rng = np.random.default_rng(13)
    w = rng.standard_normal((20, 20)).astype(np.float32)
    r = (rng.standard_normal((3, 3, 4, 4, 4, 3)) + 1j * rng.standard_normal((3, 3, 4, 4, 4, 3))).astype(np.complex64)
    for p0 in (w, r):
        as_real = p0.view(np.float32).ravel() if np.iscomplexobj(p0) else p0.ravel()
        n = as_real.size
        p = dev(as_real.copy())
        m = torch.zeros(n, device="cuda")
        v = torch.zeros(n, device="cuda")
        po, mo, vo = as_real.astype(np.float64), np.zeros(n), np.zeros(n)
        for step in (1, 2, 3):
            g = (rng.standard_normal(n) * (10.0 ** rng.integers(-3, 2))).astype(np.float32)
            B.fno_adam_step(n, p, dev(g), m, v, 1e-3, 0.9, 0.999, 1e-8, step)
            before = po
            po, mo, vo = O.adam_step(po, g, mo, vo, step)
            torch.cuda.synchronize()
            assert rel(host(m), mo) <= TOL and rel(host(v), vo) <= TOL
            assert rel(host(p), po) <= TOL
            # the update itself, not only the updated parameter
            assert rel(host(p).astype(np.float64) - before, po - before) <= 1e-3


@pytest.mark.parametrize("shape", [
    # batch, c_in, hidden, c_out, points
    (2, 3, 5, 2, 77),                 # ragged tile, hidden below one chunk
    (1, 20, 128, 1, 3000),            # the projection of the benchmark network, several tiles
    (2, 5, 20, 4, 1024),              # whole tiles, four outputs
    (2, 5, 32, 1, 200),               # one 32-row block of hidden units on the matrix cores, ragged tile
    (2, 9, 64, 3, 1000),              # two blocks, three outputs, two batch elements
    (1, 24, 192, 4, 333),             # more than 21 input channels, six blocks
    (1, 20, 128, 1, 64 * 512 * 17 + 7),  # 17 and more tiles a block
])
def test_pointwise_adjoints_match_oracle(shape):
    batch, c_in, hidden, c_out, npts = shape
    rng = np.random.default_rng([19, c_in, hidden, c_out, npts])
    grid = (npts, 1, 1, 1)
    x = rng.standard_normal((batch, c_in) + grid).astype(np.float32)
    w1 = (rng.standard_normal((hidden, c_in)) / np.sqrt(c_in)).astype(np.float32)
    b1 = (0.1 * rng.standard_normal(hidden)).astype(np.float32)
    w2 = (rng.standard_normal((c_out, hidden)) / np.sqrt(hidden)).astype(np.float32)
    gu = rng.standard_normal((batch, c_out) + grid).astype(np.float32)
    nbytes = max(B.fno_pointwise_bwd_workspace_bytes(c_in, hidden, c_out),
                 B.fno_pointwise_bwd_workspace_bytes(c_in, 0, min(hidden, 32)))
    ws = torch.empty(nbytes // 4 + 2, dtype=torch.float32, device="cuda")
    # the linear map (lift): hidden plays the output width
    gh_in = rng.standard_normal((batch, hidden) + grid).astype(np.float32)
    gx = torch.empty((batch, c_in) + grid, device="cuda")
    gW = torch.empty((hidden, c_in), device="cuda")
    gb = torch.empty(hidden, device="cuda")
    if hidden <= 32:
        B.fno_pointwise_linear_bwd(batch, c_in, hidden, npts, dev(x), dev(w1), dev(gh_in), gx, gW, gb, ws)
        torch.cuda.synchronize()
        want = O.pointwise_linear_bwd(x, w1, gh_in)
        assert rel(host(gx), want["gx"]) <= TOL and rel(host(gW), want["gW"]) <= TOL
        assert rel(host(gb), want["gb"]) <= TOL
    # the two-layer projection: forward, then its adjoint
    b2 = (0.1 * rng.standard_normal(c_out)).astype(np.float32)
    u = torch.empty((batch, c_out) + grid, device="cuda")
    B.fno_pointwise_mlp2(batch, c_in, hidden, c_out, npts, dev(x), dev(w1), dev(b1), dev(w2), dev(b2), u)
    torch.cuda.synchronize()
    assert rel(host(u), O.pointwise_mlp2(x, w1, b1, w2, b2)) <= TOL
    B.fno_pointwise_mlp2(batch, c_in, hidden, c_out, npts, dev(x), dev(w1), None, dev(w2), None, u)
    torch.cuda.synchronize()
    assert rel(host(u), O.pointwise_mlp2(x, w1, np.zeros(hidden), w2, np.zeros(c_out))) <= TOL
    gW1 = torch.empty((hidden, c_in), device="cuda")
    gb1 = torch.empty(hidden, device="cuda")
    gW2 = torch.empty((c_out, hidden), device="cuda")
    gb2 = torch.empty(c_out, device="cuda")
    B.fno_pointwise_mlp2_bwd(batch, c_in, hidden, c_out, npts, dev(x), dev(w1), dev(b1), dev(w2), dev(gu),
                             gx, gW1, gb1, gW2, gb2, ws)
    torch.cuda.synchronize()
    want = O.pointwise_mlp2_bwd(x, w1, b1, w2, gu)
    for name, got in (("gx", gx), ("gW1", gW1), ("gb1", gb1), ("gW2", gW2), ("gb2", gb2)):
        assert rel(host(got), want[name]) <= TOL, name
    # identical bits on a second run
    gW1b, gW2b = torch.empty_like(gW1), torch.empty_like(gW2)
    B.fno_pointwise_mlp2_bwd(batch, c_in, hidden, c_out, npts, dev(x), dev(w1), dev(b1), dev(w2), dev(gu),
                             None, gW1b, None, gW2b, None, ws)
    torch.cuda.synchronize()
    assert torch.equal(gW1, gW1b) and torch.equal(gW2, gW2b)
    # without the hidden bias
    B.fno_pointwise_mlp2_bwd(batch, c_in, hidden, c_out, npts, dev(x), dev(w1), None, dev(w2), dev(gu),
                             gx, gW1b, gb1, gW2b, gb2, ws)
    torch.cuda.synchronize()
    want0 = O.pointwise_mlp2_bwd(x, w1, np.zeros(hidden), w2, gu)
    for name, got in (("gx", gx), ("gW1", gW1b), ("gb1", gb1), ("gW2", gW2b), ("gb2", gb2)):
        assert rel(host(got), want0[name]) <= TOL, name


def _projection(batch, ci, h, co, npts, seed, sx=1.0, sg=1.0, sw2=1.0):
    """Inputs of a projection, its float32 results and the float64 ones (torch, on the device)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    normal = lambda *shape: torch.randn(shape, device="cuda", generator=gen)
    x, g = normal(batch, ci, npts) * sx, normal(batch, co, npts) * sg
    W1, b1, W2, b2 = normal(h, ci) * ci ** -0.5 / (sx.T if torch.is_tensor(sx) else sx), normal(h) * 0.1, \
        normal(co, h) * h ** -0.5 * sw2, normal(co) * 0.1
    u, gx = torch.empty(batch, co, npts, device="cuda"), torch.empty_like(x)
    grads = [torch.empty_like(p) for p in (W1, b1, W2, b2)]
    ws = torch.empty(B.fno_pointwise_bwd_workspace_bytes(ci, h, co) // 4 + 2, device="cuda")
    B.fno_pointwise_mlp2(batch, ci, h, co, npts, x, W1, b1, W2, b2, u)
    B.fno_pointwise_mlp2_bwd(batch, ci, h, co, npts, x, W1, b1, W2, g, gx, *grads, ws)
    torch.cuda.synchronize()
    xd = x.double().transpose(0, 1).reshape(ci, -1)
    gd = g.double().transpose(0, 1).reshape(co, -1)
    z = W1.double() @ xd + b1.double()[:, None]
    cdf = 0.5 * torch.erfc(-z / 2 ** 0.5)
    gh = (W2.double().T @ gd) * (cdf + z * torch.exp(-0.5 * z * z) / (2 * np.pi) ** 0.5)
    wide = lambda a: a.reshape(a.shape[0], batch, npts).transpose(0, 1)
    want = dict(u=wide(W2.double() @ (z * cdf) + b2.double()[:, None]), gx=wide(W1.double().T.contiguous() @ gh),
                gW1=gh @ xd.T.contiguous(), gb1=gh.sum(1), gW2=gd @ (z * cdf).T.contiguous(), gb2=gd.sum(1))
    # what the errors go with: the values themselves, and the root sum square of the terms of a sum over points
    act, sq = z * cdf, lambda a, b: float((a ** 2 @ (b ** 2).T.contiguous()).sum().sqrt())
    scale = dict(u=float(want["u"].norm()), gx=float(want["gx"].norm()), gW1=sq(gh, xd), gb1=float(gh.norm()),
                 gW2=sq(gd, act), gb2=float(gd.norm()))
    return dict(u=u, gx=gx, gW1=grads[0], gb1=grads[1], gW2=grads[2], gb2=grads[3]), want, scale


# every tile of channels (1 .. 7, .. 15, .. 23, .. 31, 32) at its ends, hidden widths on and off the groups of 32 with one
# and two waves each, ragged and single points, several batch entries and channels
@pytest.mark.parametrize("batch, ci, h, co, npts", [
    (1, 1, 32, 1, 33), (2, 7, 40, 1, 65), (1, 8, 64, 1, 64), (3, 15, 96, 1, 127), (1, 16, 128, 1, 2000), (1, 23, 100, 4, 31),
    (1, 24, 160, 1, 1), (2, 31, 256, 1, 200), (1, 32, 32, 1, 63), (1, 32, 250, 1, 1000), (1, 20, 1, 1, 129), (1, 5, 300, 2, 70),
    # the most channels that four and three waves stage in their rounds
    (1, 7, 128, 1, 65), (1, 15, 128, 1, 66), (2, 23, 128, 1, 200), (1, 31, 128, 1, 130), (1, 23, 96, 1, 129)])
def test_projection_on_split_products(batch, ci, h, co, npts):
    got, want, scale = _projection(batch, ci, h, co, npts, 7)
    for name, ref in want.items():
        # a hidden value and its slope are within about 2 units of 2^-23 (products of 24 bits, the fits of GELU); the sum over
        # the hidden units may cancel to a quarter of its terms' size
        assert float((got[name].double() - ref).norm()) <= 8 * 2.0 ** -23 * scale[name], name


def test_projection_adjoint_with_channels_and_points_of_very_different_size():
    # channels of x from 1e-9 to 1e2 (and weights to match), hidden units weighted 1e-4 to 1e4, cotangents that grow by 1e12
    # along the points.  Every channel by itself, as above
    sx = torch.logspace(-9, 2, 20, device="cuda")[:, None]
    got, want, _ = _projection(1, 20, 128, 1, 100000, 8, sx=sx, sg=torch.logspace(-20, -8, 100000, device="cuda"),
                               sw2=torch.logspace(-4, 4, 128, device="cuda"))
    for name, dim in (("gx", 2), ("gW1", 0)):
        err = (got[name].double() - want[name]).norm(dim=dim) / want[name].norm(dim=dim)
        assert float(err.max()) <= 8 * 2.0 ** -23, name
    first = slice(0, 5000)                              # the small cotangents alone
    err = (got["gx"].double() - want["gx"])[..., first].norm(dim=2) / want["gx"][..., first].norm(dim=2)
    assert float(err.max()) <= 8 * 2.0 ** -23


@pytest.mark.parametrize("batch, ci, h", [
    (1, 20, 128), (1, 7, 128), (1, 31, 128),               # four waves, two column blocks each
    (1, 20, 96), (1, 23, 96),                              # three waves
    (1, 32, 128), (1, 32, 96), (1, 20, 64), (2, 15, 32),   # two waves a group of hidden units
    (1, 32, 256), (2, 24, 160),                            # eight and five waves
])
def test_projection_adjoint_tile_by_tile(batch, ci, h):
    """512 blocks of several tiles of 64 points each, past a flush of the sums (32 tiles) with two waves a group: the
    cotangents of a block's tiles differ by 2^20 from one to the next, and every tile's gx is held against its own size."""
    npts = 64 * 512 * (35 if h <= 64 else 5) // batch + 7
    tiles = (npts + 63) // 64
    turn = (torch.arange(batch, device="cuda")[:, None] * tiles + torch.arange(npts, device="cuda") // 64) // 512
    got, want, _ = _projection(batch, ci, h, 1, npts, 9, sg=torch.where(turn % 2 == 0, 1.0, 2.0 ** -20)[:, None])
    pad = lambda t: torch.nn.functional.pad(t, (0, tiles * 64 - npts)).reshape(batch, ci, tiles, 64).norm(dim=(1, 3))
    err = pad(got["gx"].double() - want["gx"]) / pad(want["gx"])
    # as for the whole field above: the smallest tile has 7 points of at least 7 channels
    assert float(err.max()) <= 8 * 2.0 ** -23


@pytest.mark.parametrize("ci, h", [(20, 128), (32, 128), (9, 64)])
@pytest.mark.parametrize("kind", ["off by 3", "off by 5", "off by 7", "a heavy unit without weights", "light units", "a plume"])
def test_projection_adjoint_value_by_value(kind, ci, h):
    """Units that are all but off, a large W2 beside weights W1 of zero, units 2^-25 as heavy as one that is off at the point, and
    units that are off where the values are large and on where these are 2^-20 as large.  Every value by itself, against
    the sum of the sizes of its terms: a term is off by its slope's fit and roundings (as for a block's), by what the
    rounding of the hidden value makes of it, and by eight roundings of products and sums; forty in the sums over points."""
    npts, eps = 3001, 2.0 ** -24
    gen = torch.Generator(device="cuda")
    gen.manual_seed(ci)
    normal = lambda *shape: torch.randn(shape, device="cuda", generator=gen)
    x, g = normal(1, ci, npts), normal(1, 1, npts) * 1e-3
    W1, b1, W2 = normal(h, ci) * ci ** -0.5, normal(h) * 0.1, normal(1, h) * h ** -0.5
    if kind.startswith("off"):
        W1 *= 0.2
        b1 -= float(kind[-1])
    elif kind == "a heavy unit without weights":
        W2[0, 3], W1[3] = 1e5, 0.0
    elif kind == "light units":
        W2[0, 1:] *= 2.0 ** -25
        W1[0] = 0.0
        W1[0, 0] = 8.0
        x[:, 0] = torch.where(x[:, 0] < 0, -1.0, 1.0)
    else:
        W1[:, 0] = 8.0
        x[:, 0], x[:, 1:, npts // 16:] = 1.0, x[:, 1:, npts // 16:] * 2.0 ** -20
        x[:, 0, :npts // 16] = -1.0
    gx, grads = torch.empty_like(x), [torch.empty_like(p) for p in (W1, b1, W2)]
    ws = torch.empty(B.fno_pointwise_bwd_workspace_bytes(ci, h, 1) // 4 + 2, device="cuda")
    B.fno_pointwise_mlp2_bwd(1, ci, h, 1, npts, x, W1, b1, W2, g, gx, *grads, torch.empty(1, device="cuda"), ws)
    torch.cuda.synchronize()
    x, g, W1, b1, W2 = x[0].double(), g[0].double(), W1.double(), b1.double(), W2.double()
    z, z_off = W1 @ x + b1[:, None], 6 * eps * (W1.abs() @ x.abs() + b1.abs()[:, None])
    a, dens = z.abs(), torch.exp(-0.5 * z * z) / (2 * np.pi) ** 0.5
    tail = 0.5 * torch.erfc(a / 2 ** 0.5)
    slope = torch.where(z < 0, tail, 1 - tail) + z * dens
    off = torch.minimum(3.6e-8 / a.clamp(min=1), 1.75e-3 * tail) + eps * (1.5 * a * a + 8) * (tail + a * dens) + \
        (2 - z * z).abs() * dens * z_off * 1.1 + torch.where(z < 0, 0.0, 2 * eps)
    M, Y = W1 * W2.T, torch.cat([x, torch.ones_like(x[:1])]) * g
    pairs = [(gx[0], M.T.contiguous() @ slope * g, (M.abs().T.contiguous() @ (off + 8 * eps * slope.abs())) * g.abs())]
    sums, bound = slope @ Y.T.contiguous() * W2.T, (off + 40 * eps * slope.abs()) @ Y.abs().T.contiguous() * W2.abs().T
    pairs += [(grads[0], sums[:, :ci], bound[:, :ci]), (grads[1], sums[:, ci], bound[:, ci])]
    for got, want, most in pairs:
        worst = float(((got.double() - want).abs() / most.clamp(min=1e-40)).max())
        assert worst <= 1.0


@pytest.mark.parametrize("ci, h", [(20, 128), (32, 128), (32, 160), (20, 64), (7, 32)])
def test_projection_adjoint_over_many_points(ci, h):
    # 66 and more tiles a block: two flushes of the weight gradients and a rest, on one and two waves to a group of units
    got, want, scale = _projection(1, ci, h, 1, 64 * 512 * 66 + 7, 11)
    for name in ("gx", "gW1", "gb1", "gW2", "gb2"):
        assert float((got[name].double() - want[name]).norm()) <= 8 * 2.0 ** -23 * scale[name], name


@pytest.mark.parametrize("ci, h", [(1, 128), (32, 128), (32, 160), (3, 32)])
def test_projection_adjoint_adds_up_equal_points(ci, h):
    # 2^25 equal points, 1024 tiles a block: every lane adds one number again and again, whose roundings do not scatter.  Sums in
    # fp32 of at most 32 tiles, 64 terms, are off by at most 32 x 2^-24; the term itself by eight roundings and a tile's products
    # by eight more
    npts, gen = 1 << 25, torch.Generator(device="cuda")
    gen.manual_seed(h)
    x1, W1 = [0.1 * torch.randn(s, device="cuda", generator=gen) for s in (ci, (h, ci))]
    W2, b1, c = torch.ones(1, h, device="cuda"), torch.linspace(0.5, 4.0, h, device="cuda") - W1 @ x1, 0.3
    x = x1[None, :, None].expand(1, ci, npts).contiguous()
    g = torch.full((1, 1, npts), c, device="cuda")
    grads = [torch.empty_like(p) for p in (W1, b1, W2)]
    ws = torch.empty(B.fno_pointwise_bwd_workspace_bytes(ci, h, 1) // 4 + 2, device="cuda")
    B.fno_pointwise_mlp2_bwd(1, ci, h, 1, npts, x, W1, b1, W2, g, None, *grads, torch.empty(1, device="cuda"), ws)
    torch.cuda.synchronize()
    z = W1.double() @ x1.double() + b1.double()
    cdf, dens = 0.5 * torch.erfc(-z / 2 ** 0.5), torch.exp(-0.5 * z * z) / (2 * np.pi) ** 0.5
    total = float(g[0, 0, 0].double()) * npts
    for got, want in ((grads[2][0], total * z * cdf), (grads[1], total * (cdf + z * dens))):
        worst = float(((got.double() - want) / want).abs().max())
        assert worst <= (32 + 16) * 2.0 ** -24


def test_whole_network_training_step_matches_oracle():
    """Lift, two blocks, projection; relative L2 loss; backward through all of it; one Adam step.

    Every stage runs through the C ABI; the float64 oracle differentiates its own forward."""
    grid, modes, c_in, width, hidden, nblocks = (8, 8, 8, 8), (2, 2, 2, 3), 3, 8, 16, 2
    spec = O.LayerSpec(grid, modes, 0)
    counts = tuple(len(k) for k in O.mode_lists(spec))
    npts = int(np.prod(grid))
    a = synth.normal_field(0, synth.T_X, 1, c_in, grid)
    y = synth.normal_field(1, synth.T_TARGET, 1, 1, grid)
    lw, lb = synth.linear_weights(0, width, c_in, synth.T_LIFT), synth.bias(0, width, synth.T_LIFT)
    blocks = [(synth.spectral_weights(k, width, width, counts), synth.linear_weights(10 + k, width, width),
               synth.bias(10 + k, width)) for k in range(nblocks)]
    w1, b1 = synth.linear_weights(1, hidden, width, synth.T_PROJ), synth.bias(1, hidden, synth.T_PROJ)
    w2, b2 = synth.linear_weights(2, 1, hidden, synth.T_PROJ), synth.bias(2, 1, synth.T_PROJ)

    # ---- GPU: forward
    desc = B.make_desc(1, width, width, grid, modes, 0, B.FNO_ACT_GELU)
    ws = B.alloc_workspace(desc, B.FNO_OP_BLOCK_BWD)
    d = {k: dev(v) for k, v in dict(a=a, y=y, lw=lw, lb=lb, w1=w1, b1=b1, w2=w2, b2=b2).items()}
    dblocks = [tuple(dev(t) for t in blk) for blk in blocks]
    vs = [torch.empty((1, width) + grid, device="cuda")]
    B.fno_pointwise_linear(1, c_in, width, npts, d["a"], d["lw"], d["lb"], vs[0])
    zs, xhs = [], []
    for (R, W, b) in dblocks:
        out = torch.empty_like(vs[0])
        z = torch.empty_like(vs[0])
        xh = torch.empty((1, width) + counts, dtype=torch.complex64, device="cuda")
        B.fno_block_fwd(desc, vs[-1], R, W, b, out, z, xh, ws)
        vs.append(out); zs.append(z); xhs.append(xh)
    u = torch.empty((1, 1) + grid, device="cuda")
    B.fno_pointwise_mlp2(1, width, hidden, 1, npts, vs[-1], d["w1"], d["b1"], d["w2"], d["b2"], u)
    # ---- loss and its gradient
    lws = torch.empty(B.fno_rel_l2_workspace_bytes() // 4, dtype=torch.float32, device="cuda")
    loss = torch.empty(1, device="cuda")
    gu = torch.empty_like(u)
    B.fno_rel_l2_loss(npts, u, d["y"], loss, gu, lws)
    # ---- backward
    pws = torch.empty(max(B.fno_pointwise_bwd_workspace_bytes(width, hidden, 1),
                          B.fno_pointwise_bwd_workspace_bytes(c_in, 0, width)) // 4 + 2,
                      dtype=torch.float32, device="cuda")
    gv = torch.empty_like(vs[0])
    g = {"w1": torch.empty_like(d["w1"]), "b1": torch.empty_like(d["b1"]), "w2": torch.empty_like(d["w2"]),
         "b2": torch.empty_like(d["b2"]), "lw": torch.empty_like(d["lw"]), "lb": torch.empty_like(d["lb"])}
    B.fno_pointwise_mlp2_bwd(1, width, hidden, 1, npts, vs[-1], d["w1"], d["b1"], d["w2"], gu, gv,
                             g["w1"], g["b1"], g["w2"], g["b2"], pws)
    gblocks = [None] * nblocks
    for k in reversed(range(nblocks)):
        R, W, b = dblocks[k]
        gx = torch.empty_like(vs[0])
        gR, gW, gb = torch.empty_like(R), torch.empty_like(W), torch.empty_like(b)
        B.fno_block_bwd(desc, vs[k], R, W, zs[k], xhs[k], gv, gx, gR, gW, gb, ws)
        gblocks[k] = (gR, gW, gb)
        gv = gx
    B.fno_pointwise_linear_bwd(1, c_in, width, npts, d["a"], d["lw"], gv, None, g["lw"], g["lb"], pws)
    torch.cuda.synchronize()

    # ---- oracle
    uo = O.fno_forward(a, lw, lb, blocks, (w1, b1, w2, b2), spec)
    assert rel(host(u), uo) <= TOL
    assert abs(float(loss.cpu()) - O.rel_l2_loss(uo, y)) <= TOL * O.rel_l2_loss(uo, y)
    ref = O.fno_backward(a, lw, lb, blocks, (w1, b1, w2, b2), spec, O.rel_l2_grad(uo, y))
    GT = 5 * TOL     # gradients pass through 2 blocks and 3 pointwise stages
    assert rel(host(g["w1"]), ref["proj"]["gW1"]) <= GT and rel(host(g["b1"]), ref["proj"]["gb1"]) <= GT
    assert rel(host(g["w2"]), ref["proj"]["gW2"]) <= GT and rel(host(g["b2"]), ref["proj"]["gb2"]) <= GT
    for k in range(nblocks):
        gR, gW, gb = gblocks[k]
        assert rel(host(gR), ref["blocks"][k]["gR"]) <= GT, k
        assert rel(host(gW), ref["blocks"][k]["gW"]) <= GT, k
        assert rel(host(gb), ref["blocks"][k]["gb"]) <= GT, k
    assert rel(host(g["lw"]), ref["lift"]["gW"]) <= GT and rel(host(g["lb"]), ref["lift"]["gb"]) <= GT

    # ---- one Adam step on every parameter (complex weights as pairs of floats)
    params = [(d["lw"], g["lw"], lw, ref["lift"]["gW"]), (d["w1"], g["w1"], w1, ref["proj"]["gW1"])]
    R0 = dblocks[0][0]
    params.append((torch.view_as_real(R0).reshape(-1), torch.view_as_real(gblocks[0][0]).reshape(-1),
                   np.ascontiguousarray(blocks[0][0]).view(np.float32).ravel(),
                   np.ascontiguousarray(ref["blocks"][0]["gR"].astype(np.complex128)).view(np.float64).ravel()))
    for p, grad, p_host, g_ref in params:
        n = p.numel()
        m = torch.zeros(n, device="cuda")
        v = torch.zeros(n, device="cuda")
        B.fno_adam_step(n, p, grad, m, v, 1e-3, 0.9, 0.999, 1e-8, 1)
        torch.cuda.synchronize()
        po, _, _ = O.adam_step(p_host.astype(np.float64).ravel(), np.asarray(g_ref).ravel(), np.zeros(n), np.zeros(n), 1)
        assert rel(host(p).ravel(), po) <= TOL


def test_network_with_time_lift_training_gradients_match_oracle():
    """The paper's input stage (eqs. (8)-(9)) in front of the network: time + channel lift of an
    input without a time axis, one block, projection, relative L2 loss, and the gradients of all
    four lift parameters through the whole chain."""
    sgrid, nt, modes, c_in, width, hidden = (6, 4, 8), 8, (2, 2, 2, 3), 2, 8, 32
    grid = sgrid + (nt,)
    spec = O.LayerSpec(grid, modes, 0)
    counts = tuple(len(k) for k in O.mode_lists(spec))
    nspace, npts = int(np.prod(sgrid)), int(np.prod(grid))
    rng = np.random.default_rng(41)
    a = rng.standard_normal((1, c_in) + sgrid + (1,)).astype(np.float32)
    wt, bt = rng.standard_normal(nt).astype(np.float32), (0.3 * rng.standard_normal(nt)).astype(np.float32)
    wc = (rng.standard_normal((width, c_in)) / np.sqrt(c_in)).astype(np.float32)
    bc = (0.1 * rng.standard_normal(width)).astype(np.float32)
    y = synth.normal_field(1, synth.T_TARGET, 1, 1, grid)
    R, W, b = (synth.spectral_weights(3, width, width, counts), synth.linear_weights(13, width, width),
               synth.bias(13, width))
    w1, b1 = synth.linear_weights(1, hidden, width, synth.T_PROJ), synth.bias(1, hidden, synth.T_PROJ)
    w2, b2 = synth.linear_weights(2, 1, hidden, synth.T_PROJ), synth.bias(2, 1, synth.T_PROJ)

    desc = B.make_desc(1, width, width, grid, modes, 0, B.FNO_ACT_GELU)
    ws = B.alloc_workspace(desc, B.FNO_OP_BLOCK_BWD)
    d = {k: dev(v) for k, v in dict(a=a, wt=wt, bt=bt, wc=wc, bc=bc, y=y, R=R, W=W, b=b, w1=w1, b1=b1, w2=w2,
                                    b2=b2).items()}
    v0 = torch.empty((1, width) + grid, device="cuda")
    B.fno_time_lift(1, c_in, width, nspace, nt, d["a"], d["wt"], d["bt"], d["wc"], d["bc"], v0)
    v1, z = torch.empty_like(v0), torch.empty_like(v0)
    xh = torch.empty((1, width) + counts, dtype=torch.complex64, device="cuda")
    B.fno_block_fwd(desc, v0, d["R"], d["W"], d["b"], v1, z, xh, ws)
    u = torch.empty((1, 1) + grid, device="cuda")
    B.fno_pointwise_mlp2(1, width, hidden, 1, npts, v1, d["w1"], d["b1"], d["w2"], d["b2"], u)
    lws = torch.empty(B.fno_rel_l2_workspace_bytes() // 4, dtype=torch.float32, device="cuda")
    loss, gu = torch.empty(1, device="cuda"), torch.empty_like(u)
    B.fno_rel_l2_loss(npts, u, d["y"], loss, gu, lws)
    pws = torch.empty(B.fno_pointwise_bwd_workspace_bytes(width, hidden, 1) // 4 + 2, dtype=torch.float32,
                      device="cuda")
    gv1, gv0 = torch.empty_like(v0), torch.empty_like(v0)
    B.fno_pointwise_mlp2_bwd(1, width, hidden, 1, npts, v1, d["w1"], d["b1"], d["w2"], gu, gv1,
                             None, None, None, None, pws)
    B.fno_block_bwd(desc, v0, d["R"], d["W"], z, xh, gv1, gv0, torch.empty_like(d["R"]), torch.empty_like(d["W"]),
                    torch.empty_like(d["b"]), ws)
    tws = torch.empty(B.fno_time_lift_bwd_workspace_bytes(c_in, width, nt) // 4 + 2, dtype=torch.float32,
                      device="cuda")
    gwt, gbt = torch.empty(nt, device="cuda"), torch.empty(nt, device="cuda")
    gwc, gbc = torch.empty((width, c_in), device="cuda"), torch.empty(width, device="cuda")
    B.fno_time_lift_bwd(1, c_in, width, nspace, nt, d["a"], d["wt"], d["bt"], d["wc"], gv0, gwt, gbt, gwc, gbc, tws)
    torch.cuda.synchronize()

    # oracle: the same chain in float64
    v0o = O.time_lift(a, wt, bt, wc, bc)
    v1o = O.block_fwd(v0o, R, W, b, spec, "gelu")[0]
    uo = O.pointwise_mlp2(v1o, w1, b1, w2, b2)
    assert rel(host(v0), v0o) <= TOL and rel(host(u), uo) <= TOL
    gvo = O.pointwise_mlp2_bwd(v1o, w1, b1, w2, O.rel_l2_grad(uo, y))["gx"]
    gvo = O.block_bwd(v0o, R, W, b, gvo, spec, "gelu")["gx"]
    ref = O.time_lift_bwd(a, wt, bt, wc, gvo)
    GT = 5 * TOL
    for name, got in (("gWt", gwt), ("gbt", gbt), ("gWc", gwc), ("gbc", gbc)):
        assert rel(host(got), ref[name]) <= GT, name


@pytest.mark.parametrize("nz,mz,nt,mt,rule", [
    (1, 0, 5, 3, 1),          # one row, paired with itself; a row shorter than the tail's four lane groups x 2
    (2, 1, 1, 1, 0),          # one pair, one time step
    (8, 3, 35, 15, 0),        # four planes of 4 pairs per tile, 74 planes: the last tile is half empty
    (5, 2, 6, 3, 1),          # four planes of 3 pairs, the middle row its own pair
    (12, 4, 20, 10, 1),       # two planes of 6 pairs per tile, 37 planes, 20 columns
    (15, 3, 7, 4, 0),         # odd z: the middle row at half weight, two planes of 8 pairs per tile
    (31, 7, 13, 7, 1),        # exactly one tile of 16 pairs
    (33, 15, 17, 9, 0),       # one pair into a second tile, all 16 frequency rows; a tail of one step; 18 columns
    (34, 16, 20, 10, 0),      # 17 frequency rows: two row tiles, the second nearly empty
    (71, 33, 33, 16, 1),      # 34 frequency rows: two groups of row tiles; 32 columns
    (70, 5, 63, 32, 0),       # 64 columns: two column groups; three whole runs of 16 steps and a tail of 15
    (263, 24, 45, 3, 0),      # long axes on both sides
])
def test_folded_forward_transform_at_the_edges_of_its_tiles(nz, mz, nt, mt, rule):
    """Forward (t, z) stage for lengths without a fast split, at the edges of the row tiles, frequency
    tiles, column tiles and of the tail of a row; 37 planes are no multiple of a block's or an XCD's share."""
    grid = (37, 2, nz, nt) if rule == 0 else (37, 1, nz, nt)
    L = Layer(1, 1, 1, grid, (1, 1, mz, mt) if rule == 0 else (1, 0, mz, mt), rule)
    y, xh = gpu_spectral_fwd(L)
    yo, xho = O.spectral_conv_fwd(L.x, L.R, L.spec, return_xhat=True)
    assert rel(xh, xho) <= TOL
    assert rel(y, yo) <= TOL


@pytest.mark.parametrize("c, nz, mz, nt, mt, rule", [
    (1, 1, 0, 1, 1, 1),         # one point per column
    (3, 5, 2, 3, 2, 1),         # half a tile: three pairs and their mirrored rows, the middle row its own pair
    (8, 16, 4, 8, 3, 0),        # eight pairs and eight channels: the generic kernel
    (9, 18, 9, 17, 9, 0),       # nine pairs: one past the half tile; a second tile of t with one new step; 17 of 20 columns
    (20, 33, 8, 16, 8, 1),      # one pair past a whole tile, symmetric rule
    (20, 49, 12, 30, 8, 0),     # two tiles (nine pairs in the second), overlapping runs of four steps at the end of a row
    (17, 64, 12, 20, 6, 0),     # runs of three steps; three empty channels in the last group
    (21, 40, 6, 24, 8, 1),      # more than 20 channels: one row of a pair at a time, then runs of three steps
    (32, 35, 17, 31, 16, 0),    # every channel, the largest column count, one row of a pair at a time; odd z
    (24, 40, 5, 10, 5, 0),      # 24 channels, runs of three: both rows again
    (5, 70, 33, 63, 32, 0),     # folded spectrum of four channels past half a CU's LDS: the generic kernel
    (5, 70, 33, 20, 8, 0),      # more than eight K steps
    (4, 40, 5, 63, 32, 0),      # 63 columns in 16 tiles, four tiles of t
    (4, 128, 60, 48, 24, 0),    # as the case of 70: the generic kernel, with a 16-point FFT
    (3, 12, 3, 70, 5, 0),       # t axis past the folded kernel: the generic one
    (2, 35, 6, 66, 4, 1),       # same, dense z stage
    (20, 256, 128, 10, 1, 0),   # table of the folded kernel past the LDS: the per-tile one, rows padded to 16
])
def test_inverse_transform_at_the_edges_of_its_tiles(c, nz, mz, nt, mt, rule):
    """Inverse (z, t) stage with every epilogue (forward, forward with the pre-activation, adjoint, none) at the edges of
    the tiles of row pairs, of t, of columns and of channels; 7 and 14 columns are no multiple of a block's share.
    A batch entry of NaNs leaves the other entry, whose columns share blocks with it, as it was."""
    L = Layer(1, c, c, (7, 1, nz, nt), (2, 0, mz, mt), 1) if rule else Layer(1, c, c, (7, 2, nz, nt), (2, 1, mz, mt))
    out, z, xh = gpu_block_fwd(L)
    oo, zo, xho = O.block_fwd(L.x, L.R, L.W, L.b, L.spec)
    assert rel(out, oo) <= TOL and rel(z, zo) <= TOL
    y, _ = gpu_spectral_fwd(L)
    assert rel(y, O.spectral_conv_fwd(L.x, L.R, L.spec)) <= TOL
    g = synth.normal_field(3, synth.T_GOUT, 1, c, L.spec.grid)
    ref = O.block_bwd(L.x, L.R, L.W, L.b, g, L.spec)
    gx = torch.empty((1, c) + L.spec.grid, device="cuda")
    B.fno_block_bwd(L.desc, dev(L.x), dev(L.R), dev(L.W), dev(z), dev(xh), dev(g), gx, None, None, None,
                    B.alloc_workspace(L.desc, B.FNO_OP_BLOCK_BWD))
    torch.cuda.synchronize()
    assert rel(host(gx), ref["gx"]) <= TOL

    two = B.make_desc(2, c, c, L.spec.grid, L.spec.modes, rule, B.FNO_ACT_GELU)
    x2 = dev(np.concatenate([np.full_like(L.x, np.nan), L.x]))
    out2 = torch.empty_like(x2)
    B.fno_block_fwd(two, x2, dev(L.R), dev(L.W), dev(L.b), out2, None, None, B.alloc_workspace(two, B.FNO_OP_BLOCK_FWD))
    torch.cuda.synchronize()
    assert np.isnan(host(out2[0])).all()
    assert np.array_equal(host(out2[1]), out[0])


@pytest.mark.parametrize("c, nz, mz, nt, mt, rule", [
    (20, 5, 2, 17, 6, 0),       # half a tile alone, the middle row its own pair, one step in the second tile of t
    (6, 40, 7, 24, 8, 1),       # a whole tile and a half one; runs of three steps, none to spare
    (7, 47, 9, 25, 9, 0),       # a half tile of exactly eight pairs, odd z; overlapping runs of four
    (10, 33, 6, 29, 3, 0),      # an odd axis whose middle row opens the half tile
    (20, 44, 8, 32, 11, 0),     # whole runs of four
    (2, 21, 4, 18, 1, 1),       # one group of channels; the last lanes of the second tile of t have no step of their own
])
def test_inverse_transform_of_rows_in_two_tiles(c, nz, mz, nt, mt, rule):
    """Folded inverse (z, t) stage, one task over both tiles of t: whole and half tiles of row pairs."""
    test_inverse_transform_at_the_edges_of_its_tiles(c, nz, mz, nt, mt, rule)


@pytest.mark.parametrize("c, nz, mz, nt, mt, rule", [
    # per-tile kernel: one residue class; padded channels; rows padded from 30 and 24 to 32 and from 12 to 16 points of t;
    # eight channel tiles; several groups of residue classes, most z frequencies kept; an odd number of them
    (20, 16, 4, 32, 8, 0), (7, 128, 30, 16, 9, 0), (18, 64, 12, 30, 9, 0), (13, 16, 8, 24, 11, 0), (24, 16, 3, 20, 7, 0),
    (3, 256, 128, 12, 7, 0), (8, 512, 140, 16, 2, 0), (6, 32, 9, 16, 8, 1),
    # generic kernel: 20 channels; a 32-channel convolution whose rows take V's place in LDS (its block folded); 32 and 24
    # channels under a t axis past the folded kernel
    (20, 8, 3, 24, 6, 0), (32, 8, 3, 16, 5, 0), (32, 7, 3, 66, 4, 0), (24, 8, 3, 66, 4, 0),
    # folded: short z axes without an FFT of eight points
    (8, 12, 4, 48, 12, 0), (32, 9, 3, 20, 5, 1), (6, 27, 6, 33, 9, 1), (32, 7, 3, 6, 3, 1),
    (4, 16, 4, 8, 3, 0),        # folded: eight pairs, a half tile with every lane at work
])
def test_inverse_transform_on_the_tile_and_generic_kernels(c, nz, mz, nt, mt, rule):
    test_inverse_transform_at_the_edges_of_its_tiles(c, nz, mz, nt, mt, rule)


@pytest.mark.parametrize("c, nz, mz, nt, mt", [
    # folded spectra that leave a block of the folded kernel one column, on more columns than fill the chip: fewer tasks
    # than waves; two blocks per CU
    (20, 64, 12, 16, 9), (6, 128, 64, 16, 9),
])
def test_many_columns_of_a_large_folded_spectrum(c, nz, mz, nt, mt):
    test_block_fwd_and_bwd_match_oracle((1, c, c, (28, 28, nz, nt), (1, 1, mz, mt), 0), B.FNO_ACT_GELU)


@pytest.mark.parametrize("nx, ny", [(48, 32), (29, 53), (64, 32), (50, 41)])
def test_short_last_tiles_of_columns_that_fill_the_chip_once(nx, ny):
    """Folded inverse (z, t) stage with 12 channels, three tasks a column: on two waves at three quarters of the 2048 columns that
    one wave each has on the chip at a time (1536) and past them (2050), on one wave between (1537, 2048)."""
    test_block_fwd_and_bwd_match_oracle((1, 12, 12, (nx, ny, 35, 18), (1, 1, 5, 4), 0), B.FNO_ACT_GELU)


@pytest.mark.parametrize("c, nz, mz, nt, mt", [
    (2, 611, 30, 4, 2), (1, 1215, 300, 3, 2), (2, 609, 304, 5, 3),      # folded, one row tile per block
    (3, 128, 64, 10, 5), (2, 160, 30, 24, 4), (2, 256, 100, 20, 9),     # mixed radix: many frequencies
    (2, 512, 40, 14, 4), (3, 640, 20, 8, 3),
])
def test_forward_transform_of_long_z_axes(c, nz, mz, nt, mt):
    L = Layer(2, c, c, (3, 2, nz, nt), (1, 1, mz, mt))
    y, xh = gpu_spectral_fwd(L)
    yo, xho = O.spectral_conv_fwd(L.x, L.R, L.spec, return_xhat=True)
    assert rel(xh, xho) <= TOL and rel(y, yo) <= TOL


@pytest.mark.parametrize("nz, mz, nt, mt", [
    (16, 3, 16, 9), (128, 20, 16, 9), (64, 12, 32, 17), (8, 2, 64, 33), (32, 5, 64, 33), (64, 9, 30, 16),      # every bin of t
    (64, 12, 32, 9), (64, 30, 64, 12), (64, 9, 30, 15), (128, 16, 32, 8), (128, 3, 64, 10), (128, 20, 30, 7),  # 4 and 8 residues
    (256, 20, 16, 5), (64, 32, 16, 8), (128, 1, 16, 3), (32, 4, 32, 5),                                        # any count of them
])
def test_forward_transform_of_whole_rows(nz, mz, nt, mt):
    """The kernel with a row per thread; 15 planes: blocks of several have one left over."""
    L = Layer(1, 1, 1, (5, 3, nz, nt), (2, 1, mz, mt))
    y, xh = gpu_spectral_fwd(L)
    yo, xho = O.spectral_conv_fwd(L.x, L.R, L.spec, return_xhat=True)
    assert rel(xh, xho) <= TOL and rel(y, yo) <= TOL


@pytest.mark.parametrize("nz, mz, nt, mt", [(12, 2, 4, 2), (20, 4, 5, 2), (8, 2, 6, 3), (24, 4, 7, 3), (16, 3, 8, 3),
                                            (32, 5, 5, 2), (10, 3, 5, 2)])
@pytest.mark.parametrize("nx, ny", [(63, 61), (24, 32)])
def test_forward_transform_of_short_rows(nx, ny, nz, mz, nt, mt):
    """Many planes of short rows on the mixed-radix kernel, M = 4, 8, 16 and 32 (M = 2 is folded), few of them folded;
    3072 planes are the most that are few."""
    L = Layer(2, 2, 2, (nx, ny, nz, nt), (1, 1, mz, mt))
    y, xh = gpu_spectral_fwd(L)
    yo, xho = O.spectral_conv_fwd(L.x, L.R, L.spec, return_xhat=True)
    assert rel(xh, xho) <= TOL and rel(y, yo) <= TOL


@pytest.mark.parametrize("case", [
    # x and y axes on the kernels with an FFT of M points in registers: M = 4, 2 and 1 with more than 48 folded
    # frequencies or a folded table past 40 KiB, 8 and 16
    (1, 2, 2, (204, 202, 2, 3), (50, 49, 1, 2), 0),
    (2, 1, 2, (156, 101, 3, 4), (34, 49, 1, 2), 1),
    (1, 2, 1, (80, 72, 3, 4), (13, 20, 1, 2), 0),
    (1, 3, 2, (144, 40, 4, 5), (30, 20, 1, 2), 0),
    # M = 4 and 2 with few residues and frequencies under rows of 48 (80) values and more; one value less is folded
    (2, 3, 2, (12, 20, 20, 16), (2, 3, 5, 8), 0),
    (1, 2, 3, (20, 12, 12, 16), (3, 2, 3, 8), 0),
    (1, 2, 2, (14, 10, 12, 16), (1, 1, 3, 8), 1),
    (1, 2, 2, (6, 2, 12, 16), (2, 1, 3, 8), 0),
    (1, 2, 2, (4, 12, 47, 3), (1, 2, 23, 1), 1),
    # inverse: more frequencies than bins (M = 32, 16); rows of 84 values, off the 64-byte grid, in 4096 wide tiles
    (1, 2, 2, (64, 96, 3, 4), (31, 40, 1, 2), 1),
    (1, 2, 1, (48, 16, 5, 6), (23, 7, 2, 3), 1),
    (2, 8, 8, (128, 16, 22, 8), (2, 3, 10, 4), 1),
])
def test_fft_axis_kernels_match_oracle(case):
    test_spectral_conv_fwd_matches_oracle(case)
    test_spectral_conv_bwd_matches_oracle(case)


@pytest.mark.parametrize("case", [
    # x stages and mode mix in one launch: tiles of four columns with one to spare, of eight; one and two points, every
    # frequency kept; odd and even axes; more and fewer channels out than in; one to four entries
    (1, 3, 5, (1, 3, 4, 5), (0, 1, 1, 1), 1),
    (4, 2, 2, (2, 4, 4, 4), (1, 1, 1, 3), 0),
    (3, 4, 4, (9, 6, 5, 6), (4, 2, 2, 3), 1),
    (2, 5, 3, (14, 7, 6, 5), (7, 3, 2, 3), 0),
    (2, 3, 5, (11, 6, 5, 6), (3, 2, 1, 2), 1),
    (1, 2, 2, (10, 17, 17, 10), (2, 8, 8, 5), 1),
    (1, 17, 32, (6, 5, 4, 4), (1, 1, 1, 2), 0),
    # one step inside it: many sums in an adjoint, many products of the mix
    (1, 20, 10, (36, 4, 8, 6), (4, 1, 2, 2), 0),
    (4, 29, 29, (16, 5, 5, 4), (3, 1, 1, 2), 1),
    # one step past it: kernels of their own for one to five entries
    (1, 12, 16, (30, 9, 8, 6), (7, 2, 2, 3), 0),
    (2, 12, 16, (30, 9, 8, 6), (7, 2, 2, 3), 0),
    (3, 6, 6, (32, 9, 8, 6), (8, 2, 2, 3), 0),
    (5, 2, 3, (9, 6, 5, 6), (2, 2, 2, 3), 1),
    # past it by the products of the mix alone, by the weights' size, and (adjoint) by the points of all entries
    (1, 32, 32, (11, 5, 4, 4), (5, 1, 1, 2), 1),
    (1, 28, 28, (6, 24, 16, 8), (2, 6, 4, 4), 1),
    (3, 2, 2, (33, 6, 5, 6), (2, 2, 1, 3), 0),
])
def test_x_stages_and_mode_mix_of_small_layers(case):
    test_spectral_conv_fwd_matches_oracle(case)
    test_spectral_conv_bwd_matches_oracle(case)
    if case[1] == case[2]:
        test_block_fwd_and_bwd_match_oracle(case, B.FNO_ACT_GELU)


@pytest.mark.parametrize("n, m", [(80, 13), (12, 2), (20, 3), (14, 1), (6, 2), (4, 1), (36, 6), (45, 10), (28, 5), (16, 4)])
def test_x_stage_kernels_of_five_entries(n, m):
    """Short x axes on the kernels of the stage itself: batches above four are never in one launch with the mix."""
    test_fft_axis_kernels_match_oracle((5, 2, 2, (n, 5, 12, 16), (m, 1, 3, 8), 0))


@pytest.mark.parametrize("case", [
    (1, 3, 5, (1, 3, 4, 5), (0, 1, 1, 1), 1),          # x stages and mode mix in one launch, forward and adjoint
    (2, 4, 4, (9, 6, 5, 6), (4, 2, 2, 3), 1),
    (4, 16, 16, (12, 9, 8, 6), (3, 2, 2, 3), 0),       # the forward alone
    (2, 3, 5, (11, 6, 5, 6), (3, 2, 1, 2), 1),         # the adjoint alone
    (2, 12, 16, (30, 9, 8, 6), (7, 2, 2, 3), 0),       # neither
])
def test_weight_gradient_from_a_spectrum_saved_and_worked_out_again(case):
    """The adjoint without the forward's spectrum takes the forward's kernels: the same bits."""
    L = Layer(*case)
    gy = dev(synth.normal_field(1, synth.T_GOUT, case[0], case[2], L.spec.grid))
    x, R = dev(L.x), dev(L.R)
    ws = B.alloc_workspace(L.desc, B.FNO_OP_SPECTRAL_CONV_BWD)
    xh = torch.empty((case[0], case[1]) + L.counts, dtype=torch.complex64, device="cuda")
    B.fno_spectral_conv_fwd(L.desc, x, R, torch.empty_like(gy), xh, ws)
    gR = [torch.empty_like(R) for _ in range(2)]
    B.fno_spectral_conv_bwd(L.desc, x, xh, R, gy, None, gR[0], ws)
    B.fno_spectral_conv_bwd(L.desc, x, None, R, gy, None, gR[1], ws)
    torch.cuda.synchronize()
    assert torch.equal(gR[0], gR[1])
    assert rel(host(gR[1]), O.spectral_conv_bwd(L.x, L.R, host(gy), L.spec)[1]) <= TOL


def test_one_launch_adds_to_the_weight_gradient():
    """FNO_FLAG_ACCUMULATE_GRADS on a small layer: gR is added to what the buffer holds, gx is not."""
    L = Layer(2, 3, 4, (8, 6, 5, 6), (2, 2, 1, 2))
    gy = dev(synth.normal_field(1, synth.T_GOUT, 2, 4, L.spec.grid))
    ws = B.alloc_workspace(L.desc, B.FNO_OP_SPECTRAL_CONV_BWD)
    got = []
    for flags in (0, B.FNO_FLAG_ACCUMULATE_GRADS):
        gx = torch.full((2, 3) + L.spec.grid, 7.0, device="cuda")
        gR = torch.full((3, 4) + L.counts, 0.5 - 2j, dtype=torch.complex64, device="cuda")
        desc = B.make_desc(2, 3, 4, L.spec.grid, L.spec.modes, 0, 0, flags)
        B.fno_spectral_conv_bwd(desc, dev(L.x), None, dev(L.R), gy, gx, gR, ws)
        torch.cuda.synchronize()
        got.append((host(gx), host(gR)))
    assert np.array_equal(got[0][0], got[1][0])
    # two fp32 additions more, each within 2^-24 of a sum of size 2
    assert np.abs(got[1][1] - got[0][1] - (0.5 - 2j)).max() <= 4 * 2.0 ** -24 * max(2.1, np.abs(got[1][1]).max())


@pytest.mark.parametrize("c_in, c_out, npts, batch", [
    (1, 1, 3, 1), (8, 8, 64, 2), (5, 20, 65, 2), (8, 32, 127, 1), (9, 12, 66, 3), (24, 24, 193, 1), (7, 25, 640, 2),
    (25, 8, 130, 1), (26, 16, 129, 2), (32, 32, 1001, 1), (32, 17, 64, 1),
    (5, 8, 64 * (2048 * 32 + 700) + 13, 1),      # more than one fp32 chain per wave, ragged end
])
def test_sums_over_points_of_every_tile_shape(c_in, c_out, npts, batch):
    """gW = sum g x^T and gb = sum g (the adjoint of a pointwise linear map) at the edges of the kernel's channel
    tiles and point steps, on tensors that are only 4-byte aligned where a row's length makes them so."""
    gen = torch.Generator(device="cuda").manual_seed(c_in * 1000 + c_out)
    x = torch.randn((batch, c_in, npts), device="cuda", generator=gen)
    g = torch.randn((batch, c_out, npts), device="cuda", generator=gen) + 0.1
    w = torch.randn((c_out, c_in), device="cuda", generator=gen)
    gW, gb = torch.empty_like(w), torch.empty(c_out, device="cuda")
    ws = torch.empty(B.fno_pointwise_bwd_workspace_bytes(c_in, 0, c_out) // 4 + 2, device="cuda")
    B.fno_pointwise_linear_bwd(batch, c_in, c_out, npts, x, w, g, None, gW, gb, ws)
    torch.cuda.synchronize()
    xd, gd = x.cpu().double().numpy(), g.cpu().double().numpy()
    want = sum(gd[k] @ xd[k].T for k in range(batch))
    # fp32 chains of at most 128 terms (then doubles): an entry is off by a few 2^-24 of its terms' root sum square
    scale = np.sqrt(sum((gd[k] ** 2) @ (xd[k] ** 2).T for k in range(batch)))
    assert np.max(np.abs(host(gW) - want) / np.maximum(scale, np.abs(want))) <= TOL
    assert rel(host(gb), gd.sum(axis=(0, 2))) <= TOL


@pytest.mark.parametrize("c_in, c_out", [(24, 24), (17, 13), (32, 32), (27, 25)])
def test_sums_over_points_of_a_short_last_step(c_in, c_out):
    """Widths whose waves share a step: entries of fewer points than a lane takes at once, and last steps whose points
    end 1, 2 or 3 into a lane's four, before and after the first step, so that lanes read points in front of theirs."""
    for npts in (1, 2, 3, 4, 5, 6, 7, 61, 62, 63, 65, 66, 67, 68, 190):
        test_sums_over_points_of_every_tile_shape(c_in, c_out, npts, 2)


@pytest.mark.parametrize("npts", [2 ** 27, 2 ** 27 + 1])
@pytest.mark.parametrize("c_in, c_out", [(9, 13), (9, 25)])
def test_sums_over_points_of_the_longest_entries(c_in, c_out, npts):
    """The most points that four rows of a tensor may have for 32-bit offsets (two and four waves a step), and one more (every
    wave reads all of x, at 64-bit addresses), against float64 sums made piece by piece on the device."""
    gen = torch.Generator(device="cuda").manual_seed(c_out)
    x = torch.randn((1, c_in, npts), device="cuda", generator=gen)
    g = torch.randn((1, c_out, npts), device="cuda", generator=gen)
    gW, gb = torch.empty((c_out, c_in), device="cuda"), torch.empty(c_out, device="cuda")
    ws = torch.empty(B.fno_pointwise_bwd_workspace_bytes(c_in, 0, c_out) // 4 + 2, device="cuda")
    B.fno_pointwise_linear_bwd(1, c_in, c_out, npts, x, torch.ones_like(gW), g, None, gW, gb, ws)
    want, sq, wantb, sqb = (torch.zeros(*shape, device="cuda", dtype=torch.float64)
                            for shape in ((c_out, c_in), (c_out, c_in), (c_out,), (c_out,)))
    for p in range(0, npts, 2 ** 22):
        gd, xd = g[0, :, p:p + 2 ** 22].double(), x[0, :, p:p + 2 ** 22].double()
        for i in range(c_in):
            term = gd * xd[i]
            want[:, i] += term.sum(1)
            sq[:, i] += term.square_().sum(1)
        wantb += gd.sum(1)
        sqb += gd.square().sum(1)
    # as above: an entry is off by a few 2^-24 of its terms' root sum square
    assert float(((gW - want).abs() / torch.maximum(sq.sqrt(), want.abs())).max()) <= TOL
    assert float(((gb - wantb).abs() / torch.maximum(sqb.sqrt(), wantb.abs())).max()) <= TOL


@pytest.mark.parametrize("case", [
    (2, 32, 32, (3, 3, 9, 5), (1, 1, 2, 2), 0),        # 405 points: 5 lanes of four and a point in the last step
    (2, 27, 27, (3, 3, 5, 3), (1, 1, 1, 1), 0),        # 135: a lane and 3 points, a ragged channel tile
    (1, 24, 24, (1, 2, 11, 3), (0, 0, 2, 1), 1),       # 66: 2 points
    (3, 18, 18, (1, 1, 2, 3), (0, 0, 0, 1), 1),        # 6: less than a step
])
def test_block_adjoint_of_a_short_last_step(case):
    for activation in (B.FNO_ACT_GELU, B.FNO_ACT_IDENTITY):
        test_block_fwd_and_bwd_match_oracle(case, activation)


@pytest.mark.parametrize("c_in, c_out", [(5, 8), (24, 24), (32, 7)])
def test_sums_over_points_reach_doubles_after_128_terms(c_in, c_out):
    """Whole numbers whose 128-term chains stay below 2^24 (128 x 255 x 255 < 8.4e6) and are therefore exact in fp32,
    while the 2048 terms of a wave's 16 lane blocks are not: every sum of products comes out exact, where the halves of
    the points cancel to what a rounding of the partial sums would drown."""
    npts = 64 * 2048 * 32                                # one chain per wave
    gen = torch.Generator(device="cuda").manual_seed(c_in)
    x = torch.randint(0, 256, (1, c_in, npts), device="cuda", generator=gen).float()
    g = torch.randint(0, 256, (1, c_out, npts), device="cuda", generator=gen).float()
    g[:, :, npts // 2:] *= -1.0
    gW, gb = torch.empty((c_out, c_in), device="cuda"), torch.empty(c_out, device="cuda")
    ws = torch.empty(B.fno_pointwise_bwd_workspace_bytes(c_in, 0, c_out) // 4 + 2, device="cuda")
    B.fno_pointwise_linear_bwd(1, c_in, c_out, npts, x, torch.zeros_like(gW), g, None, gW, gb, ws)
    torch.cuda.synchronize()
    want = torch.stack([(g[0, o].double() * x[0].double()).sum(1) for o in range(c_out)])
    assert torch.equal(gW, want.float())
    assert torch.equal(gb, g[0].double().sum(1).float())


def test_sums_over_points_of_a_streamed_gradient():
    """A gradient above 256 MiB with an odd point count: the nontemporal variant on rows that are 4-byte aligned."""
    c_in, c_out, npts = 3, 17, 4_100_003
    gen = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn((1, c_in, npts), device="cuda", generator=gen)
    x[:, 0] = torch.linspace(0.0, 1.0, npts, device="cuda")          # a coordinate channel
    g = torch.randn((1, c_out, npts), device="cuda", generator=gen) + 0.1
    w = torch.randn((c_out, c_in), device="cuda", generator=gen)
    gW, gb = torch.empty_like(w), torch.empty(c_out, device="cuda")
    ws = torch.empty(B.fno_pointwise_bwd_workspace_bytes(c_in, 0, c_out) // 4 + 2, device="cuda")
    B.fno_pointwise_linear_bwd(1, c_in, c_out, npts, x, w, g, None, gW, gb, ws)
    torch.cuda.synchronize()
    gd, xd = g[0].double(), x[0].double()
    want = torch.stack([(gd * xd[i]).sum(1) for i in range(c_in)], 1)
    scale = torch.stack([(gd * xd[i]).square().sum(1) for i in range(c_in)], 1).sqrt()
    assert float(((gW - want).abs() / torch.maximum(scale, want.abs())).max()) <= TOL
    assert rel(host(gb), host(gd.sum(1))) <= TOL


@pytest.mark.parametrize("c", [13, 32])
def test_block_adjoint_of_streamed_tensors(c):
    """A block backward whose gradient with respect to the pre-activation is above 256 MiB, at an odd width and at 32:
    gW and gb against products in float64 on the device, gx against the same call on halves of the batch that stay
    below."""
    grid, modes = (624 // c, 40, 21, 17), (2, 2, 2, 3)
    batch = 10
    counts = tuple(2 * m for m in modes[:3]) + (modes[3],)
    gen = torch.Generator(device="cuda").manual_seed(c)
    randn = lambda *s: torch.randn(s, device="cuda", generator=gen)
    x, z, g = (randn(batch, c, *grid) for _ in range(3))
    assert g.numel() * 4 >= 256 << 20
    W, R = randn(c, c), torch.view_as_complex(randn(c, c, *counts, 2) / c)
    gx, gW, gb = torch.empty_like(x), torch.empty_like(W), torch.empty(c, device="cuda")
    desc = B.make_desc(batch, c, c, grid, modes, 0, B.FNO_ACT_GELU)
    B.fno_block_bwd(desc, x, R, W, z, None, g, gx, None, gW, gb, B.alloc_workspace(desc, B.FNO_OP_BLOCK_BWD))
    half = B.make_desc(batch // 2, c, c, grid, modes, 0, B.FNO_ACT_GELU)
    parts = torch.empty_like(x)
    ws = B.alloc_workspace(half, B.FNO_OP_BLOCK_BWD)
    for h in (slice(0, batch // 2), slice(batch // 2, batch)):
        B.fno_block_bwd(half, x[h], R, W, z[h], None, g[h], parts[h], None, None, None, ws)
    torch.cuda.synchronize()
    assert rel(host(gx), host(parts)) <= TOL
    want, scale, wb = (torch.zeros((c, c), device="cuda", dtype=torch.float64) for _ in range(3))
    for b in range(batch):
        zd = z[b].reshape(c, -1).double()
        slope = 0.5 * (1 + torch.erf(zd / 2 ** 0.5)) + zd * torch.exp(-zd * zd / 2) / (2 * np.pi) ** 0.5
        gz, xd = g[b].reshape(c, -1).double() * slope, x[b].reshape(c, -1).double()
        want += gz @ xd.T
        scale += gz.square() @ xd.square().T
        wb[0] += gz.sum(1)
    assert float(((gW - want).abs() / torch.maximum(scale.sqrt(), want.abs())).max()) <= TOL
    assert rel(host(gb), host(wb[0])) <= TOL


@pytest.mark.parametrize("batch", [1, 2])
def test_mode_mix_adjoint_of_a_streamed_weight(batch):
    """The adjoint of the mode mix with a weight above 256 MiB, one and two batch entries: gR and gx of a convolution
    that keeps every mode of its x axis, at sampled channel pairs and on the whole gradient."""
    c, grid, modes, counts = 32, (64, 33, 8, 6), (32, 16, 4, 3), (64, 32, 8, 3)
    gen = torch.Generator(device="cuda").manual_seed(batch)
    randn = lambda *s: torch.randn(s, device="cuda", generator=gen)
    R = torch.view_as_complex(randn(c, c, *counts, 2) / c)
    assert R.numel() * 8 >= 256 << 20
    x, g = randn(batch, c, *grid), randn(batch, c, *grid)
    desc = B.make_desc(batch, c, c, grid, modes, 0, B.FNO_ACT_IDENTITY)
    ws = B.alloc_workspace(desc, B.FNO_OP_SPECTRAL_CONV_BWD)
    gx, gR = torch.empty_like(x), torch.empty_like(R)
    B.fno_spectral_conv_bwd(desc, x, None, R, g, gx, gR, ws)
    torch.cuda.synchronize()
    spec = O.LayerSpec(grid, modes, 0)
    for i, o in ((0, 0), (5, 31), (31, 7)):
        _, gRo = O.spectral_conv_bwd(host(x[:, i:i + 1]), host(R[i:i + 1, o:o + 1]), host(g[:, o:o + 1]), spec)
        assert rel(host(gR[i:i + 1, o:o + 1]), gRo) <= TOL
    # <gx, x'> = <g, K x'> for a random x'
    xp, y = randn(batch, c, *grid), torch.empty_like(x)
    B.fno_spectral_conv_fwd(desc, xp, R, y, None, ws)
    torch.cuda.synchronize()
    lhs, rhs = float((gx.double() * xp.double()).sum()), float((g.double() * y.double()).sum())
    assert abs(lhs - rhs) <= TOL * float(gx.double().norm()) * float(xp.double().norm())


@pytest.mark.parametrize("case", [
    (1, 32, 32, (3, 2, 32, 16), (1, 1, 4, 4), 0),      # width 32, 48 whole steps
    (2, 20, 20, (3, 3, 12, 7), (1, 1, 3, 3), 0),       # width 20, 756 points: a ragged last step
    (1, 28, 28, (3, 5, 6, 7), (1, 2, 2, 3), 0),        # a padded channel tile, rows that are not 16-byte aligned
    (1, 13, 13, (3, 3, 9, 5), (1, 1, 2, 2), 0),        # odd width
])
def test_block_adjoint_for_widths_and_point_counts_off_the_tiles(case):
    for activation in (B.FNO_ACT_GELU, B.FNO_ACT_IDENTITY):
        test_block_fwd_and_bwd_match_oracle(case, activation)


@pytest.mark.parametrize("case", [
    # x and y axes at the edges of the folded products' tiles: 1, 8, 16, 17, 33 and 48 folded frequencies
    (1, 2, 3, (45, 118, 4, 5), (7, 16, 1, 2), 0),      # odd length; 2 x 59 with 17 folded frequencies
    (1, 2, 2, (31, 33, 3, 4), (15, 16, 1, 1), 1),      # every frequency kept, symmetric rule: 16 and 17, inner of 3
    (1, 1, 1, (106, 94, 2, 3), (47, 32, 1, 2), 0),     # 48 and 33 folded frequencies
    (2, 2, 2, (64, 32, 4, 8), (12, 15, 2, 3), 0),      # 32 points folded, 64 on the FFT kernels
    (1, 1, 2, (2, 66, 4, 4), (1, 33, 1, 2), 0),        # two points; every frequency of an even length
    (1, 1, 1, (1, 7, 4, 4), (0, 0, 1, 2), 1),          # one point; one frequency
    (3, 4, 2, (96, 72, 9, 6), (9, 10, 2, 3), 0),       # 32- and 8-point FFTs
    (2, 20, 2, (44, 60, 9, 16), (9, 10, 3, 8), 0),     # two tiles per wave
])
def test_folded_axis_products_match_oracle(case):
    test_spectral_conv_fwd_matches_oracle(case)
    test_spectral_conv_bwd_matches_oracle(case)


@pytest.mark.parametrize("n, m", [(12, 2), (13, 6), (20, 4), (28, 5), (32, 15), (36, 17), (44, 8), (45, 22), (60, 12),
                                  (68, 16), (100, 40), (118, 16), (150, 25)])
def test_folded_axis_products_round_only_their_table_and_their_result(n, m):
    """The sums over an axis without a large power of two are formed in double from float data and a float table.
    What is left are two roundings of relative size up to 2^-24 (rms 0.42 x 2^-24 each over uniform mantissas), a third
    one in the mode mix before the inverse: 0.6 and 0.73 x 2^-24 of the norm expected, 2^-24 asserted.  Chains in fp32
    are off by 1.1 x 2^-24 at 12 points and 2.7 x at 150."""
    L = Layer(256, 1, 1, (n, 1, 1, 1), (m, 0, 0, 1), 1)
    L.R = np.ones_like(L.R)
    y, xh = gpu_spectral_fwd(L)
    k = np.array(O.mode_lists(L.spec)[0])
    wave = np.exp(2j * np.pi * (np.outer(k, np.arange(n)) % n) / n)
    x = L.x.astype(np.float64).reshape(256, n)
    assert rel(xh.reshape(256, -1), x @ wave.conj().T) <= 2.0 ** -24
    # the mix scales by 1 / N as a float
    want = (xh.astype(np.complex128).reshape(256, -1) * float(np.float32(1.0 / n)) @ wave).real
    assert rel(y.reshape(256, n), want) <= 2.0 ** -24


@pytest.mark.parametrize("nz, mz, nt, mt", [(21, 3, 14, 5), (40, 7, 14, 5), (64, 11, 20, 8), (80, 14, 24, 9),
                                            (100, 18, 10, 4), (128, 23, 40, 16), (160, 28, 48, 16), (263, 47, 20, 8), (611, 30, 4, 2),
                                            (801, 30, 8, 2)])
def test_folded_forward_transform_sums_in_short_chains(nz, mz, nt, mt):
    """The error of the forward (t, z) stage is that of two chains of Nt / 2 terms over t and of blocks of eight pairs
    over z.  A rounding has an rms of 0.42 x 2^-24 of its value; a chain of n terms of equal size rounds partial sums
    whose squares add up to (n + 1) / 2 of the total's.  Beside the chains: table and fold, the joined chains, the
    table over z, the phase.  A tenth is added for the scatter of the inputs; a single chain over z is 1.2 times
    (40 points) to 1.6 times (160 points) further off."""
    L = Layer(64, 1, 1, (1, 1, nz, nt), (0, 0, mz, mt), 1)
    _, xh = gpu_spectral_fwd(L)
    n = np.arange(nz)
    k = np.array(O.mode_lists(L.spec)[2])
    bins = np.fft.rfft(L.x.astype(np.float64).reshape(64, nz, nt), axis=2)[:, :, :mt]
    want = np.einsum("kn,bnt->bkt", np.exp(-2j * np.pi * (np.outer(k, n) % nz) / nz), bins)
    roundings = 2 + (nt / 2 + 1) / 2 + 1 + 1 + 4.5 + (np.ceil(nz / 16) + 1) / 2 + 1
    assert rel(xh.reshape(want.shape), want) <= 1.1 * 0.42 * 2.0 ** -24 * np.sqrt(roundings)


@pytest.mark.parametrize("nz, mz, nt, mt", [
    (33, 5, 13, 5), (34, 6, 26, 8), (45, 8, 64, 7),         # one tile of frequencies: a K step of four values, of eight, two
    (17, 5, 17, 9), (90, 16, 24, 12), (150, 30, 48, 16),    # two tiles of bins; of frequencies too
    (99, 17, 1, 1), (118, 20, 20, 8),                       # two tiles of frequencies
    (263, 24, 16, 8), (181, 20, 5, 2),                      # long tables
])
def test_forward_transform_on_split_products(nz, mz, nt, mt):
    """Products of exact three-way splits leave out less than 2^-25 of each, and an instruction sums 32 of them to its
    accumulator; two roundings are counted for it.  Rounded are the fold, the table over t, the large products of at most
    two K steps, the table over z, a tile's sum, the tiles' sum (a chain), and the phase: rms 0.42 x 2^-24 each, a fifth
    for the scatter of the inputs.  Chains in fp32 (four terms an instruction) are a sixth (20 points of t, 118) to a half
    (64 and 45) further off."""
    L = Layer(64, 1, 1, (1, 1, nz, nt), (0, 0, mz, mt), 1)
    _, xh = gpu_spectral_fwd(L)
    n, k = np.arange(nz), np.array(O.mode_lists(L.spec)[2])
    bins = np.fft.rfft(L.x.astype(np.float64).reshape(64, nz, nt), axis=2)[:, :, :mt]
    want = np.einsum("kn,bnt->bkt", np.exp(-2j * np.pi * (np.outer(k, n) % nz) / nz), bins)
    roundings = 1 + 1 + (3 if nt > 32 else 2) + 1 + 2 + (np.ceil(nz / 32) + 1) / 2 + 1
    assert rel(xh.reshape(want.shape), want) <= 1.2 * 0.42 * 2.0 ** -24 * np.sqrt(roundings)


@pytest.mark.parametrize("planes, nz, mz, nt, mt", [
    (2047, 181, 20, 5, 2), (2048, 181, 20, 5, 2), (2304, 263, 24, 16, 8),       # blocks of four waves, of eight
    (16000, 263, 24, 16, 8), (24000, 118, 20, 24, 12), (38000, 60, 12, 30, 8),  # 256 MiB and more: streamed
])
def test_forward_transform_on_split_products_of_many_planes(planes, nz, mz, nt, mt):
    """The bound of the test above, against torch in float64."""
    desc = B.make_desc(planes, 1, 1, (1, 1, nz, nt), (0, 0, mz, mt), 1, 0)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(planes)
    x = torch.randn((planes, 1, 1, 1, nz, nt), device="cuda", generator=gen)
    xh = torch.empty((planes, 1, 1, 1, 2 * mz + 1, mt), dtype=torch.complex64, device="cuda")
    R = torch.zeros((1, 1, 1, 1, 2 * mz + 1, mt), dtype=torch.complex64, device="cuda")
    B.fno_spectral_conv_fwd(desc, x, R, torch.empty_like(x), xh, B.alloc_workspace(desc, B.FNO_OP_SPECTRAL_CONV_FWD))
    want = torch.fft.fft(torch.fft.rfft(x.double(), dim=5)[..., :mt], dim=4)
    want = torch.cat([want[..., :mz + 1, :], want[..., nz - mz:, :]], dim=4)
    roundings = 1 + 1 + (3 if nt > 32 else 2) + 1 + 2 + (np.ceil(nz / 32) + 1) / 2 + 1
    assert float((xh.to(torch.complex128) - want).norm() / want.norm()) <= 1.2 * 0.42 * 2.0 ** -24 * np.sqrt(roundings)


@pytest.mark.parametrize("nz, nt", [(108, 33), (270, 14)])
def test_split_products_leave_no_bias_in_the_lowest_frequencies(nz, nt):
    """Planes add up over y and x.  An entry's error scatters with that of the norm (1.5e-7 of the bins' size; 6 times that
    over 512 entries); a bias of each plane's sums, which the 16-bit instructions have, would add up to 3e-6 here."""
    grid, m = (48, 32, nz, nt), 2
    L_desc = B.make_desc(1, 8, 8, grid, (m, m, m, m), 0, 0)
    gen = torch.Generator(device="cuda").manual_seed(nz)
    x = torch.randn((1, 8) + grid, device="cuda", generator=gen)
    xh = torch.empty((1, 8, 2 * m, 2 * m, 2 * m, m), dtype=torch.complex64, device="cuda")
    R = torch.zeros((8, 8, 2 * m, 2 * m, 2 * m, m), dtype=torch.complex64, device="cuda")
    B.fno_spectral_conv_fwd(L_desc, x, R, torch.empty_like(x), xh, B.alloc_workspace(L_desc, B.FNO_OP_SPECTRAL_CONV_FWD))
    want = torch.fft.rfft(x.double(), dim=5)[..., :m]
    for d in (4, 3, 2):
        want = torch.fft.fft(want, dim=d)
        want = torch.cat([want.narrow(d, 0, m), want.narrow(d, want.shape[d] - m, m)], dim=d)
    size = float(want.abs().square().mean().sqrt())
    assert float((xh.to(torch.complex128) - want).abs().max()) <= 9e-7 * size


@pytest.mark.parametrize("nz, mz, nt, mt", [(64, 11, 20, 8), (96, 17, 20, 8), (128, 23, 10, 4), (160, 28, 24, 9),
                                            (263, 47, 20, 8)])
def test_folded_inverse_transform_sums_in_short_chains(nz, mz, nt, mt):
    """The same count for the inverse (z, t) stage of a convolution: four chains over the folded frequencies, one over
    the 2 mt - 1 columns of t; beside them the mode mix, the folded spectrum, the two tables, the joined chains and the
    two rows of a pair.  One chain over z and a phase in fp32 are 1.15 to 1.4 times further off."""
    L = Layer(64, 1, 1, (1, 1, nz, nt), (0, 0, mz, mt), 1)
    L.R = np.ones_like(L.R)
    y, xh = gpu_spectral_fwd(L)
    k, n = np.array(O.mode_lists(L.spec)[2]), np.arange(nz)
    theta = 2 * np.pi * (np.outer(np.arange(mt), np.arange(nt)) % nt) / nt
    c = np.where((np.arange(mt) == 0) | (2 * np.arange(mt) == nt), 1.0, 2.0) * float(np.float32(1.0 / (nz * nt)))
    rows = np.einsum("kn,bkt->bnt", np.exp(2j * np.pi * (np.outer(k, n) % nz) / nz),
                     xh.astype(np.complex128).reshape(64, len(k), mt) * c)
    want = rows.real @ np.cos(theta) - rows.imag @ np.sin(theta)
    roundings = 6 + ((mz + 1) / 4 + 1) / 2 + mt
    assert rel(y.reshape(want.shape), want) <= 1.1 * 0.42 * 2.0 ** -24 * np.sqrt(roundings)


@pytest.mark.parametrize("c, grid, modes, rule", [
    (32, (5, 2, 35, 31), (1, 1, 17, 16), 0),     # channel groups in several blocks per column, overlapping runs of t
    (20, (7, 2, 49, 30), (2, 1, 12, 8), 0),      # overlapping runs of t
    (20, (6, 4, 64, 20), (1, 1, 12, 8), 0),
    (20, (6, 3, 128, 16), (1, 1, 16, 9), 0),     # column kernels: 16 and 32 points of t
    (20, (6, 3, 64, 32), (1, 1, 12, 9), 0),
    (6, (5, 3, 12, 70), (1, 1, 3, 5), 0),        # generic kernel
    (32, (3, 2, 7, 6), (1, 1, 3, 3), 0),
    (32, (5, 2, 32, 20), (1, 1, 2, 10), 0),      # per-tile kernel: no room for the generic one
    (24, (5, 2, 64, 12), (1, 1, 8, 5), 0),
])
@pytest.mark.parametrize("over", ["out", "z"])
def test_block_in_place_matches_oracle(c, grid, modes, rule, over):
    """out (or the saved pre-activation) over x itself: every point is read before it is written."""
    L = Layer(1, c, c, grid, modes, rule)
    oo, zo, _ = O.block_fwd(L.x, L.R, L.W, L.b, L.spec)
    x, other = dev(L.x), torch.empty((1, c) + L.spec.grid, device="cuda")
    out, z = (x, other) if over == "out" else (other, x)
    B.fno_block_fwd(L.desc, x, dev(L.R), dev(L.W), dev(L.b), out, z, None, B.alloc_workspace(L.desc, B.FNO_OP_BLOCK_FWD))
    torch.cuda.synchronize()
    assert rel(host(out), oo) <= TOL and rel(host(z), zo) <= TOL

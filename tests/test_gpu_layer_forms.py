"""Layers at the sizes where the recurrent loop or its products change form: one compute unit per four rows up to 128 units, the
widths where the bfloat16 loops change their split, products with tile edges and K ranges.  Every optional input, NaN in padded
frames and in untouched workspace, against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import lstm_oracle as O
from tests import test_gpu_parity as P
from tests.gpu_util import TOL, check, dev, host


def _lens(rng, T, B):
    lens = rng.integers(0, T + 1, B)
    lens[0], lens[-1] = T, min(1, T)
    return lens


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("T,B,n_in,n,bidir", [
    (2, 1, 1, 5, False), (2, 4, 33, 64, True), (9, 5, 40, 65, False), (6, 3, 7, 63, True), (5, 8, 130, 128, True), (7, 2, 31, 127, False),
    (3, 260, 12, 20, True),                                                 # bias gradient: more slices than the workspace keeps
    (65, 64, 128, 128, False),                                              # products too large for the tiny ones
    (40, 2, 64, 64, False), (21, 17, 100, 96, True),
    (70, 40, 130, 16, True),                                                # the data gradient: a stage per direction
])
def test_narrow_layer(T, B, n_in, n, bidir, dt):
    _layer(T, B, n_in, n, bidir, dt)


@pytest.mark.parametrize("T,B,n_in,n,bidir", [
    (4, 1, 200, 256, True), (4, 9, 64, 257, True), (5, 17, 250, 512, True), (4, 3, 500, 513, True), (3, 33, 130, 136, False),
    (60, 7, 333, 264, True),
    (52, 32, 60, 1000, True),                                               # the input projection: many tiles, over listed frames, rows of W_x past the last one
    (3, 1, 40, 1025, False), (5, 17, 72, 1160, False), (4, 33, 33, 1027, True), (5, 32, 64, 2048, False), (6, 20, 40, 1900, False),
])
def test_wider_layer(T, B, n_in, n, bidir):
    _layer(T, B, n_in, n, bidir, "bf16")


@pytest.mark.parametrize("T,B,n,bidir", [(3, 1, 500, True), (4, 4, 330, False), (6, 29, 134, True), (3, 40, 200, False), (2, 2, 330, True)])
def test_float_calls_of_few_steps_keep_their_bits(T, B, n, bidir):
    """Where few steps go to the per-step kernels, sums of gradients past 2^32 have all 24 bits and every result repeats: bit for bit as with FLAG_PER_STEP."""
    from paper_1805_05225_amd import binding as Bn
    g = torch.Generator(device="cuda").manual_seed(n)
    D = 2 if bidir else 1
    r = lambda w, *s: (torch.rand(*s, generator=g, device="cuda") * 2 - 1) * w
    sq = lambda t: t if bidir else t[0]
    x, Wx, Wh, b = r(1., T, B, 24), sq(r(.3, D, 24, 4 * n)), sq(r(.3, D, n, 4 * n)), sq(r(.1, D, 4 * n))
    dy = r(2. ** 40, T, B, D * n)

    def run(flags):
        f = Bn.forward(x, Wx, Wh, b, bidirectional=bidir, flags=flags)
        return dict(Bn.backward(f, x, Wx, Wh, None, None, None, dy), **{k: f[k].clone() for k in ("y", "c", "hT", "cT")})
    got, want = run(0), run(Bn.FLAG_PER_STEP)
    for k in want:
        assert torch.isfinite(want[k]).all() and torch.equal(got[k], want[k]), k


@pytest.mark.parametrize("T,B,n_in,n,bidir", [
    (60, 7, 333, 263, True), (30, 21, 200, 443, True), (9, 3, 8, 1003, False), (40, 10, 123, 201, False),
    (52, 64, 60, 1001, True),                                               # the input projection in many tiles
    (200, 32, 2100, 131, False),                                            # the data gradient
    (12, 9, 2100, 1001, True),                                              # the weight gradients
])
def test_odd_width(T, B, n_in, n, bidir):
    """Rows of W_x and DZ are whole 8 bytes, not 16, and the data gradient's K ends in half a chunk."""
    _layer(T, B, n_in, n, bidir, "bf16")


@pytest.mark.parametrize("T,B,n_in,n", [(9, 5, 37, 201), (1, 20, 40, 133)])
def test_odd_width_in_the_smallest_workspace(T, B, n_in, n):
    """Products at any alignment, for workspaces of the size that sufficed while odd widths had no others."""
    from paper_1805_05225_amd import binding as Bn
    rng = np.random.default_rng(n)
    r = lambda *shape: torch.from_numpy(rng.uniform(-0.3, 0.3, shape)).to(torch.bfloat16).cuda()
    x, Wx, Wh, dy = r(T, B, n_in), r(2, n_in, 4 * n), r(2, n, 4 * n), r(T, B, 2 * n)
    lens = torch.from_numpy(_lens(rng, T, B).astype(np.int32)).cuda()
    args = (x, Wx, Wh, None, None, None, lens)
    flags = Bn.FLAG_INFERENCE if T == 1 else 0
    want = Bn.forward(*args, bidirectional=True, flags=flags)
    lo, hi = 0, want["workspace"].numel()                                    # the smallest size that is not refused
    while hi - lo > 256:
        mid = (lo + hi) // 2
        try:
            Bn.forward(*args, bidirectional=True, flags=flags, workspace=torch.empty(mid, dtype=torch.uint8, device="cuda"))
            hi = mid
        except Bn.LstmError as e:
            assert e.status == -6
            lo = mid
    assert hi < want["workspace"].numel()                                    # (neither the padded operands nor, in a step, the packed weights)
    f = Bn.forward(*args, bidirectional=True, flags=flags, workspace=torch.empty(hi, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    check("y", f["y"], want["y"].double().cpu().numpy(), TOL["bf16"])
    check("y (oracle)", f["y"], O.blstm_fwd(host(x), host(Wx), host(Wh), None, None, None, host(lens).astype(np.int64))[0], TOL["bf16"])
    if T > 1:
        g, h = (Bn.backward(k, x, Wx, Wh, None, None, lens, dy) for k in (f, want))
        torch.cuda.synchronize()
        for name in ("dx", "dW_x", "dW_h", "db"):
            check(name, g[name], h[name].double().cpu().numpy(), TOL["bf16"])


@pytest.mark.parametrize("T,B,n_in,n,bidir", [
    (5, 1, 37, 132, False), (6, 17, 30, 256, True), (4, 40, 101, 257, True), (7, 70, 33, 131, True), (3, 300, 8, 130, False),
    (5, 33, 64, 513, True), (4, 64, 41, 1001, True), (90, 12, 30, 140, False),
])
def test_wider_float_layer(T, B, n_in, n, bidir):
    """Rows in any order of length over several row tiles, widths that are no multiple of a tile or a chunk."""
    _layer(T, B, n_in, n, bidir, "f32")


@pytest.mark.parametrize("T,B,n,bidir", [(2, 3, 129, True), (3, 8, 130, False), (4, 25, 255, True), (5, 9, 258, False), (9, 2, 511, True), (6, 7, 1002, False), (13, 16, 1024, True)])
def test_eight_row_loops(T, B, n, bidir):
    """Frames fetched two and four together: any number of steps, also fewer; units that end inside a tile, and inside the four units of a
    load; the last row's last units at the end of a frame."""
    _layer(T, B, 32, n, bidir, "bf16")


@pytest.mark.parametrize("T,B,n_in,n,bidir", [(13, 4, 1296, 648, True), (30, 64, 100, 200, True), (25, 9, 130, 203, True), (2, 3, 33, 130, False), (90, 21, 300, 140, False)])
def test_gradient_products_in_one_launch(T, B, n_in, n, bidir):
    """More tiles than run at a time and dX in sixteen ranges; dX whole; half a chunk at the end of its K; a stage in all; every product in ranges."""
    _layer(T, B, n_in, n, bidir, "bf16")


@pytest.mark.parametrize("T,B,n,bidir", [(9, 5, 136, True), (8, 17, 256, False), (7, 9, 513, True), (9, 20, 640, True), (8, 3, 641, False), (9, 30, 768, True), (6, 8, 769, False),
                                         (12, 48, 768, True)])
def test_eight_row_loop_forms(T, B, n, bidir):
    """The first and last width of each form, W_h packed and (inference) as it lies in memory; the last batch takes another form's packing."""
    _layer(T, B, 24, n, bidir, "bf16")
    from paper_1805_05225_amd import binding as Bn
    g = torch.Generator(device="cuda").manual_seed(n)
    r = lambda *shape: (torch.randn(*shape, generator=g, device="cuda") * n ** -0.5).bfloat16()
    D = 2 if bidir else 1
    x, W_x, W_h = r(T, B, 24), r(*(D, 24, 4 * n)[2 - D:]), r(*(D, n, 4 * n)[2 - D:])
    lens = torch.linspace(1, T, B, device="cuda").int()
    got, ref = (Bn.forward(x, W_x, W_h, None, None, None, lens, bidirectional=bidir, flags=f)["y"] for f in (Bn.FLAG_INFERENCE, Bn.FLAG_PER_STEP))
    check("y", got, host(ref), TOL["bf16"])


@pytest.mark.parametrize("T,B,n,bidir", [(7, 40, 1000, True), (3, 70, 1022, False), (9, 100, 514, True), (5, 200, 520, False), (2, 49, 900, True)])
def test_rows_one_behind_the_other(T, B, n, bidir):
    """More rows than places, lengths from 0 to T, every optional state, against the oracle."""
    _layer(T, B, 24, n, bidir, "bf16")


@pytest.mark.parametrize("T,B,n,shortest,longest", [(600, 100, 520, 0, 600), (600, 100, 520, 0, 9), (40, 37, 1024, 0, 0), (30, 64, 1000, 1, 1),
                                                    (40, 64, 1000, 38, 40), (40, 64, 1000, 26, 40), (40, 33, 1000, 0, 40)])
def test_rows_one_behind_the_other_per_step(T, B, n, shortest, longest):
    """More steps than the table in LDS holds, groups that are done at once, batches without any frame, lengths for which neither loop or only
    the forward one takes rows so: the per-step path's results."""
    from paper_1805_05225_amd import binding
    P.Bn = binding
    rng = np.random.default_rng(n + longest)
    lens = rng.integers(shortest, longest + 1, B)
    lens[3] = longest
    c = P.rnd_case(rng, T, B, 16, n, 2, lens, "bf16", scale=1.0 / np.sqrt(n))
    f1, g1 = P.run_gpu(c, "bf16", True)
    f2, g2 = P.run_gpu(c, "bf16", True, flags=binding.FLAG_PER_STEP)
    for got, ref, names in ((f1, f2, ("y", "c", "hT", "cT")), (g1, g2, ("dx", "dW_x", "dW_h", "db", "dh0", "dc0"))):
        for k in names:
            if longest == 0 or float(ref[k].abs().max()) == 0.0:
                assert torch.equal(got[k], ref[k]), k
            else:
                check(k, got[k], host(ref[k]), 1e-2)


def _layer(T, B, n_in, n, bidir, dt):
    from paper_1805_05225_amd import binding
    P.Bn = binding
    rng = np.random.default_rng(T * 1000 + B + n)
    for lens in (None, _lens(rng, T, B)):
        c = P.rnd_case(rng, T, B, n_in, n, 2 if bidir else 1, lens, dt, scale=2.0 / np.sqrt(n + n_in))
        x, dy = c["x"].copy(), c["dy"].copy()
        if lens is not None:
            for b in range(B):
                x[lens[b]:, b], dy[lens[b]:, b] = np.nan, np.nan
        print("  layer", dt, T, B, n_in, n, bidir, lens is not None, flush=True)
        for direction in ((1,) if bidir else (1, -1)):
            f, g = P.run_gpu(c, dt, bidir, direction, x_override=x, dy_override=dy, poison=True)
            P.compare(f, g, *P.run_oracle(c, bidir, direction), TOL[dt])


@pytest.mark.parametrize("dt,T,B,n", [("bf16", 24, 20, 1040), ("bf16", 16, 33, 2048), ("bf16", 5, 9, 330), ("bf16", 9, 5, 1000), ("bf16", 40, 20, 200), ("bf16", 6, 140, 1000), ("bf16", 4, 6, 64), ("f32", 40, 33, 331),
                                      ("f32", 4, 6, 64), ("f32", 3, 5, 1100)])
@pytest.mark.parametrize("direction", [1, -1])
def test_state_in_place(dt, T, B, n, direction):
    """hT = h0 and cT = c0; rows of length 1 begin in the last step of the reversed direction, rows of length 0 keep their state."""
    from paper_1805_05225_amd import binding as Bn
    rng = np.random.default_rng(n + T)
    lens = rng.integers(0, T + 1, B)
    lens[::3], lens[1] = 1, 0
    c = P.rnd_case(rng, T, B, 40, n, 1, lens, dt, scale=2.0 / np.sqrt(n + 40))
    x, Wx, Wh, b, ln = dev(c["x"], dt), dev(c["W_x"][0], dt), dev(c["W_h"][0], dt), dev(c["b"][0]), dev(c["lens"])
    h, cc = dev(c["h0"][0]), dev(c["c0"][0])
    s = Bn.forward(x, Wx, Wh, b, h, cc, ln, bidirectional=False, direction=direction, flags=Bn.FLAG_INFERENCE, want_c=False)
    assert not Bn.sync_status(s["workspace"])
    y, p = torch.empty_like(s["y"]), lambda t: t.data_ptr()
    assert Bn.lib.lstm_fwd(Bn.ctypes.byref(s["desc"]), p(x), p(Wx), p(Wh), p(b), p(h), p(cc), p(ln), p(y), None, p(h), p(cc), None, p(s["workspace"]),
                           Bn._stream()) == 0
    assert not Bn.sync_status(s["workspace"])
    for name, got, ref in (("y", y, s["y"]), ("hT", h, s["hT"]), ("cT", cc, s["cT"])):
        check(name, got, host(ref), TOL[dt])


@pytest.mark.parametrize("T,B,n,bidir,lengths", [(12, 48, 1000, True, None), (9, 100, 1000, False, None),
                                                 (30, 64, 1000, True, (30, 18))])      # (32 places: 48 steps, which only the forward loop takes so)
def test_rows_one_behind_the_other_in_place(T, B, n, bidir, lengths):
    """A training call with hT = h0 and cT = c0: the reversed direction's padded frames hold the state that the call began with, and the backward call,
    which may read the state entering a row from there, gets the oracle's gradients."""
    from paper_1805_05225_amd import binding as Bn
    P.Bn = Bn
    rng = np.random.default_rng(n + T)
    lens = _lens(rng, T, B) if lengths is None else np.repeat(lengths, B // 2)
    c = P.rnd_case(rng, T, B, 24, n, 2 if bidir else 1, lens, "bf16", scale=2.0 / np.sqrt(n))
    d = -1
    sq = (lambda a: a) if bidir else (lambda a: a[0])
    x, dy, Wx, Wh = dev(c["x"], "bf16"), dev(c["dy"], "bf16"), dev(sq(c["W_x"]), "bf16"), dev(sq(c["W_h"]), "bf16")
    b, h0, c0, dhT, dcT, ln = (dev(sq(c[k])) if k != "lens" else dev(c[k]) for k in ("b", "h0", "c0", "dhT", "dcT", "lens"))
    f = Bn.forward(x, Wx, Wh, b, h0, c0, ln, bidirectional=bidir, direction=d, poison=True)      # (buffers and their sizes)
    f["hT"], f["cT"] = h0.clone(), c0.clone()
    for k in ("y", "c"):
        f[k].fill_(float("nan"))
    p = lambda t: t.data_ptr()
    call = Bn.lib.blstm_fwd if bidir else Bn.lib.lstm_fwd
    assert call(Bn.ctypes.byref(f["desc"]), p(x), p(Wx), p(Wh), p(b), p(f["hT"]), p(f["cT"]), p(ln), p(f["y"]), p(f["c"]), p(f["hT"]), p(f["cT"]),
                p(f["reserve"]), p(f["workspace"]), Bn._stream()) == 0
    assert not Bn.sync_status(f["workspace"])
    g = Bn.backward(f, x, Wx, Wh, h0, c0, ln, dy, dhT, dcT)
    assert not Bn.sync_status(f["workspace"])
    P.compare(f, g, *P.run_oracle(c, bidir, d), TOL["bf16"])


# Outside the range of what the loops exchange: the result is the per-step kernels', which exchange nothing between work-groups of a launch.
@pytest.mark.parametrize("what", ["nan_x", "nan_W", "large_W", "inf_dy", "large_dy"])
@pytest.mark.parametrize("dt,T,B,n", [("bf16", 24, 9, 1040), ("bf16", 24, 33, 2048), ("f32", 24, 9, 331), ("f32", 24, 40, 200), ("f32", 16, 17, 1000), ("f32", 16, 70, 1001)])
def test_values_outside_the_exchange_range(dt, T, B, n, what):
    from paper_1805_05225_amd import binding as Bn
    P.Bn = Bn
    rng = np.random.default_rng(n)
    c = P.rnd_case(rng, T, B, 24, n, 1, None, dt, scale=2.0 / np.sqrt(n))
    if what == "nan_x":
        c["x"][1, 1, 0] = c["x"][1, 2, 3] = np.nan
    elif what == "nan_W":
        c["W_h"][0, 5, 7] = np.nan
    elif what == "large_W":
        # Pre-activations of the i, f, o gates beyond 2^33, of either sign but far from 0, where 16 bits of a share would decide the
        # gate: h and a column's weights do not change sign (g = tanh(4 + ...), c > 0).
        for k in ("h0", "c0"):
            c[k] = np.abs(c[k])
        c["b"][0, 2 * n:3 * n] += 4
        for gate in (0, 1, 3):
            cols = slice(gate * n + gate % 2, (gate + 1) * n, 3)
            c["W_h"][0, :, cols] = np.abs(c["W_h"][0, :, cols]) * 2.0 ** 44
            c["W_h"][0, :, cols][:, ::2] *= -1
    elif what == "inf_dy":
        c["dy"][2, 1, 3] = np.inf
    else:                                                 # dz and partial sums of Dh beyond 2^33 in some rows, in tagged units and others
        c["dy"][:, 1::4, 3::4] *= 2.0 ** 40
        c["dy"][:, 2::8, 1::8] *= -2.0 ** 45
    for direction in (1, -1):
        Bn.profile_enable(1)
        f, g = P.run_gpu(c, dt, False, direction)
        Bn.profile_enable(0)
        launches = Bn.profile_read()
        assert launches["loop_fwd"][1] < T and launches["loop_bwd"][1] < T       # (the loops it is about)
        fs, gs = P.run_gpu(c, dt, False, direction, flags=Bn.FLAG_PER_STEP)
        for name, got, ref in [(k, f[k], fs[k]) for k in ("y", "c", "hT", "cT")] + [(k, g[k], gs[k]) for k in ("dx", "dW_x", "dW_h", "db", "dh0", "dc0")]:
            got, ref = host(got), host(ref)
            print("  ", name, "not finite: %d" % (~np.isfinite(ref)).sum(), flush=True)
            assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(got)], ref[np.isinf(ref)]), name
            ok = np.isfinite(ref)
            # by row where there are rows: the large ones must not hide the others
            ax = -1 if name in ("dx", "dh0", "dc0", "c", "cT") else None
            size = np.abs(np.where(ok, ref, 0)).max(axis=ax, keepdims=True)
            err = np.abs(np.where(ok, got, 0) - np.where(ok, ref, 0)) / np.maximum(size, 1e-30)
            assert err.max() < TOL[dt], (name, err.max())


@pytest.mark.parametrize("what", ["ordinary", "huge_W", "huge_dy", "tiny_W"])
@pytest.mark.parametrize("T,B,n", [(24, 9, 200), (24, 17, 500), (24, 140, 500), (24, 70, 1001), (24, 12, 1024)])
def test_float_loops_in_parts(T, B, n, what):
    """Slabs of one and of two row tiles in each width: three bfloat16 parts, and the float MFMAs for what these cannot hold (weights from 2^76 on; dz from
    2^100 on); weights whose parts end below the smallest bfloat16.  Against the per-step kernels, which multiply floats; by row and column."""
    from paper_1805_05225_amd import binding as Bn
    P.Bn = Bn
    rng = np.random.default_rng(n + B)
    c = P.rnd_case(rng, T, B, 24, n, 1, _lens(rng, T, B), "f32", scale=1.0 / np.sqrt(n))
    if what == "huge_W":
        c["W_h"][0, 3::16, 5] = 1e25
        c["W_h"][0, 7, n + 9] = -1e30
    elif what == "huge_dy":
        c["dy"][:, 1::4, 3::4] *= 2.0 ** 105
    elif what == "tiny_W":
        c["W_h"][0, :, 1::2] *= 2.0 ** -120
        c["W_h"][0, 1::2, :] *= 2.0 ** -20
    Bn.profile_enable(1)
    f, g = P.run_gpu(c, "f32", False, flags=Bn.FLAG_PLAIN_LAUNCH, poison=True)
    Bn.profile_enable(0)
    launches = Bn.profile_read()
    assert launches["loop_fwd"][1] < T and launches["loop_bwd"][1] < T
    fs, gs = P.run_gpu(c, "f32", False, flags=Bn.FLAG_PER_STEP)
    for name, got, ref in [(k, f[k], fs[k]) for k in ("y", "c", "hT", "cT")] + [(k, g[k], gs[k]) for k in ("dx", "dW_x", "dW_h", "db", "dh0", "dc0")]:
        got, ref = host(got), host(ref)
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(got)], ref[np.isinf(ref)]), name
        ok = np.isfinite(ref)
        size = np.abs(np.where(ok, ref, 0)).max(axis=-1, keepdims=True)
        err = np.abs(np.where(ok, got, 0) - np.where(ok, ref, 0)) / np.maximum(size, 1e-30)
        assert err.max() < 5e-5, (name, err.max())


@pytest.mark.parametrize("B,n,bidir", [(9, 257, True), (190, 384, True), (12, 640, False), (64, 513, True), (7, 641, True), (70, 768, True), (10, 896, False), (64, 770, True),
                                       (5, 897, False)])
def test_float_loop_forms(B, n, bidir):
    """As many chunks and column tiles as the width needs, in twos: the first and last width of a form, slabs of one and of two row tiles."""
    _layer(9, B, 24, n, bidir, "f32")
    for what in ("huge_W", "huge_dy"):
        test_float_loops_in_parts(24, B, n, what)


@pytest.mark.parametrize("dy_exp,w_exp", [(-118, 60), (60, -120)])
@pytest.mark.parametrize("T,B,n", [(24, 9, 200), (24, 140, 500), (24, 12, 1024)])
def test_float_backward_loop_small_operands(T, B, n, dy_exp, w_exp):
    """Gate gradients and weights whose parts would end below the smallest bfloat16, against partners that make the product an ordinary number.  Every fourth
    unit's output gate is shut, so its row of W_h, the only one that is not zero, has no effect but on dh0: 4 n products of one step (2^-23 of their
    size, root mean square, as for a float product)."""
    from paper_1805_05225_amd import binding as Bn
    P.Bn = Bn
    rng = np.random.default_rng(n + B)
    c = P.rnd_case(rng, T, B, 24, n, 1, _lens(rng, T, B), "f32", scale=0.3)
    shut = np.arange(n) % 4 == 0
    c["b"][0, 3 * n:][shut] = -300.0
    c["W_h"][0] *= shut[:, None] * 2.0 ** w_exp
    c["h0"][0][:, shut] = 0.0
    for k in ("dy", "dhT", "dcT"):
        c[k] *= 2.0 ** dy_exp
    Bn.profile_enable(1)
    f, g = P.run_gpu(c, "f32", False, flags=Bn.FLAG_PLAIN_LAUNCH, poison=True)
    Bn.profile_enable(0)
    assert Bn.profile_read()["loop_bwd"][1] < T
    fs, gs = P.run_gpu(c, "f32", False, flags=Bn.FLAG_PER_STEP)
    live = c["lens"] > 0
    got, ref = host(g["dh0"])[live][:, shut], host(gs["dh0"])[live][:, shut]
    assert np.isfinite(ref).all() and np.abs(ref).max(axis=1).min() > 0
    err = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
    print("    dh0 err", err.max(), flush=True)
    assert err.max() < 4 * 2.0 ** -23 * (4 * n / 64) ** 0.5      # (gate gradients of either loop: another order of sums)


@pytest.mark.parametrize("T,B,n,bidir", [(150, 5, 1032, False), (64, 32, 1536, True), (90, 33, 2048, False), (40, 64, 2048, True), (33, 17, 1921, False)])
def test_wide_loops_over_many_steps(T, B, n, bidir):
    """The rings of the wide loops are used over and over: many steps, ordinary and cooperative launch, against the per-step kernels; the same
    call gives the same bits every time."""
    from paper_1805_05225_amd import binding as Bn
    P.Bn = Bn
    rng = np.random.default_rng(T + n)
    D = 2 if bidir else 1
    c = P.rnd_case(rng, T, B, 24, n, D, _lens(rng, T, B), "bf16", scale=2.0 / np.sqrt(n))
    grads = ("dx", "dW_x", "dW_h", "db", "dh0", "dc0")
    fs, gs = P.run_gpu(c, "bf16", bidir, flags=Bn.FLAG_PER_STEP)
    first = None
    for flags in (Bn.FLAG_PLAIN_LAUNCH, 0, Bn.FLAG_PLAIN_LAUNCH, Bn.FLAG_PLAIN_LAUNCH):
        Bn.profile_enable(1)
        f, g = P.run_gpu(c, "bf16", bidir, flags=flags, poison=True)
        Bn.profile_enable(0)
        launches = Bn.profile_read()
        assert launches["loop_fwd"][1] == launches["loop_bwd"][1] == 2 * D      # (a launch per step otherwise)
        got = [f[k] for k in ("y", "c", "hT", "cT")] + [g[k] for k in grads]
        if first is None:
            first = [t.clone() for t in got]
            for name, a, b in zip(("y", "c", "hT", "cT") + grads, got, [fs[k] for k in ("y", "c", "hT", "cT")] + [gs[k] for k in grads]):
                check(name, a, host(b), TOL["bf16"])
        for a, b in zip(got, first):
            assert torch.equal(a, b)


@pytest.mark.parametrize("B,n,bidir", [(64, 1032, True), (96, 1280, False), (64, 1536, True), (256, 2048, True), (3, 2048, False)])
@pytest.mark.parametrize("T", [2, 60])
def test_wide_layer_on_either_side_of_the_rule(T, B, n, bidir):
    """Forward and backward choose their loop by themselves: any pairing gives the per-step result."""
    from paper_1805_05225_amd import binding as Bn
    P.Bn = Bn
    rng = np.random.default_rng(T + B + n)
    if T * B > 4000:
        T = 9
    c = P.rnd_case(rng, T, B, 24, n, 2 if bidir else 1, _lens(rng, T, B), "bf16", scale=2.0 / np.sqrt(n))
    fs, gs = P.run_gpu(c, "bf16", bidir, flags=Bn.FLAG_PER_STEP)
    for flags in (0, Bn.FLAG_PLAIN_LAUNCH):
        f, g = P.run_gpu(c, "bf16", bidir, flags=flags, poison=True)
        for k in ("y", "c", "hT", "cT"):
            check(k, f[k], host(fs[k]), TOL["bf16"])
        for k in ("dx", "dW_x", "dW_h", "db", "dh0", "dc0"):
            check(k, g[k], host(gs[k]), TOL["bf16"])


@pytest.mark.parametrize("T,B,n,bidir,loops", [(60, 100, 1000, True, True), (100, 5, 700, False, True), (30, 20, 300, True, True), (2, 40, 300, False, False),
                                               (20, 300, 700, True, False), (9, 256, 200, True, None)])
def test_float_layer_on_either_side_of_the_rule(T, B, n, bidir, loops):
    """The single-launch loops where they pay (several launches of row tiles among them), the per-step kernels elsewhere; any lengths, against the
    per-step result (another order of the float sums)."""
    from paper_1805_05225_amd import binding as Bn
    P.Bn = Bn
    rng = np.random.default_rng(T + B + n)
    c = P.rnd_case(rng, T, B, 24, n, 2 if bidir else 1, _lens(rng, T, B), "f32", scale=1.0 / np.sqrt(n))
    fs, gs = P.run_gpu(c, "f32", bidir, flags=Bn.FLAG_PER_STEP)
    for flags in (0, Bn.FLAG_PLAIN_LAUNCH):
        Bn.profile_enable(1)
        f, g = P.run_gpu(c, "f32", bidir, flags=flags, poison=True)
        Bn.profile_enable(0)
        launches = Bn.profile_read()
        if loops is not None and not flags:       # (a plain launch costs the loops less: the rule may choose them then)
            assert launches["loop_fwd"][1] == (1 if loops else T)
        for k in ("y", "c", "hT", "cT"):
            check(k, f[k], host(fs[k]), 5e-5)
        for k in ("dx", "dW_x", "dW_h", "db", "dh0", "dc0"):
            check(k, g[k], host(gs[k]), 5e-5)


@pytest.mark.parametrize("dt,T,B,n_in,n", [("bf16", 40, 21, 123, 330), ("f32", 20, 4, 32, 64), ("f32", 30, 16, 100, 200), ("bf16", 60, 32, 40, 1024)])
def test_phase_times_name_every_product(dt, T, B, n_in, n):
    """Products that share a launch share its time, and none of them goes without."""
    from paper_1805_05225_amd import binding as Bn
    P.Bn = Bn
    rng = np.random.default_rng(n)
    c = P.rnd_case(rng, T, B, n_in, n, 2, _lens(rng, T, B), dt, scale=2.0 / np.sqrt(n))
    P.run_gpu(c, dt, True)
    total = {}
    for level in (1, 2):
        Bn.profile_enable(level)
        P.run_gpu(c, dt, True)
        Bn.profile_enable(0)
        p = Bn.profile_read()
        print("  ", {k: "%.1f us, %d" % (v[0] * 1e3, v[1]) for k, v in p.items()}, flush=True)
        assert all(p[k][0] > 0 for k in ("gemm_zx", "gemm_dx", "gemm_dwx", "gemm_dwh", "loop_fwd", "loop_bwd"))
        total[level] = sum(v[1] for k, v in p.items() if k.startswith("gemm"))
    assert total[1] == total[2]


def test_phase_times_count_the_fill_of_padded_frames():
    """Rows one behind the other: the launch that fills the padded frames is part of the forward recurrence."""
    from paper_1805_05225_amd import binding as Bn
    P.Bn = Bn
    rng = np.random.default_rng(3)
    c = P.rnd_case(rng, 12, 48, 24, 1000, 2, _lens(rng, 12, 48), "bf16", scale=2.0 / np.sqrt(1000))
    Bn.profile_enable(1)
    P.run_gpu(c, "bf16", True)
    Bn.profile_enable(0)
    assert Bn.profile_read()["loop_fwd"][1] == 2


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("n", [128, 124, 72, 62, 60, 56, 8, 4, 3])
def test_narrow_layer_widths(dt, n):
    """W_h of a narrow layer is read by 16 bytes where its rows allow it, by single elements elsewhere; one step more than inputs are asked for ahead."""
    _layer(5, 6, 24, n, True, dt)


@pytest.mark.parametrize("M,N", [(3600, 3592), (4088, 3608)])
@pytest.mark.parametrize("K", [1, 16, 17, 48, 63, 64, 65, 127, 128, 129, 250])
def test_weight_gradient_product_stages(M, N, K):
    """Products of more than 200 tiles of 256 x 256, both operands k-major: one to four stages, k-steps that are part or all past K, ragged tiles."""
    import torch
    from paper_1805_05225_amd import binding as Bn
    g = torch.Generator().manual_seed(M + K)
    A, B = torch.randn(K, M, generator=g).bfloat16().cuda(), torch.randn(K, N, generator=g).bfloat16().cuda()
    got = Bn.gemm(A, B, a_kcontig=False, b_kcontig=False, M=M, N=N, K=K)
    ref = A.double().t().contiguous() @ B.double()
    assert float((got.double() - ref).abs().max()) < 1e-5 * float(ref.abs().max())          # (exact inputs: the order of float sums)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("T", [1, 2, 3, 4, 5, 6, 7, 8, 9])
@pytest.mark.parametrize("n,B,bidir", [(64, 5, True), (100, 4, False)])
def test_narrow_layer_rounds(dt, T, n, B, bidir):
    """Narrow loops walk rounds of four steps, those past the end without effect, and store a frame's outputs a step later."""
    _layer(T, B, 16, n, bidir, dt)


@pytest.mark.parametrize("T,B,n_in,n,bidir", [(2, 1, 2, 104, True), (3, 5, 34, 200, False), (16, 1, 620, 328, True), (17, 1, 256, 1000, True), (4, 8, 94, 264, False),
                                              (11, 3, 1000, 1000, False), (8, 8, 310, 512, True), (13, 5, 288, 520, True), (16, 32, 30, 136, False), (27, 19, 64, 128, True),
                                              (9, 1, 33, 200, True), (2, 3, 40, 201, True), (40, 20, 40, 1000, True), (4, 300, 64, 200, True), (3, 40, 48, 1024, True)])
def test_projection_with_the_set_up(T, B, n_in, n, bidir):
    """Inference over few frames: row tiles of 16, 32 and 64, several of them, the last piece of a row of x reaching into the next, a last chunk of k and a last tile of
    units in part; odd n_in and n, and up to 128 units, which go other ways; more frames, where only W_h is read as it lies in memory, and several launches and
    sixteen rows a group, where it is not.  Padded frames of x hold NaN.  Against a training call, whose sums come in another order; the test below has the oracle."""
    from paper_1805_05225_amd import binding as Bn
    g = torch.Generator().manual_seed(T * B + n_in)
    D = 2 if bidir else 1
    W_x, W_h = (torch.randn(D, k, 4 * n, generator=g).mul(0.7 / k ** 0.5).bfloat16().cuda() for k in (n_in, n))
    b, h0, c0 = (torch.randn(D, *s, generator=g).cuda() for s in ((4 * n,), (B, n), (B, n)))
    lens = torch.randint(1, T + 1, (B,), generator=g, dtype=torch.int32)
    x = torch.randn(T, B, n_in, generator=g).bfloat16()
    x[torch.arange(T)[:, None] >= lens[None, :]] = float("nan")
    for state in ((None, None), (h0, c0)):
        runs = [Bn.forward(x.cuda(), W_x, W_h, b, *state, lens.cuda(), bidirectional=bidir, flags=flags) for flags in (0, Bn.FLAG_INFERENCE)]
        for what in ("y", "c", "hT", "cT"):
            want, got = (r[what].float() for r in runs)
            assert torch.isfinite(got).all() and float((got - want).norm()) <= 1e-2 * float(want.norm()), what       # (roundings of h and y that fall the other way)


@pytest.mark.parametrize("T,B,n_in,n,bidir,together", [
    (2, 1, 2, 136, True, True), (2, 3, 6, 200, True, True), (3, 1, 34, 1000, False, True),             # fewer k than a piece of a row, and one more chunk than a whole one
    (32, 16, 64, 136, True, True), (27, 19, 64, 136, True, False),                                      # 512 rows, and one more
    (40, 8, 40, 1000, True, True), (41, 8, 40, 1000, True, False), (48, 8, 44, 1000, True, True),       # five rounds of work-groups, six; six of rows that would be copied
    (24, 8, 2000, 520, True, True), (32, 8, 2000, 520, True, False), (8, 8, 4000, 520, True, True), (9, 15, 4000, 520, True, False)])      # K times rounds
def test_projection_with_the_set_up_against_the_oracle(T, B, n_in, n, bidir, together):
    """Both sides of the rule that puts the projection into the set-up launch; which side it is shows in the launches that are counted."""
    from paper_1805_05225_amd import binding as Bn
    from oracle import lstm_oracle as O
    rng = np.random.default_rng(n_in + T)
    c = P.rnd_case(rng, T, B, n_in, n, 2 if bidir else 1, _lens(rng, T, B), "bf16", scale=2.0 / np.sqrt(n + n_in))
    sq = (lambda a: a) if bidir else (lambda a: a[0])
    x, Wx, Wh, b, ln = dev(c["x"], "bf16"), dev(sq(c["W_x"]), "bf16"), dev(sq(c["W_h"]), "bf16"), dev(sq(c["b"])), dev(c["lens"])
    for state in (False, True):
        h0, c0 = (sq(c[k]) if state else None for k in ("h0", "c0"))
        Bn.profile_enable(2)
        f = Bn.forward(x, Wx, Wh, b, dev(h0), dev(c0), ln, bidirectional=bidir, flags=Bn.FLAG_INFERENCE)
        Bn.profile_enable(0)
        launches = {k: v[1] for k, v in Bn.profile_read().items()}
        assert state or (launches["prep"] == 0) == together, launches
        want = O.blstm_fwd(c["x"], c["W_x"], c["W_h"], c["b"], h0, c0, c["lens"]) if bidir else O.lstm_fwd(c["x"], sq(c["W_x"]), sq(c["W_h"]), sq(c["b"]), h0, c0, c["lens"], 1)
        for name, ref in zip(("y", "c", "hT", "cT"), want):
            check(name, f[name], ref, TOL["bf16"])


@pytest.mark.parametrize("T,B,n,bidir", [(4, 136, 1000, False), (8, 72, 1024, True), (3, 240, 520, True), (2, 824, 136, False)])
def test_inference_in_several_launches(T, B, n, bidir):
    """More rows than a launch holds: W_h is packed, as in training.  Two calls add some sums in another order (the order in which other work-groups' values
    arrive: below one in a thousand of c); W_h as it lies in memory adds all of them in another (a third of c and more)."""
    from paper_1805_05225_amd import binding as Bn
    g = torch.Generator().manual_seed(B)
    D = 2 if bidir else 1
    lead = (D,) if bidir else ()
    W_x, W_h = (torch.randn(*lead, k, 4 * n, generator=g).mul(0.7 / k ** 0.5).bfloat16().cuda() for k in (96, n))
    b, x = torch.randn(*lead, 4 * n, generator=g).cuda(), torch.randn(T, B, 96, generator=g).bfloat16().cuda()
    want, got = (Bn.forward(x, W_x, W_h, b, bidirectional=bidir, flags=flags) for flags in (0, Bn.FLAG_INFERENCE))
    # (where a last place makes an h fall to the other bfloat16 beside it, 2^-8 of 1, a gate moves by at most 2^-8 times the largest weight, 0.7 / n^0.5 times five, and c by no
    # more than twice that a step; such an h moves its row from there on, a hundredth of c)
    assert torch.isfinite(got["c"]).all() and float((got["c"] - want["c"]).abs().max()) < 2 * T * 2 ** -8 * 3.5 / n ** 0.5
    assert float((got["c"] != want["c"]).float().mean()) < 0.05


@pytest.mark.parametrize("M,N", [(1100, 136), (1153, 513), (136, 1160), (129, 128), (2400, 2440), (1040, 5560), (1640, 3072)])
@pytest.mark.parametrize("K", [8, 64, 72, 128, 184, 256, 312, 2120, 4104])
def test_product_of_few_tiles_stages(M, N, K):
    """128 x 128 tiles, all three layouts: one to five stages (the ring of two is walked by both parities), ragged last ones, more tile rows than columns (several
    bands, the last one lower; work-groups of the grid that have no tile) and fewer; 352 to 511 work-groups,
    which have less on its way from some K on, or another order where tile columns do not come in whole eights."""
    import torch
    from paper_1805_05225_amd import binding as Bn
    g = torch.Generator().manual_seed(M + K)
    A, B = torch.randn(M, K, generator=g).bfloat16().cuda(), torch.randn(K, N, generator=g).bfloat16().cuda()
    ref = A.double() @ B.double()
    forms = {"NT": (A, B.t().contiguous(), True, True)}
    if N % 8 == 0:
        forms["NN"] = (A, B, True, False)
    if M % 8 == 0 and N % 8 == 0:
        forms["TN"] = (A.t().contiguous(), B, False, False)
    for form, (a, b, ak, bk) in forms.items():
        got = Bn.gemm(a, b, a_kcontig=ak, b_kcontig=bk, M=M, N=N, K=K)
        assert float((got.double() - ref).abs().max()) < 1e-5 * float(ref.abs().max()), form          # (exact inputs: the order of float sums)


@pytest.mark.parametrize("M,N", [(4100, 4104), (2049, 8320), (3329, 7944), (2305, 14344), (104, 51464), (51300, 104), (7681, 4096), (6145, 7632), (6145, 7640)])
@pytest.mark.parametrize("K", [8, 64, 72, 128, 136, 200, 320])
def test_product_of_many_tiles_b_k_major(M, N, K):
    """B as it lies in memory: one to five stages, ragged last ones, tiles of 256 x 256 of which a row or eight columns are left; 289 and 297 of them, which tiles of
    128 x 128 take, 448, and 570, which K chooses for; a row and a column of them that would be half empty, which tiles of 128 x 128 take;
    496, 750 with rows of whole runs of 64 bytes, and not."""
    import torch
    from paper_1805_05225_amd import binding as Bn
    g = torch.Generator(device="cuda").manual_seed(M + K)
    A, B = (torch.randn(*s, generator=g, device="cuda").bfloat16() for s in ((M, K), (K, N)))
    got = Bn.gemm(A, B, a_kcontig=True, b_kcontig=False, M=M, N=N, K=K)
    ref = A.float() @ B.float()
    assert float((got - ref).abs().max()) < 2e-5 * float(ref.abs().max())          # (exact inputs: the order of float sums, twice)


@pytest.mark.parametrize("n_in", [20800, 20803])
def test_inputs_past_2_gib(n_in):
    """More than 32-bit byte offsets reach: the generic product, on W_x as the caller holds it, with whole rows of x and with padded ones; the first rows and the last."""
    from paper_1805_05225_amd import binding as Bn
    from oracle import lstm_oracle as O
    B, n, g = 52000, 2, torch.Generator(device="cuda").manual_seed(n_in)
    x = torch.randn(1, B, n_in, generator=g, device="cuda", dtype=torch.bfloat16)
    Wx, Wh = (torch.randn(k, 4 * n, generator=g, device="cuda").mul(0.7 / k ** 0.5).bfloat16() for k in (n_in, n))
    lens = torch.ones(B, dtype=torch.int32, device="cuda")
    lens[7] = 0
    f = Bn.forward(x, Wx, Wh, None, None, None, lens, bidirectional=False)
    for rows in (slice(0, 40), slice(B - 40, B)):
        want = O.lstm_fwd(host(x[:, rows]), host(Wx), host(Wh), None, None, None, lens[rows].cpu().numpy(), 1)
        check("y", f["y"][:, rows], want[0], TOL["bf16"])
        check("c", f["c"].view(1, B, n)[:, rows], want[1], TOL["bf16"])


@pytest.mark.parametrize("T,B", [(1, 16), (5, 13), (9, 16), (13, 16), (30, 16)])
def test_weight_gradients_over_listed_frames(T, B):
    """The same product walking the list of real frames: fewer than a stage, one, and several."""
    _layer(T, B, 2048, 1024, True, "bf16")


@pytest.mark.parametrize("n,n_in", [(1024, 1024), (1000, 40), (512, 72)])
def test_weight_gradients_in_ranges_of_frames(n, n_in):
    """Few tiles and many frames: K ranges on the 256 x 256 kernel (for n = 512 four of them), of real frames that end inside one.  Rows do not interact, so the weight
    gradients are the sums of those of four quarters, which are too short for ranges; a value in bfloat16 may round the other way."""
    import torch
    from paper_1805_05225_amd import binding as Bn
    T, B = 840, 32
    g = torch.Generator(device="cuda").manual_seed(n)
    rnd = lambda *shape: torch.randn(*shape, generator=g, device="cuda")
    x, dy = rnd(T, B, n_in).bfloat16(), rnd(T, B, 2 * n).bfloat16()
    W_x, W_h = (0.5 / n_in ** 0.5 * rnd(2, n_in, 4 * n)).bfloat16(), (0.5 / n ** 0.5 * rnd(2, n, 4 * n)).bfloat16()
    lens = torch.randint(T // 2, T + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    lens[0] = T

    def grads(rows):
        xs, dys, ls = x[:, rows].contiguous(), dy[:, rows].contiguous(), lens[rows].contiguous()
        f = Bn.forward(xs, W_x, W_h, None, None, None, ls, bidirectional=True)
        r = Bn.backward(f, xs, W_x, W_h, None, None, ls, dys)
        assert not Bn.sync_status(f["workspace"])
        return r
    whole, lo, hi = grads(slice(0, B)), grads(slice(0, B // 4)), grads(slice(B // 4, B // 2))
    hi2, hi3 = grads(slice(B // 2, 3 * B // 4)), grads(slice(3 * B // 4, B))
    for k in ("dW_x", "dW_h"):
        ref = lo[k].double() + hi[k].double() + hi2[k].double() + hi3[k].double()
        assert float((whole[k].double() - ref).norm() / ref.norm()) < 2e-3, k

"""The kernels for a handful of rows (stepped cell, readout, plain product) at the row counts where the dispatch changes kernel and
at column counts and pieces that end inside a tile or a chunk, against float64 products of the same bfloat16 values."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import decoder_oracle as D
from oracle import lstm_oracle as O
from tests.gpu_util import check, dev

TOL = 2e-2


def _bf(rng, *shape, w=1.0):
    return torch.from_numpy(rng.uniform(-w, w, shape)).to(torch.bfloat16)


@pytest.mark.parametrize("B,n_in,n", [(1, 37, 50), (16, 300, 104), (17, 300, 104), (32, 1100, 36), (33, 40, 1000), (64, 2620, 130),
                                      (65, 77, 34), (192, 1200, 66), (193, 1200, 66), (12, 4100, 24), (1025, 300, 104), (1300, 77, 34),
                                      # every tile of gemm_skinny.hip, rows and units that end inside one: 96 x 128 (twice), 128 x 128, 64 x 128, 96 x 64, 64 x 64
                                      (767, 40, 1000), (765, 64, 1021), (1001, 40, 1000), (500, 40, 700), (333, 100, 901), (640, 300, 512), (257, 64, 330), (1024, 8, 250),
                                      (64, 40, 1000), (66, 40, 1000), (129, 40, 481), (130, 40, 480), (200, 32, 504),
                                      (1, 37, 51), (16, 300, 105), (17, 301, 107), (64, 40, 131), (193, 33, 67), (500, 41, 701), (1030, 45, 203)])   # odd widths; either side of few_cell_pays; 32 x 64
def test_stepped_cell(B, n_in, n):
    from paper_1805_05225_amd import binding as Bn
    rng = np.random.default_rng(B + n_in)
    Wx, Wh = _bf(rng, n_in, 4 * n, w=0.1), _bf(rng, n, 4 * n, w=0.1)
    b, h, c = rng.uniform(-.1, .1, 4 * n), rng.uniform(-1, 1, (B, n)), rng.standard_normal((B, n))
    x = _bf(rng, 1, B, n_in)
    f64 = lambda t: t.float().numpy().astype(np.float64)
    ws = None
    for flags in (Bn.FLAG_INFERENCE, Bn.FLAG_INFERENCE | Bn.FLAG_WEIGHTS_PACKED):
        s = Bn.forward(x.cuda(), Wx.cuda(), Wh.cuda(), dev(b), dev(h), dev(c), None, bidirectional=False, flags=flags, workspace=ws)
        ws = s["workspace"]
        y, _, ho, co = O.lstm_fwd(f64(x), f64(Wx), f64(Wh), b, h, c, None, 1)
        torch.cuda.synchronize()
        check("y", s["y"], y, TOL)
        check("hT", s["hT"], ho, TOL)
        check("cT", s["cT"], co, TOL)


@pytest.mark.parametrize("B,n_in,n", [(1, 30, 1021), (16, 300, 1024), (16, 40, 1028), (17, 40, 720), (64, 77, 724), (193, 40, 201), (368, 64, 560), (361, 150, 552), (835, 58, 520), (1024, 9, 333)])
def test_stepped_cell_of_both_directions(B, n_in, n):
    """One launch steps both directions: either side of few_cell_pays for 16 rows and more, and tiles chosen for the rounds of both."""
    from paper_1805_05225_amd import binding as Bn
    rng = np.random.default_rng(B + n)
    Wx, Wh = _bf(rng, 2, n_in, 4 * n, w=0.1), _bf(rng, 2, n, 4 * n, w=0.1)
    b, h, c = rng.uniform(-.1, .1, (2, 4 * n)), rng.uniform(-1, 1, (2, B, n)), rng.standard_normal((2, B, n))
    x = _bf(rng, 1, B, n_in)
    lens = (np.arange(B) % 7 > 0).astype(np.int32)           # (a row without a frame keeps its state)
    f64 = lambda t: t.float().numpy().astype(np.float64)
    y, _, ho, co = O.blstm_fwd(f64(x), f64(Wx), f64(Wh), b, h, c, lens)
    ws = None
    for flags in (Bn.FLAG_INFERENCE, Bn.FLAG_INFERENCE | Bn.FLAG_WEIGHTS_PACKED):
        s = Bn.forward(x.cuda(), Wx.cuda(), Wh.cuda(), dev(b), dev(h), dev(c), dev(lens), bidirectional=True, flags=flags, workspace=ws)
        ws = s["workspace"]
        torch.cuda.synchronize()
        check("y", s["y"], y, TOL)
        check("hT", s["hT"], ho, TOL)
        check("cT", s["cT"], co, TOL)


@pytest.mark.parametrize("B,n,bidir", [(12, 40, False), (12, 41, True), (64, 40, True), (64, 41, False), (300, 200, False), (300, 201, True), (1300, 34, True), (1300, 35, False)])
def test_stepped_cell_clears_the_status(B, n, bidir):
    """A workspace on record for a wait that expired: one step, in every kernel that takes one, clears the record, weights kept or not."""
    from paper_1805_05225_amd import binding as Bn
    g = torch.Generator(device="cuda").manual_seed(n)
    r = lambda *s: (torch.randn(*s, generator=g, device="cuda") * 0.1).bfloat16()
    D = 2 if bidir else 1
    x, Wx, Wh = r(1, B, 24), r(*(D, 24, 4 * n)[2 - D:]), r(*(D, n, 4 * n)[2 - D:])
    ws = None
    for flags in (Bn.FLAG_INFERENCE, Bn.FLAG_INFERENCE, Bn.FLAG_INFERENCE | Bn.FLAG_WEIGHTS_PACKED):
        if ws is not None:
            ws[:512].fill_(1)                                # (the word, at the first 256 bytes' boundary)
            assert Bn.sync_status(ws)
        ws = Bn.forward(x, Wx, Wh, bidirectional=bidir, flags=flags, want_c=False, workspace=ws)["workspace"]
        assert not Bn.sync_status(ws)


@pytest.mark.parametrize("n,nt,E,R", [(104, 62, 130, 20), (1000, 620, 2000, 1000), (5, 3, 8, 33), (104, 62, 130, 4001), (104, 62, 106, 31), (24, 16, 24, 2050)])
def test_readout_packed_once_for_any_row_count(n, nt, E, R):
    """FLAG_WEIGHTS_PACKED speaks of the weights and the workspace, not of the number of rows."""
    from paper_1805_05225_amd import binding as Bn
    rng = np.random.default_rng(n)
    W, br = _bf(rng, R, n + nt + E, w=0.1), rng.uniform(-.1, .1, R)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    for k, B in enumerate((300, 1, 16, 17, 64, 192, 193, 1024, 1025, 1300)):
        s, t, a = _bf(rng, B, n), _bf(rng, B, nt), _bf(rng, B, E)
        out = Bn.readout(s.cuda(), t.cuda(), a.cuda(), W.cuda(), dev(br), workspace=ws, flags=Bn.FLAG_WEIGHTS_PACKED if k else 0)
        f64 = lambda v: v.float().numpy().astype(np.float64)
        torch.cuda.synchronize()
        check("readout B=%d" % B, out, D.readout(f64(s), f64(t), f64(a), f64(W).T, br), 5e-3)


@pytest.mark.parametrize("M,N,K", [(1, 20001, 1000), (16, 4097, 72), (17, 33, 2048), (32, 1000, 1000), (33, 1000, 1000),
                                   # gemm_skinny.hip: 64 x 128, 128 x 128 (one row of tiles, several), 64 x 64, 96 x 128, more work-groups than the device holds at once
                                   (200, 8000, 4000), (104, 22051, 96), (1000, 3001, 200), (193, 33, 608), (350, 6000, 1000), (130, 16500, 264), (1024, 7169, 8),
                                   # 32 x 64; either side of few_rows_pay
                                   (64, 1000, 1000), (130, 2001, 72), (17, 8193, 896), (17, 8200, 904), (32, 8192, 40), (32, 24577, 904)])
def test_product(M, N, K):
    from paper_1805_05225_amd import binding as Bn
    rng = np.random.default_rng(M + N)
    A, B, bias = _bf(rng, M, K), _bf(rng, N, K), rng.uniform(-1, 1, N)
    C = Bn.gemm(A.cuda(), B.cuda(), a_kcontig=True, b_kcontig=True, M=M, N=N, K=K, bias=dev(bias))
    torch.cuda.synchronize()
    check("C", C, A.double().numpy() @ B.double().numpy().T + bias, 1e-4)


@pytest.mark.parametrize("M,N,K", [(65, 31001, 272), (224, 20000, 448), (385, 14002, 268), (480, 20000, 800), (300, 5000, 800), (900, 5001, 104), (1024, 16001, 60), (1024, 3000, 2000)])
def test_product_on_each_side_of_the_route(M, N, K):
    """64 rows and up: few-rows tiles, 128 x 128 or 256 x 256, whichever is expected to end first; float and bfloat16 results."""
    from paper_1805_05225_amd import binding as Bn
    test_product(M, N, K)
    g = torch.Generator(device="cuda").manual_seed(M)
    A, B = (torch.randn(r, K, generator=g, device="cuda").bfloat16() for r in (M, N))
    C = Bn.gemm(A, B, a_kcontig=True, b_kcontig=True, M=M, N=N, K=K, out_dtype=torch.bfloat16)
    want = A.double() @ B.double().T
    assert ((C.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-4 * K ** 0.5).all()


@pytest.mark.parametrize("M,N,K,gap,at", [(1, 20, 8, 0, 0), (7, 401, 9, 0, 1), (16, 1000, 334, 0, 0), (17, 401, 333, 2, 3), (32, 2787, 505, 0, 0), (33, 700, 510, 4, 2), (64, 1000, 1003, 1, 1),
                                          (65, 263, 1012, 0, 0), (192, 700, 31, 0, 0), (4, 8000, 612, 0, 0), (12, 50, 1025, 1, 0), (16, 33, 2046, 3, 1), (16, 33, 2051, 0, 0), (24, 40, 1999, 0, 1),
                                          (40, 70, 4001, 0, 0), (17, 300, 1027, 0, 0), (32, 61, 4099, 2, 1), (33, 300, 1050, 0, 1), (64, 60, 2049, 1, 0), (300, 257, 130, 8, 5), (768, 1000, 334, 0, 0), (1000, 1000, 701, 0, 0)])
def test_product_of_rows_at_any_element(M, N, K, gap, at):
    """Rows of any length, distance and first element, either side of few_any_ok; what lies between and around the rows is NaN and takes no part."""
    from paper_1805_05225_amd import binding as Bn
    rng = np.random.default_rng(M + N + K)

    def rows(count):
        v, ld = _bf(rng, count, K), K + gap
        flat = torch.full((at + count * ld + 16,), float("nan"), dtype=torch.bfloat16)
        flat[at:at + count * ld].view(count, ld)[:, :K] = v
        return v.double().numpy(), flat.cuda()
    (a, A), (b, B), bias = rows(M), rows(N), rng.uniform(-1, 1, N)
    bias_d, want = dev(bias), a @ b.T + bias
    for out in (torch.float32, torch.bfloat16):
        C = torch.full((M, N + 1), 7., dtype=out, device="cuda")
        assert Bn.lib.lstm_gemm(1, out == torch.bfloat16, 1, 1, M, N, K, A.data_ptr() + 2 * at, K + gap, B.data_ptr() + 2 * at, K + gap, C.data_ptr(), N + 1,
                                bias_d.data_ptr(), 0, None, 1, 0, Bn._stream()) == 0
        torch.cuda.synchronize()
        check("C", C[:, :N].contiguous(), want, 1e-4 if out == torch.float32 else 5e-3)
        assert (C[:, N] == 7.).all()


@pytest.mark.parametrize("ak,bk", [(1, 1), (1, 0), (0, 0)])
@pytest.mark.parametrize("M,N,K", [(129, 4, 12), (260, 8, 68), (1684, 16, 76), (2004, 32, 96), (3000, 12, 100), (129, 36, 20), (128, 4, 20), (8104, 24, 20)])
def test_product_of_a_handful_of_columns(M, N, K, ak, bk):
    """Results in bfloat16, rows of whole 8 bytes but not 16, either side of narrow_result; what lies between the rows is NaN."""
    from paper_1805_05225_amd import binding as Bn
    g = torch.Generator(device="cuda").manual_seed(M + N + K)

    def rows(r, k):
        ld = k + (4 if k % 8 == 0 else 8)
        return torch.cat([torch.randn(r, k, generator=g, device="cuda"), torch.full((r, ld - k), float("nan"), device="cuda")], 1).bfloat16()
    A, B = rows(M, K) if ak else rows(K, M), rows(N, K) if bk else rows(K, N)
    a, b = (A[:, :K] if ak else A[:, :M].T).double(), (B[:, :K].T if bk else B[:, :N]).double()
    C = torch.full((M, N + 1), 7., dtype=torch.bfloat16, device="cuda")
    assert Bn.lib.lstm_gemm(1, 1, ak, bk, M, N, K, A.data_ptr(), A.shape[1], B.data_ptr(), B.shape[1], C.data_ptr(), N + 1, None, 0, None, 1, 0, Bn._stream()) == 0
    want = a @ b
    # (K sums of float, then rounded once)
    assert ((C[:, :N].double() - want).abs() <= K * 2.0 ** -24 * (a.abs() @ b.abs()) + 2.0 ** -8 * want.abs()).all() and (C[:, N] == 7.).all()


@pytest.mark.parametrize("dt,bk", [(torch.bfloat16, 1), (torch.bfloat16, 0), (torch.float32, 1), (torch.float32, 0)])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (1, 300, 2), (17, 5, 3), (64, 1000, 1), (255, 1025, 3), (2037, 515, 2), (4100, 257, 1), (70001, 17, 3),
                                   (3, 1000001, 1), (9, 300001, 3), (2113, 1025, 3), (250001, 9, 1)])
def test_product_of_less_than_a_chunk(M, N, K, dt, bk):
    """K below 16 bytes of a k-contiguous A; an element a thread, then tiles of 16 to 256 columns with one, four and sixteen rows a thread, remainders of both; what lies behind the rows is NaN."""
    from paper_1805_05225_amd import binding as Bn
    K += 4 if dt == torch.bfloat16 and N % 2 else 0
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    rows = lambda r, k: torch.cat([torch.randn(r, k, generator=g, device="cuda"), torch.full((r, 1), float("nan"), device="cuda")], 1).to(dt)
    A, B, bias = rows(M, K), rows(N, K) if bk else rows(K, N), torch.randn(N, generator=g, device="cuda")
    a, b = A[:, :K].double(), (B[:, :K].T if bk else B[:, :N]).double()
    for out, acc in ((torch.float32, 0), (torch.float32, 1)) + (((torch.bfloat16, 0),) if dt == torch.bfloat16 else ()):
        C = torch.full((M, N + 1), 7., dtype=out, device="cuda")
        assert Bn.lib.lstm_gemm(dt == torch.bfloat16, out == torch.bfloat16, 1, bk, M, N, K, A.data_ptr(), K + 1, B.data_ptr(), (K if bk else N) + 1, C.data_ptr(), N + 1,
                                bias.data_ptr(), acc, None, 1, 0, Bn._stream()) == 0
        want = a @ b + bias + (7. if acc else 0.)
        # (at most seven products, the bias and what was there: eight sums of float; a result in bfloat16 is rounded once more)
        bound = 9 * 2.0 ** -24 * (a.abs() @ b.abs() + bias.abs() + (7. if acc else 0.)) + (2.0 ** -8 * want.abs() if out == torch.bfloat16 else 0.)
        assert ((C[:, :N].double() - want).abs() <= bound).all() and (C[:, N] == 7.).all()


def test_product_of_less_than_a_chunk_over_more_than_2_to_32_elements():
    from paper_1805_05225_amd import binding as Bn
    M, N, K = 65600, 65552, 4
    g = torch.Generator(device="cuda").manual_seed(1)
    A, B = (torch.randn(r, K, generator=g, device="cuda").bfloat16() for r in (M, N))
    C = Bn.gemm(A, B, a_kcontig=True, b_kcontig=True, M=M, N=N, K=K, out_dtype=torch.bfloat16)
    for m0 in (0, 32768, M - 64):
        want = A[m0:m0 + 64].double() @ B.double().T
        assert ((C[m0:m0 + 64].double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-6).all()


@pytest.mark.parametrize("B,n_in,n", [(1, 64, 64), (12, 2620, 1000), (16, 300, 104), (17, 300, 104), (193, 64, 66)])
def test_stepped_cell_in_place(B, n_in, n):
    """hT = h0 and cT = c0: every work-group needs all of h, so none may store its part before the others have read it."""
    from paper_1805_05225_amd import binding as Bn
    rng = np.random.default_rng(B + n)
    Wx, Wh, x = _bf(rng, n_in, 4 * n, w=0.1).cuda(), _bf(rng, n, 4 * n, w=0.1).cuda(), _bf(rng, 1, B, n_in).cuda()
    b, h, c = dev(rng.uniform(-.1, .1, 4 * n)), dev(rng.uniform(-1, 1, (B, n))), dev(rng.standard_normal((B, n)))
    lens = torch.ones(B, dtype=torch.int32, device="cuda")
    lens[B // 2] = 0                                         # this row keeps its state
    for step in range(6):                                    # (the weights stay packed, the state moves on)
        s = Bn.forward(x, Wx, Wh, b, h, c, lens, bidirectional=False, flags=Bn.FLAG_INFERENCE, want_c=False)
        d = Bn.make_desc(1, B, n_in, n, Bn.LSTM_BF16_F32STATE, 1, Bn.FLAG_INFERENCE)
        d.workspace_bytes = s["workspace"].numel()
        y = torch.empty_like(s["y"])
        p = lambda t: t.data_ptr()
        assert Bn.lib.lstm_fwd(Bn.ctypes.byref(d), p(x), p(Wx), p(Wh), p(b), p(h), p(c), p(lens), p(y), None, p(h), p(c), None, p(s["workspace"]),
                               Bn._stream()) == 0
        torch.cuda.synchronize()
        # (in place K is summed in another order for up to 16 rows: float sums of bf16 products, y may round the other way: one unit in 8 bits)
        check("hT", h, s["hT"].double().cpu().numpy(), 1e-5)
        check("cT", c, s["cT"].double().cpu().numpy(), 1e-5)
        check("y", y, s["y"].double().cpu().numpy(), 2 ** -7)


@pytest.mark.parametrize("B", [1, 12, 16, 17])
def test_readout_over_its_inputs(B):
    from paper_1805_05225_amd import binding as Bn
    rng = np.random.default_rng(B)
    n, nt, E = 200, 62, 136
    W, br = _bf(rng, n, n + nt + E, w=0.1).cuda(), dev(rng.uniform(-.1, .1, n))
    wide = _bf(rng, B, n + nt + E).cuda()                    # s | trg | att, one row after the other
    s, trg, att = wide[:, :n], wide[:, n:n + nt], wide[:, n + nt:]
    want = Bn.readout(s, trg, att, W, br)
    Bn.readout(s, trg, att, W, br, out=s)                    # the result where s was
    torch.cuda.synchronize()
    check("readout", s, want.double().cpu().numpy(), 2 ** -7)

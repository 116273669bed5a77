"""The work that a user of this library has it do, as measurable cases.

Five kinds, all through paper_1805_05225_amd.binding:

  train     one training pass through a stack of (B)LSTM layers: forward and backward, optionally with max-pooling in time
            behind the lower layers (speech) and one bidirectional layer below unidirectional ones (mixed);
  stateful  the same for unidirectional layers whose state is carried from one piece of text to the next (no padding);
  encode    forward only: what an encoder does before a search;
  decode    one decoder step of a search: cell, attention, readout, for all hypotheses;
  choose    the other half of the search step: output layer, choice of the best hypotheses, their state, their embeddings.

Lengths are spread evenly over [len_lo, len_hi] and dealt to the rows at random, so the number of real frames belongs to the
case and not to the seed.  Padded frames hold noise, as in a batch that was assembled from longer buffers.
"""
import math
import random

import torch

from paper_1805_05225_amd import binding as lstm

BF16, F32 = "bf16", "f32"


# ------------------------------------------------------------------------------------------------ cases

def train(name, dtype, stack, layers, n_in, n, B, len_lo, len_hi, pooled=0, owns_device=True):
    """stack: "lstm", "blstm" or "mixed" (first layer bidirectional, the others forward in time); pooled: this many of the lower
    layers are followed by a maximum over pairs of frames; owns_device: a training process, alone on its GPU, says so."""
    return dict(name=name, kind="train", dtype=dtype, stack=stack, layers=layers, n_in=n_in, n=n, B=B, len_lo=len_lo, len_hi=len_hi,
                pooled=pooled, owns_device=owns_device)


def listed():
    return [
        # the smallest training call there is: one narrow float layer on four short rows (configuration 1); launches and host work
        train("narrow-f32-train", F32, "lstm", 1, 32, 64, 4, 20, 20, owns_device=False),
        # float storage at the paper's layer size (configuration 2): embedding 620, 1000 units per direction, 64 sentences
        train("blstm-f32-train", F32, "blstm", 1, 620, 1000, 64, 10, 50),
        # the translation encoder, six bidirectional layers (configuration 3)
        train("translation-train", BF16, "blstm", 6, 620, 1000, 64, 20, 80),
        # the headline: the speech encoder on long utterances (configuration 4), the largest case
        train("speech-train", BF16, "blstm", 6, 40, 1024, 32, 200, 1500),
        # the attention model's speech encoder: the input shortened by 8 between the lower layers (configuration 6)
        train("speech-pooled-train", BF16, "blstm", 6, 40, 1024, 32, 200, 1500, pooled=3),
        # sizes nobody rounded: feature, unit and row counts that are multiples of nothing convenient, rows of length 1
        train("ragged-train", BF16, "blstm", 2, 123, 330, 21, 1, 97, owns_device=False),
        # a wide unidirectional network over running text, state carried between the pieces
        dict(name="wide-stateful-train", kind="stateful", dtype=BF16, layers=2, n_in=620, n=2048, B=32, T=35),
        # one sentence arrives and is encoded (six bidirectional layers): nothing but latency
        dict(name="encode-one", kind="encode", dtype=BF16, stack="blstm", layers=6, n_in=620, n=1000, B=1, len_lo=27, len_hi=27),
        # a batch of 50 sentences is encoded before its search: one bidirectional layer below five unidirectional ones
        dict(name="encode-batch", kind="encode", dtype=BF16, stack="mixed", layers=6, n_in=620, n=1000, B=50, len_lo=5, len_hi=60),
        # decoder step for one sentence, beam 12
        dict(name="decode-one", kind="decode", Q=1, beam=12, S=27, n=1000, n_trg=620, E=2000, A=1000, R=1000),
        # decoder step for 64 sentences, beam 12 (configuration 8)
        dict(name="decode-batch", kind="decode", Q=64, beam=12, S=60, n=1000, n_trg=620, E=2000, A=1000, R=1000),
        # output layer over 20000 labels, choice, gather and embedding for the same batch (the rest of configuration 9)
        dict(name="choose-batch", kind="choose", Q=64, beam=12, S=60, n=1000, n_trg=620, E=2000, R=1000, V=20000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _units(rng, lo, hi):
    """A layer width: most people take multiples of 8, some take what comes."""
    v = _log(rng, lo, hi)
    return max(lo, v // 8 * 8) if rng.random() < 0.75 else v


def _seconds(c):
    """A rough upper estimate of a training pass, for keeping drawn cases within the largest listed one."""
    steps = c["layers"] * (c["T"] if c["kind"] == "stateful" else c["len_hi"])
    ragged = c["n"] % 8 != 0
    rate = 4e14 if c["dtype"] == BF16 and not ragged else 5e13
    step = 4e-6 if c["dtype"] == BF16 and not ragged and c["n"] <= 1024 else 60e-6
    return steps * step + work(c)["flops"] / rate


def draw(rng):
    kind = rng.choice(["train", "train", "train", "stateful", "encode", "decode", "choose"])
    if kind in ("train", "encode"):
        c = dict(kind=kind, dtype=rng.choice([BF16, BF16, F32]), stack=rng.choice(["lstm", "blstm", "blstm", "mixed"]),
                 layers=rng.randint(1, 6), n_in=_log(rng, 24, 1024), n=_units(rng, 64, 1024), B=_log(rng, 1, 64),
                 len_lo=1, len_hi=_log(rng, 8, 1500 if kind == "train" else 200))
        if kind == "train":
            c.update(pooled=rng.choice([0, 0, 1, 3]), owns_device=rng.random() < 0.5)
            while _seconds(c) > 0.03:
                c["len_hi"] = max(8, c["len_hi"] * 3 // 4)
                if c["len_hi"] == 8:
                    c["layers"] = max(1, c["layers"] - 1)
            c["pooled"] = min(c["pooled"], c["layers"] - 1)
        c["len_lo"] = max(1, int(c["len_hi"] * rng.uniform(0.05, 1.0)))
        return c
    if kind == "stateful":
        c = dict(kind=kind, dtype=rng.choice([BF16, BF16, F32]), layers=rng.randint(1, 3), n_in=_log(rng, 64, 1024),
                 n=_units(rng, 256, 2048), B=_log(rng, 8, 64), T=_log(rng, 16, 128))
        while _seconds(c) > 0.03 and c["T"] > 8:
            c["T"] = c["T"] * 3 // 4
        return c
    c = dict(kind=kind, Q=_log(rng, 1, 64), beam=rng.randint(4, 16), S=_log(rng, 5, 120), n=_units(rng, 256, 1024),
             n_trg=2 * _units(rng, 64, 320), E=2 * _units(rng, 256, 1024), R=_units(rng, 256, 1024))
    c.update(dict(A=_units(rng, 256, 1024)) if kind == "decode" else dict(V=_log(rng, 1000, 32000)))
    return c


# ------------------------------------------------------------------------------------------------ inputs

class Draws:
    """Random tensors on the GPU from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        self.rng = random.Random(seed)

    def normal(self, *shape, dtype=torch.float32):
        return torch.randn(*shape, generator=self.g, device="cuda").to(dtype)

    def uniform(self, w, *shape, dtype=torch.float32):
        return ((torch.rand(*shape, generator=self.g, device="cuda") * 2 - 1) * w).to(dtype)

    def lengths(self, lo, hi, count):
        lens = _lengths(lo, hi, count)
        self.rng.shuffle(lens)
        return torch.tensor(lens, dtype=torch.int32, device="cuda")

    def layer(self, D, n_in, n, dtype):
        """Weights of a layer with D directions as the calls take them: (W_x, W_h, b), without the leading axis if D = 1."""
        w = min(0.3, 2.5 / math.sqrt(n))
        W_x, W_h, b = self.uniform(w, D, n_in, 4 * n, dtype=dtype), self.uniform(w, D, n, 4 * n, dtype=dtype), self.uniform(0.1, D, 4 * n)
        return (W_x, W_h, b) if D == 2 else (W_x[0].contiguous(), W_h[0].contiguous(), b[0].contiguous())


def _lengths(lo, hi, count):
    return [hi] if count == 1 else [lo + round((hi - lo) * k / (count - 1)) for k in range(count)]


def _directions(c):
    return {"lstm": [1], "blstm": [2], "mixed": [2]}[c["stack"]] + [2 if c["stack"] == "blstm" else 1] * (c["layers"] - 1)


def _layer_inputs(c):
    """Input width of every layer."""
    ds = _directions(c) if "stack" in c else [1] * c["layers"]
    return [c["n_in"]] + [d * c["n"] for d in ds[:-1]]


def _storage(c):
    return torch.bfloat16 if c["dtype"] == BF16 else torch.float32


def _flags(c):
    return lstm.FLAG_PLAIN_LAUNCH if c.get("owns_device") else 0


def _workspace(c, directions, T, B, flags):
    """One workspace for every layer of a stack: the calls of a stack follow each other."""
    dt = lstm.LSTM_BF16_F32STATE if c["dtype"] == BF16 else lstm.LSTM_F32
    need = [lstm.query(lstm.make_desc(T, B, k, c["n"], dt, 1, flags), d == 2)[1] for k, d in zip(_layer_inputs(c), directions)]
    return torch.empty(max(need), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    r, c = Draws(seed), case
    s = dict(case=case, kind=c["kind"])
    if c["kind"] in ("train", "encode", "stateful"):
        dt, B = _storage(c), c["B"]
        T = c["T"] if c["kind"] == "stateful" else c["len_hi"]
        ds = [1] * c["layers"] if c["kind"] == "stateful" else _directions(c)
        s["flags"] = lstm.FLAG_INFERENCE if c["kind"] == "encode" else _flags(c)
        s["lens"] = None if c["kind"] == "stateful" else r.lengths(c["len_lo"], c["len_hi"], B)
        s["x"] = r.normal(T, B, c["n_in"], dtype=dt)
        s["layers"] = [r.layer(d, k, c["n"], dt) for d, k in zip(ds, _layer_inputs(c))]
        s["directions"] = ds
        s["workspace"] = _workspace(c, ds, T, B, s["flags"])
        if c["kind"] != "encode":
            Tp = T
            for _ in range(c.get("pooled", 0)):
                Tp = -(-Tp // 2)
            s["dy"] = r.normal(Tp, B, ds[-1] * c["n"], dtype=dt)
        if c["kind"] == "stateful":      # the state the previous piece of text ended with
            s["h0"] = [r.uniform(0.7, B, c["n"]) for _ in ds]
            s["c0"] = [r.normal(B, c["n"]) for _ in ds]
        return s
    Q, beam, n, nt, E, R, S, bf = c["Q"], c["beam"], c["n"], c["n_trg"], c["E"], c["R"], c["S"], torch.bfloat16
    B = Q * beam
    s["h"], s["c"], s["xin"] = r.uniform(0.7, B, n), r.normal(B, n), torch.cat([r.normal(B, nt), r.uniform(0.7, B, E)], 1).to(bf)
    s["xin_next"] = torch.zeros(B, nt + E, dtype=bf, device="cuda")     # trg | att of the next step's cell input
    if c["kind"] == "decode":
        A = c["A"]
        s["src_lens"] = r.lengths(max(1, S // 3), S, Q)
        s["enc"], s["enc_ctx"] = r.uniform(0.7, S, Q, E, dtype=bf), r.normal(S, Q, A, dtype=bf)
        # attention weights handed out so far: zero at padded positions
        s["accum"] = r.uniform(0.5, B, S).abs() * (torch.arange(S, device="cuda")[None] < s["src_lens"].repeat_interleave(beam)[:, None])
        s["cell"] = r.layer(1, nt + E, n, bf)
        s["att"] = (r.uniform(0.08, A, n, dtype=bf), r.uniform(0.1, A), r.uniform(0.5, A), r.uniform(0.1, A), r.uniform(0.3, A), 0.1)
        s["readout"] = (r.uniform(0.05, R, n + nt + E, dtype=bf), r.uniform(0.1, R))
        # the search has been going on: the cell's and the readout's packed weights are in their workspaces
        s["cell_ws"] = lstm.forward(s["xin"].view(1, B, nt + E), *s["cell"], s["h"], s["c"], None, bidirectional=False,
                                    flags=lstm.FLAG_INFERENCE, want_c=False)["workspace"]
        s["att_ws"] = torch.empty(lstm.attention_query(S, Q, beam, A, E, n).workspace_bytes, dtype=torch.uint8, device="cuda")
        rq = lstm.ctypes.c_uint64(0)
        assert lstm.lib.lstm_readout_query(B, R, n, nt, E, lstm.ctypes.byref(rq)) == 0
        s["readout_ws"] = torch.empty(rq.value, dtype=torch.uint8, device="cuda")
        lstm.readout(s["h"].to(bf), s["xin"][:, :nt], s["xin"][:, nt:], *s["readout"], workspace=s["readout_ws"])
    else:
        V = c["V"]
        # Readout and output weights lie on a coarse grid (6 bits each): every logit is then an exact float whatever the order
        # of summation, and the choice between close candidates does not hang on it.
        s["ro"] = (r.normal(B, R).clamp(-3, 3) * 16).round().div(16).relu().to(bf)
        s["W_o"] = (r.uniform(0.2, V, R) * 256).round().div(256).to(bf)
        s["b_o"] = (r.normal(V) * 256).round().div(256)
        s["score"] = (-4.0 - 2.0 * r.uniform(1.0, Q, beam).abs()).sort(1, descending=True).values
        s["accum"] = r.uniform(0.5, B, S).abs()
        s["att_now"] = r.uniform(0.7, B, E, dtype=bf)
        s["W_trg"] = r.normal(V, nt, dtype=bf)
        need = lstm.ctypes.c_uint64(0)
        assert lstm.lib.lstm_beam_query(Q, beam, V, lstm.ctypes.byref(need)) == 0
        s["beam_ws"] = torch.empty(need.value, dtype=torch.uint8, device="cuda")
        s["next"] = [torch.empty_like(s["h"]), torch.empty_like(s["c"]), torch.empty_like(s["accum"]), s["xin_next"][:, nt:]]
    return s


# ------------------------------------------------------------------------------------------------ one pass

def _train(s):
    pooled = s["case"].get("pooled", 0)
    carried = "h0" in s
    cur, lens, saved, out = s["x"], s["lens"], [], {}
    for k, ((W_x, W_h, b), d) in enumerate(zip(s["layers"], s["directions"])):
        h0, c0 = (s["h0"][k], s["c0"][k]) if carried else (None, None)
        f = lstm.forward(cur, W_x, W_h, b, h0, c0, lens, bidirectional=d == 2, flags=s["flags"], workspace=s["workspace"],
                         want_state=carried)
        saved.append((f, cur, lens, None))
        if carried:
            out["hT%d" % k], out["cT%d" % k] = f["hT"], f["cT"]
        cur = f["y"]
        if k < pooled:
            T = cur.shape[0]
            p = lstm.time_pool_fwd(cur, lens, 2)
            saved[-1] = (f, saved[-1][1], lens, (p["arg"], T))
            cur, lens = p["out"], p["lens"]
    out["y"] = cur
    grad = s["dy"]
    for k in range(len(saved) - 1, -1, -1):
        f, x, lens, pool = saved[k]
        W_x, W_h, b = s["layers"][k]
        h0, c0 = (s["h0"][k], s["c0"][k]) if carried else (None, None)
        if pool is not None:
            grad = lstm.time_pool_bwd(grad, pool[0], lens, 2, pool[1])
        g = lstm.backward(f, x, W_x, W_h, h0, c0, lens, grad, want_dstate=False)
        out["dW_x%d" % k], out["dW_h%d" % k], out["db%d" % k] = g["dW_x"], g["dW_h"], g["db"]
        grad = g["dx"]
    out["dx"] = grad
    return out


def _encode(s):
    cur = s["x"]
    for (W_x, W_h, b), d in zip(s["layers"], s["directions"]):
        cur = lstm.forward(cur, W_x, W_h, b, None, None, s["lens"], bidirectional=d == 2, flags=s["flags"], workspace=s["workspace"],
                           want_c=False, want_state=False)["y"]
    return cur


def _decode(s):
    c, nt = s["case"], s["case"]["n_trg"]
    B = c["Q"] * c["beam"]
    f = lstm.forward(s["xin"].view(1, B, -1), *s["cell"], s["h"], s["c"], None, bidirectional=False,
                     flags=lstm.FLAG_INFERENCE | lstm.FLAG_WEIGHTS_PACKED, workspace=s["cell_ws"], want_c=False)
    cell = f["y"][0]
    a = lstm.attention_step(s["enc"], s["enc_ctx"], s["src_lens"], c["beam"], cell, *s["att"][:2], *s["att"][2:5], s["att"][5], s["accum"],
                            att=s["xin_next"][:, nt:], workspace=s["att_ws"], want_a=False)
    ro = lstm.readout(cell, s["xin"][:, :nt], a["att"], *s["readout"], workspace=s["readout_ws"], flags=lstm.FLAG_WEIGHTS_PACKED)
    return dict(h=f["hT"], c=f["cT"], accum=a["accum"], att=a["att"], readout=ro)


def _choose(s):
    c, nt = s["case"], s["case"]["n_trg"]
    logits = lstm.gemm(s["ro"], s["W_o"], a_kcontig=True, b_kcontig=True, M=c["Q"] * c["beam"], N=c["V"], K=c["R"], bias=s["b_o"])
    best = lstm.beam_step(logits, s["score"], workspace=s["beam_ws"])
    state = lstm.beam_gather_many([s["h"], s["c"], s["accum"], s["att_now"]], best["src"], outs=s["next"])
    lstm.embed(best["label"], s["W_trg"], out=s["xin_next"][:, :nt])
    return dict(score=best["score"], src=best["src"], label=best["label"], h=state[0], c=state[1], accum=state[2], xin=s["xin_next"])


def run(state):
    return {"train": _train, "stateful": _train, "encode": _encode, "decode": _decode, "choose": _choose}[state["kind"]](state)


# ------------------------------------------------------------------------------------------------ what a pass cannot do without

def _frames(c, halvings=0):
    if c["kind"] == "stateful":
        return c["B"] * c["T"]
    return sum(-(-v // (1 << halvings)) for v in _lengths(c["len_lo"], c["len_hi"], c["B"]))


def work(case):
    c = case
    if c["kind"] in ("train", "encode", "stateful"):
        e, n = (2 if c["dtype"] == BF16 else 4), c["n"]
        ds = [1] * c["layers"] if c["kind"] == "stateful" else _directions(c)
        pooled, grad = c.get("pooled", 0), c["kind"] != "encode"
        flops = bytes_ = 0
        for k, (d, k_in) in enumerate(zip(ds, _layer_inputs(c))):
            F = _frames(c, min(k, pooled))
            flops += d * F * (24 if grad else 8) * n * (k_in + n)
            weights = d * 4 * n * (k_in + n)
            bytes_ += weights * e + d * 4 * n * 4 + (weights * 4 + d * 4 * n * 4 if grad else 0)
        top = _frames(c, pooled) * ds[-1] * n * e
        bytes_ += _frames(c) * c["n_in"] * e * (2 if grad else 1) + top * (2 if grad else 1)
        if c["kind"] == "stateful":
            bytes_ += c["layers"] * 4 * c["B"] * n * 4
        return {"bytes": bytes_, "flops": flops}
    B, n, nt, E, R, S = c["Q"] * c["beam"], c["n"], c["n_trg"], c["E"], c["R"], c["S"]
    if c["kind"] == "decode":
        A = c["A"]
        positions = sum(_lengths(max(1, S // 3), S, c["Q"]))
        valid = positions * c["beam"]
        flops = 2 * B * (4 * n * (nt + E + n) + n * A + R * (n + nt + E)) + valid * (11 * A + 2 * E)
        weights = 2 * (4 * n * (nt + E + n) + n * A + R * (n + nt + E)) + 4 * (4 * n + 4 * A + R)
        return {"bytes": weights + positions * (E + A) * 2 + B * (nt + E) * 2 + 4 * B * n * 4 + valid * 4 + B * S * 4 + B * (E + R) * 2, "flops": flops}
    V = c["V"]
    state = B * (2 * n * 4 + S * 4 + E * 2)
    return {"bytes": 2 * V * R + 4 * V + 2 * B * R + 2 * state + 2 * 2 * B * nt + 6 * 4 * B, "flops": 2 * B * V * R}


def tolerance(case):
    """bfloat16 passes round h, dz and the layer outputs at every frame, and another order of summation moves those roundings;
    float passes differ by the order of sums over n, n_in and the frames, carried through the recurrence."""
    if case["kind"] == "choose":       # moved rows are exact; scores carry a log-sum-exp over V labels
        return {"rel": 1e-5, "differ": 2e-3}
    return {"rel": 1e-2} if case.get("dtype") != F32 else {"rel": 2e-5}

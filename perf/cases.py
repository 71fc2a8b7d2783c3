"""Cases that time the sketch-linear library through its public entry points, as a serving or conversion
program calls them: decode of one token or a small batch, whole decoder blocks, prompts, and the construction
of the sketches.  Every layer is made as a user makes it -- weights on the GPU, states built by
sketch_linear_build_states, a handle from sketch_linear_create -- with the value distributions of the
benchmark: weights N(0, 0.02^2), one percent of the input channels scaled by 20 and given four times the
sketch width, activations N(0, 1).

A case is a dict of plain values:
  kind      "gemv" (decode), "gate_up" (decode of a gate/up pair with SiLU), "block" (decode of the seven
            layers of a decoder block), "gemm" (prefill), "build" (sketch construction)
  in, out   features; for "block" the hidden and the feed-forward size
  tile      0: one sketch per input channel; otherwise the side of the square groups
  d         sketch rows
  bpw       bits per weight spent on states
  bits      16, or 8 / 4: low-bit states (same bits per weight, so 2x / 4x as many states)
  rows      batch (decode) or tokens (prefill)
  x, y      element types of the activations and of the result
"""
import math
import random

import numpy as np
import torch

import paper_2506_17255_amd as skl

DTYPE = {"f16": (torch.float16, skl.SKL_F16), "bf16": (torch.bfloat16, skl.SKL_BF16), "f32": (torch.float32, skl.SKL_F32)}
OUTLIERS, OUTLIER_SCALE, OUTLIER_WIDTH = 0.01, 20.0, 4.0


def _case(kind, n_in, n_out, tile=0, d=4, bpw=0.5, bits=16, rows=1, x="f16", y="f16", **name):
    return dict(name, kind=kind, **{"in": n_in, "out": n_out}, tile=tile, d=d, bpw=bpw, bits=bits, rows=rows, x=x, y=y)


def listed():
    return [
        # the smallest call: one 256 x 256 group, batch 1; two launches and their latency
        _case("gemv", 256, 256, tile=256, d=2, name="decode_group_256_b1"),
        # attention projection of a 7B-sized model, one token
        _case("gemv", 4096, 4096, d=3, name="decode_4096x4096_b1"),
        # up projection, one token: the step that bench.py reports
        _case("gemv", 4096, 11008, name="decode_4096x11008_b1"),
        # down projection, a small batch of sequences
        _case("gemv", 11008, 4096, rows=8, name="decode_11008x4096_b8"),
        # first half of the feed-forward block, the largest batch a decode call takes
        _case("gate_up", 4096, 11008, rows=16, name="gate_up_4096x11008_b16"),
        # one token through a whole decoder block: q/k/v, o, gate/up, down -- seven layers, nothing re-used
        _case("block", 4096, 11008, name="block_4096_11008_b1"),
        # the paper's own recipe for 0.5 bit per weight: 4-bit states, four times as many
        _case("gemv", 4096, 11008, bits=4, name="decode_4096x11008_4bit_b1"),
        # a short prompt (or a chunk of one) through the up projection
        _case("gemm", 4096, 11008, rows=100, name="prefill_4096x11008_t100"),
        # a long prompt through the attention projection
        _case("gemm", 4096, 4096, rows=2048, x="bf16", y="bf16", name="prefill_4096x4096_t2048"),
        # a long prompt through the up projection at 0.75 bit per weight
        _case("gemm", 4096, 11008, bpw=0.75, rows=2048, x="bf16", y="bf16", name="prefill_4096x11008_t2048"),
        # the largest: a long prompt through the feed-forward layer of a 70B-sized model
        _case("gemm", 8192, 28672, rows=2048, x="bf16", y="bf16", name="prefill_8192x28672_t2048"),
        # conversion of a layer: the states of its sketch from its weights
        _case("build", 4096, 11008, name="build_4096x11008"),
    ]


def _log_int(rng, lo, hi, step=1):
    return max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step)


def draw(rng):
    kind = rng.choice(["gemv", "gemv", "gemv", "gemm", "gemm", "gemm", "gate_up", "block", "build"])
    step = rng.choice([64, 64, 8, 1])                  # mostly the sizes of real models, odd ones among them
    d = rng.choice([2, 3, 4, 4])
    bpw = rng.choice([0.5, 0.5, 0.75])
    if kind == "block":
        h = _log_int(rng, 1024, 6144, 128)
        return _case("block", h, _log_int(rng, 2 * h, 3 * h, 64), d=4, bpw=bpw, rows=_log_int(rng, 1, 16), y="f16")
    if kind in ("gemv", "gemm") and rng.random() < 0.25:       # square groups
        side = rng.choice([128, 256])
        n_in, n_out = (_log_int(rng, 256, 2048, side) for _ in range(2))
        rows = _log_int(rng, 1, 16) if kind == "gemv" else _log_int(rng, 17, 512)
        x = "f16" if kind == "gemv" else rng.choice(["f16", "bf16"])
        return _case(kind, n_in, n_out, tile=side, d=min(d, 3), bpw=bpw, rows=rows, x=x, y=x)
    n_in, n_out = _log_int(rng, 512, 8192, step), _log_int(rng, 1024, 28672, step)
    if kind == "build":
        return _case(kind, n_in, min(n_out, 16384), d=d, bpw=bpw)
    bits = rng.choice([16, 16, 16, 8, 4])
    if bits < 16:                                      # wider sketches: the tables of larger layers do not fit a compute unit
        n_out, d = min(n_out, 11008), 4
    if kind == "gemm":
        x = rng.choice(["f16", "bf16", "bf16"])
        return _case(kind, n_in, n_out, d=d, bpw=bpw, bits=bits, rows=_log_int(rng, 17, 2048), x=x, y=rng.choice([x, x, "f32"]))
    return _case(kind, n_in, n_out, d=d, bpw=bpw, bits=bits, rows=_log_int(rng, 1, 16), y=rng.choice(["f16", "f16", "f32"]))


class _Sketch:
    """Weights, geometry and widths of one layer."""

    def __init__(self, case, n_in, n_out, rng, gen):
        tile = case["tile"]
        self.n_in, self.n_out, self.d = n_in, n_out, case["d"]
        self.tile_in, self.tile_out = (tile, tile) if tile else (1, n_out)
        self.W = torch.randn(n_in, n_out, device="cuda", dtype=torch.float16, generator=gen) * 0.02
        groups = (n_in // self.tile_in) * (n_out // self.tile_out)
        importance = np.ones(groups)
        if not tile:
            outliers = sorted(rng.sample(range(n_in), math.ceil(OUTLIERS * n_in)))
            self.W[torch.tensor(outliers, device="cuda")] *= OUTLIER_SCALE
            importance[outliers] = OUTLIER_WIDTH
        # a state of `bits` bits per bpw bits of weight, divided over the groups by importance
        budget = int(n_in * n_out * case["bpw"] / case["bits"])
        self.widths = np.maximum(1, np.floor(importance / importance.sum() * budget / self.d)).astype(np.uint32)
        self.a = np.array([2 * rng.randrange(1 << 23) + 1 for _ in range(self.d)], dtype=np.uint32)
        self.c = np.array([rng.randrange(1 << 24) for _ in range(self.d)], dtype=np.uint32)
        self.n_states = self.d * int(self.widths.sum())

    def desc(self, states=None, **low_bit):
        return skl.make_desc(self.n_in, self.n_out, self.tile_in, self.tile_out, self.d, self.a, self.c, self.widths, states,
                             n_states=self.n_states, **low_bit)

    def build(self):
        """The states of the sketch, on the GPU."""
        desc = self.desc()
        states = torch.empty(self.n_states, dtype=torch.int16, device="cuda")
        ws = torch.empty(skl.sketch_linear_build_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
        skl.sketch_linear_build_states(desc, self.W.data_ptr(), states.data_ptr(), ws.data_ptr(), ws.numel(), _stream())
        return states


class _Layer:
    """A layer resident on the GPU."""

    def __init__(self, case, n_in, n_out, rng, gen):
        sk = _Sketch(case, n_in, n_out, rng, gen)
        states = sk.build()
        if case["bits"] == 16:
            desc = sk.desc(states.cpu().numpy().view(np.uint16))
        else:
            desc = sk.desc(None, state_bits=case["bits"], **_quantize(states, sk, case["bits"]))
        n = skl.sketch_linear_device_bytes(desc)
        self.buf = torch.empty(n, dtype=torch.uint8, device="cuda")
        self.handle = None
        self.handle = skl.sketch_linear_create(desc, self.buf.data_ptr(), n, _stream())

    def __del__(self, destroy=skl.sketch_linear_destroy):
        if getattr(self, "handle", None):
            destroy(self.handle)


def _quantize(states, sk, bits):
    """Signed codes and one binary16 scale per sketch row of a group: the largest magnitude of the row."""
    qmax = 127 if bits == 8 else 7
    v = states.view(torch.float16).float()
    width = torch.from_numpy(sk.widths.astype(np.int64)).cuda().repeat_interleave(sk.d)        # of every (group, row)
    row = torch.repeat_interleave(torch.arange(width.numel(), device="cuda"), width)
    scale = torch.zeros(width.numel(), device="cuda").scatter_reduce_(0, row, v.abs(), "amax")
    s = scale[row]
    q = torch.where(s > 0, torch.round(v * qmax / torch.where(s > 0, s, torch.ones_like(s))), torch.zeros_like(s)).to(torch.int8)
    if bits == 4:
        n = torch.nn.functional.pad(q, (0, q.numel() % 2)).view(torch.uint8) & 15
        q = n[0::2] | (n[1::2] << 4)
    return {"codes": q.cpu().numpy().view(np.uint8), "scales": scale.half().cpu().numpy().view(np.uint16)}


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _bytes(n):
    return torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")


class _State:
    pass


def prepare(case, seed):
    rng = random.Random(seed)
    gen = torch.Generator("cuda").manual_seed(seed)
    n_in, n_out, rows, kind = case["in"], case["out"], case["rows"], case["kind"]
    (x_t, x_c), (y_t, y_c) = DTYPE[case["x"]], DTYPE[case["y"]]
    s = _State()
    s.case, s.rows, s.x_code, s.y_code, s.stream = case, rows, x_c, y_c, _stream()

    def act(n):
        return torch.randn(rows, n, device="cuda", generator=gen).to(x_t)

    def out(n):
        return torch.empty(rows, n, dtype=y_t, device="cuda")

    if kind == "build":
        s.sk = _Sketch(case, n_in, n_out, rng, gen)
        s.desc = s.sk.desc()
        s.y = torch.empty(s.sk.n_states, dtype=torch.int16, device="cuda")
        s.ws = _bytes(skl.sketch_linear_build_workspace_bytes(s.desc))
    elif kind == "block":
        mk = lambda i, o: _Layer(case, i, o, rng, gen)  # noqa: E731
        s.qkv, s.o = [mk(n_in, n_in) for _ in range(3)], mk(n_in, n_in)
        s.gate, s.up, s.down = mk(n_in, n_out), mk(n_in, n_out), mk(n_out, n_in)
        s.x, s.attn, s.x2 = act(n_in), act(n_in), act(n_in)
        s.ys, s.yo, s.h, s.y = [out(n_in) for _ in range(3)], out(n_in), out(n_out), out(n_in)
        s.qkv_handles, s.qkv_ptrs = [l.handle for l in s.qkv], [y.data_ptr() for y in s.ys]
        s.ws = _bytes(max(skl.sketch_linear_gemv_group_workspace_bytes(s.qkv_handles, rows),
                          skl.sketch_linear_workspace_bytes(s.o.handle, 0, rows),
                          skl.sketch_linear_gemv_group_workspace_bytes([s.gate.handle, s.up.handle], rows),
                          skl.sketch_linear_workspace_bytes(s.down.handle, 0, rows)))
    elif kind == "gate_up":
        s.gate, s.up = (_Layer(case, n_in, n_out, rng, gen) for _ in range(2))
        s.x, s.y = act(n_in), out(n_out)
        s.ws = _bytes(skl.sketch_linear_gemv_group_workspace_bytes([s.gate.handle, s.up.handle], rows))
    else:
        s.layer = _Layer(case, n_in, n_out, rng, gen)
        s.x, s.y = act(n_in), out(n_out)
        s.ws = _bytes(skl.sketch_linear_workspace_bytes(s.layer.handle, 0 if kind == "gemv" else 1, rows))
    s.ws_ptr, s.ws_bytes = s.ws.data_ptr(), s.ws.numel()
    return s


def run(s):
    c, rows, ws, nws, st = s.case, s.rows, s.ws_ptr, s.ws_bytes, s.stream
    kind, n_in, n_out = c["kind"], c["in"], c["out"]
    if kind == "gemv":
        skl.sketch_linear_gemv(s.layer.handle, s.x.data_ptr(), s.x_code, n_in, s.y.data_ptr(), s.y_code, n_out, rows, ws, nws, st)
        return s.y
    if kind == "gemm":
        skl.sketch_linear_gemm(s.layer.handle, s.x.data_ptr(), s.x_code, n_in, s.y.data_ptr(), s.y_code, n_out, rows, ws, nws, st)
        return s.y
    if kind == "gate_up":
        skl.sketch_linear_gemv_gate_up(s.gate.handle, s.up.handle, s.x.data_ptr(), s.x_code, n_in, s.y.data_ptr(), s.y_code, n_out,
                                       rows, ws, nws, st)
        return s.y
    if kind == "block":
        xc, yc = s.x_code, s.y_code
        skl.sketch_linear_gemv_group(s.qkv_handles, s.x.data_ptr(), xc, n_in, s.qkv_ptrs, yc, n_in, rows, ws, nws, st)
        skl.sketch_linear_gemv(s.o.handle, s.attn.data_ptr(), xc, n_in, s.yo.data_ptr(), yc, n_in, rows, ws, nws, st)
        skl.sketch_linear_gemv_gate_up(s.gate.handle, s.up.handle, s.x2.data_ptr(), xc, n_in, s.h.data_ptr(), yc, n_out, rows, ws, nws, st)
        skl.sketch_linear_gemv(s.down.handle, s.h.data_ptr(), xc, n_out, s.y.data_ptr(), yc, n_in, rows, ws, nws, st)
        return [*s.ys, s.yo, s.h, s.y]
    skl.sketch_linear_build_states(s.desc, s.sk.W.data_ptr(), s.y.data_ptr(), ws, nws, st)
    return s.y


def work(case):
    n_in, n_out, rows, kind = case["in"], case["out"], case["rows"], case["kind"]
    per = {"f16": 2, "bf16": 2, "f32": 4}
    states = n_in * n_out * case["bpw"] / 8                     # bytes of one in x out layer's sketch
    if kind == "build":
        return {"bytes": 2 * n_in * n_out + states, "flops": 0}
    if kind == "block":
        weights = 4 * n_in * n_in + 3 * n_in * n_out
        return {"bytes": weights * case["bpw"] / 8 + 2 * rows * (8 * n_in + 2 * n_out), "flops": 2 * rows * weights}
    n = 2 if kind == "gate_up" else 1
    return {"bytes": n * states + rows * (n_in * per[case["x"]] + n_out * per[case["y"]]), "flops": 2 * n * rows * n_in * n_out}


def tolerance(case):
    # Weights are reconstructed exactly and products of binary16 values are exact in float32; what differs is
    # the order of the float32 sums and the final rounding.  Measured against a product in 64 bits: float32
    # 7e-8 to 8e-8 (a longer serial chain would show several times that), binary16 2.1e-4, bfloat16 1.7e-3.
    if case["kind"] == "build":
        return "exact"
    return {"f32": {"rel": 1e-6}, "f16": {"rel": 8e-4}, "bf16": {"rel": 6.6e-3}}[case["y"]]

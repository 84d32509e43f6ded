"""The GEMM calls a user of this library times: squares, decoding, prefill,
sizes off every tile and B stored K x N, in the three precisions.

A case is a dict:
  entry   "plain" (GEMM[dtype]: raw sums), "scaled" (gemm_scaled) or "bt"
          (gemm_bt, B stored K x N)
  dtype   "f16" (FP32 sums), "s8" or "s4" (INT32 sums)
  m, n, k C is m x n, the sums run over k
  ws      whether the call is given a workspace kept across calls, as a
          serving loop does
  out     scaled calls: "f16", "bf16" or "f32"
  zero    scaled calls: zero points, "" (none), "a" or "ab"
  values  "uniform" (the full range of the type, U[-1, 1] for FP16) or
          "model" (bell-shaped, as activations and weights are)
"""
import math

import torch

import paper_2608_10103_amd as mp

_OUT = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}


def _case(entry, dtype, m, n, k, ws=False, out="", zero="", values="uniform", name=None):
    c = {"entry": entry, "dtype": dtype, "m": m, "n": n, "k": k, "ws": ws, "out": out, "zero": zero,
         "values": values}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The square sweep's ends and middles: its smallest point (launch
        # bound), its largest, and INT8 and INT4 at 4096 (INT4 with the
        # workspace its conversion pre-pass takes).
        _case("plain", "f16", 512, 512, 512, name="f16_square_512"),
        _case("plain", "f16", 8192, 8192, 8192, name="f16_square_8192"),
        _case("plain", "s8", 4096, 4096, 4096, name="s8_square_4096"),
        _case("plain", "s4", 4096, 4096, 4096, ws=True, name="s4_square_4096"),
        # Decoding: a few tokens times a weight matrix. A batch of 16 in FP16,
        # one token with INT8 weights and activations (the smallest call of a
        # quantised model), a batch of 32 with INT4 ones, both scaled back to
        # 16 bits.
        _case("plain", "f16", 16, 8192, 8192, ws=True, values="model", name="f16_decode_16"),
        _case("scaled", "s8", 1, 14336, 4096, out="f16", values="model", name="s8_decode_1_scaled"),
        _case("scaled", "s4", 32, 4096, 14336, ws=True, out="f16", values="model", name="s4_decode_32_scaled"),
        # Prefill: prompts of whatever length times a weight matrix. FP16 to
        # FP16 at an odd length, INT8 with asymmetric activations (a zero point
        # per row) to BF16, INT4 without a workspace.
        _case("scaled", "f16", 300, 11008, 4096, ws=True, out="f16", values="model", name="f16_prefill_300"),
        _case("scaled", "s8", 2048, 4096, 4096, ws=True, out="bf16", zero="a", values="model",
              name="s8_prefill_zero_points"),
        _case("scaled", "s4", 1000, 11008, 4096, out="f16", values="model", name="s4_prefill_1000"),
        # A size that nobody chose for the hardware: K fills no whole K-slice.
        _case("plain", "f16", 1000, 1000, 1000, name="f16_ragged_1000"),
        # Weights stored K x N, as frameworks that keep them (in, out) do.
        _case("bt", "s8", 1024, 4096, 4096, values="model", name="s8_b_k_by_n"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _to(x, q, lo, hi):
    return max(lo, min(hi, (x + q // 2) // q * q))


def draw(rng):
    kind = rng.choice(["square", "decode", "prefill", "ragged", "bt"])
    dtype = rng.choice(["f16", "s8", "s4"])
    ints = dtype != "f16"
    if kind == "square":
        n = _to(_log(rng, 512, 8192), 128, 512, 8192)
        return _case("plain", dtype, n, n, n, ws=rng.random() < 0.5)
    if kind == "ragged":
        # any sizes, most of them odd (INT4's K is even)
        m, n, k = (_log(rng, 33, 3000) for _ in range(3))
        return _case("plain", dtype, m, n, k + (k & 1) if dtype == "s4" else k, ws=rng.random() < 0.5)
    if kind == "bt":
        return _case("bt", dtype, _log(rng, 64, 4096), _to(_log(rng, 1024, 8192), 256, 1024, 8192),
                     _to(_log(rng, 512, 8192), 256, 512, 8192), values="model")
    m = _log(rng, 1, 128) if kind == "decode" else _log(rng, 129, 4096)
    n = _to(_log(rng, 2048, 14336), 64, 2048, 14336)
    k = _to(_log(rng, 2048, 14336), 256, 2048, 14336)
    if m * n * k > 8192 ** 3:
        k = 4096
    ws = rng.random() < 0.5
    if rng.random() < 0.3:
        return _case("plain", dtype, m, n, k, ws=ws, values="model")
    zero = rng.choice(["", "", "a", "ab"]) if ints and ws else ""
    return _case("scaled", dtype, m, n, k, ws=ws, out=rng.choice(["f16", "bf16", "f32"]), zero=zero,
                 values="model")


def _operand(g, dtype, rows, cols, values, std):
    """rows x cols values of the type (INT4: packed two per byte along cols)."""
    if dtype == "f16":
        if values == "uniform":
            return (torch.rand(rows, cols, generator=g, device="cuda") * 2 - 1).half()
        return (torch.randn(rows, cols, generator=g, device="cuda") * std).half()
    if values == "uniform":
        x = torch.randint(0, 256, (rows, cols if dtype == "s8" else cols // 2), generator=g, device="cuda",
                          dtype=torch.uint8)
        return x.view(torch.int8) if dtype == "s8" else x
    # quantised with the largest magnitude (about four deviations) at the end
    # of the type's range
    top = 127 if dtype == "s8" else 7
    x = torch.randn(rows, cols, generator=g, device="cuda").mul_(top / 4).round_().clamp_(-top - 1, top)
    x = x.to(torch.int8)
    if dtype == "s8":
        return x
    x = x.view(torch.uint8) & 0xF
    return (x[:, 0::2] | (x[:, 1::2] << 4)).contiguous()


def prepare(case, seed):
    """Operands, scales, zero points, an output buffer and (where the case
    says so) a workspace, on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    d, m, n, k = case["dtype"], case["m"], case["n"], case["k"]
    s = dict(case)
    s["A"] = _operand(g, d, m, k, case["values"], 1.0)
    s["B"] = _operand(g, d, *((k, n) if case["entry"] == "bt" else (n, k)), case["values"], 0.02)
    epi = None
    if case["entry"] == "scaled":
        if d != "f16":
            s["scale_a"] = torch.rand(m, generator=g, device="cuda") * 0.02 + 0.01
            s["scale_b"] = torch.rand(n, generator=g, device="cuda") * 0.002 + 0.001
            top = 20 if d == "s8" else 3
            if "a" in case["zero"]:
                s["zero_a"] = torch.randint(-top, top + 1, (m,), generator=g, device="cuda", dtype=torch.int32)
            if "b" in case["zero"]:
                s["zero_b"] = torch.randint(-top, top + 1, (n,), generator=g, device="cuda", dtype=torch.int32)
        out = _OUT[case["out"]]
        vec = [s[x].data_ptr() if x in s else None for x in ("scale_a", "scale_b", "zero_a", "zero_b")]
        epi = mp.gemm.Epilogue(*vec, mp.gemm.OUT_TYPE[out])
    else:
        out = torch.float32 if d == "f16" else torch.int32
    s["C"] = torch.empty(m, n, dtype=out, device="cuda")
    if case["ws"]:
        s["workspace"] = mp.new_workspace(mp.workspace_size(d, m, n, k, epi=epi), torch.device("cuda", 0))
    return s


def run(s):
    d = s["dtype"]
    if s["entry"] == "bt":
        return mp.gemm_bt(d, s["A"], s["B"], C=s["C"])
    ws = s.get("workspace")
    if s["entry"] == "plain":
        return mp.GEMM[d](s["A"], s["B"], C=s["C"], workspace=ws)
    return mp.gemm_scaled(d, s["A"], s["B"], scale_a=s.get("scale_a"), scale_b=s.get("scale_b"),
                          zero_a=s.get("zero_a"), zero_b=s.get("zero_b"), out_dtype=_OUT[s["out"]], C=s["C"],
                          workspace=ws)


def work(case):
    m, n, k = case["m"], case["n"], case["k"]
    per = {"f16": 2.0, "s8": 1.0, "s4": 0.5}[case["dtype"]]
    c = 2 if case["out"] in ("f16", "bf16") else 4
    vec = (m + n) * 4 if case["entry"] == "scaled" and case["dtype"] != "f16" else 0
    vec += 4 * (("a" in case["zero"]) * m + ("b" in case["zero"]) * n)
    return {"bytes": (m + n) * k * per + m * n * c + vec, "flops": 2.0 * m * n * k}


def tolerance(case):
    """About four times what two orders of the same FP32 sums differ by:
    5.5e-7 (2-norm) and 6e-6 (largest) measured at K = 8192, one K range
    against two. Narrow outputs: a sum that differs by 5.5e-7 rounds the other
    way with probability 5.5e-7 / ulp, each time by one ulp of at most 2^-10
    (FP16) or 2^-7 (BF16): sqrt(5.5e-7 * ulp) in the 2-norm. Integer sums are
    exact; scaling them takes three FP32 roundings, below those 5.5e-7."""
    if case["entry"] != "scaled" and case["dtype"] != "f16":
        return "exact"
    if case["out"] == "f16":
        return {"rel": 1e-4, "max": 2e-3}
    if case["out"] == "bf16":
        return {"rel": 3e-4, "max": 1.6e-2}
    return {"rel": 3e-6, "max": 3e-5}


def _decode(x, dtype):
    """The operand's values in 64 bits (INT4: unpacked along the last axis)."""
    if dtype != "s4":
        return x.double()
    lo, hi = (x & 0xF).to(torch.int16), (x >> 4).to(torch.int16)
    v = torch.stack([lo, hi], dim=-1).reshape(x.shape[0], -1)
    return ((v ^ 8) - 8).double()


def exact(case, seed):
    s = prepare(case, seed)
    a, b = _decode(s["A"], case["dtype"]), _decode(s["B"], case["dtype"])
    if case["entry"] != "bt":
        b = b.t().contiguous()
    if case["entry"] == "scaled":
        if "zero_a" in s:
            a -= s["zero_a"].double()[:, None]
        if "zero_b" in s:
            b -= s["zero_b"].double()[None, :]
        if "scale_a" in s:
            a *= s["scale_a"].double()[:, None]
            b *= s["scale_b"].double()[None, :]
    c = a @ b
    if case["entry"] != "scaled" and case["dtype"] != "f16":
        return c.round().to(torch.int32)
    return c

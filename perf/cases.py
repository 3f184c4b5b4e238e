"""The work a user of this package has it do, as timed cases over its public entry points.

A case is a dict of plain values.  ``listed()`` holds the named ones, ``draw(rng)`` gives another
of the same ranges, ``prepare(case, seed)`` makes what a program holds before the call (inputs,
weights in the kernels' layout, calibrated static scales, kept output and workspace buffers) and
``run(state)`` is one pass.  Five kinds of work:

  linear       one linear layer through the no-allocation prefill entry
  decode       the linears of decoder layers for a few new rows: one launch per group of linears
               at one row, rotate + quantize followed by the grouped GEMV for more
  prefill      a prefill step: mask remap and row permute of the embeddings, then qkv, o, gate_up
               and down with static scales, per-token dynamic scales, or the flagged-channel split
               of Rotation Magnitude Suppression on down
  attention    attention on AIFS-ordered tokens, on its own or behind the qkv linear and RoPE
  weight_only  the four linears with 16-bit activations and group-128 int4 weights

Shapes are those of the package's workloads: 7B-class (3584 channels, 28 heads on 4) and 72B-class
(8192 channels, 64 heads on 8).
"""
import math

import numpy as np
import torch

from paper_2502_00425_amd import binding as mq
from paper_2502_00425_amd import workloads as wl

HEAD_DIM = 128
# name -> (Hadamard block, query heads, key/value heads, {projection: (K, N)})
MODELS = {
    "7b": (512, 28, 4, wl.workload(1).projections),
    "72b": (128, 64, 8, wl.workload(4).projections),
}


def listed():
    return [
        # The smallest call: one 512 x 512 linear on a 64-token prompt; launches and host time count.
        {"name": "linear_512_t64", "kind": "linear", "T": 64, "K": 512, "N": 512, "block": 512, "spans": 1},
        # Token-by-token generation of one sequence: four decoder layers, one new row.
        {"name": "decode_7b_t1", "kind": "decode", "model": "7b", "T": 1, "layers": 4},
        # Batched generation on the large shapes: sixteen sequences, one new row each.
        {"name": "decode_72b_t16", "kind": "decode", "model": "72b", "T": 16, "layers": 1},
        # A short mixed prompt (a thumbnail and a question), ragged length.
        {"name": "prompt_7b_t77", "kind": "prefill", "model": "7b", "T": 77, "scheme": "static", "n_split": 0, "spans": 1},
        # One image and a question: the usual multimodal prompt on the 7B shapes.
        {"name": "prefill_7b_t1280", "kind": "prefill", "model": "7b", "T": 1280, "scheme": "static", "n_split": 0, "spans": 1},
        # A high-resolution image or a short video.
        {"name": "prefill_7b_t4096", "kind": "prefill", "model": "7b", "T": 4096, "scheme": "static", "n_split": 0, "spans": 1},
        # Several images in a long context on the large shapes, the largest single-GPU step.
        {"name": "prefill_72b_t16384", "kind": "prefill", "model": "72b", "T": 16384, "scheme": "static", "n_split": 0, "spans": 4},
        # A model with layers flagged by Rotation Magnitude Suppression; odd length, several spans.
        {"name": "prefill_7b_t1003_rms", "kind": "prefill", "model": "7b", "T": 1003, "scheme": "rms", "n_split": 4, "spans": 3},
        # The attention half of a layer at the usual prompt: qkv linear, RoPE, attention.
        {"name": "attention_7b_t1280", "kind": "attention", "model": "7b", "T": 1280, "spans": 1, "project": True},
        # Attention alone over a long context of several images.
        {"name": "attention_7b_t8192", "kind": "attention", "model": "7b", "T": 8192, "spans": 4, "project": False},
        # Weight-only checkpoints: one new row, and a usual prompt.
        {"name": "weight_only_7b_t1", "kind": "weight_only", "model": "7b", "T": 1},
        {"name": "weight_only_7b_t1280", "kind": "weight_only", "model": "7b", "T": 1280},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("linear", "decode", "decode", "prefill", "prefill", "prefill", "attention", "weight_only"))
    model = rng.choice(("7b", "7b", "72b"))
    if kind == "linear":
        block = rng.choice((128, 512))
        return {"kind": kind, "T": _log_int(rng, 16, 2048), "K": block * _log_int(rng, 1, 8192 // block),
                "N": 8 * _log_int(rng, 16, 1280), "block": block, "spans": rng.randint(0, 3)}
    if kind == "decode":
        return {"kind": kind, "model": model, "T": _log_int(rng, 1, 32), "layers": 4 if model == "7b" else 1}
    if kind == "prefill":
        scheme = rng.choice(("static", "static", "dynamic", "rms"))
        return {"kind": kind, "model": model, "T": _log_int(rng, 33, 8192 if model == "7b" else 4096), "scheme": scheme,
                "n_split": rng.randint(1, 37) if scheme == "rms" else 0, "spans": rng.randint(0, 4)}
    if kind == "attention":
        return {"kind": kind, "model": model, "T": _log_int(rng, 64, 16384 if model == "7b" else 8192),
                "spans": rng.randint(0, 4), "project": rng.random() < 0.5}
    return {"kind": kind, "model": model, "T": _log_int(rng, 1, 2048)}


# ------------------------------------------------------------------------------------ inputs

def _spans(T, n):
    """n visual spans that take three quarters of the sequence, text before, between and behind."""
    if n == 0:
        return []
    vis, gap = (3 * T) // (4 * n), T // (4 * (n + 1))
    out, at = [], gap
    for _ in range(n):
        out.append((at, vis))
        at += vis + gap
    return out


def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    return gen


def _activations(gen, rows, K, is_vis):
    """Text rows N(0, 1); visual rows twenty times wider with four outlier channels."""
    gain = torch.full((K,), wl.VIS_SIGMA, dtype=torch.float32, device="cuda")
    for c in wl.OUTLIER_CHANNELS:
        if c < K:
            gain[c] *= wl.OUTLIER_GAIN
    out = torch.empty((rows, K), dtype=torch.float16, device="cuda")
    for r in range(0, rows, 2048):
        x = torch.randn((min(2048, rows - r), K), dtype=torch.float32, device="cuda", generator=gen)
        out[r:r + 2048] = torch.where(is_vis[r:r + 2048, None], x * gain, x).half()
    return out


def _scales(gen, K, block):
    """Static scales of both modalities from 256 calibration rows each."""
    rows = torch.ones(wl.CALIB_ROWS, dtype=torch.bool, device="cuda")
    absmax = torch.zeros(2, device="cuda")
    mq.hadamard_absmax(_activations(gen, wl.CALIB_ROWS, K, rows), block, absmax[0:1])
    mq.hadamard_absmax(_activations(gen, wl.CALIB_ROWS, K, ~rows), block, absmax[1:2])
    return [mq.static_scale_from_absmax(a, block) for a in absmax.tolist()]


def _weight(gen, K, N, scale=0.0125):
    """Uniform int4 codes, drawn in the layout the kernels stream, and per-channel scales."""
    wp = torch.randint(0, 256, (mq.w4_prepacked_bytes(N, K),), dtype=torch.uint8, device="cuda", generator=gen)
    return wp, (scale * (0.4 + 1.2 * torch.rand(N, device="cuda", generator=gen))).half()


def _half(*shape):
    return torch.empty(shape, dtype=torch.float16, device="cuda")


def _layout(T, spans):
    perm, _, n_vis = mq.aifs_build_perm(T, spans)
    is_vis = torch.zeros(T, dtype=torch.bool)
    for s, n in spans:
        is_vis[s:s + n] = True
    return torch.from_numpy(perm).cuda(), n_vis, is_vis.cuda()


def prepare(case, seed):
    gen, T, kind = _generator(seed), case["T"], case["kind"]
    st = {"case": case, "T": T}
    if kind == "linear":
        K, N, block = case["K"], case["N"], case["block"]
        st["perm"], st["n_vis"], is_vis = _layout(T, _spans(T, case["spans"]))
        st["x"] = _activations(gen, T, K, is_vis)
        st["s"] = _scales(gen, K, block)
        st["w"] = _weight(gen, K, N)
        st["y"] = _half(T, N)
        return st

    block, hq, hkv, proj = MODELS[case["model"]]
    st["block"] = block
    if kind == "decode":
        # New rows are text.  The projections of a group share their input and keep their own
        # weights and outputs.
        groups = (("qkv", (hq * HEAD_DIM, hkv * HEAD_DIM, hkv * HEAD_DIM)), ("o", (proj["o"][1],)),
                  ("gate_up", (proj["gate_up"][1] // 2,) * 2), ("down", (proj["down"][1],)))
        text = torch.zeros(T, dtype=torch.bool, device="cuda")
        scale = {K: _scales(gen, K, block)[1] for K in {k for k, _ in proj.values()}}
        st["groups"] = []
        for _ in range(case["layers"]):
            for p, outs in groups:
                K = proj[p][0]
                lin = [(*_weight(gen, K, N), N, _half(T, N)) for N in outs]
                st["groups"].append((_activations(gen, T, K, text), scale[K], lin,
                                     torch.empty((T, K), dtype=torch.int8, device="cuda")))
        return st

    if kind == "weight_only":
        text = torch.zeros(T, dtype=torch.bool, device="cuda")
        st["lin"] = []
        for K, N in proj.values():
            codes = torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, device="cuda", generator=gen)
            sc = (0.002 + 0.008 * torch.rand((N, K // 128), device="cuda", generator=gen)).half()
            st["lin"].append((_activations(gen, T, K, text), mq.w4g128_prepack(codes, sc), N, _half(T, N)))
        return st

    spans = _spans(T, case["spans"])
    st["perm"], st["n_vis"], is_vis = _layout(T, spans)
    if kind == "attention":
        st["heads"] = hq, hkv
        st["ws"] = torch.empty(mq.aifs_attention_workspace_bytes(T, hkv), dtype=torch.uint8, device="cuda")
        st["o"] = _half(T, hq * HEAD_DIM)
        K, N = proj["qkv"]
        if case["project"]:
            # weight scales that leave queries and keys of a visual row at a few units
            st["x"], st["s"] = _activations(gen, T, K, is_vis), _scales(gen, K, block)
            st["w"], st["qkv"] = _weight(gen, K, N, 1e-4), _half(T, N)
            st["lws"] = torch.empty(mq.w4a8_linear_prefill_workspace_bytes(T, N, K), dtype=torch.uint8, device="cuda")
        else:
            st["qkv"] = torch.randn((T, N), device="cuda", generator=gen).half()
        return st

    # prefill
    st["mask"] = torch.tril(torch.ones((T, T), dtype=torch.uint8, device="cuda"))
    st["mask_u"] = torch.empty_like(st["mask"])
    st["lin"], need = [], 256
    scale = {K: _scales(gen, K, block) for K in {k for k, _ in proj.values()}}
    for name, (K, N) in proj.items():
        split = None
        if case["scheme"] == "rms" and name == "down":
            n = case["n_split"]
            split = (np.arange(n, dtype=np.int32) * block,
                     torch.randint(-8, 8, (n, N), dtype=torch.int8, device="cuda", generator=gen),
                     np.linspace(0.05, 0.35, n, dtype=np.float32))
        st["lin"].append((_activations(gen, T, K, is_vis), *_weight(gen, K, N), N, scale[K], _half(T, N), split))
        need = max(need, mq.w4a8_linear_prefill_workspace_bytes(T, N, K))
    st["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    st["x_u"] = torch.empty_like(st["lin"][0][0])
    if case["scheme"] != "static":
        st["xq"] = {K: torch.empty((T, K), dtype=torch.int8, device="cuda") for K, _ in proj.values()}
        st["row_scale"] = torch.empty(T, dtype=torch.float32, device="cuda")
    return st


# -------------------------------------------------------------------------------------- pass

def run(st):
    return _RUN[st["case"]["kind"]](st)


def _run_linear(st):
    case = st["case"]
    (wp, ws), (s_vis, s_txt) = st["w"], st["s"]
    return mq.w4a8_linear_prefill_static(st["x"], st["perm"], wp, ws, case["N"], st["n_vis"], s_vis, s_txt,
                                         case["block"], st["y"])


def _run_decode(st):
    block, out = st["block"], []
    for x, s, lin, xq in st["groups"]:
        if st["T"] == 1:
            if len(lin) == 1:
                wp, ws, N, y = lin[0]
                mq.w4a8_linear_decode(x, wp, ws, N, 0, s, s, block, out=y)
            else:
                mq.w4a8_linear_decode_grouped(x, lin, 0, s, s, block)
        else:
            mq.hadamard_quant_act(x, 0, s, s, block, out=xq)
            mq.w4a8_gemv_grouped(xq, lin, 0, s, s)
        out += [l[3] for l in lin]
    return out


def _run_prefill(st):
    scheme, block, n_vis, perm, ws = st["case"]["scheme"], st["block"], st["n_vis"], st["perm"], st["ws"]
    out = [mq.aifs_remap_mask(st["mask"], perm, out=st["mask_u"]),
           mq.aifs_permute(st["lin"][0][0], perm, out=st["x_u"])]
    for x, wp, wsc, N, (s_vis, s_txt), y, split in st["lin"]:
        if scheme == "dynamic":
            xq, rs = mq.hadamard_dynquant_act(x, block, perm_dev=perm, out=st["xq"][x.shape[1]], row_scale=st["row_scale"])
            mq.w4a8_gemm_rowscale(xq, wp, wsc, rs, N, out=y, workspace=ws)
        elif split is not None:
            xq = mq.hadamard_quant_act(x, n_vis, s_vis, s_txt, block, perm_dev=perm, out=st["xq"][x.shape[1]])
            mq.w4a8_gemm_rms(xq, wp, wsc, N, n_vis, s_vis, s_txt, *split, out=y, workspace=ws)
        else:
            mq.w4a8_linear_prefill(x, perm, wp, wsc, N, n_vis, s_vis, s_txt, block, ws, out=y)
        out.append(y)
    return out


def _run_attention(st):
    hq, hkv = st["heads"]
    qkv = st["qkv"]
    if st["case"]["project"]:
        (wp, wsc), (s_vis, s_txt) = st["w"], st["s"]
        mq.w4a8_linear_prefill(st["x"], st["perm"], wp, wsc, qkv.shape[1], st["n_vis"], s_vis, s_txt, st["block"],
                               st["lws"], out=qkv)
        mq.rope_apply(qkv[:, :(hq + hkv) * HEAD_DIM], st["perm"], hq + hkv)
    q, k, v = qkv[:, :hq * HEAD_DIM], qkv[:, hq * HEAD_DIM:(hq + hkv) * HEAD_DIM], qkv[:, (hq + hkv) * HEAD_DIM:]
    o = mq.aifs_attention(q, k, v, st["perm"], hq, hkv, out=st["o"], workspace=st["ws"])
    return (qkv, o) if st["case"]["project"] else o


def _run_weight_only(st):
    return [mq.w4g128_gemm(x, wp, N, out=y) for x, wp, N, y in st["lin"]]


_RUN = {"linear": _run_linear, "decode": _run_decode, "prefill": _run_prefill, "attention": _run_attention,
        "weight_only": _run_weight_only}


# ---------------------------------------------------------------------------- what it must cost

def work(case):
    """16-bit inputs and outputs and 4-bit weights once each; two operations per multiply-add."""
    T, kind = case["T"], case["kind"]

    def linears(shapes):
        return (sum(K * N / 2 + 2 * N + 2 * T * N for K, N in shapes),
                sum(2.0 * T * K * N for K, N in shapes))

    if kind == "linear":
        K, N = case["K"], case["N"]
        b, f = linears([(K, N)])
        return {"bytes": b + 2 * T * K + 4 * T, "flops": f}
    _, hq, hkv, proj = MODELS[case["model"]]
    if kind == "attention":
        b, f = 2 * T * (2 * hq + 2 * hkv) * HEAD_DIM + 4 * T, 2.0 * HEAD_DIM * hq * T * (T + 1)
        if case["project"]:
            K, N = proj["qkv"]
            lb, lf = linears([(K, N)])
            b, f = 2 * T * hq * HEAD_DIM + 4 * T + lb + 2 * T * K, f + lf
        return {"bytes": b, "flops": f}
    b, f = linears(proj.values())
    x = 2 * T * sum(K for K, _ in proj.values())
    if kind == "decode":
        return {"bytes": case["layers"] * (b + x), "flops": case["layers"] * f}
    if kind == "weight_only":
        return {"bytes": b + x + sum(2 * N * (K // 128) for K, N in proj.values()), "flops": f}
    split = case["n_split"] * proj["down"][1]
    return {"bytes": b + x + split + 2 * T * T + 2 * T * proj["qkv"][0] + 4 * T, "flops": f + 2.0 * T * split}


def tolerance(case):
    kind = case["kind"]
    if kind in ("linear", "decode") or (kind == "prefill" and case["scheme"] != "rms"):
        # integer sums, then a defined sequence of roundings: every output bit is specified
        return "exact"
    # Four times what the path is off a 64-bit evaluation of the same operands by (2.1e-4 and 4.9e-4
    # with fp32 sums and an fp16 result: weight-only linears, flagged-channel terms, RoPE; 2.6e-4 and
    # 3.1e-3 with the fp16 probabilities of attention).
    if kind == "attention":
        return {"rel": 1e-3, "max": 1.2e-2}
    return {"rel": 8e-4, "max": 2e-3}

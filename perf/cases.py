"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is a dict of plain values.  ``listed()`` gives the fixed ones, ``draw(rng)`` another one of the same ranges;
``prepare(case, seed)`` makes what a program has in hand before the call, ``run(state)`` makes one pass through the
public entry points.  Kinds of case:

  core_prefill     conv1d + selective scan of one layer over a context (the repository's headline measurement)
  core_decode      draft steps of the layer core: every step forks the states of all live branches by parent index and
                   advances them, layer by layer; replayed as a HIP graph, or launched call by call
  drafter_prefill  a whole 24-block drafter encodes a prompt
  drafter_draft    the whole drafter drafts one token tree (captured once per tree shape, as MambaDrafter does)
  block_prefill    one whole Mamba block over a batch of contexts
  ssd_prefill      scalar-decay (Mamba-2 style) layer core over a context
  ssd_step         one scalar-decay state update of all live branches

Distributions are those of ``paper_2506_01206_amd.synth`` and ``bench.py``, drawn on the device.
"""
import math

import torch

from paper_2506_01206_amd import binding as m
from paper_2506_01206_amd.drafter import MambaDrafter

DEV = "cuda:0"
K = 4                                  # conv taps
N = 16                                 # states per channel
VOCAB, LAYERS, D_MODEL, D_INNER, DT_RANK = 50280, 24, 768, 1536, 48
SSD_H, SSD_P, SSD_N = 24, 64, 128
LARGEST = 8 * 8192 * 4096              # channel-tokens of the largest context
TYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # a small layer in float32, short context: what a unit test or a tiny drafter calls; launches and host work count
        dict(name="core_prefill_256_f32", kind="core_prefill", io="f32", batch=1, L=256, D=256),
        # the context length of an ordinary chat prompt on a 130M-shaped layer
        dict(name="core_prefill_2k", kind="core_prefill", io="bf16", batch=1, L=2048, D=1536),
        # long-context encoding, the headline prefill
        dict(name="core_prefill_32k", kind="core_prefill", io="bf16", batch=1, L=32768, D=1536),
        # a batch of contexts on a 1.4B-shaped layer: the largest call
        dict(name="core_prefill_8x8k_wide", kind="core_prefill", io="bf16", batch=8, L=8192, D=4096),
        # tree decode over all layers, the headline decode: fixed shapes, so the program keeps a graph of it
        dict(name="core_decode_32x24", kind="core_decode", io="bf16", branches=32, layers=24, steps=5, D=1536, graph=True),
        # decode of one wide layer launched call by call, as a program does whose branch count changes as it goes
        dict(name="core_decode_64_wide", kind="core_decode", io="bf16", branches=64, layers=1, steps=8, D=4096, graph=False),
        # a short prompt of no particular length, and a long one
        dict(name="drafter_prefill_333", kind="drafter_prefill", L=333),
        dict(name="drafter_prefill_8000", kind="drafter_prefill", L=8000),
        # one draft round of the default tree
        dict(name="drafter_draft_3_2_2_1_1", kind="drafter_draft", tree="3,2,2,1,1"),
        # one block of a long-context encoding
        dict(name="block_prefill_32k", kind="block_prefill", batch=1, L=32768),
        # a Mamba-2 style drafter's layer: an ordinary context, and one draft step of 64 branches
        dict(name="ssd_prefill_2k", kind="ssd_prefill", batch=1, L=2048),
        dict(name="ssd_step_64", kind="ssd_step", branches=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("core_prefill", "core_prefill", "core_decode", "drafter_prefill", "drafter_prefill", "drafter_draft",
                       "block_prefill", "ssd_prefill", "ssd_step"))
    if kind == "core_prefill":
        # widths in steps of 8 channels (what d_inner of a real layer is a multiple of), any number of tokens
        D = 8 * _log_int(rng, 32, 512)
        batch = _log_int(rng, 1, 16)
        L = _log_int(rng, 64, min(32768, LARGEST // (2 * D * batch)))
        return dict(kind=kind, io=rng.choice(("bf16", "bf16", "bf16", "f32")), batch=batch, L=L, D=D)
    if kind == "core_decode":
        graph = rng.random() < 0.5
        return dict(kind=kind, io="bf16", branches=_log_int(rng, 1, 128), layers=rng.choice((4, 12, 24)) if graph else 1,
                    steps=rng.randint(3, 8), D=8 * _log_int(rng, 96, 512), graph=graph)
    if kind == "drafter_prefill":
        return dict(kind=kind, L=_log_int(rng, 32, 8000))
    if kind == "drafter_draft":
        tree, width = [], 1
        for _ in range(rng.randint(3, 6)):
            n = rng.choice((1, 1, 2, 2, 3))
            n = n if width * n <= 32 else 1
            width *= n
            tree.append(n)
        return dict(kind=kind, tree=",".join(str(n) for n in tree))
    if kind == "block_prefill":
        batch = _log_int(rng, 1, 8)
        return dict(kind=kind, batch=batch, L=_log_int(rng, 256, 32768 // batch))
    if kind == "ssd_prefill":
        batch = _log_int(rng, 1, 4)
        return dict(kind=kind, batch=batch, L=_log_int(rng, 128, 32768 // batch))
    return dict(kind="ssd_step", branches=_log_int(rng, 1, 128))


# ----------------------------------------------------------------------------------------------------------- inputs
class _Draws:
    def __init__(self, seed):
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(int(seed))

    def normal(self, *shape, std=1.0, dtype=torch.float32):
        return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=self.gen)

    def uniform(self, lo, hi, *shape):
        return torch.empty(shape, device=DEV).uniform_(lo, hi, generator=self.gen)

    def ints(self, hi, *shape):
        return torch.randint(0, hi, shape, device=DEV, generator=self.gen, dtype=torch.int32)

    def dt_bias(self, D):
        dt0 = torch.exp(self.uniform(math.log(1e-3), math.log(0.1), D))
        return dt0 + torch.log(-torch.expm1(-dt0))

    def layer(self, D):
        """Parameters of one layer core: A = -(1..16) perturbed as training does, D = 1, conv weights U(-0.5, 0.5)."""
        A = -torch.arange(1, N + 1, device=DEV, dtype=torch.float32) * torch.exp(0.1 * self.normal(D, N))
        return dict(A=A.contiguous(), Dskip=torch.ones(D, device=DEV), dt_bias=self.dt_bias(D),
                    conv_w=self.uniform(-0.5, 0.5, D, K), conv_bias=0.1 * self.normal(D))

    def tokens(self, lead, D, dtype):
        """x, z, B, C ~ N(0,1), dt ~ N(0, std 0.1) for the layer core."""
        return dict(x=self.normal(*lead, D, dtype=dtype), z=self.normal(*lead, D, dtype=dtype),
                    Bm=self.normal(*lead, N, dtype=dtype), Cm=self.normal(*lead, N, dtype=dtype),
                    dt=self.normal(*lead, D, std=0.1, dtype=dtype))

    def block(self):
        bf = torch.bfloat16
        p = self.layer(D_INNER)
        return m.Block(dict(
            norm_w=1 + 0.1 * self.normal(D_MODEL), conv_w=p["conv_w"], conv_b=p["conv_bias"], dt_bias=p["dt_bias"],
            A=p["A"], Dskip=p["Dskip"],
            in_proj_w=self.normal(2 * D_INNER, D_MODEL, std=D_MODEL ** -0.5, dtype=bf),
            x_proj_w=self.normal(DT_RANK + 2 * N, D_INNER, std=D_INNER ** -0.5, dtype=bf),
            dt_proj_w=self.normal(D_INNER, DT_RANK, std=DT_RANK ** -0.5, dtype=bf),
            out_proj_w=self.normal(D_MODEL, D_INNER, std=D_INNER ** -0.5, dtype=bf)))

    def drafter(self):
        """A 24-block drafter.  A trained model's next-token distribution is peaked; random weights alone would leave the
        candidates of a draft tree within rounding of each other.  So the LM head is given every token's likely
        successors: row w is a weighted sum of the embeddings of the tokens that w tends to follow."""
        bf = torch.bfloat16
        emb = self.normal(VOCAB, D_MODEL, std=2.0)
        head = torch.zeros_like(emb)
        for j in range(3):
            order = torch.randperm(VOCAB, device=DEV, generator=self.gen)
            head += emb[order] * (0.7 ** j / 2.0 / D_MODEL ** 0.5)
        return MambaDrafter(emb.to(bf), [self.block() for _ in range(LAYERS)], torch.ones(D_MODEL, device=DEV), head.to(bf))


def prepare(case, seed):
    r = _Draws(seed)
    kind = case["kind"]
    s = dict(case=dict(case))
    if kind == "core_prefill":
        B, L, D, dtype = case["batch"], case["L"], case["D"], TYPES[case["io"]]
        s["p"], s["t"] = r.layer(D), r.tokens((B, L), D, dtype)
        s["xc"], s["out"] = torch.empty_like(s["t"]["x"]), torch.empty_like(s["t"]["x"])
        s["conv_state"] = torch.empty((B, D, K - 1), dtype=dtype, device=DEV)
        s["h"] = torch.empty((B, D, N), device=DEV)
        s["ws"] = torch.empty(max(m.mamba_scan_workspace_bytes(B, L, D, N), 16), dtype=torch.uint8, device=DEV)
    elif kind == "core_decode":
        nb, nl, ns, D, dtype = case["branches"], case["layers"], case["steps"], case["D"], TYPES[case["io"]]
        s["p"] = [r.layer(D) for _ in range(nl)]
        s["ssm"] = [r.normal(nl, nb, D, N)] + [torch.empty((nl, nb, D, N), device=DEV) for _ in range(2)]
        s["conv"] = [r.normal(nl, nb, D, K - 1, dtype=dtype)] + [torch.empty((nl, nb, D, K - 1), dtype=dtype, device=DEV)
                                                                 for _ in range(2)]
        s["parents"] = [r.ints(nb, nb) for _ in range(ns)]
        s["t"] = [[r.tokens((nb,), D, dtype) for _ in range(nl)] for _ in range(ns)]
        s["out"] = torch.empty((ns, nl, nb, D), dtype=dtype, device=DEV)
        if case["graph"]:
            _decode(s)
            graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                with torch.cuda.graph(graph, stream=side):
                    _decode(s)
            torch.cuda.current_stream().wait_stream(side)
            s["graph"] = graph
    elif kind == "drafter_prefill":
        s["drafter"], s["prompt"] = r.drafter(), r.ints(VOCAB, case["L"])
    elif kind == "drafter_draft":
        s["drafter"] = r.drafter()
        s["drafter"].prefill(r.ints(VOCAB, 64))
        s["tree"] = tuple(int(n) for n in case["tree"].split(","))
        s["drafter"].draft(s["tree"])                       # captures the round
    elif kind == "block_prefill":
        B, L = case["batch"], case["L"]
        s["block"] = r.block()
        s["hidden"] = r.normal(B, L, D_MODEL, dtype=torch.bfloat16)
        s["out"] = torch.empty_like(s["hidden"])
        s["conv_state"] = torch.empty((B, D_INNER, K - 1), dtype=torch.bfloat16, device=DEV)
        s["h"] = torch.empty((B, D_INNER, N), device=DEV)
        s["ws"] = torch.empty(max(m.mamba_block_workspace_bytes(s["block"], B, L), 16), dtype=torch.uint8, device=DEV)
    else:
        bf = torch.bfloat16
        lead = (case["batch"], case["L"]) if kind == "ssd_prefill" else (case["branches"],)
        s["x"], s["z"] = r.normal(*lead, SSD_H, SSD_P, dtype=bf), r.normal(*lead, SSD_H, SSD_P, dtype=bf)
        s["dt"] = r.normal(*lead, SSD_H, std=0.5, dtype=bf)
        s["Bm"], s["Cm"] = r.normal(*lead, SSD_N, dtype=bf), r.normal(*lead, SSD_N, dtype=bf)
        s["A"] = r.uniform(-1.5, -0.05, SSD_H)
        s["Dskip"], s["dt_bias"] = torch.ones(SSD_H, device=DEV), torch.full((SSD_H,), -2.5, device=DEV)
        s["out"] = torch.empty_like(s["x"])
        s["h"] = torch.empty((lead[0], SSD_H, SSD_P, SSD_N), device=DEV)
        if kind == "ssd_prefill":
            s["ws"] = torch.empty(max(m.mamba2_ssd_workspace_bytes(*lead, SSD_H, SSD_P, SSD_N), 16), dtype=torch.uint8, device=DEV)
        else:
            s["h_in"], s["parents"] = r.normal(*s["h"].shape), r.ints(lead[0], lead[0])
    return s


# ------------------------------------------------------------------------------------------------------------ passes
def _decode(s):
    src = 0
    for i, parents in enumerate(s["parents"]):
        dst = 1 + (i & 1)
        for l, p in enumerate(s["p"]):
            t = s["t"][i][l]
            m.mamba_conv_state_step(s["ssm"][src][l], s["conv"][src][l], t["x"], p["conv_w"], p["conv_bias"], t["dt"], p["A"],
                                    t["Bm"], t["Cm"], p["Dskip"], t["z"], p["dt_bias"], parent_idx=parents,
                                    h_out=s["ssm"][dst][l], conv_state_out=s["conv"][dst][l], out=s["out"][i, l])
        src = dst
    return src


def run(s):
    kind = s["case"]["kind"]
    if kind == "core_prefill":
        p, t = s["p"], s["t"]
        m.mamba_conv1d_fwd(t["x"], p["conv_w"], p["conv_bias"], y=s["xc"], conv_state_out=s["conv_state"])
        m.mamba_scan_fwd(s["xc"], t["dt"], p["A"], t["Bm"], t["Cm"], p["Dskip"], t["z"], p["dt_bias"], out=s["out"],
                         h_final=s["h"], workspace=s["ws"])
        return s["xc"], s["conv_state"], s["out"], s["h"]
    if kind == "core_decode":
        if "graph" in s:
            s["graph"].replay()
        else:
            _decode(s)
        last = 1 + ((len(s["parents"]) - 1) & 1)
        return s["out"], s["ssm"][last], s["conv"][last]
    if kind == "drafter_prefill":
        d = s["drafter"]
        return d.prefill(s["prompt"]), d.root_conv, d.root_ssm
    if kind == "drafter_draft":
        return s["drafter"].draft(s["tree"])
    if kind == "block_prefill":
        return m.mamba_block_fwd(s["block"], s["hidden"], hidden_out=s["out"], conv_state_out=s["conv_state"],
                                 h_final=s["h"], workspace=s["ws"])
    if kind == "ssd_prefill":
        return m.mamba2_ssd_fwd(s["x"], s["dt"], s["A"], s["Bm"], s["Cm"], s["Dskip"], s["z"], s["dt_bias"], out=s["out"],
                                h_final=s["h"], workspace=s["ws"])
    return m.mamba2_state_step(s["h_in"], s["x"], s["dt"], s["A"], s["Bm"], s["Cm"], s["Dskip"], s["z"], s["dt_bias"],
                               parent_idx=s["parents"], h_out=s["h"], out=s["out"])


# ------------------------------------------------------------------------------------------------------- bare minimum
def _update_flops(channel_tokens):
    """One state update is 7 operations (delta A, exp, delta x B, two fused multiply-adds), a token of a channel 15."""
    return channel_tokens * (7 * N + 15)


_BLOCK_MACS = 2 * D_INNER * D_MODEL + (DT_RANK + 2 * N) * D_INNER + D_INNER * DT_RANK + D_MODEL * D_INNER
_BLOCK_BYTES = 2 * _BLOCK_MACS + 4 * D_INNER * (N + K + 3) + 4 * D_MODEL


def _block_flops(tokens):
    return 2 * _BLOCK_MACS * tokens + _update_flops(tokens * D_INNER) + 2 * K * tokens * D_INNER


def work(case):
    kind = case["kind"]
    e = 4 if case.get("io") == "f32" else 2
    state = lambda D: 4 * D * N                           # bytes of one branch's SSM state
    if kind == "core_prefill":
        B, L, D = case["batch"], case["L"], case["D"]
        # conv: x in, x_c out; scan: dt, z in, out written, B and C; the final states
        return dict(bytes=B * L * (5 * D + 2 * N) * e + B * (state(D) + D * (K - 1) * e) + 4 * D * (N + K + 3),
                    flops=_update_flops(B * L * D) + 2 * K * B * L * D)
    if kind == "core_decode":
        nb, nl, ns, D = case["branches"], case["layers"], case["steps"], case["D"]
        # every step reads and writes all states (they do not stay on the chip between calls)
        per = nb * (2 * state(D) + (2 * (K - 1) * D + 4 * D + 2 * N) * e) + 4 * D * (N + K + 3)
        return dict(bytes=ns * nl * per, flops=ns * nl * (_update_flops(nb * D) + 2 * K * nb * D))
    if kind == "drafter_prefill":
        L = case["L"]
        return dict(bytes=LAYERS * (_BLOCK_BYTES + state(D_INNER) + 2 * D_INNER * (K - 1)) + 2 * VOCAB * D_MODEL
                    + 2 * L * D_MODEL + 4 * L, flops=LAYERS * _block_flops(L) + 2 * VOCAB * D_MODEL)
    if kind == "drafter_draft":
        total, width, nbytes = 0, 1, 0
        for n in case["tree"].split(","):
            width *= int(n)
            total += width
            nbytes += LAYERS * (_BLOCK_BYTES + 2 * width * (state(D_INNER) + 2 * D_INNER * (K - 1))) + 2 * VOCAB * (D_MODEL + width)
        return dict(bytes=nbytes, flops=LAYERS * _block_flops(total) + 2 * VOCAB * D_MODEL * total)
    if kind == "block_prefill":
        T = case["batch"] * case["L"]
        return dict(bytes=4 * T * D_MODEL + _BLOCK_BYTES + case["batch"] * (state(D_INNER) + 2 * D_INNER * (K - 1)),
                    flops=_block_flops(T))
    T = case["batch"] * case["L"] if kind == "ssd_prefill" else case["branches"]
    rows = case["batch"] if kind == "ssd_prefill" else 2 * case["branches"]
    return dict(bytes=2 * T * (3 * SSD_H * SSD_P + SSD_H + 2 * SSD_N) + 4 * rows * SSD_H * SSD_P * SSD_N,
                flops=T * SSD_H * (6 * SSD_P * SSD_N + 10 * SSD_P))


def tolerance(case):
    """float32 arithmetic in another order, then what the storage type of the results rounds away; in the whole drafter the
    tensors between the stages are stored too, and 24 blocks add up what that rounds away (an input changed by less than a
    bf16 step moves the results by 1e-2).  Draft tokens are whole numbers and stay the same."""
    if case["kind"] in ("drafter_prefill", "drafter_draft"):
        return {"rel": 2e-2}
    if case.get("io") == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2}

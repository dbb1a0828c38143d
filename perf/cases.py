"""The work that programs built on this library have it do, as cases that can be timed and compared.

Four kinds of pass, each through the public C ABI as its binding exposes it:

  train       one step of the registered training instance: forward, loss, backward, update
  infer       a group of inference requests from submission to the last completed ticket, no training beside them
  collocated  training steps with their communication bubbles, and offline requests that are filled into these
  stack       a training step of a layer stack without embedding (a pipeline stage's or tensor shard's share)

All states of one process share one pair of streams, as one program does, so passes follow each other on the device.
Model sizes are those of the configurations in synth_inputs.py and of the tests, or generic ones of their kind.
"""
import ctypes as C
import math

import torch

import paper_2503_02550_amd as B
from paper_2503_02550_amd import params as P

DEV = "cuda:0"


# ---- cases -------------------------------------------------------------------------------------------------------
def _mlp(**kw):
    return dict(dict(model="mlp", d_in=256, d_hidden=256, d_out=256), **kw)


def _encoder(**kw):
    return dict(dict(model="encoder", n_layers=12, d_model=768, n_heads=12, d_head=64, d_ffn=3072, vocab=30522, max_pos=512), **kw)


def _decoder(**kw):
    return dict(dict(model="decoder", n_layers=12, d_model=768, n_heads=12, d_head=64, d_ffn=3072, vocab=50257, max_pos=1024, micro=1), **kw)


def listed():
    return [
        # the Tiny configuration's training step and inference batch: a handful of launches, nothing but latency
        _mlp(name="mlp_train", kind="train", batch=32),
        _mlp(name="mlp_infer", kind="infer", online=False, requests=1, batch=8, seq_min=1, seq_max=1),
        # one online request as it arrives at an idle instance: batch 1, an odd length in the middle of 32..256
        _encoder(name="online_one", kind="infer", online=True, requests=1, batch=1, seq_min=77, seq_max=77),
        # what piles up while a bubble is awaited: eight online requests of different lengths
        _encoder(name="online_eight", kind="infer", online=True, requests=8, batch=1, seq_min=32, seq_max=256),
        # one offline batch of the fill encoder, and a deep queue of them (as the benchmark keeps it)
        _encoder(name="offline_one", kind="infer", online=False, requests=1, batch=32, seq_min=128, seq_max=128),
        _encoder(name="offline_queue", kind="infer", online=False, requests=32, batch=32, seq_min=128, seq_max=128),
        # a small decoder with heads of 32 (attention through its three separate kernels): launch-bound training
        _decoder(name="train_small", kind="train", n_layers=2, d_model=128, n_heads=4, d_head=32, d_ffn=512, vocab=300, max_pos=64, batch=4, seq=64),
        # a middle-sized step whose tokens, vocabulary and widths fall on no tile boundary
        _decoder(name="train_odd", kind="train", n_layers=6, d_model=520, n_heads=8, d_head=64, d_ffn=2056, vocab=10007, max_pos=512, batch=8, seq=251),
        # the data-parallel rank share: the benchmark's training step without its bubble
        _decoder(name="train_dp", kind="train", batch=8, seq=1024),
        # a pipeline stage's share: six wide layers, heads of 128, gradients accumulated over two micro-batches
        _decoder(name="stack_pp", kind="stack", n_layers=6, d_model=2048, n_heads=16, d_head=128, d_ffn=8192, vocab=0, max_pos=0, batch=2, seq=2048, micro=2),
        # a tensor shard's share: d 4096 with an eighth of the heads and of the feed-forward columns
        _decoder(name="stack_tp", kind="stack", n_layers=24, d_model=4096, n_heads=4, d_head=128, d_ffn=2048, vocab=0, max_pos=0, batch=4, seq=2048),
        # the whole idea: two data-parallel steps, each with its 4.98 ms bubble, and five offline batches served inside these
        _decoder(name="collocated_dp", kind="collocated", batch=8, seq=1024, steps=2, requests=5, fill_batch=32, fill_seq=128),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw(rng):
    pick = rng.random()
    if pick < 0.12:
        return _mlp(kind="train", d_in=_log(rng, 64, 1024), d_hidden=_log(rng, 64, 1024), d_out=_log(rng, 64, 1024), batch=_log(rng, 1, 512))
    if pick < 0.2:
        return _mlp(kind="infer", online=False, requests=rng.randint(1, 4), batch=_log(rng, 1, 256), seq_min=1, seq_max=1,
                    d_in=_log(rng, 64, 1024), d_hidden=_log(rng, 64, 1024), d_out=_log(rng, 64, 1024))
    if pick < 0.55:
        heads = rng.choice((4, 8, 12, 16))
        enc = dict(n_layers=rng.randint(2, 12), n_heads=heads, d_model=64 * heads, d_ffn=256 * heads)
        if rng.random() < 0.5:
            lo = _log(rng, 16, 256)
            return _encoder(kind="infer", online=True, requests=rng.randint(1, 8), batch=1, seq_min=lo, seq_max=min(512, lo + _log(rng, 1, 256)), **enc)
        seq = _log(rng, 16, 512)
        batch = _log(rng, 1, 64)
        return _encoder(kind="infer", online=False, requests=_log(rng, 1, 32), batch=batch, seq_min=seq, seq_max=seq, **enc)
    if pick < 0.8:
        d_head = rng.choice((32, 64, 64, 128))
        heads = rng.choice((2, 4, 8, 12)) * (2 if d_head == 32 else 1)
        d = 8 * rng.randint(max(1, heads * d_head // 10), heads * d_head // 6)      # not always the heads' whole width
        seq = _log(rng, 32, 512 if d_head == 32 else 2048)
        batch = 8 // math.gcd(8, seq) * rng.randint(1, max(1, 8 * math.gcd(8, seq) // 8))
        vocab = _log(rng, 200, 50257)
        return _decoder(kind="train", n_layers=rng.randint(1, 12), d_model=d, n_heads=heads, d_head=d_head, d_ffn=8 * rng.randint(d // 4, d // 2), vocab=vocab,
                        max_pos=seq, batch=batch, seq=seq)
    if pick < 0.93:
        heads = rng.choice((2, 4, 8, 16))
        seq = 8 * _log(rng, 16, 256)
        return _decoder(kind="stack", n_layers=rng.randint(1, 6), d_model=128 * rng.randint(4, 32), n_heads=heads, d_head=128, d_ffn=128 * rng.randint(8, 64),
                        vocab=0, max_pos=0, batch=rng.randint(1, 4), seq=seq, micro=rng.randint(1, 4))
    return _decoder(kind="collocated", n_layers=rng.randint(8, 12), batch=rng.randint(2, 8), seq=8 * _log(rng, 16, 128), steps=2, requests=rng.randint(1, 4),
                    fill_batch=_log(rng, 4, 24), fill_seq=_log(rng, 16, 144))


def draw(rng):
    most = max(work(c)["flops"] for c in listed())
    while True:
        c = _draw(rng)
        tokens = c["batch"] * c.get("seq", c.get("seq_max", 1)) * c.get("requests", 1) * c.get("micro", 1)
        if work(c)["flops"] <= 0.8 * most and tokens <= 131072:
            return c


# ---- shapes, and the work a pass cannot do without ----------------------------------------------------------------
def _shape(c):
    if c["model"] == "mlp":
        return P.make_shape(B.SIF_MODEL_MLP, B.SIF_F32, d_in=c["d_in"], d_hidden=c["d_hidden"], d_out=c["d_out"], batch=c["batch"])
    return P.make_shape(B.SIF_MODEL_DECODER if c["model"] == "decoder" else B.SIF_MODEL_ENCODER, B.SIF_BF16, n_layers=c["n_layers"], d_model=c["d_model"],
                        n_heads=c["n_heads"], d_head=c["d_head"], d_ffn=c["d_ffn"], vocab=c["vocab"], max_pos=c["max_pos"], batch=c["batch"],
                        seq=c.get("seq", c.get("seq_max")))


def _fill_case(c):
    return _encoder(kind="infer", online=False, requests=c["requests"], batch=c["fill_batch"], seq_min=c["fill_seq"], seq_max=c["fill_seq"])


def _lengths(c):
    n = c["requests"]
    return [c["seq_min"] + (c["seq_max"] - c["seq_min"]) * i // max(1, n - 1) for i in range(n)]


def work(c):
    """Every parameter, input and output once (a training step: fp32 master read and written, gradient written), and the
    products of the model's definition; backward counts twice forward.  A bubble's waiting is no work."""
    n = B.sif_model_n_params(_shape(c))
    if c["model"] == "mlp":
        w1, w2, b = c["d_in"] * c["d_hidden"], c["d_hidden"] * c["d_out"], c["batch"]
        if c["kind"] == "train":
            return {"bytes": 12.0 * n + 4.0 * b * (c["d_in"] + c["d_out"]), "flops": 2.0 * b * (2 * w1 + 3 * w2)}
        return {"bytes": 4.0 * n + 4.0 * b * c["requests"] * (c["d_in"] + c["d_out"]), "flops": 2.0 * b * c["requests"] * (w1 + w2)}
    d, da, f = c["d_model"], c["n_heads"] * c["d_head"], c["d_ffn"]
    per_token = 2.0 * c["n_layers"] * (4 * d * da + 2 * d * f)
    if c["kind"] == "infer":
        seqs = [s * c["batch"] for s in _lengths(c)]
        attention = sum(4.0 * c["n_layers"] * da * s * t for s, t in zip(_lengths(c), seqs))
        tokens = sum(seqs)
        layers = n - (c["vocab"] + c["max_pos"]) * d
        return {"bytes": 2.0 * layers + tokens * (4.0 + 2.0 * d) + 2.0 * d * min(tokens, c["vocab"]), "flops": per_token * tokens + attention}
    tokens = c["batch"] * c["seq"] * c["micro"]
    forward = tokens * (per_token + 2.0 * c["n_layers"] * da * c["seq"] + 2.0 * d * c["vocab"])
    got = {"bytes": 10.0 * n + tokens * (8.0 if c["vocab"] else 8.0 * d), "flops": 3.0 * forward}
    if c["kind"] == "collocated":
        fill = work(_fill_case(c))
        got = {k: c["steps"] * got[k] + fill[k] for k in got}
    return got


def tolerance(c):
    if c["model"] == "mlp":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 2e-2, "max": 0.5}


# ---- what a program has in hand -----------------------------------------------------------------------------------
_pair = []


class Program:
    """A context with its registered models and the device memory it works in; gives the context back when dropped."""

    def __init__(self, cfg):
        self.ctx, self.keep = None, []
        need = B.sif_ctx_workspace_bytes()
        ws = self.bytes(need)
        for _ in range(16):
            if not _pair:
                _pair[:] = [torch.cuda.Stream(device=DEV), torch.cuda.Stream(device=DEV)]
            try:
                self.ctx = B.sif_create(cfg, _pair[0], _pair[1], ws, need)
                return
            except B.SifError as e:
                if e.status != B.SIF_E_AGAIN:
                    raise
                _pair.clear()      # the two streams share a hardware queue
        raise RuntimeError("no pair of concurrent streams found")

    def bytes(self, n):
        t = torch.zeros(int(n) + 256, dtype=torch.uint8, device=DEV)
        self.keep.append(t)
        off = -t.data_ptr() % 256
        return t[off:off + int(n)]

    def train(self, shape, master, par_mode=B.SIF_PAR_NONE, micro=1, bw=0):
        d = B.sif_train_desc()
        d.struct_size = C.sizeof(d)
        d.par_mode, d.shape, d.lr, d.bw_bytes_per_s = par_mode, shape, 0.01, bw
        if par_mode == B.SIF_PAR_PP:
            d.pp_stages, d.pp_micro, d.pp_stage = 1, micro, 0
        d.workspace_bytes = B.sif_train_workspace_bytes(d)
        ws = self.bytes(d.workspace_bytes)
        torch.cuda.synchronize()
        d.master_dev, d.workspace_dev = master.data_ptr(), ws.data_ptr()
        self.step = B.sif_register_training_step(self.ctx, d)
        self.keep.append(master)
        self.outputs = {"master": master}
        kind = torch.float32 if shape.kind == B.SIF_MODEL_MLP else torch.bfloat16
        for name in ("grads",) + (("y_all", "dx_all") if par_mode == B.SIF_PAR_PP else ()):
            addr, n = B.sif_train_tensor(self.ctx, self.step, name)
            raw = ws[addr - ws.data_ptr():]
            self.outputs[name] = raw[:n * torch.empty((), dtype=kind).element_size()].view(kind)

    def serve(self, shape, master, online, coalesce):
        d = B.sif_infer_desc()
        d.struct_size = C.sizeof(d)
        d.online, d.shape, d.coalesce = int(online), shape, coalesce
        d.workspace_bytes = B.sif_infer_workspace_bytes(d)
        ws = self.bytes(d.workspace_bytes)
        torch.cuda.synchronize()
        d.master_dev, d.workspace_dev, d.peak_bytes = master.data_ptr(), ws.data_ptr(), d.workspace_bytes + 4 * master.numel()
        self.keep.append(master)
        return B.sif_register_inference_model(self.ctx, d)

    def __del__(self):
        if self.ctx is not None:
            B.sif_destroy(self.ctx)
            self.ctx = None


def _weights(shape, gen):
    """fp32 parameters: N(0, 0.02) around 0, LayerNorm gains around 1."""
    flat = torch.randn(B.sif_model_n_params(shape), device=DEV, generator=gen) * 0.02
    at = 0
    for path, extent in P.layout(shape):
        n = math.prod(extent)
        if (path if isinstance(path, str) else path[2]).endswith("_g"):
            flat[at:at + n] += 1.0
        at += n
    return flat


def _ids(gen, vocab, *extent):
    return torch.randint(0, vocab, extent, device=DEV, dtype=torch.int32, generator=gen)


def _requests(c, gen):
    """[(input, output, batch, seq)] of a case's inference requests."""
    got = []
    for s in _lengths(c):
        if c["model"] == "mlp":
            got.append((torch.randn(c["batch"], c["d_in"], device=DEV, generator=gen), torch.zeros(c["batch"], c["d_out"], device=DEV), c["batch"], 1))
        else:
            got.append((_ids(gen, c["vocab"], c["batch"], s), torch.zeros(c["batch"], s, c["d_model"], device=DEV, dtype=torch.bfloat16), c["batch"], s))
    return got


def prepare(c, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    cfg = B.sif_default_config()
    cfg.kernel_us_max = 1200      # as the benchmark sets it for long bubbles
    p = Program(cfg)
    shape = _shape(c)
    state = {"case": c, "program": p}
    if c["kind"] == "infer":
        state["model"] = p.serve(shape, _weights(shape, gen), c["online"], min(32, c["requests"]))
        state["requests"] = _requests(c, gen)
    else:
        mode = B.SIF_PAR_PP if c["kind"] == "stack" else B.SIF_PAR_DP if c["kind"] == "collocated" else B.SIF_PAR_NONE
        p.train(shape, _weights(shape, gen), mode, c.get("micro", 1), 50_000_000_000 if mode == B.SIF_PAR_DP else 0)
        state["loss"] = torch.zeros(1, device=DEV)
        if c["model"] == "mlp":
            state["in"] = torch.randn(c["batch"], c["d_in"], device=DEV, generator=gen)
            state["target"] = torch.randn(c["batch"], c["d_out"], device=DEV, generator=gen)
        elif c["vocab"]:
            state["in"], state["target"] = (_ids(gen, c["vocab"], c["batch"], c["seq"]) for _ in range(2))
        else:
            extent = (c["micro"], c["batch"], c["seq"], c["d_model"])
            state["in"] = torch.randn(extent, device=DEV, generator=gen).to(torch.bfloat16)
            state["target"] = (torch.randn(extent, device=DEV, generator=gen) / math.sqrt(math.prod(extent[1:]))).to(torch.bfloat16)
        if c["kind"] == "collocated":
            fill = _fill_case(c)
            eshape = _shape(fill)
            state["model"] = p.serve(eshape, _weights(eshape, gen), False, 8)
            state["requests"] = _requests(fill, gen)
            torch.cuda.synchronize()
            B.sif_calibrate(p.ctx, 1, state["in"], state["target"])
    torch.cuda.synchronize()
    return state


# ---- one pass -----------------------------------------------------------------------------------------------------
def _submit(state):
    ctx, model = state["program"].ctx, state["model"]
    if state["case"].get("online"):
        return [B.sif_submit_online_request(ctx, model, i, o, s) for i, o, _, s in state["requests"]]
    return [B.sif_submit_offline_batch(ctx, model, i, o, b, s) for i, o, b, s in state["requests"]]


def run(state):
    p, kind = state["program"], state["case"]["kind"]
    outputs = {}
    if kind in ("infer", "collocated"):
        tickets = _submit(state)
        outputs["answers"] = [o for _, o, _, _ in state["requests"]]
    if kind != "infer":
        for _ in range(state["case"].get("steps", 1)):
            B.sif_run_training_step(p.ctx, p.step, state["in"], state["target"], None if kind == "stack" else state["loss"])
        outputs.update(p.outputs)
        if kind != "stack":
            outputs["loss"] = state["loss"]
    while kind != "train" and kind != "stack" and tickets:
        try:
            B.sif_wait(p.ctx, tickets[0], 10_000_000_000 if kind == "infer" else 100_000_000)
            tickets.pop(0)
        except B.SifError as e:
            if kind == "infer" or e.status != B.SIF_E_TIMEOUT:
                raise
            # training goes on while requests wait for a bubble with room for them
            B.sif_run_training_step(p.ctx, p.step, state["in"], state["target"], state["loss"])
    return outputs

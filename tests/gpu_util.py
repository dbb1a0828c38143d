"""Helpers for the GPU parity tests: tensor marshalling and the comparison bars.

Bars (per tensor): max|gpu - ref| / max|ref| <= 2e-2 for bf16 results and <= 1e-4 for fp32 results.  For single
kernels an element-wise bar is checked as well: one bf16 rounding step (2^-8 relative) plus fp32-accumulation
noise, which catches a wrong index or a dropped term that the per-tensor bar could hide."""
import numpy as np
import torch

from oracle.numerics import bf16_round

DEV = "cuda:0"


def bf(x):
    """numpy -> bf16 device tensor (values are rounded to bf16)."""
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(DEV).to(torch.bfloat16).contiguous()


def f32(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(DEV).contiguous()


def i32(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).to(DEV).contiguous()


def up(t):
    """device tensor -> float64 numpy."""
    return t.detach().float().cpu().double().numpy()


def q(x):
    """The value a bf16 tensor made from x holds, as float64."""
    return bf16_round(np.asarray(x, dtype=np.float32))


def rel_err(got, ref):
    ref = np.asarray(ref, dtype=np.float64)
    den = np.max(np.abs(ref))
    return float(np.max(np.abs(np.asarray(got, np.float64) - ref)) / (den if den > 0 else 1.0))


def assert_bf16_close(got, ref, name="", elem_slack=2e-3):
    got, ref = np.asarray(got, np.float64), np.asarray(ref, np.float64)
    assert got.shape == ref.shape, (name, got.shape, ref.shape)
    assert np.all(np.isfinite(got)), name
    e = rel_err(got, ref)
    assert e <= 2e-2, (name, e)
    bound = 2.0 ** -7 * np.abs(ref) + elem_slack * np.max(np.abs(ref)) + 1e-30
    bad = np.abs(got - ref) > bound
    assert not bad.any(), (name, int(bad.sum()), np.argwhere(bad)[:5].tolist(), got[bad][:5], ref[bad][:5])


def assert_deep_bf16_close(got, ref, ref_unrounded, name=""):
    """The output of a deep bf16 network (twelve layers) against the oracle with bf16 storage.  Storing every tensor in
    bf16 is itself a perturbation of that size: the oracle with bf16 storage and the oracle that rounds nothing (same
    bf16 weights) differ by 1.7-1.9 % of the largest output and 1.2 % in the root mean square for the twelve-layer
    d 768 encoder, and two correct bf16 pipelines that round in a different order somewhere differ by as much.  So the
    bar of 2e-2 is applied to the root-mean-square error, and the largest single error may reach 2e-2 or one and a half
    times what the oracle's own rounding does to this sample, whichever is larger."""
    got, ref, exact = (np.asarray(x, np.float64) for x in (got, ref, ref_unrounded))
    assert got.shape == ref.shape == exact.shape, (name, got.shape, ref.shape)
    assert np.all(np.isfinite(got)), name
    rms = float(np.sqrt(np.mean((got - ref) ** 2)) / np.sqrt(np.mean(ref ** 2)))
    assert rms <= 2e-2, (name, "rms", rms)
    own = rel_err(ref, exact)
    e = rel_err(got, ref)
    assert e <= max(2e-2, 1.5 * own), (name, e, own)


def assert_f32_close(got, ref, name="", tol=1e-4):
    got, ref = np.asarray(got, np.float64), np.asarray(ref, np.float64)
    assert got.shape == ref.shape, (name, got.shape, ref.shape)
    assert np.all(np.isfinite(got)), name
    e = rel_err(got, ref)
    assert e <= tol, (name, e)


def lse_reference(qkv64, h, dh, causal=True):
    """log sum exp of the scaled, masked scores, written out from its definition on the bf16-rounded inputs."""
    b, s, _ = qkv64.shape
    da = h * dh
    qh = qkv64[..., 0:da].reshape(b, s, h, dh).transpose(0, 2, 1, 3)
    kh = qkv64[..., da:2 * da].reshape(b, s, h, dh).transpose(0, 2, 1, 3)
    sc = qh @ kh.transpose(0, 1, 3, 2) / np.sqrt(dh)
    if causal:
        sc = np.where(np.tril(np.ones((s, s), dtype=bool)), sc, -np.inf)
    mx = sc.max(axis=-1, keepdims=True)
    return (mx + np.log(np.exp(sc - mx).sum(axis=-1, keepdims=True)))[..., 0].reshape(b * h, s)


def stream_beside(side, busy):
    """A stream whose work does not wait for what is queued on `side` (two streams can share a hardware queue); `busy` queues
    some milliseconds of work there."""
    x = torch.zeros(1, device=DEV)
    for _ in range(16):
        main = torch.cuda.Stream()
        torch.cuda.synchronize()
        busy()
        with torch.cuda.stream(main):
            x.add_(1.0)
        main.synchronize()
        beside = not side.query()
        torch.cuda.synchronize()
        if beside:
            return main
    raise RuntimeError("no stream found that runs beside the other")

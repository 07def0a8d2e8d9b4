"""Where a prefill chunk's rows go: a full head's into its store before the attention launch (which reads them there), a
compressed head's into the staging buffer and, behind it, into its ring.  Chunks that begin and end around the edges of the
32-slot tiles; the stores afterwards hold the bits that an append of the same rows leaves."""
import numpy as np
import pytest
import torch

import harness
import paper_2510_08525_amd as rl
from harness import Case
from inputs import synth

pytestmark = pytest.mark.gpu
KW = dict(dtype=rl.RLKV_BF16, kernel=rl.RLKV_KERNEL_MFMA, arena_fill=0xFF)


def rows(c, counts):
    T = max(counts)
    k = torch.zeros(c.B, c.Hkv, T, 128, dtype=torch.bfloat16)
    v = torch.zeros_like(k)
    for b, t in enumerate(counts):
        n = int(c.n[b])
        k[b, :, :t] = c.k_hist[b, :, n:n + t]
        v[b, :, :t] = c.v_hist[b, :, n:n + t]
    return k.to(c.device), v.to(c.device)


@pytest.mark.parametrize("page", [0, 32])
@pytest.mark.parametrize("mask", [[1, 1], [1, 0], [0, 0]], ids=["full", "mixed", "compressed"])
@pytest.mark.parametrize("cached", [0, 1, 31, 32, 33])
def test_chunks_around_tile_edges(gpu_device, cached, mask, page):
    kw = dict(Hq=14, Hkv=2, B=5, S=3, R=40, mask=mask, cap=260, seed=11 + cached, prefill_tokens=97, page_tokens=page,
              pool_pages=5 * 9 if page else 0, **KW)
    a, b = Case(**kw), Case(**kw)
    if cached:
        a.append([cached] * 5)
        b.append([cached] * 5)
    for step, counts in enumerate([[1, 31, 32, 33, 0], [97, 1, 64, 30, 65]]):
        k, v = rows(b, counts)
        b.cache.append_ragged(0, k, v, counts)
        b.n = b.n + np.asarray(counts, dtype=b.n.dtype)
        a.check_prefill(counts, step, f"{cached} cached, chunk {step}")
        a.check_indices()
    q = synth.normal(3, synth.T_Q, 0, range(5), range(14), 0, 1, 128, dtype=torch.bfloat16)[:, :, 0].contiguous().to(a.device)
    outs = [torch.zeros_like(q) for _ in range(2)]
    for c, out in zip((a, b), outs):
        c.cache.decode_attention(0, q, out, c.scale)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])
    a.close()
    b.close()


@pytest.mark.parametrize("n_compressed", [64, 65])
def test_more_compressed_heads_than_travel_in_the_arguments(gpu_device, n_compressed):
    H = n_compressed + 1
    c = Case(Hq=H, Hkv=H, B=2, S=2, R=5, mask=[0] * 30 + [1] + [0] * (H - 31), cap=80, seed=4, prefill_tokens=35, **KW)
    for step, counts in enumerate([[35, 4], [7, 33]]):
        c.check_prefill(counts, step, f"chunk {step}")
        c.check_indices()
    c.check_decode(0, "decode behind the chunks")
    c.close()


@pytest.mark.parametrize("B", [64, 65, 128, 129])
def test_batches_around_those_that_travel_in_the_arguments(gpu_device, B):
    """Chunks of unlike lengths, a few without tokens: the order of up to 64 sequences comes to the lanes of one register, of up to
    128 to those of two, of more through memory."""
    c = Case(Hq=8, Hkv=2, B=B, S=4, R=20, mask=[1, 0], cap=150, seed=B, prefill_tokens=100, **KW)
    rng = np.random.default_rng(B)
    for step in range(2):
        counts = rng.integers(1, [100, 50][step], size=B)
        counts[rng.integers(0, B, size=step)] = 0
        counts[-1] = [99, 1][step]
        c.check_prefill(counts, step, f"chunk {step}")
    np.testing.assert_array_equal(c.cache.lengths(0), c.n.astype(np.int32))
    c.close()


@pytest.mark.parametrize("offset", [0, 1, 2, 4, 8])
def test_output_that_starts_at_any_element(gpu_device, offset):
    """Output rows go out in 8-byte stores where the caller's buffer lies on 8 bytes, else in 2-byte ones: the same bits."""
    B, Hq, Hkv, T = 2, 8, 2, 70
    c = Case(Hq=Hq, Hkv=Hkv, B=B, S=4, R=20, mask=[1, 0], cap=T, seed=6, prefill_tokens=T, **KW)
    q = synth.normal(6, synth.T_Q, 0, range(B), range(Hq), 0, T, 128, dtype=torch.bfloat16).to(c.device)
    k, v = rows(c, [T, T - 5])
    want = torch.zeros_like(q)
    room = torch.zeros(want.numel() + 16, dtype=torch.bfloat16, device=c.device)
    got = room[offset:offset + want.numel()].view(want.shape)
    for out in (want, got):
        c.cache.reset()
        c.cache.prefill_attention(0, q, k, v, [T, T - 5], out, c.scale)
    torch.cuda.synchronize()
    assert torch.equal(want, got)
    assert not room[:offset].any() and not room[offset + want.numel():].any()
    c.close()


@pytest.mark.parametrize("gated", [False, True], ids=["plain", "blending"])
@pytest.mark.parametrize("form", [0, 1], ids=["form by size", "two-group form"])
def test_every_form_writes_the_same_rows_at_any_element(gpu_device, form, gated, monkeypatch):
    """A wavefront's outputs pass through LDS, in each form through another part of it: the rows of the last, partly filled block,
    of the first one and of heads of either class, at offsets of 0, 2, 8 and 16 bytes, against the oracle and bit for bit."""
    monkeypatch.setattr(harness, "TUNING", {"prefill_two_group_only": form})
    B, Hq, Hkv, T = 2, 21, 3, 75
    c = Case(Hq=Hq, Hkv=Hkv, B=B, S=4, R=20, mask=[1, 0, 1], cap=T, seed=8, prefill_tokens=T, **KW)
    g = None
    if gated:
        g = np.asarray([0.5, 1.0, 1.0], dtype=np.float32)
        c.cache.set_gates(g)
    c.check_prefill([T, T - 6], 0, "aligned", gates=g)
    q = synth.normal(8, synth.T_Q, 0, range(B), range(Hq), 100000, T, 128, dtype=torch.float32).to(torch.bfloat16).to(c.device)
    want = c.last_out
    c.n[:] = 0
    k, v = rows(c, [T, T - 6])
    for offset in (0, 1, 4, 8):
        room = torch.full((want.numel() + 16,), 7.0, dtype=torch.bfloat16, device=c.device)
        got = room[offset:offset + want.numel()].view(want.shape)
        c.cache.reset()
        c.cache.prefill_attention(0, q, k, v, [T, T - 6], got, c.scale)
        torch.cuda.synchronize()
        assert torch.equal(want, got), offset
        assert (room[:offset] == 7.0).all() and (room[offset + want.numel():] == 7.0).all()
    c.close()

"""GPU parity of ff_packed_attention (every chunk of one stage in one launch,
the renderer rows of the packed block-causal training mask) against the
oracle's packed mask, and against the sequential ring path on the same
inputs.  Bars as in test_gpu_parity: bf16 within max-abs 2e-2 and relative-L2
5e-3 of float64, float32 within 1e-5."""
import math

import numpy as np
import pytest
import torch

import synth
from oracle import ff_oracle as fo
from paper_2609_32540_amd import ff

from gpu_util import anchor_frames, check_attention, exact, make_cache, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ff.lib()


def clip(w, n_chunks, stage=0, layer=0):
    """Packed Q, K, V of chunks 0 .. n_chunks-1 at (stage, layer)."""
    parts = [[synth.chunk_tensor(w, t, c, stage, layer) for c in range(n_chunks)]
             for t in (synth.T_Q, synth.T_K, synth.T_V)]
    return [torch.cat(p, 0) for p in parts]


def oracle_packed(w, q, k, v, ak, av, table, window, scale):
    Nq, G = w.chunk_tokens, w.tokens_per_frame
    n = q.shape[0] // Nq
    Qs = [exact(q[c * Nq:(c + 1) * Nq]) for c in range(n)]
    Ks = [exact(k[c * Nq:(c + 1) * Nq]) for c in range(n)]
    Vs = [exact(v[c * Nq:(c + 1) * Nq]) for c in range(n)]
    frames = {}
    if ak is not None:
        for f in range(ak.shape[0] // G):
            frames[f] = (exact(ak[f * G:(f + 1) * G]), exact(av[f * G:(f + 1) * G]))
    return fo.packed_stage_attention(Qs, Ks, Vs, frames, table if ak is not None else [[]] * n,
                                     window, scale)


def run_and_check(w, n_chunks, window, table, n_frames):
    q, k, v = (to_dev(t) for t in clip(w, n_chunks))
    ak = av = None
    if n_frames:
        a_k, a_v = synth.anchor_tensors(w, list(range(n_frames)), 0)
        ak, av = to_dev(a_k), to_dev(a_v)
    scale = 1.0 / math.sqrt(w.head_dim)
    out = ff.packed_attention(q, k, v, n_chunks=n_chunks, window=window, anchor_k=ak, anchor_v=av,
                              frame_tokens=w.tokens_per_frame, anchors_of_chunk=table, scale=scale)
    torch.cuda.synchronize()
    ref = oracle_packed(w, q, k, v, ak, av, table, window, scale)
    Nq = w.chunk_tokens
    got = exact(out)
    for c in range(n_chunks):
        check_attention(got[c * Nq:(c + 1) * Nq], ref[c], w.dtype, f"chunk {c}")
    return out


def small(dtype, head_dim, grid=(6, 11), **kw):
    base = dict(dtype=dtype, heads=2, head_dim=head_dim, grid_h=grid[0], grid_w=grid[1],
                ring_chunks=2, stages=1, layers=1, n_chunks=6, anchor_rule="none",
                max_anchor_frames=3)
    base.update(kw)
    return synth.small_workload("packed", **base)


# anchor tables with unsorted entries, gaps (several runs), empty rows and a full row
TABLE6 = [[], [2, 0], [0, 1, 2], [1], [2, 1], [0, 2]]


@pytest.mark.parametrize("dtype,d,grid", [("f32", 64, (8, 8)), ("bf16", 64, (6, 11)),
                                          ("bf16", 128, (6, 11)), ("bf16", 128, (10, 20))])
@pytest.mark.parametrize("window", [0, 1, 2, 9])
def test_packed_matches_oracle(dtype, d, grid, window):
    w = small(dtype, d, grid)
    run_and_check(w, 6, window, TABLE6, 3)


def test_packed_without_anchors_tiny_workload():
    w = synth.WORKLOADS["tiny-f32"]
    run_and_check(w, w.n_chunks, w.ring_chunks, None, 0)


def test_packed_single_chunk_and_short_chunks():
    # one chunk (only its own keys), and 1-frame chunks of 18 tokens (a single partial tile)
    w = small("bf16", 128)
    run_and_check(w, 1, 3, [[0]], 1)
    w2 = small("bf16", 64, grid=(3, 6), frames_per_chunk=1)
    run_and_check(w2, 5, 2, [[0], [], [0], [0], []], 1)
    # 1-token chunks and 1-token anchor frames (a 1x1 grid)
    w3 = small("bf16", 128, grid=(1, 1), frames_per_chunk=1)
    run_and_check(w3, 5, 2, [[0], [], [1, 0], [1], []], 2)


def test_packed_largest_launch_shape():
    # FF_MAX_PACKED_CHUNKS = 128 chunks in one launch, the widest window W = 8,
    # 2-token chunks and 1-token anchor frames from a bank of 9; chunk c lists
    # frames c // 16 .. c // 16 + c % 3 (1-3 frames, each frame seen by one run
    # of chunks) and chunk 127 all eight frames it can list
    w = small("bf16", 64, grid=(1, 2), frames_per_chunk=1)
    n = 128
    tab = [[f for f in range(c // 16, min(9, c // 16 + c % 3 + 1))] for c in range(n)]
    tab[127] = list(range(1, 9))
    run_and_check(w, n, 8, tab, 9)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 128)])
def test_packed_equals_sequential_ring(dtype, d):
    """Chunk i of the packed launch against ff_chunk_attention of chunk i after
    chunks 0 .. i-1 were published into a ring of W = window, anchors set to
    chunk i's frames: both within the bar of the oracle, and (f32) equal to
    each other within 1e-5."""
    w = small(dtype, d, grid=(6, 11), ring_chunks=2)
    n, W = 6, 2
    q, k, v = (to_dev(t) for t in clip(w, n))
    a_k, a_v = synth.anchor_tensors(w, [0, 1, 2], 0)
    ak, av = to_dev(a_k), to_dev(a_v)
    scale = 1.0 / math.sqrt(d)
    packed = ff.packed_attention(q, k, v, n_chunks=n, window=W, anchor_k=ak, anchor_v=av,
                                 frame_tokens=w.tokens_per_frame, anchors_of_chunk=TABLE6,
                                 scale=scale)
    cache = make_cache(w, stages=1, layers=1)
    Nq, G = w.chunk_tokens, w.tokens_per_frame
    seq = torch.empty_like(q)
    for c in range(n):
        fr = TABLE6[c]
        if fr:
            kk = torch.cat([ak[f * G:(f + 1) * G] for f in fr])
            vv = torch.cat([av[f * G:(f + 1) * G] for f in fr])
            cache.anchor_set(0, fr, kk.contiguous(), vv.contiguous())
        else:
            cache.anchor_set(0, [], None, None)
        sl = slice(c * Nq, (c + 1) * Nq)
        cache.chunk_attention(0, 0, c, q[sl], k[sl], v[sl], seq[sl], scale=scale)
        cache.kv_publish(0, 0, c, k[sl], v[sl])
    torch.cuda.synchronize()
    ref = oracle_packed(w, q, k, v, ak, av, TABLE6, W, scale)
    gp, gs = exact(packed), exact(seq)
    for c in range(n):
        sl = slice(c * Nq, (c + 1) * Nq)
        check_attention(gp[sl], ref[c], dtype, f"packed chunk {c}")
        check_attention(gs[sl], ref[c], dtype, f"sequential chunk {c}")
    if dtype == "f32":
        assert np.abs(gp - gs).max() <= 1e-5


@pytest.mark.parametrize("d", [128, 64])
def test_packed_log_sum_exp_reference_far_below_the_max(d):
    """The launch that also writes the log-sum-exp (the training forward) when a
    chunk's first block sets a reference far below its largest scores: chunk 0's
    keys are tiny and the first block of every chunk's read set is chunk 0's;
    keys scaled by 8 give probabilities up to ~2^35 relative to that reference,
    keys scaled by 24 go past 2^56, where the key-split kernel, which this small
    launch runs, raises its reference (the 256-query kernel's checked pass:
    test_gpu_256_row_kernels.py).  Output and base-2 log-sum-exp against the
    oracle (log2_sum_exp2 over the packed mask)."""
    n, W = 5, 4
    w = small("bf16", d, grid=(6, 11), ring_chunks=W, n_chunks=n)
    q, k, v = clip(w, n)
    Nq = w.chunk_tokens
    factors = [0.01, 8.0, 8.0, 24.0, 1.0]
    k = torch.cat([(k[c * Nq:(c + 1) * Nq].float() * f).to(torch.bfloat16)
                   for c, f in enumerate(factors)])
    q, k, v = to_dev(q), to_dev(k), to_dev(v)
    scale = 1.0 / math.sqrt(d)
    lse = torch.empty((n * Nq, w.heads), dtype=torch.float32, device=q.device)
    out = ff.packed_attention(q, k, v, n_chunks=n, window=W, anchor_k=None, anchor_v=None,
                              frame_tokens=w.tokens_per_frame, anchors_of_chunk=None,
                              scale=scale, lse=lse)
    torch.cuda.synchronize()
    ref = oracle_packed(w, q, k, v, None, None, None, W, scale)
    got = exact(out)
    for c in range(n):
        check_attention(got[c * Nq:(c + 1) * Nq], ref[c], "bf16",
                        f"chunk {c} (key scale {factors[c]:g})")
    M = fo.packed_visibility(n, Nq, w.tokens_per_frame, 0, [[]] * n, W)
    rlse = fo.log2_sum_exp2(exact(q), exact(k), M, scale)
    err = float(np.abs(exact(lse) - rlse).max())
    assert err <= 2e-3, f"log-sum-exp off by {err:.2e} (log2 units)"


@pytest.mark.parametrize("name", ["1.3b-480p", "14b-720p"])
def test_packed_full_size_sampled_rows(name):
    """A whole clip of one stage (27 chunks, W = 4, anchor windows Gamma(i)) at
    the 1.3B 480p shape (4680-token chunks, 12 heads) and at the 14B 720p shape
    the benchmark times (10800-token chunks, 40 heads): one launch, checked on
    sampled rows (incl. the ragged last query tile) of chunks at the start, the
    middle and the end against the float64 oracle over the visible keys (the
    renderer rows of the packed mask M, Alg. 2); inputs seeded N(0,1) drawn on
    the device."""
    w = synth.WORKLOADS[name]
    n, W, Nq, G = w.n_chunks, w.ring_chunks, w.chunk_tokens, w.tokens_per_frame
    dev = torch.device("cuda", 0)
    g = torch.Generator(device=dev)
    g.manual_seed(1234)
    shape = (n * Nq, w.heads, w.head_dim)
    q, k, v = (torch.randn(shape, generator=g, device=dev).to(torch.bfloat16) for _ in range(3))
    frames = sorted({f for c in range(n) for f in anchor_frames(w, c)})
    a_shape = (len(frames) * G, w.heads, w.head_dim)
    ak, av = (torch.randn(a_shape, generator=g, device=dev).to(torch.bfloat16) for _ in range(2))
    table = [[frames.index(f) for f in anchor_frames(w, c)] for c in range(n)]
    scale = 1.0 / math.sqrt(w.head_dim)
    out = ff.packed_attention(q, k, v, n_chunks=n, window=W, anchor_k=ak, anchor_v=av,
                              frame_tokens=G, anchors_of_chunk=table, scale=scale)
    torch.cuda.synchronize()
    rows = np.concatenate([np.arange(0, 256), np.arange(Nq - 200, Nq)])
    for c in (0, 3, 13, n - 1):
        keys = [slice(f * G, (f + 1) * G) for f in table[c]]
        chunks = slice(max(0, c - W) * Nq, (c + 1) * Nq)
        for h in (0, w.heads - 1):
            Kh = np.concatenate([exact(ak[s, h]) for s in keys] + [exact(k[chunks, h])])
            Vh = np.concatenate([exact(av[s, h]) for s in keys] + [exact(v[chunks, h])])
            Qh = exact(q[c * Nq + rows, h])
            ref = fo.attend(Qh.astype(np.float64), Kh.astype(np.float64), Vh.astype(np.float64),
                            scale)
            check_attention(exact(out[c * Nq + rows, h]), ref, "bf16", f"chunk {c} head {h}")

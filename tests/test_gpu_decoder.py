"""GPU parity of the decoder loop around the MoE layer against the decoder
oracle: the dense projection, rotary embedding with the cache append,
causal grouped-query attention (every group size, several positions),
arg max and embedding gather, and a two-layer decoder (prefill then greedy
decode, prediction and prefetch on) whose every layer is checked
teacher-forced: the oracle gets each layer's GPU input and builds its own
key/value caches from them."""
import numpy as np
import pytest

import synth
from gpu_helpers import check_close

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _bf16(a):
    """(device bf16 tensor, exact fp64 values) of an fp32 array."""
    from workload import to_device
    raw, f = synth.storage(np.ascontiguousarray(a, np.float32), "bf16")
    return to_device(raw, "bf16"), f.astype(np.float64)


# n_in a multiple of 64 takes the staged matrix-core kernels, an odd multiple
# of 32 with T >= 16 the register-staged one (ragged 64-token and 64-output
# tiles); the rest the fma-chain kernels (four tokens at a time up to n_in 4096,
# two above)
@pytest.mark.parametrize("T,n_in,n_out", [(1, 256, 13), (3, 4096, 100), (9, 512, 64), (2, 8192, 24),
                                          (16, 256, 13), (17, 1024, 70), (64, 4096, 100), (130, 512, 200),
                                          (40, 8192, 24), (20, 264, 33), (17, 1056, 70), (130, 8160, 24), (3, 4088, 17),
                                          (1, 4104, 13), (5, 8184, 30), (20, 8184, 9)])
def test_dense_matches_numpy(T, n_in, n_out):
    from paper_2509_08342_amd import moesplit as ms
    rng = np.random.default_rng(T + n_in)
    x, xf = _bf16(rng.standard_normal((T, n_in)))
    w, wf = _bf16(0.02 * rng.standard_normal((n_out, n_in)))
    add = torch.from_numpy(rng.standard_normal((T, n_out)).astype(np.float32)).cuda()
    y = torch.empty(T, n_out, dtype=torch.float32, device="cuda")
    ms.ms_dense(x, w, T, n_in, n_out, y, add, torch.cuda.current_stream())
    torch.cuda.synchronize()
    ref = xf @ wf.T + add.cpu().numpy()
    bound = 1e-5 * (np.abs(xf) @ np.abs(wf).T).max() + 1e-6
    assert np.max(np.abs(y.cpu().numpy() - ref)) <= bound


# n_in a multiple of 64: the staged matrix-core kernels (96: the others).  Fewer than 16
# tokens (in four waves; in eight from n_in 2048 on up to 256 blocks of 16 outputs); then every tile of the larger ones (32 x 32 ... 256 x 192 tokens x
# outputs) with remainders, outputs that are no multiple of 4, and y rows that
# are not 16-byte aligned, with `add` separate, aliasing y or absent.  The
# sums are 32-bit in 32-wide steps at worst: n_in / 32 roundings of at most
# the sum of magnitudes, 2^-23 each.
@pytest.mark.parametrize("T,n_in,n_out", [(1, 64, 1), (15, 64, 17), (2, 192, 100), (15, 8192, 16), (7, 2112, 4096),
                                          (1, 2048, 4097), (16, 64, 1),
                                          (33, 448, 30), (100, 64, 3000), (250, 128, 6144), (511, 64, 6100),
                                          (990, 64, 6141), (2047, 64, 6140), (70, 96, 65), (9, 96, 65)])
@pytest.mark.parametrize("add", ["none", "apart", "alias"])
@pytest.mark.parametrize("shift", [0, 1])
def test_dense_staged_tiles(T, n_in, n_out, add, shift):
    from paper_2509_08342_amd import moesplit as ms
    rng = np.random.default_rng(T + n_in)
    x, xf = _bf16(rng.standard_normal((T, n_in)))
    w, wf = _bf16(0.02 * rng.standard_normal((n_out, n_in)))
    a = torch.from_numpy(rng.standard_normal((T, n_out)).astype(np.float32)).cuda()
    buf = torch.full((T * n_out + 2,), -7.0, dtype=torch.float32, device="cuda")
    y = buf[shift:shift + T * n_out].view(T, n_out)
    if add == "alias":
        y.copy_(a)
    ms.ms_dense(x, w, T, n_in, n_out, y, {"none": None, "apart": a, "alias": y}[add], torch.cuda.current_stream())
    torch.cuda.synchronize()
    ref = xf @ wf.T
    mags = np.abs(xf) @ np.abs(wf).T
    if add != "none":
        ref = ref + a.cpu().numpy()
        mags = mags + np.abs(a.cpu().numpy())
    assert np.all(np.abs(y.cpu().numpy() - ref) <= (n_in / 32 + 2) * 2.0 ** -23 * mags)
    out = buf.cpu().numpy()
    assert np.all(out[:shift] == -7.0) and np.all(out[shift + T * n_out:] == -7.0)


@pytest.mark.parametrize("pos0,T", [(0, 1), (7, 3), (200, 2)])
def test_rope_kv_matches_oracle(pos0, T):
    from oracle import decoder as od
    from paper_2509_08342_amd import moesplit as ms
    Hq, Hkv, D, base, max_ctx = 4, 2, 64, 1e4, 256
    rng = np.random.default_rng(pos0)
    qkv = rng.standard_normal((T, (Hq + 2 * Hkv) * D)).astype(np.float32)
    q = torch.empty(T, Hq, D, dtype=torch.bfloat16, device="cuda")
    kc = torch.zeros(Hkv, max_ctx, D, dtype=torch.bfloat16, device="cuda")
    vc = torch.zeros_like(kc)
    ms.ms_rope_kv(torch.from_numpy(qkv).cuda(), T, Hq, Hkv, D, pos0, base, q, kc, vc, max_ctx,
                  torch.cuda.current_stream())
    torch.cuda.synchronize()
    qg, kg, vg = q.float().cpu().numpy(), kc.float().cpu().numpy(), vc.float().cpu().numpy()
    for t in range(T):
        p = pos0 + t
        rq = od.bf16_round(od.rope(qkv[t, :Hq * D].reshape(Hq, D), p, base))
        rk = od.bf16_round(od.rope(qkv[t, Hq * D:(Hq + Hkv) * D].reshape(Hkv, D), p, base))
        rv = od.bf16_round(qkv[t, (Hq + Hkv) * D:].reshape(Hkv, D))
        # fp32 products against fp64: at most one bf16 rounding step apart
        for got, ref in ((qg[t], rq), (kg[:, p], rk)):
            assert np.all(np.abs(got - ref) <= 2.0 ** -7 * np.abs(ref) + 1e-30)
        assert np.array_equal(vg[:, p], rv)
    untouched = np.ones(max_ctx, bool)
    untouched[pos0:pos0 + T] = False
    assert not np.any(kg[:, untouched]) and not np.any(vg[:, untouched])


# angles of the thread's own (few rows, few heads, half width 515) and shared ones:
# four pairs per thread or one (widths, addresses), one block per token or
# several, angles on either side of what a block computes at once (half 256, 260)
@pytest.mark.parametrize("Hq,Hkv,D,T,shift", [(4, 2, 64, 5, 1), (1, 1, 6, 2, 0), (3, 1, 1030, 2, 0), (32, 8, 128, 3, 0),
                                              (1, 1, 64, 700, 0), (32, 8, 128, 42, 0), (32, 8, 128, 43, 0), (4, 2, 64, 400, 1),
                                              (8, 8, 8, 2100, 0), (7, 7, 6, 300, 0), (2, 1, 512, 3, 0), (2, 1, 520, 3, 1)])
def test_rope_kv_widths(Hq, Hkv, D, T, shift):
    from oracle import decoder as od
    from paper_2509_08342_amd import moesplit as ms
    base, pos0 = 1e6, 3
    max_ctx = pos0 + T
    rng = np.random.default_rng(D)
    qkv = rng.standard_normal((T, (Hq + 2 * Hkv) * D)).astype(np.float32)
    src = torch.empty(qkv.size + 4, dtype=torch.float32, device="cuda")[shift:shift + qkv.size].view(qkv.shape)
    src.copy_(torch.from_numpy(qkv))
    q = torch.empty(T, Hq, D, dtype=torch.bfloat16, device="cuda")
    kc = torch.zeros(Hkv, max_ctx, D, dtype=torch.bfloat16, device="cuda")
    vc = torch.zeros_like(kc)
    ms.ms_rope_kv(src, T, Hq, Hkv, D, pos0, base, q, kc, vc, max_ctx, torch.cuda.current_stream())
    torch.cuda.synchronize()
    qg, kg, vg = q.float().cpu().numpy(), kc.float().cpu().numpy(), vc.float().cpu().numpy()
    for t in range(0, T, max(1, T // 5)):
        p = pos0 + t
        rq = od.bf16_round(od.rope(qkv[t, :Hq * D].reshape(Hq, D), p, base))
        rk = od.bf16_round(od.rope(qkv[t, Hq * D:(Hq + Hkv) * D].reshape(Hkv, D), p, base))
        for got, ref in ((qg[t], rq), (kg[:, p], rk)):  # as above; a sum near zero by its terms' rounding
            assert np.all(np.abs(got - ref) <= 2.0 ** -7 * np.abs(ref) + 2.0 ** -22 * np.abs(qkv[t]).max())
        assert np.array_equal(vg[:, p], od.bf16_round(qkv[t, (Hq + Hkv) * D:].reshape(Hkv, D)))


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("pos0,T", [(0, 1), (5, 3), (300, 2)])
def test_attention_matches_oracle(G, pos0, T):
    from oracle import decoder as od
    from paper_2509_08342_amd import moesplit as ms
    Hkv, D, max_ctx = 2, 128, 512
    Hq = G * Hkv
    rng = np.random.default_rng(100 * G + pos0)
    q, qf = _bf16(rng.standard_normal((T, Hq, D)))
    kc, kf = _bf16(rng.standard_normal((Hkv, max_ctx, D)))
    vc, vf = _bf16(rng.standard_normal((Hkv, max_ctx, D)))
    out = torch.empty(T, Hq, D, dtype=torch.bfloat16, device="cuda")
    ms.ms_attention(q, kc, vc, T, Hq, Hkv, D, pos0, max_ctx, out, torch.cuda.current_stream())
    torch.cuda.synchronize()
    got = out.float().cpu().numpy()
    for t in range(T):
        ref = od.attend(qf[t], kf, vf, pos0 + t + 1)
        check_close(got[t], ref, "bf16", "attention t=%d" % t)


def _attention(qf, kf, vf, pos0):
    """Causal grouped-query attention in 64 bits: qf [T][Hq][D], caches [Hkv][ctx][D]."""
    T, Hq, D = qf.shape
    G = Hq // kf.shape[0]
    out = np.empty_like(qf)
    for h in range(Hq):
        n = pos0 + T
        s = qf[:, h] @ kf[h // G, :n].T / np.sqrt(D)
        s[np.arange(n)[None, :] > pos0 + np.arange(T)[:, None]] = -np.inf
        p = np.exp(s - s.max(axis=1, keepdims=True))
        out[:, h] = (p / p.sum(axis=1, keepdims=True)) @ vf[h // G, :n]
    return out


def attention_route(G, Hkv, D, pos0, T):
    """The kernel of a call at D = 64 or 128: few tokens in 8 or 4 waves (a
    work-group per token, head and 32 columns), prompts in blocks of 64 or 128 rows."""
    wgs = T * Hkv * D // 32
    if wgs <= 512 or (pos0 + T >= 256 and wgs <= (1024 if Hkv * D <= 1024 else 768)):
        return "few8" if wgs <= 256 else "few4"
    return "rows128" if -(-T * G // 64) * Hkv >= 1024 else "rows64"


# every group size and head width on each route, with remainders of tokens, rows,
# key steps of 32 and key tiles of 64, fewer key steps than waves, and long
# prefixes that nothing masks; q and out 2-byte aligned only
ATTENTION_SHAPES = [
    ("few8", [(1, 2, 64, 0, 1), (1, 3, 64, 130, 17), (1, 2, 128, 0, 5), (2, 2, 64, 255, 2), (2, 2, 128, 63, 3),
              (4, 2, 64, 40, 3), (4, 8, 128, 31, 1), (4, 8, 128, 70, 8), (8, 1, 64, 7, 31), (8, 4, 128, 1000, 1),
              (8, 2, 128, 500, 16)]),
    ("few4", [(1, 16, 64, 512, 24), (1, 2, 128, 0, 64), (2, 4, 64, 100, 40), (2, 2, 128, 63, 33), (4, 4, 64, 33, 33),
              (4, 8, 128, 290, 9), (4, 2, 128, 1, 61), (8, 1, 64, 7, 131), (8, 2, 128, 77, 40), (2, 4, 128, 500, 50),
              (8, 1, 64, 7, 500), (4, 2, 128, 1500, 97), (8, 2, 128, 500, 98), (1, 16, 128, 300, 12)]),
    ("rows64", [(1, 16, 64, 20, 25), (1, 8, 128, 300, 65), (2, 8, 64, 63, 50), (2, 4, 128, 500, 70), (4, 2, 64, 0, 200),
                (4, 2, 128, 1, 100), (4, 2, 128, 1500, 140), (8, 3, 64, 30, 128), (8, 1, 64, 7, 520), (8, 2, 128, 500, 130),
                (1, 16, 128, 300, 13), (4, 2, 128, 1, 65)]),
    ("rows128", [(1, 64, 64, 5, 1025), (1, 64, 128, 0, 1021), (2, 32, 64, 100, 1025), (2, 32, 128, 60, 1025),
                 (4, 16, 64, 0, 1030), (4, 16, 128, 1000, 1010), (8, 16, 64, 3, 520), (8, 16, 128, 3, 520)]),
]


@pytest.mark.parametrize("route,G,Hkv,D,pos0,T", [(r, *c) for r, cs in ATTENTION_SHAPES for c in cs])
@pytest.mark.parametrize("shift", [0, 1])
def test_attention_prompts(route, G, Hkv, D, pos0, T, shift):
    from paper_2509_08342_amd import moesplit as ms
    assert attention_route(G, Hkv, D, pos0, T) == route
    max_ctx, Hq = pos0 + T + 3, G * Hkv
    rng = np.random.default_rng(T + pos0)
    q, qf = _bf16(2 * rng.standard_normal((T, Hq, D)))
    kc, kf = _bf16(2 * rng.standard_normal((Hkv, max_ctx, D)))
    vc, vf = _bf16(rng.standard_normal((Hkv, max_ctx, D)))
    qs = torch.empty(T * Hq * D + 8, dtype=torch.bfloat16, device="cuda")[shift:shift + q.numel()].view(q.shape)
    qs.copy_(q)
    buf = torch.full((T * Hq * D + 2,), -7.0, dtype=torch.bfloat16, device="cuda")
    out = buf[shift:shift + q.numel()].view(q.shape)
    ms.ms_attention(qs, kc, vc, T, Hq, Hkv, D, pos0, max_ctx, out, torch.cuda.current_stream())
    torch.cuda.synchronize()
    ref = _attention(qf, kf, vf, pos0)
    # the result's rounding to bf16 (2^-9), and 2^-15 of the largest value for
    # scores and probabilities (32-bit sums, 16 bits of each probability)
    got = out.float().cpu().numpy()
    assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 2.0 ** -15 * np.abs(vf).max())
    rest = buf.float().cpu().numpy()
    assert np.all(rest[:shift] == -7.0) and np.all(rest[shift + q.numel():] == -7.0)


# the other head widths: 1024 threads for one token where its scores and partial
# sums fit, else 256; one thread per position up to a wave of them (D = 8 ... 512)
@pytest.mark.parametrize("G,Hkv,D,pos0,T", [(1, 2, 8, 0, 1), (8, 2, 8, 300, 1), (2, 3, 8, 40, 9), (4, 2, 16, 100, 1),
                                            (2, 3, 32, 1000, 1), (8, 1, 32, 60, 7), (1, 2, 256, 130, 1), (8, 1, 256, 600, 1),
                                            (2, 2, 256, 50, 5), (1, 2, 512, 70, 1), (2, 1, 512, 10, 1), (4, 1, 512, 900, 3)])
def test_attention_other_widths(G, Hkv, D, pos0, T):
    from paper_2509_08342_amd import moesplit as ms
    ctx, Hq = pos0 + T + 3, G * Hkv
    rng = np.random.default_rng(T + pos0)
    q, qf = _bf16(2 * rng.standard_normal((T, Hq, D)))
    kc, kf = _bf16(2 * rng.standard_normal((Hkv, ctx, D)))
    vc, vf = _bf16(rng.standard_normal((Hkv, ctx, D)))
    out = torch.full((T * Hq * D + 8,), -7.0, dtype=torch.bfloat16, device="cuda")
    ms.ms_attention(q, kc, vc, T, Hq, Hkv, D, pos0, ctx, out, torch.cuda.current_stream())
    torch.cuda.synchronize()
    got = out.float().cpu().numpy()
    ref = _attention(qf, kf, vf, pos0)
    assert np.all(np.abs(got[:ref.size].reshape(ref.shape) - ref) <= 2.0 ** -8 * np.abs(ref) + 2.0 ** -15 * np.abs(vf).max())
    assert np.all(got[ref.size:] == -7.0)


# scores of 1e8 to 1e33 whose products and sums are exact: the largest keys of a
# row share its weight, whatever the rounding of their scaled score.  Both
# few-token variants (one key; eight waves; four) and both row block heights.
@pytest.mark.parametrize("G,Hkv,D,pos0,T", [(1, 1, 64, 0, 1), (4, 8, 128, 700, 1), (4, 8, 64, 100, 30), (4, 8, 128, 100, 40),
                                            (8, 16, 64, 64, 520)])
@pytest.mark.parametrize("exponent", [20, 27, 36, 60, 100])
@pytest.mark.parametrize("sign", [1, -1])
def test_attention_large_scores(G, Hkv, D, pos0, T, exponent, sign):
    from paper_2509_08342_amd import moesplit as ms
    ctx, Hq = pos0 + T, G * Hkv
    rng = np.random.default_rng(T + exponent)
    q, qf = _bf16(np.full((T, Hq, D), 1.5 * 2.0 ** (exponent // 2)))
    steps = rng.integers(0, 3, (Hkv, ctx, 1)) / 8.0  # three distinct scores, apart by a sixteenth of them or more
    kc, kf = _bf16(np.broadcast_to(sign * (1.25 + steps) * 2.0 ** (exponent - exponent // 2), (Hkv, ctx, D)).copy())
    vc, vf = _bf16(rng.standard_normal((Hkv, ctx, D)))
    out = torch.empty_like(q)
    ms.ms_attention(q, kc, vc, T, Hq, Hkv, D, pos0, ctx, out, torch.cuda.current_stream())
    torch.cuda.synchronize()
    ref = _attention(qf, kf, vf, pos0)
    assert np.all(np.abs(out.float().cpu().numpy() - ref) <= 2.0 ** -8 * np.abs(ref) + 2.0 ** -15 * np.abs(vf).max())


# probabilities of 24 bits: per column three values that cancel to about 2^-18 of
# their terms, for all tokens alike (one query, exact scores between 0 and
# -1).  Left over: the scale's and the exponential's rounding, 2^-22 of
# the terms each; 16 bits of a probability would leave up to 2^-18.
@pytest.mark.parametrize("G,Hkv,D,pos0,T", [(4, 2, 128, 200, 1), (4, 8, 64, 100, 30), (4, 8, 128, 100, 40),
                                            (8, 16, 64, 64, 520), (4, 16, 128, 64, 1030)])
def test_attention_cancelling_values(G, Hkv, D, pos0, T):
    from paper_2509_08342_amd import moesplit as ms
    ctx, Hq = pos0 + T, G * Hkv
    rng = np.random.default_rng(T + D)
    q, qf = _bf16(np.ones((T, Hq, D)))
    keys = np.zeros((Hkv, ctx, D))  # one column each: every score is the key's value there
    keys[:, 1:, 0] = -rng.random((Hkv, ctx - 1)) * np.sqrt(D)
    kc, kf = _bf16(keys)
    p = np.exp(kf[:, :, 0] / np.sqrt(D))
    vf = np.zeros((Hkv, ctx, D))
    for h in range(Hkv):
        for c in range(D):
            a, b, e = rng.choice(np.arange(1, pos0), 3, replace=False)
            vf[h, a, c] = 1.0
            vf[h, b, c] = -synth.storage(np.float32([p[h, a] / p[h, b]]), "bf16")[1][0]
            vf[h, e, c] = -(p[h, a] + p[h, b] * vf[h, b, c]) / p[h, e]
    vc, vf = _bf16(vf)
    out = torch.empty_like(q)
    ms.ms_attention(q, kc, vc, T, Hq, Hkv, D, pos0, ctx, out, torch.cuda.current_stream())
    torch.cuda.synchronize()
    ref, mags = _attention(qf, kf, vf, pos0), _attention(qf, kf, np.abs(vf), pos0)
    assert np.all(np.abs(out.float().cpu().numpy() - ref) <= 2.0 ** -8 * np.abs(ref) + 2.0 ** -21 * mags)


# few tokens in eight waves and in four, prompts in row blocks of 64 and of 128;
# the value that is not finite among the call's own tokens (some row blocks mask
# it, later ones see it whole) or before them
@pytest.mark.parametrize("G,Hkv,D,T,pos0,at", [(4, 2, 128, 1, 500, 100), (8, 1, 64, 3, 40, 41), (4, 2, 128, 60, 0, 35),
                                               (4, 2, 128, 150, 20, 95), (4, 2, 64, 300, 10, 160), (4, 2, 128, 300, 10, 5),
                                               (8, 16, 64, 520, 100, 250), (2, 32, 128, 1025, 60, 30)])
@pytest.mark.parametrize("what", [np.nan, np.inf, -np.inf])
def test_attention_values_that_are_not_finite(G, Hkv, D, T, pos0, at, what):
    """A value of infinity or NaN gives its column infinity or NaN for every token
    that sees it, a key of NaN gives NaN for the whole head; neither reaches the
    tokens before.  Finite values whose unnormalized sum would pass the largest
    float give a finite mean."""
    from paper_2509_08342_amd import moesplit as ms
    ctx, Hq, pos = pos0 + T, G * Hkv, np.arange(pos0, pos0 + T)
    rng = np.random.default_rng(T)
    q, qf = _bf16(rng.standard_normal((T, Hq, D)))
    kc, kf = _bf16(rng.standard_normal((Hkv, ctx, D)))
    vc, vf = _bf16(rng.standard_normal((Hkv, ctx, D)))
    big = float(torch.tensor(3e38, dtype=torch.bfloat16))
    vc[0, :, 5], vf[0, :, 5] = big, big
    vc[:, at, 3] = what
    nan_key = min(at + 5, ctx - 1)
    kc[Hkv - 1, nan_key] = np.nan
    out = torch.empty_like(q)
    ms.ms_attention(q, kc, vc, T, Hq, Hkv, D, pos0, ctx, out, torch.cuda.current_stream())
    torch.cuda.synchronize()
    got, ref = out.float().cpu().numpy(), _attention(qf, kf, vf, pos0)
    ref[pos >= at, :, 3] = what
    ref[pos >= nan_key, (Hkv - 1) * G:] = np.nan
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    infinite = np.isinf(ref)
    assert np.array_equal(got[infinite], ref[infinite])
    fine = np.isfinite(ref)
    tail = np.where(np.arange(D) == 5, big, np.abs(np.delete(vf, 5, axis=2)).max())  # largest value of a column
    bound = 2.0 ** -8 * np.abs(ref) + 2.0 ** -15 * tail
    assert np.all(np.abs(got[fine] - ref[fine]) <= bound[fine])


@pytest.mark.parametrize("G,Hkv,D,pos0,T", [(4, 8, 128, 700, 1), (4, 8, 64, 100, 30), (4, 8, 128, 100, 40), (2, 2, 32, 9, 5)])
def test_attention_in_place(G, Hkv, D, pos0, T):
    """out may be q: the rows that a work-group writes are no other's input."""
    from paper_2509_08342_amd import moesplit as ms
    ctx, Hq = pos0 + T, G * Hkv
    rng = np.random.default_rng(T)
    q, qf = _bf16(2 * rng.standard_normal((T, Hq, D)))
    kc, kf = _bf16(2 * rng.standard_normal((Hkv, ctx, D)))
    vc, vf = _bf16(rng.standard_normal((Hkv, ctx, D)))
    ms.ms_attention(q, kc, vc, T, Hq, Hkv, D, pos0, ctx, q, torch.cuda.current_stream())
    torch.cuda.synchronize()
    ref = _attention(qf, kf, vf, pos0)
    assert np.all(np.abs(q.float().cpu().numpy() - ref) <= 2.0 ** -8 * np.abs(ref) + 2.0 ** -15 * np.abs(vf).max())


def test_attention_rejects_what_it_cannot_hold():
    from paper_2509_08342_amd import moesplit as ms
    q = torch.zeros(1, 8, 128, dtype=torch.bfloat16, device="cuda")
    kc = torch.zeros(1, 8192, 128, dtype=torch.bfloat16, device="cuda")
    out = torch.empty_like(q)
    with pytest.raises(ms.MoeSplitError) as ei:
        ms.ms_attention(q, kc, kc, 1, 8, 1, 128, 4000, 8192, out)
    assert ei.value.status == ms.MS_E_UNSUPPORTED
    with pytest.raises(ms.MoeSplitError) as ei:
        ms.ms_attention(q, kc, kc, 1, 8, 1, 128, 8192, 8192, out)
    assert ei.value.status == ms.MS_E_INVALID


def test_argmax_and_embed():
    from paper_2509_08342_amd import moesplit as ms
    x = torch.tensor([[1.0, 5.0, 5.0, -1.0], [0.0, 0.0, 0.0, 0.0], [-3.0, -2.0, -9.0, -2.0]], device="cuda")
    idx = torch.empty(3, dtype=torch.int32, device="cuda")
    ms.ms_argmax(x, 3, 4, idx)
    torch.cuda.synchronize()
    assert idx.cpu().tolist() == [1, 0, 1]
    rng = np.random.default_rng(9)
    big = torch.from_numpy(rng.standard_normal((2, 70001)).astype(np.float32)).cuda()
    ms.ms_argmax(big, 2, 70001, idx)
    torch.cuda.synchronize()
    assert idx[:2].cpu().tolist() == np.argmax(big.cpu().numpy(), axis=1).tolist()
    table, tf = _bf16(rng.standard_normal((50, 64)))
    ids = torch.tensor([3, 49, 0], dtype=torch.int32, device="cuda")
    out = torch.empty(3, 64, dtype=torch.bfloat16, device="cuda")
    ms.ms_embed(ids, table, 50, 3, 64, out)
    torch.cuda.synchronize()
    assert np.array_equal(out.float().cpu().numpy(), tf[[3, 49, 0]])


def test_decoder_layers_match_oracle():
    import oracle
    from oracle import decoder as od
    from decoder import Decoder
    from paper_2509_08342_amd import moesplit as ms
    from workload import top_bytes
    shape = synth.ModelShape("dec-tiny", 2, 256, 512, 8, 2, "bf16")
    attn = synth.TINY_ATTN
    P, n_dec = 12, 3
    with Decoder(shape, attn, seed=4, n_sets=2, max_tokens=P, max_ctx=64,
                 budget_total=2 * 8 * shape.expert_bytes) as dec:
        rig = dec.stack.rig
        dec.stack.configure(0.5, 2 * 4 * top_bytes(rig, 0.5))
        for l in range(2):
            rig.load_tops(l, [0, 1, 2, 3])
        ms.ms_sync(dec.ctx)
        cfg = dict(Hq=attn.n_heads, Hkv=attn.n_kv_heads, D=attn.head_dim, base=attn.rope_base)
        caches = [od.Cache(attn.n_kv_heads, 64, attn.head_dim) for _ in range(2)]
        prompt = synth.prompt_tokens(attn, 4, P)
        ids = torch.from_numpy(prompt).cuda()
        x = torch.empty(P, shape.d_model, dtype=torch.bfloat16, device="cuda")
        dec.embed_ids(ids, P, x)
        torch.cuda.synchronize()
        assert np.array_equal(x.float().cpu().numpy(), dec.embed_f32[prompt])
        x1 = torch.empty(1, shape.d_model, dtype=torch.bfloat16, device="cuda")
        for step in range(1 + n_dec):
            T = P if step == 0 else 1
            pos0 = dec.pos
            cap = dec.step(x if step == 0 else x1, T, capture=(0, 1))
            torch.cuda.synchronize()
            for l in range(2):
                c = cap[l]
                qf, of = dec.f32[l % dec.n_sets]
                moe = od.moe_from_layer_oracle(rig.routers[l], rig.layer_experts(l), shape.top_k, bias=rig.biases[l])
                xo, h = od.layer(c["x"], dict(w_qkv=qf, w_o=of), caches[l], pos0, cfg, moe)
                check_close(c["h"], h, "bf16", "step %d layer %d h" % (step, l))
                # routing of the GPU's own h is exact; its output within tolerance
                ref = oracle.moe_layer(c["h"].astype(np.float32), rig.routers[l], rig.layer_experts(l), shape.top_k,
                                       bias=rig.biases[l])
                assert np.array_equal(c["idx"], ref["idx"])
                check_close(c["x_out"], od.bf16_round(od.rmsnorm(c["h"] + ref["y"])), "bf16",
                            "step %d layer %d x_out" % (step, l))
            # head on the GPU's final state; the greedy token where the top two are apart
            last = dec.final[T - 1:T].float().cpu().numpy()
            logits, am = od.head_argmax(last, dec.head_f32)
            got = dec.logits.cpu().numpy()
            check_close(got, logits, "bf16", "logits")
            top2 = np.sort(logits[0])[-2:]
            if top2[1] - top2[0] > 1e-3 * np.abs(logits).max():
                assert int(dec.ids[0].item()) == int(am[0])
            dec.embed_ids(dec.ids, 1, x1)
        assert dec.pos == P + n_dec

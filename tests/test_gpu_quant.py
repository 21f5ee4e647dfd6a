"""GPU parity of the layer over b-bit expert codes (the HQQ format of the
paper's 2-bit Mixtral setting) against the quantized-expert oracle: 2- and
4-bit codes at hidden widths that take every lane layout of the kernel
(d = 256 ... 4096), ragged token counts (many tokens per expert loop over
the kernel's token tile), outputs bitwise independent of residency and split
ratio, and the entry points' error codes."""
import numpy as np
import pytest

import synth
from gpu_helpers import check_layer

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [
    synth.ModelShape("q2-d256", 1, 256, 512, 8, 2, "bf16", expert_bits=2),
    synth.ModelShape("q4-d512", 1, 512, 256, 8, 2, "bf16", expert_bits=4),
    synth.ModelShape("q2-d1024", 1, 1024, 384, 16, 4, "bf16", expert_bits=2),
    synth.ModelShape("q4-d2048", 2, 2048, 256, 16, 4, "bf16", expert_bits=4),
    synth.ModelShape("q2-d4096", 1, 4096, 256, 8, 2, "bf16", expert_bits=2),
]


def _rig(shape, max_tokens=70):
    from workload import SplitRig, top_bytes
    r = SplitRig(shape, seed=2, max_tokens=max_tokens,
                 budget_bytes=shape.n_layers * shape.n_experts * shape.expert_bytes)
    tb = top_bytes(r, 0.5)
    r.configure([shape.n_experts * tb] * shape.n_layers, [0.5] * shape.n_layers)
    r.load_tops(0, list(range(0, shape.n_experts, 2)))
    return r


@pytest.fixture(scope="module", params=SHAPES, ids=lambda s: s.name)
def rig(request):
    r = _rig(request.param)
    yield r
    r.close()


def _run(rig, h, T, flags=0):
    y, idx, w = rig.outputs(T)
    rig.forward(0, h, T, y, idx, w, flags)
    torch.cuda.synchronize()
    return y, idx, w


@pytest.mark.parametrize("T", [1, 3, 17, 70])
def test_quantized_layer_parity(rig, T):
    h, hf = rig.hidden(T, tag=300 + T)
    y, idx, w = _run(rig, h, T)
    check_layer(rig, 0, hf, y, idx, w)


def test_quantized_outputs_independent_of_residency(rig):
    """Each chunk is computed the same way whether its codes sit in the top
    cache, in a prefetched staging slot or arrive after routing."""
    from paper_2509_08342_amd import moesplit as ms
    from workload import top_bytes
    s = rig.shape
    h, hf = rig.hidden(5, tag=9)
    y0, idx0, w0 = _run(rig, h, 5)
    check_layer(rig, 0, hf, y0, idx0, w0)
    y0 = y0.cpu().numpy()
    for r, tops in ((0.5, []), (0.25, list(range(s.n_experts))), (1.0, [1, 2]), (0.0, [])):
        tb = top_bytes(rig, r)
        rig.configure([s.n_experts * max(tb, 1)] * s.n_layers, [r] * s.n_layers)
        rig.load_tops(0, tops if r > 0 else [])
        ms.ms_drop_buffer(rig.ctx)
        y, idx, w = _run(rig, h, 5, ms.MS_FWD_PREDICT_NEXT if s.n_layers > 1 else 0)
        assert np.array_equal(idx.cpu().numpy(), idx0.cpu().numpy())
        assert np.array_equal(y.cpu().numpy(), y0), "r=%s tops=%s" % (r, tops)


def test_quantized_entry_points_reject_the_other_format():
    from paper_2509_08342_amd import moesplit as ms
    shape = SHAPES[0]
    with _rig(shape, max_tokens=4) as r:
        d, F = shape.d_model, shape.d_ff
        with pytest.raises(ms.MoeSplitError) as ei:
            ms.ms_set_expert(r.ctx, 0, 0, np.zeros((d, F), np.uint16), np.zeros((d, F), np.uint16),
                             np.zeros((F, d), np.uint16))
        assert ei.value.status == ms.MS_E_STATE
    from workload import SplitRig
    plain = synth.ModelShape("bf16-d256", 1, 256, 512, 8, 2, "bf16")
    with SplitRig(plain, seed=1, max_tokens=2, budget_bytes=0) as r2:
        qe = synth.quant_expert(SHAPES[0], 0, 0, 0, 2)
        with pytest.raises(ms.MoeSplitError) as ei:
            ms.ms_set_expert_q(r2.ctx, 0, 0, qe.codes, qe.meta)
        assert ei.value.status == ms.MS_E_STATE


@pytest.mark.parametrize("T", [3, 64, 70])
def test_quantized_matrix_core_and_chunk_paths_match_oracle(rig, T):
    """The matrix-core prefill over b-bit chunks (code pairs as bf16 B
    fragments, scale and zero folded per group) and the chunk kernel both
    match the oracle at partial and full row tiles."""
    from paper_2509_08342_amd import moesplit as ms
    h, hf = rig.hidden(T, tag=600 + T)
    for flag in (ms.MS_FWD_MATRIX_CORES, ms.MS_FWD_NO_MATRIX_CORES):
        y, idx, w = _run(rig, h, T, flag)
        check_layer(rig, 0, hf, y, idx, w)


# the staged matrix-core kernels (d a multiple of 256): row tiles of every
# height and experts over several tiles, one and two groups of four per row,
# an odd number of chunks, chunk ranges of the down projection that are no
# multiple of four; and the register-staged kernels (d = 320)
@pytest.mark.parametrize("bits,d,chunks", [(2, 256, 33), (4, 256, 5), (2, 512, 6), (4, 1024, 34), (2, 320, 5)])
def test_quantized_prefill_tiles(bits, d, chunks):
    from paper_2509_08342_amd import moesplit as ms
    from workload import top_bytes
    shape = synth.ModelShape("q%d-d%d-c%d" % (bits, d, chunks), 1, d, 64 * chunks, 4, 2, "bf16", expert_bits=bits)
    with _rig(shape, max_tokens=480) as r:
        for T in (3, 30, 62, 120, 180, 240, 310, 370, 480):
            h, hf = r.hidden(T, tag=T)
            r.configure([0], [0.0])
            ms.ms_drop_buffer(r.ctx)
            y0, idx, w = _run(r, h, T, ms.MS_FWD_MATRIX_CORES)
            small = d * chunks <= 256 * 33  # else some of the tokens, for the oracle's time
            check_layer(r, 0, hf, y0, idx, w, tokens=None if small else sorted({0, 1, T // 3, T // 2, T - 2, T - 1}))
            # whole experts and half of each resident: the same bits
            for ratio in (1.0, 0.5):
                r.configure([4 * top_bytes(r, ratio)], [ratio])
                r.load_tops(0, range(4))
                y, _, _ = _run(r, h, T, ms.MS_FWD_MATRIX_CORES)
                assert torch.equal(y, y0), "T=%d r=%s" % (T, ratio)


@pytest.mark.parametrize("bits,d,T,rows", [(2, 256, 4, 8), (4, 256, 15, 8), (2, 512, 8, 8), (4, 512, 16, 8),
                                           (4, 1024, 7, 4), (2, 1024, 8, 4), (2, 2048, 3, 2), (4, 2048, 4, 2), (2, 768, 16, 8)])
def test_quantized_path_choice(bits, d, T, rows):
    """Around the row count from which b-bit experts take the matrix cores (two
    rows per expert from width 2048 on, four from 1024, else eight; 4 experts,
    top-2): an unflagged forward gives the bits of the path the rule names, and
    matches the oracle."""
    from paper_2509_08342_amd import moesplit as ms
    from workload import top_bytes
    shape = synth.ModelShape("q%d-d%d-choice" % (bits, d), 1, d, 320, 4, 2, "bf16", expert_bits=bits)
    with _rig(shape, max_tokens=16) as r:
        r.configure([4 * top_bytes(r, 0.5)], [0.5])
        r.load_tops(0, range(4))
        h, hf = r.hidden(T, tag=T)
        y, idx, w = _run(r, h, T, 0)
        check_layer(r, 0, hf, y, idx, w)
        if d == 768:  # no chunk kernel
            named, _, _ = _run(r, h, T, ms.MS_FWD_MATRIX_CORES)
            assert torch.equal(y, named)
            return
        paths = [_run(r, h, T, f)[0] for f in (ms.MS_FWD_NO_MATRIX_CORES, ms.MS_FWD_MATRIX_CORES)]
        assert not torch.equal(paths[0], paths[1])  # (else nothing would be told apart)
        assert torch.equal(y, paths[T * 2 >= rows * 4])

"""GPU parity of the prefill path (matrix-core gate/up with a SwiGLU
epilogue, then the down projection over all of an expert's chunks) on small
bf16 shapes: ragged row tiles, shared experts, agreement with the decode
path, and outputs bitwise independent of split ratio and residency."""
import numpy as np
import pytest

import synth
from gpu_helpers import check_layer

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TINY_BF16 = synth.ModelShape("tiny-bf16", 1, 256, 512, 8, 2, "bf16")
TINY_SHARED = synth.ModelShape("tiny-bf16-shared", 2, 256, 384, 16, 4, "bf16", n_shared=2, d_ff_shared=320)
# 32 chunks per expert and a skewed router: at T = 300 and 400 the experts
# hold 0 .. 389 rows, so the LDS-staged gate/up launch (at least 256 tiles of
# up to 192 rows) runs 64-, 128- and 192-row tiles and hot experts span two
# and three tiles
SKEWED = synth.ModelShape("skewed-bf16", 1, 256, 2048, 8, 2, "bf16", zipf=0.8)


def _ms():
    from paper_2509_08342_amd import moesplit as ms
    return ms


@pytest.fixture(scope="module")
def rig():
    from workload import SplitRig
    r = SplitRig(TINY_BF16, seed=4, max_tokens=160, budget_bytes=8 * TINY_BF16.expert_bytes)
    yield r
    r.close()


def _configure(rig, ratio, tops, layer_count=1):
    from workload import top_bytes
    tb = top_bytes(rig, ratio)
    rig.configure([8 * tb] * layer_count, [ratio] * layer_count)
    for l in range(layer_count):
        rig.load_tops(l, tops)


def _run(rig, h, T, flags, layer=0):
    y, idx, w = rig.outputs(T)
    rig.forward(layer, h, T, y, idx, w, flags)
    torch.cuda.synchronize()
    return y, idx, w


@pytest.mark.parametrize("T", [1, 5, 64, 65, 130, 160])
def test_prefill_path_parity(rig, T):
    ms = _ms()
    _configure(rig, 0.5, [0, 1, 2, 3])
    h, hf = rig.hidden(T, tag=T)
    y, idx, w = _run(rig, h, T, ms.MS_FWD_MATRIX_CORES)
    check_layer(rig, 0, hf, y, idx, w)


def test_prefill_and_decode_paths_agree(rig):
    ms = _ms()
    _configure(rig, 0.5, [0, 2, 4, 6])
    h, hf = rig.hidden(48, tag=3)
    y1, i1, _ = _run(rig, h, 48, ms.MS_FWD_MATRIX_CORES)
    y2, i2, _ = _run(rig, h, 48, ms.MS_FWD_NO_MATRIX_CORES)
    assert torch.equal(i1, i2)
    ref = np.abs(y2.cpu().numpy()).max()
    assert np.abs(y1.cpu().numpy() - y2.cpu().numpy()).max() <= 1e-2 * ref + 1e-3


def test_prefill_outputs_independent_of_residency(rig):
    ms = _ms()
    h, hf = rig.hidden(96, tag=11)
    _configure(rig, 0.5, [0, 1, 2, 3])
    y0, idx0, w0 = _run(rig, h, 96, ms.MS_FWD_MATRIX_CORES)
    check_layer(rig, 0, hf, y0, idx0, w0)
    cases = [(0.5, [e for e in range(8) if (m >> e) & 1]) for m in (0, 1, 0x0f, 0xf0, 0x55, 0xff)]
    cases += [(0.0, []), (0.25, [1, 3]), (0.75, [0, 5, 6]), (1.0, list(range(8))), (1.0, [2])]
    for ratio, tops in cases:
        _configure(rig, ratio, tops)
        y, idx, w = _run(rig, h, 96, ms.MS_FWD_MATRIX_CORES)
        assert torch.equal(idx, idx0)
        assert torch.equal(y, y0), "r=%s tops=%s" % (ratio, tops)
    # a second pass reuses what the staging buffer still holds
    y, idx, w = _run(rig, h, 96, ms.MS_FWD_MATRIX_CORES)
    assert torch.equal(y, y0)


def test_prefill_with_few_buffer_slots_and_many_experts():
    """More active experts than staging slots: slots are recycled within one
    forward only after each expert's down projection."""
    ms = _ms()
    from workload import SplitRig
    shape = TINY_SHARED
    with SplitRig(shape, seed=5, max_tokens=128, n_buffer_slots=2,
                  budget_bytes=2 * 16 * shape.expert_bytes) as r:
        _configure(r, 0.5, [0, 1], layer_count=2)
        for layer in (0, 1):
            h, hf = r.hidden(128, tag=layer)
            y, idx, w = _run(r, h, 128, ms.MS_FWD_MATRIX_CORES | ms.MS_FWD_PREDICT_NEXT, layer=layer)
            check_layer(r, layer, hf, y, idx, w)
            st = ms.ms_stats(r.ctx, layer)
            assert st["gamma"] > 2


def test_prefill_shared_experts_decode_and_prefill(rig):
    ms = _ms()
    from workload import SplitRig
    shape = TINY_SHARED
    with SplitRig(shape, seed=6, max_tokens=64, budget_bytes=2 * 16 * shape.expert_bytes) as r:
        _configure(r, 0.5, list(range(0, 16, 2)), layer_count=2)
        h, hf = r.hidden(64, tag=9)
        for flags in (ms.MS_FWD_MATRIX_CORES, ms.MS_FWD_NO_MATRIX_CORES):
            y, idx, w = _run(r, h, 64, flags, layer=1)
            check_layer(r, 1, hf, y, idx, w)


@pytest.mark.parametrize("T", [300, 400])
def test_prefill_tall_tiles_parity_and_residency(T):
    """All experts resident: the staged gate/up kernel's tiles of every
    height match the oracle; with experts split or streamed, their chunks
    go through the other gate/up kernel, and no output bit changes."""
    ms = _ms()
    from workload import SplitRig
    shape = SKEWED
    with SplitRig(shape, seed=7, max_tokens=400, budget_bytes=8 * shape.expert_bytes) as r:
        h, hf = r.hidden(T, tag=T)
        _configure(r, 1.0, list(range(8)))
        y0, idx0, w0 = _run(r, h, T, ms.MS_FWD_MATRIX_CORES)
        counts = np.bincount(idx0.cpu().numpy().reshape(-1), minlength=8)
        tiles = [min(192, n - t) for n in counts for t in range(0, n, 192)]
        assert counts.max() > 192 and len(tiles) * 32 >= 256
        assert {(n + 63) // 64 for n in tiles} == {1, 2, 3}  # 64-, 128- and 192-row tiles
        check_layer(r, 0, hf, y0, idx0, w0)
        for ratio, tops in ((0.5, [0, 2, 4, 6]), (0.0, []), (0.25, [1, 3, 5, 7]), (1.0, list(range(8)))):
            _configure(r, ratio, tops)
            y, idx, w = _run(r, h, T, ms.MS_FWD_MATRIX_CORES)
            assert torch.equal(idx, idx0)
            assert torch.equal(y, y0), "r=%s tops=%s" % (ratio, tops)


@pytest.mark.parametrize("d", [320, 384])
def test_prefill_widths_off_the_staged_kernels(d):
    """d % 256 != 0 keeps the down projection on the 64-row kernel, and d =
    320 (d % 128 != 0) the gate/up too; oracle parity and outputs bitwise
    independent of residency there as well."""
    ms = _ms()
    from workload import SplitRig
    shape = synth.ModelShape("odd-d-bf16", 1, d, 2048, 8, 2, "bf16", zipf=0.8)
    T = 256
    with SplitRig(shape, seed=8, max_tokens=T, budget_bytes=8 * shape.expert_bytes) as r:
        h, hf = r.hidden(T, tag=d)
        _configure(r, 1.0, list(range(8)))
        y0, idx0, w0 = _run(r, h, T, ms.MS_FWD_MATRIX_CORES)
        check_layer(r, 0, hf, y0, idx0, w0)
        for ratio, tops in ((0.5, [1, 2, 5, 6]), (0.0, [])):
            _configure(r, ratio, tops)
            y, idx, w = _run(r, h, T, ms.MS_FWD_MATRIX_CORES)
            assert torch.equal(idx, idx0)
            assert torch.equal(y, y0), "r=%s tops=%s" % (ratio, tops)


@pytest.mark.parametrize("F,dtype,T", [(F, "bf16", T) for F in (320, 1024) for T in (5, 20, 40, 60, 75, 110, 128, 200)]
                         + [(320, "f32", 40), (1024, "f32", 70), (1024, "f32", 200)])
def test_decode_path_token_tiles(F, dtype, T):
    """The few-token kernel with 1 to 13 token tiles per launch (16 tokens each,
    8 with fp32 weights), most of them empty for most experts, for experts whose
    work-groups fill a run of 32 (F = 1024) and not (F = 320): every row of every
    expert is computed, whatever the order of the tiles."""
    from workload import SplitRig, top_bytes
    ms = _ms()
    shape = synth.ModelShape("tiles-%s-%d" % (dtype, F), 1, 256, F, 4, 1, dtype, zipf=1.0)
    with SplitRig(shape, seed=7, max_tokens=200, budget_bytes=4 * shape.expert_bytes) as r:
        h, hf = r.hidden(T, tag=T)
        for ratio in (1.0, 0.5):
            r.configure([4 * top_bytes(r, ratio)], [ratio])
            r.load_tops(0, range(4))
            y, idx, w = _run(r, h, T, ms.MS_FWD_NO_MATRIX_CORES)
            check_layer(r, 0, hf, y, idx, w)

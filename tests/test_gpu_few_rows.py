"""GPU parity of calls of few queries against the fp64 oracle: the attention kernel's form whose
waves without query rows only load (from one row, through whole waves and a wave cut short, to one
idle wave and none), and the merge of rows split over many workgroups (10 partial results of a row
by a workgroup, at the latent widths from 64 on, 16 with 12 of them in tests/test_gpu_layer.py, 5 to 10
in the per-head forms; fewer take the other merge), and its second pass (63 partial results at
d_c = 512, where four slices of eight take 32 at a time)."""
import numpy as np
import pytest
import torch

from tests._build_once import ensure_built

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ensure_built()
    import paper_2605_30351_amd as m
    yield m


from oracle import videomla_oracle as O  # noqa: E402
from tests.gpu_common import Layer, assert_attention_close, bf16_to_f64, dev, host_bits  # noqa: E402
from tests.test_gpu_dense import DENSE_SMALL, DenseLayer  # noqa: E402
from workloads import SMALL, TINY, f32_to_bf16_bits, make_dense_inputs, make_layer_inputs  # noqa: E402

# (first query token, tokens); two heads: 2 rows per token
BLOCKS = [(0, 1), (7, 16), (3, 33), (0, 48), (4, 111), (0, 120)]


def _check(vm, layer, fe, wants, label, form="latent"):
    for begin, count in BLOCKS:
        if begin + count > layer.inp.dims.chunk_tokens:
            continue
        for n_wg in (0, 2, 14):
            got = layer.attend(fe, vm.AttendOpts(n_workgroups=n_wg, form=form, query_begin=begin,
                                                 query_count=count))
            for b, want in enumerate(wants):
                assert_attention_close(got[b], want[begin:begin + count],
                                       f"{label} queries {begin} + {count} wg={n_wg} b={b}")


@pytest.mark.parametrize("d_c", [16, 64, 128, 192, 256, 512])
def test_latent(vm, d_c):
    dims = TINY.replace(window_frames=12, chunk_frames=4) if d_c == 16 else SMALL.replace(d_c=d_c)
    inp = make_layer_inputs(dims, seed=91, n_frames=12, batch=2)
    layer = Layer(vm, inp, packed=True)
    last = 12 - dims.chunk_frames
    for fe in range(0, 12, dims.chunk_frames):
        layer.write(fe)
    _check(vm, layer, last, [O.chunk_attention(inp, b, last) for b in range(2)], f"d_c={d_c}")


@pytest.mark.parametrize("d_nope", [96, 128])
def test_materialized(vm, d_nope):
    dims = SMALL.replace(d_nope=d_nope)
    inp = make_layer_inputs(dims, seed=92, n_frames=6)
    layer = Layer(vm, inp, packed=True)
    for fe in (0, 2, 4):
        layer.write(fe)
    _check(vm, layer, 4, [O.chunk_attention(inp, 0, 4)], f"d_nope={d_nope}", "materialized")


def test_dense(vm):
    inp = make_dense_inputs(DENSE_SMALL, seed=93, n_frames=6, batch=2)
    layer = DenseLayer(vm, inp)
    for fe in (0, 2, 4):
        layer.write(fe)
    _check(vm, layer, 4, [O.dense_chunk_attention(inp, b, 4) for b in range(2)], "dense")


@pytest.mark.parametrize("growth", [4.0, -4.0])
def test_second_pass_of_the_merge(vm, growth):
    """One query token over 68 key tiles at d_c = 512: 63 workgroups of one or two tiles. The keys
    grow (or shrink) with their position, so that the partial results of the second pass raise the
    running max of the first (or fall far below it). Bars scaled by the output magnitude."""
    d = SMALL.replace(d_c=512, window_frames=36)
    inp = make_layer_inputs(d, seed=94, n_frames=d.chunk_frames)
    rng = np.random.default_rng(95)
    S = d.window_tokens
    size = (max(0.2, 0.2 - growth) + growth * np.arange(S) / S)[:, None]
    c = f32_to_bf16_bits((rng.standard_normal((S, d.d_c)) * size).astype(np.float32))
    k = f32_to_bf16_bits((rng.standard_normal((S, d.d_rope)) * size).astype(np.float32))
    fe, n = 34, 1
    opts = vm.AttendOpts(query_count=n)
    ws = torch.full((vm.attend_workspace_bytes(d, 1, opts),), 0xFF, dtype=torch.uint8, device="cuda")
    out = torch.zeros((1, n, d.n_heads, d.d_v), dtype=torch.bfloat16, device="cuda")
    vm.attend(d, fe, 1, dev(inp.q_nope[:, :n]), dev(inp.q_r[:, :n]), dev(inp.w_uk), dev(inp.w_uv), dev(c[None]),
              dev(k[None]), out, ws, opts=opts)
    torch.cuda.synchronize()
    q_rope = O.query_rope(bf16_to_f64(inp.q_r[0, :n]), O.query_positions(np.arange(n), fe, d), d)
    want = O.attend_absorbed(bf16_to_f64(inp.q_nope[0, :n]), q_rope, bf16_to_f64(inp.w_uk),
                             bf16_to_f64(inp.w_uv), bf16_to_f64(c), bf16_to_f64(k), d)
    assert_attention_close(bf16_to_f64(host_bits(out))[0], want, f"63 splits, growth {growth}", scaled=True)

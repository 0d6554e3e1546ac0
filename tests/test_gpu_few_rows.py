"""GPU parity of calls of few queries against the fp64 oracle: the attention kernel's form whose
waves without query rows only load (from one row, through whole waves and a wave cut short, to one
idle wave and none), and the merge of rows split over many workgroups (10 partial results of a row
by a workgroup, at every latent width, 5 to 10 in the per-head forms; fewer take the other merge)."""
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
from tests.gpu_common import Layer, assert_attention_close  # noqa: E402
from tests.test_gpu_dense import DENSE_SMALL, DenseLayer  # noqa: E402
from workloads import SMALL, TINY, make_dense_inputs, make_layer_inputs  # noqa: E402

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

"""GPU parity of the wide-latent attention kernel (d_c = 512: 64-row blocks of four waves, 32-key
tiles, a ring of four tiles) where its work split and its tiles are ragged, against the fp64
oracle. 240 query rows per video are 3 whole row blocks and one of 48 rows. Windows of 120 and 300
keys are 4 and 10 tiles, the last one ragged. The workgroup counts give segments of one tile up
to whole row blocks, and workgroups with whole blocks, the head of one and the tail of one. Query
blocks of 1, 37 and 32 tokens end inside a 16-row, 32-row and 64-row group of rows."""
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
from workloads import SMALL, make_layer_inputs  # noqa: E402

DIMS = SMALL.replace(d_c=512)


@pytest.fixture(scope="module")
def layer(vm):
    inp = make_layer_inputs(DIMS, seed=71, n_frames=8, batch=2)
    lay = Layer(vm, inp, packed=True)
    wants = {}
    for fe in (0, 2, 4, 6):
        lay.write(fe)
        if fe in (0, 6):
            lay.snap = getattr(lay, "snap", {})
            lay.snap[fe] = (lay.c_kv.clone(), lay.k_r.clone())
            wants[fe] = [O.chunk_attention(inp, b, fe) for b in range(2)]
    lay.wants = wants
    return lay


@pytest.mark.parametrize("fe", [0, 6])
@pytest.mark.parametrize("n_wg", [0, 1, 3, 7, 11, 31, 80])
def test_split(layer, vm, fe, n_wg):
    layer.c_kv, layer.k_r = layer.snap[fe]
    got = layer.attend(fe, vm.AttendOpts(n_workgroups=n_wg))
    for b in range(2):
        assert_attention_close(got[b], layer.wants[fe][b], f"fe={fe} wg={n_wg} b={b}")


@pytest.mark.parametrize("begin,count", [(0, 1), (5, 37), (88, 32)])
def test_query_block(layer, vm, begin, count):
    layer.c_kv, layer.k_r = layer.snap[6]
    got = layer.attend(6, vm.AttendOpts(query_begin=begin, query_count=count))
    for b in range(2):
        assert_attention_close(got[b], layer.wants[6][b][begin:begin + count],
                               f"queries {begin} + {count} b={b}")


def test_weighted_split(layer, vm):
    layer.c_kv, layer.k_r = layer.snap[6]
    nbytes = vm.attend_workspace_bytes(DIMS, 2, vm.AttendOpts(n_workgroups=7, partition="adaptive"))
    ws = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    for mode in ("adaptive", "adaptive", "frozen"):
        got = layer.attend(6, vm.AttendOpts(n_workgroups=7, partition=mode), ws)
        for b in range(2):
            assert_attention_close(got[b], layer.wants[6][b], f"{mode} b={b}")

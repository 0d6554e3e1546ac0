"""GPU parity of the attention kernel where its running max rises tile after tile, and where its
work split needs 64-bit arithmetic.

Rising scores: the keys grow with their position, so that every key tile raises the running max by
more than the lazy margin for most rows and the accumulators are rescaled in every step, in place
or (d_c = 256 and 512) through LDS. The softmax is peaked: bars scaled by the output magnitude.

The split: units x workgroups below 2^32 is divided in 32-bit arithmetic, above it in 64-bit.
65,536 workgroups of one unit each reach 2^32 exactly; the same call over the default workgroups
is the reference. Both are exact merges of the same fp32 partial sums in another order, so they
differ by the bf16 roundings of o_lat and the output that flip (2^-9 of the value each) and by
the probabilities' rounding under another running max (2^-9 of each term): the fixed bars.
"""
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
from tests.gpu_common import assert_attention_close, bf16_to_f64, dev, host_bits  # noqa: E402
from workloads import SMALL, TINY, f32_to_bf16_bits, make_layer_inputs  # noqa: E402


@pytest.mark.parametrize("d_c,n_wg", [(64, 0), (128, 2), (192, 1), (192, 5), (256, 2), (512, 2)])
def test_rising_scores(vm, d_c, n_wg):
    d = SMALL.replace(d_c=d_c, window_frames=8)
    inp = make_layer_inputs(d, seed=61, n_frames=d.chunk_frames)
    rng = np.random.default_rng(62)
    S = d.window_tokens
    grow = (0.2 + 4.0 * np.arange(S) / S)[:, None]
    c = f32_to_bf16_bits((rng.standard_normal((S, d.d_c)) * grow).astype(np.float32))
    k = f32_to_bf16_bits((rng.standard_normal((S, d.d_rope)) * grow).astype(np.float32))
    fe = 6  # frames 6 and 7: the window is exactly full
    opts = vm.AttendOpts(n_workgroups=n_wg)
    ws = torch.empty(vm.attend_workspace_bytes(d, 1, opts), dtype=torch.uint8, device="cuda")
    out = torch.zeros((1, d.chunk_tokens, d.n_heads, d.d_v), dtype=torch.bfloat16, device="cuda")
    vm.attend(d, fe, 1, dev(inp.q_nope), dev(inp.q_r), dev(inp.w_uk), dev(inp.w_uv), dev(c[None]),
              dev(k[None]), out, ws, opts=opts)
    torch.cuda.synchronize()
    f64 = bf16_to_f64
    q_rope = O.query_rope(f64(inp.q_r[0]), O.query_positions(np.arange(d.chunk_tokens), fe, d), d)
    want = O.attend_absorbed(f64(inp.q_nope[0]), q_rope, f64(inp.w_uk), f64(inp.w_uv), f64(c),
                             f64(k), d)
    assert_attention_close(f64(host_bits(out))[0], want, f"rising d_c={d_c} wg={n_wg}", scaled=True)


def test_split_in_64_bit_arithmetic(vm):
    d = TINY.replace(grid_h=32, grid_w=32, window_frames=32)
    B, fe = 4, 40
    gen = torch.Generator(device="cuda").manual_seed(63)

    def normal(*shape, std=1.0):
        return torch.empty(shape, device="cuda").normal_(0, std, generator=gen).bfloat16()

    q_nope = normal(B, d.chunk_tokens, d.n_heads, d.d_nope)
    q_r = normal(B, d.chunk_tokens, d.n_heads, d.d_rope)
    w_uk = normal(d.n_heads * d.d_nope, d.d_c, std=d.d_c ** -0.5)
    w_uv = normal(d.n_heads * d.d_v, d.d_c, std=d.d_c ** -0.5)
    c_kv, k_r = normal(B, d.window_tokens, d.d_c), normal(B, d.window_tokens, d.d_rope)
    # 2,048 query rows = 16 row blocks of 128 per video, 32,768 keys = 1,024 tiles: 65,536 units
    outs = []
    for n_wg in (0, 65536):
        opts = vm.AttendOpts(n_workgroups=n_wg)
        ws = torch.empty(vm.attend_workspace_bytes(d, B, opts), dtype=torch.uint8, device="cuda")
        out = torch.zeros((B, d.chunk_tokens, d.n_heads, d.d_v), dtype=torch.bfloat16, device="cuda")
        vm.attend(d, fe, B, q_nope, q_r, w_uk, w_uv, c_kv, k_r, out, ws, opts=opts)
        torch.cuda.synchronize()
        outs.append(bf16_to_f64(host_bits(out)))
    assert_attention_close(outs[1], outs[0], "65,536 workgroups")

"""The token layout's workgroup shapes (1, 2, 4 and 8 waves, blocks past a short last chunk), row
widths (octets and sixteens of channels, and neither) and pointers off 16 bytes, against the
oracle bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2310_07240_amd import workloads as W
from gpu_helpers import assert_same, torch_cuda
from test_gpu_tokens import _run

pytestmark = pytest.mark.gpu

CASES = [
    # 2112 (context, chunk, layer, K/V): one wave per workgroup; chunks of 12 tokens
    W.small(name="w1_c24", n_ctx=8, n_layers=33, n_tokens=48, chunk_len=12, n_channels=24),
    # 1056 of two blocks (the last chunk of one): two waves
    W.small(name="w2_c8", n_ctx=4, n_layers=66, n_tokens=150, chunk_len=100, n_channels=8),
    # 600 of three blocks: four waves, one of them a helper
    W.small(name="w4_c16", n_ctx=2, n_layers=75, n_tokens=300, chunk_len=150, n_channels=16),
    # few: eight waves; nine blocks and a last chunk of four; C = 72 (octets), 80 (sixteens)
    W.small(name="w8_c72", n_layers=1, n_tokens=800, chunk_len=570, n_channels=72),
    W.small(name="w8_c80_g4", n_layers=1, n_tokens=130, chunk_len=70, n_channels=80, group_size=4),
    W.small(name="w8_c200", n_layers=1, n_tokens=64, chunk_len=64, n_channels=200),
    W.small(name="w8_c129_g64", n_layers=1, n_tokens=129, chunk_len=129, n_channels=129,
            group_size=64),
    # octets of channels with few long groups a chunk: a channel a thread, and either side of it
    W.small(name="one_group_64", n_layers=1, n_tokens=64, chunk_len=64, n_channels=72, group_size=64),
    W.small(name="one_group_63", n_layers=1, n_tokens=63, chunk_len=63, n_channels=72, group_size=64),
    W.small(name="groups8_201", n_layers=1, n_tokens=1700, chunk_len=1600, n_channels=24,
            group_size=201),
    W.small(name="groups9_201", n_layers=1, n_tokens=1700, chunk_len=1609, n_channels=24,
            group_size=201),
    W.small(name="groups2_200", n_layers=1, n_tokens=400, chunk_len=400, n_channels=24,
            group_size=200),
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_workgroup_shapes_bit_exact(w):
    _run(w, W.generate(w))


@pytest.mark.parametrize("offset", [1, 4])
def test_caches_off_16_bytes(offset):
    torch = torch_cuda()
    from paper_2310_07240_amd.cachegen import Codec, CodecParams
    w = W.small(name="tok_off", n_layers=1, n_tokens=90, chunk_len=60, n_channels=64)
    kv_np = W.generate(w)
    shape, cl_np = oracle.shape_from(w), w.chunk_levels()
    ca, cd = oracle.fit_all_levels(kv_np, shape)
    ow, oo, osc = oracle.encode_tokens(kv_np, shape, cl_np, ca, cd)
    want = oracle.decode_tokens(ow, oo, osc, shape, cl_np, ca, cd)
    codec = Codec(CodecParams.of(w))
    n = kv_np.size
    kv = torch.empty(n + 8, dtype=torch.int16, device="cuda")[offset:offset + n].view(kv_np.shape)
    kv.copy_(torch.from_numpy(kv_np.view(np.int16)))
    tca, tcd = (torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).cuda() for x in (ca, cd))
    cl = torch.from_numpy(cl_np).cuda()
    words, offsets, scales = codec.encode_tokens(kv, cl, tca, tcd)
    total = int(offsets[-1])
    assert_same("words", words[:total].cpu().numpy().view(np.uint32), ow)
    assert_same("scales", scales.cpu().numpy(), osc)
    buf = torch.full((n + 8,), 77, dtype=torch.int16, device="cuda")
    out = codec.decode_tokens(words, offsets, scales, cl, tca, tcd,
                              out=buf[offset:offset + n].view(kv_np.shape))
    assert_same("decoded fp16", out.cpu().numpy().view(np.uint16), want)
    rest = torch.cat([buf[:offset], buf[offset + n:]])
    assert bool((rest == 77).all()), "written outside the output"

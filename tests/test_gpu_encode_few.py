"""The encoder where few waves are spread over the CUs, with its own scales and with the fit's (then
with helper waves, which only stage tables), the one-workgroup scan around its tiles and its limit,
and the compaction around 32 words of a stream, against the oracle."""
import numpy as np
import pytest

from paper_2310_07240_amd import workloads as W
from gpu_helpers import assert_same, compare_full, run_gpu, run_oracle, torch_cuda

pytestmark = pytest.mark.gpu

CASES = [
    # six pairs of 20 units: one wave per workgroup, seven helpers
    W.small(name="spread_1", n_ctx=3, n_layers=5, n_tokens=90, chunk_len=45, n_channels=72),
    # 16 pairs of 32 units: two pairs per workgroup; two levels
    W.small(name="spread_2", n_ctx=8, n_layers=16, n_tokens=82, chunk_len=41, n_channels=64),
    # nine pairs of 100 units, G = 7: two pairs of two units, four helpers
    W.small(name="spread_4_g7", n_ctx=9, n_layers=50, n_tokens=44, chunk_len=44, n_channels=40,
            group_size=7, level_mult=(1.0,)),
    # 1024 waves at G = 10: two pairs of two units and four units of one pair, four helpers each; 810
    # of one pair: three units, three helpers
    W.small(name="help_2x2", n_ctx=2, n_layers=16, n_tokens=43, chunk_len=43, n_channels=1024),
    W.small(name="help_1x4", n_layers=32, n_tokens=21, chunk_len=21, n_channels=1024),
    W.small(name="help_1x3", n_layers=27, n_tokens=21, chunk_len=21, n_channels=960),
    # four pairs of a unit at one level: no helpers
    W.small(name="help_none", n_ctx=4, n_layers=4, n_tokens=30, chunk_len=30, n_channels=256,
            level_mult=(1.0,)),
    # short chunks stay together
    W.small(name="short", n_ctx=6, n_layers=4, n_tokens=39, chunk_len=39, n_channels=64),
    # 4096, 4097 and 16384 streams (one workgroup's scan), 16386 (three launches)
    W.small(name="scan_4096", n_layers=2, n_tokens=30, chunk_len=30, n_channels=1024),
    W.small(name="scan_4098", n_layers=1, n_tokens=30, chunk_len=30, n_channels=2049),
    W.small(name="scan_16384", n_layers=4, n_tokens=24, chunk_len=12, n_channels=1024),
    W.small(name="scan_16386", n_layers=1, n_tokens=11, chunk_len=11, n_channels=8193),
    # streams just below and above 32 and 128 words (8 bits a token at group size 1)
    W.small(name="words_32", n_layers=1, n_tokens=128, chunk_len=128, n_channels=130, group_size=1),
    W.small(name="words_128", n_layers=1, n_tokens=512, chunk_len=512, n_channels=130,
            group_size=1),
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_few_waves_bit_exact(w):
    torch = torch_cuda()
    from paper_2310_07240_amd.cachegen import Codec, CodecParams
    kv = W.generate(w)
    want = run_oracle(w, kv)
    compare_full(w, run_gpu(w, kv), want)
    # the same payload under the fit's scales, from a buffer that holds other words before
    codec = Codec(CodecParams.of(w))
    tkv = torch.from_numpy(np.ascontiguousarray(kv).view(np.int16)).cuda()
    cl = torch.from_numpy(w.chunk_levels()).cuda()
    scales = torch.empty((codec.n_streams,), dtype=torch.float32, device="cuda")
    ca, cd = codec.fit(tkv, scales=scales)
    words = torch.full((codec.bound_words,), -1, dtype=torch.int32, device="cuda")
    words, offsets = codec.encode_with_scales(tkv, cl, ca, cd, scales, words=words)
    n = int(offsets[-1])
    assert codec.status() == 0
    assert_same("offsets", offsets.cpu().numpy().view(np.uint64), want["offsets"])
    assert_same("words", words[:n].cpu().numpy().view(np.uint32), want["words"])
    assert bool((words[n:] == -1).all()), "written past the payload"

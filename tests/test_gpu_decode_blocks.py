"""The decoder's delta search covers 16, 8 or 4 blocks of 16 symbols, chosen per wave from the
tables. Payloads coded under another cache's tables hold symbols anywhere in the table, so they
take every way out of the searched blocks; the oracle decodes the same payload."""
import numpy as np
import pytest

import oracle
from paper_2310_07240_amd import workloads as W
from gpu_helpers import assert_same, run_gpu

pytestmark = pytest.mark.gpu


# bin: the delta bin, which sets the tables' width (the narrower the bin, the wider the table:
# 0.05 needs all 16 blocks, 0.7 eight, 3 four); channels: whole blocks, a last block of whole
# octets, and of a broken one; levels over two pairs and 512 units: windowed tables
@pytest.mark.parametrize("bin_", [0.05, 0.7, 3.0])
@pytest.mark.parametrize("n_layers,n_channels,n_tokens,chunk_len,levels", [
    (2, 128, 700, 400, (1.0,)),
    (1, 72, 95, 95, (1.0,)),
    (1, 70, 64, 30, (1.0, 2.0)),
    (4, 4096, 86, 43, (1.0, 4.0)),
])
def test_symbols_outside_the_searched_blocks(bin_, n_layers, n_channels, n_tokens, chunk_len,
                                             levels):
    w = W.small(name=f"blocks_{bin_}_{n_channels}", n_layers=n_layers, n_tokens=n_tokens,
                n_channels=n_channels, chunk_len=chunk_len, level_mult=levels,
                layer_bin=(bin_,) * n_layers, outlier_frac=0.0)
    shape = oracle.shape_from(w)
    cl = w.chunk_levels()
    kv = W.generate(w)
    ca, cd = oracle.fit_all_levels(kv, shape)
    # the same cache with a tenth of its tokens replaced by noise of the channel's own range
    rng = np.random.default_rng(5)
    other = kv.copy()
    hit = rng.random(kv.shape) < 0.1
    top = np.abs(kv.astype(np.float32)).max(axis=3, keepdims=True)
    other[hit] = (rng.uniform(-1, 1, kv.shape) * top).astype(np.float16)[hit]
    words, offsets, scales = oracle.encode(other, shape, cl, ca, cd)
    want = oracle.decode(words, offsets, scales, shape, cl, ca, cd)
    g = run_gpu(w, kv, decode_oracle_payload=(words, offsets, scales, ca, cd))
    assert_same("decoded fp16", g["out_from_oracle_payload"], want)
    assert_same("decoded own payload", g["out"],
                oracle.decode(g["words"], g["offsets"], g["scales"], shape, cl, ca, cd))


# Few waves: one, two and four decoding waves per workgroup (by pairs and by units), a grid that
# is not a multiple of the XCDs, and the chunks of one cache decoded alone
@pytest.mark.parametrize("n_ctx,n_layers,n_channels,n_tokens,chunk_len,levels", [
    (5, 3, 130, 90, 45, (1.0, 2.0)),        # 180 waves, one per workgroup
    (4, 32, 64, 82, 41, (1.0,)),            # 512 waves: two pairs of a unit per workgroup
    (19, 13, 72, 44, 44, (1.0, 2.0, 4.0, 8.0)),   # 988 waves: four units of one pair
    (1, 16, 2048, 43, 43, (1.0,)),          # 1024 waves of one pair: four units
    (6, 4, 72, 25, 12, (1.0, 4.0)),         # chunks of 12 tokens and one
    (16, 32, 64, 11, 11, (1.0,)),           # 1024 waves: four pairs of a unit
])
def test_at_most_a_wave_per_simd(n_ctx, n_layers, n_channels, n_tokens, chunk_len, levels):
    w = W.small(name=f"few_{n_ctx}_{n_layers}_{n_channels}", n_ctx=n_ctx, n_layers=n_layers,
                n_channels=n_channels, n_tokens=n_tokens, chunk_len=chunk_len, level_mult=levels)
    kv = W.generate(w)
    g = run_gpu(w, kv)
    want = oracle.decode(g["words"], g["offsets"], g["scales"], oracle.shape_from(w),
                         w.chunk_levels(), g["ca"], g["cd"])
    assert_same("decoded fp16", g["out"], want)

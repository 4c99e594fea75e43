"""The decoder's delta search covers 16, 8 or 4 blocks of 16 symbols, chosen per wave from the
tables, over tables staged whole or as windows; calls of few waves read the tables in pieces.
Payloads coded under another cache's tables hold symbols anywhere in the table, so they take every
way out of the searched blocks; the oracle decodes the same payload."""
import numpy as np
import pytest

import oracle
from paper_2310_07240_amd import workloads as W
from gpu_helpers import assert_same, run_gpu, torch_cuda

pytestmark = pytest.mark.gpu

LDS_BUDGET = 160 * 1024 - 1024   # dynamic LDS of a workgroup


def decode_stage(w, n_pairs=None):
    """How a group-of-10 decode of n_pairs (context, chunk) pairs stages its delta tables, as
    cg_launch_decode decides it: "pieces", "windows" or "columns"; and the waves that decode in a
    workgroup."""
    pairs = n_pairs or w.n_ctx * -(-w.n_tokens // w.chunk_len)
    units = 2 * w.n_layers * -(-w.n_channels // 64)
    levels = len(w.level_mult)

    def lds(nw, nu):
        return nu * (nw * 10 * 64 + min(nw, levels) * 64 * 260) * 2

    def piece_lds(nw, nu):
        return nu * (nw * 10 * 64 + min(nw, levels) * 33 * 512) * 2

    nw = min(pairs, 16)
    while nw > 1 and lds(nw, 1) > LDS_BUDGET:
        nw -= 1
    groups = -(-pairs // nw)
    nu = 1
    while (nu + 1) * nw <= 16 and lds(nw, nu + 1) <= LDS_BUDGET and -(-units // (nu + 1)) * groups >= 256:
        nu += 1
    sets = min(nw, levels)
    unit_bytes = nw * 10 * 64 * 2 + 64 * 260 * 2 + sets * 64 * 4
    nuc = 1
    while ((nuc + 1) * nw <= 16 and (nuc + 1) * unit_bytes <= LDS_BUDGET
           and -(-units // (nuc + 1)) * groups >= 256):
        nuc += 1
    for waves in range(1, 5):
        for pw in range(1, min(waves, pairs) + 1):
            pu = waves // pw
            if (pu * pw == waves and piece_lds(pw, pu) <= LDS_BUDGET
                    and (pu == 1 or pairs == 1 or min(w.chunk_len, w.n_tokens) >= 40)
                    and -(-units // pu) * -(-pairs // pw) <= 256):
                return "pieces", waves
    if sets > 1 and nuc > nu:
        return "windows", nw * nuc
    return ("pieces" if nw * nu <= 4 and piece_lds(nw, nu) <= LDS_BUDGET else "columns"), nw * nu


def searched_blocks(w, cd):
    """The numbers of blocks the waves of a decode of w search, as the kernel chooses them from the
    delta tables cd [levels, L, 2, C, 256]."""
    stage, waves = decode_stage(w)
    if (stage == "pieces" or w.n_channels % 8 or min(w.chunk_len, w.n_tokens) < 256
            or (w.n_ctx > 1 and waves == 16)):
        return {16}
    cum = cd.astype(np.int64)
    cum[..., 255] = 65536
    med = np.minimum((cum[..., :255] <= 32768).sum(-1) - 1, 254)

    def out(width):
        if stage == "columns":
            a = np.clip(med - width // 2, 0, 256 - width)
        else:
            a = np.clip((med + 8 - width // 2) // 16 * 16, 0, 256 - width)
        e = a + width
        lo = np.take_along_axis(cum, a[..., None], -1)[..., 0] - a
        hi = 65281 + e - np.take_along_axis(cum, np.minimum(e, 255)[..., None], -1)[..., 0]
        mass = lo + np.where(e >= 255, 0, hi)
        pad = -w.n_channels % 64   # lanes past the last channel repeat their block's first
        mass = np.concatenate([mass, np.repeat(mass[..., w.n_channels // 64 * 64][..., None],
                                               pad, -1)], -1) if pad else mass
        return 250 * w.n_ctx * mass.reshape(*mass.shape[:-1], -1, 64).sum(-1)

    gain8, gain4 = (8 << 16) - out(128), (12 << 16) - out(64)
    kf = np.where(gain8 > 0, 8, 16)
    kf = np.where((gain4 > 0) & ((kf == 16) | (gain4 > gain8)), 4, kf)
    used = sorted(set(w.chunk_levels().reshape(-1).tolist()))
    return set(kf[used].reshape(-1).tolist())


def foreign_payload(w, kv, ca, cd):
    """The cache with a tenth of its tokens replaced by noise of the channel's own range, coded under
    the tables of the cache itself, and what the oracle decodes from it."""
    shape = oracle.shape_from(w)
    rng = np.random.default_rng(5)
    other = kv.copy()
    hit = rng.random(kv.shape, np.float32) < 0.1
    top = np.abs(kv.astype(np.float32)).max(axis=3, keepdims=True)
    other[hit] = (rng.uniform(-1, 1, kv.shape) * top).astype(np.float16)[hit]
    words, offsets, scales = oracle.encode(other, shape, w.chunk_levels(), ca, cd)
    want = oracle.decode(words, offsets, scales, shape, w.chunk_levels(), ca, cd)
    return (words, offsets, scales, ca, cd), want


def check(w, stage, blocks):
    assert decode_stage(w)[0] == stage
    shape = oracle.shape_from(w)
    kv = W.generate(w)
    ca, cd = oracle.fit_all_levels(kv, shape)
    assert searched_blocks(w, cd) == blocks
    payload, want = foreign_payload(w, kv, ca, cd)
    g = run_gpu(w, kv, decode_oracle_payload=payload)
    assert_same("decoded fp16", g["out_from_oracle_payload"], want)
    assert_same("decoded own payload", g["out"],
                oracle.decode(g["words"], g["offsets"], g["scales"], shape, w.chunk_levels(),
                              g["ca"], g["cd"]))


# The layers' delta bins set the tables' widths (the narrower the bin, the wider the table), so that
# the waves of one call search 16, 8 and 4 blocks. More than 1024 waves: whole tables at one level,
# windows at four. Rows that are not made of whole octets of channels search 16, as do several
# contexts in workgroups of 16 waves.
@pytest.mark.timeout(300)
@pytest.mark.parametrize("n_ctx,n_channels,n_tokens,levels,stage,blocks", [
    (1, 728, 3840, (1.0,), "columns", {4, 8, 16}),
    (1, 5504, 768, (1.0, 1.5, 2.0, 4.0), "windows", {4, 8, 16}),
    (3, 728, 1280, (1.0,), "columns", {4, 8, 16}),
    (1, 730, 3840, (1.0,), "columns", {16}),
    (2, 728, 2048, (1.0,), "columns", {16}),
])
def test_narrow_searches(n_ctx, n_channels, n_tokens, levels, stage, blocks):
    check(W.small(name=f"narrow_{stage}_{n_channels}", n_ctx=n_ctx, n_layers=3, n_channels=n_channels,
                  n_tokens=n_tokens, chunk_len=256, level_mult=levels, layer_bin=(0.05, 1.4, 3.0),
                  outlier_frac=0.0), stage, blocks)


# Few waves, tables in pieces (all 16 blocks): whole blocks of channels, a last block of whole octets, and of a
# broken one; two levels
@pytest.mark.parametrize("bin_", [0.05, 0.7, 3.0])
@pytest.mark.parametrize("n_layers,n_channels,n_tokens,chunk_len,levels", [
    (2, 128, 700, 400, (1.0,)),
    (1, 72, 95, 95, (1.0,)),
    (1, 70, 64, 30, (1.0, 2.0)),
    (4, 4096, 86, 43, (1.0, 4.0)),
])
def test_symbols_outside_the_searched_blocks(bin_, n_layers, n_channels, n_tokens, chunk_len, levels):
    check(W.small(name=f"blocks_{bin_}_{n_channels}", n_layers=n_layers, n_tokens=n_tokens,
                  n_channels=n_channels, chunk_len=chunk_len, level_mult=levels,
                  layer_bin=(bin_,) * n_layers, outlier_frac=0.0), "pieces", {16})


# One, two and four decoding waves per workgroup (by pairs and by units), a grid that is not a
# multiple of the XCDs, more than 1024 waves of one pair, and every chunk of a cache decoded alone
@pytest.mark.parametrize("n_ctx,n_layers,n_channels,n_tokens,chunk_len,levels", [
    (5, 3, 130, 90, 45, (1.0, 2.0)),        # 180 waves, one per workgroup
    (4, 32, 64, 82, 41, (1.0,)),            # 512 waves: two pairs of a unit per workgroup
    (19, 13, 72, 44, 44, (1.0, 2.0, 4.0, 8.0)),   # 988 waves: four units of one pair
    (1, 16, 2048, 43, 43, (1.0,)),          # 1024 waves of one pair: four units
    (1, 17, 2048, 21, 21, (1.0, 2.0)),      # 1088 waves of one pair
    (6, 4, 72, 25, 12, (1.0, 4.0)),         # chunks of 12 tokens and one
    (16, 32, 64, 11, 11, (1.0,)),           # 1024 waves: four pairs of a unit
    (3, 80, 128, 29, 29, (1.0,)),           # 960 waves: three pairs of a unit
])
def test_at_most_a_wave_per_simd(n_ctx, n_layers, n_channels, n_tokens, chunk_len, levels):
    torch = torch_cuda()
    from paper_2310_07240_amd.cachegen import Codec, CodecParams
    w = W.small(name=f"few_{n_ctx}_{n_layers}_{n_channels}", n_ctx=n_ctx, n_layers=n_layers,
                n_channels=n_channels, n_tokens=n_tokens, chunk_len=chunk_len, level_mult=levels)
    assert decode_stage(w)[0] == decode_stage(w, n_ctx)[0] == "pieces"
    kv = W.generate(w)
    g = run_gpu(w, kv)
    want = oracle.decode(g["words"], g["offsets"], g["scales"], oracle.shape_from(w),
                         w.chunk_levels(), g["ca"], g["cd"])
    assert_same("decoded fp16", g["out"], want)
    codec = Codec(CodecParams.of(w))
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (
        np.concatenate([g["words"], np.zeros(8, np.uint32)]).view(np.int32),
        g["offsets"].view(np.int64), g["scales"], w.chunk_levels(), g["ca"].view(np.int16),
        g["cd"].view(np.int16))]
    out = torch.zeros(kv.shape, dtype=torch.int16, device="cuda")
    for c in range(-(-n_tokens // chunk_len)):
        codec.decode(*dev, c, c + 1, out=out)
    assert_same("chunk by chunk", out.cpu().numpy().view(np.uint16), want)

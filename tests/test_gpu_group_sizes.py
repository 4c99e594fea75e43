"""Group sizes other than the paper's 10, bit for bit against the oracle in both stream layouts:
groups longer than every chunk, up to the largest the ABI takes."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2310_07240_amd import workloads as W
from gpu_helpers import assert_same, say, torch_cuda

pytestmark = pytest.mark.gpu


def run_all(w, oracle_group):
    """Every codec call on w, against the oracle at group size oracle_group (equal in meaning)."""
    torch = torch_cuda()
    from paper_2310_07240_amd.cachegen import Codec, CodecParams
    ow = dataclasses.replace(w, group_size=oracle_group)
    shape, cl_np, kv_np = oracle.shape_from(ow), ow.chunk_levels(), W.generate(ow)
    ca, cd = oracle.fit_all_levels(kv_np, shape)
    words, offsets, scales = oracle.encode(kv_np, shape, cl_np, ca, cd)
    want = oracle.decode(words, offsets, scales, shape, cl_np, ca, cd)
    codec = Codec(CodecParams.of(w))
    kv = torch.from_numpy(np.ascontiguousarray(kv_np).view(np.int16)).cuda()
    cl = torch.from_numpy(cl_np).cuda()
    say(f"{w.name}: fit")
    gs = torch.empty((codec.n_streams,), dtype=torch.float32, device="cuda")
    ga, gd = codec.fit(kv, scales=gs)
    assert_same("anchor tables", ga.cpu().numpy().view(np.uint16), ca)
    assert_same("delta tables", gd.cpu().numpy().view(np.uint16), cd)
    assert_same("scales", gs.cpu().numpy(), scales)
    la, ld = codec.fit_per_level(kv)
    assert_same("per-level anchor tables", la.cpu().numpy().view(np.uint16), ca)
    assert_same("per-level delta tables", ld.cpu().numpy().view(np.uint16), cd)
    say(f"{w.name}: encode, decode")
    gw, go, _ = codec.encode(kv, cl, ga, gd)
    assert_same("words", gw[:int(go[-1])].cpu().numpy().view(np.uint32), words)
    out = codec.decode(gw, go, gs, cl, ga, gd)
    assert_same("decoded fp16", out.cpu().numpy().view(np.uint16), want)
    say(f"{w.name}: token layout")
    tw, to, ts = oracle.encode_tokens(kv_np, shape, cl_np, ca, cd)
    gw, go, gts = codec.encode_tokens(kv, cl, ga, gd)
    assert_same("token words", gw[:int(go[-1])].cpu().numpy().view(np.uint32), tw)
    assert_same("token scales", gts.cpu().numpy(), ts)
    out = codec.decode_tokens(gw, go, gts, cl, ga, gd)
    assert_same("token layout's decoded fp16", out.cpu().numpy().view(np.uint16), want)


# whole blocks, even and odd channel counts: every fit kernel; 2^28 and 2^31 - 1: slice ends and
# rounded-up group counts past 32 bits unless the group is cut to the chunk
@pytest.mark.parametrize("group", [49, 1 << 28, (1 << 31) - 1])
@pytest.mark.parametrize("channels,levels", [(64, (1.0,)), (72, (1.0, 2.0)), (65, (1.0, 2.0)),
                                             (65, (1.0,))])
def test_groups_longer_than_the_chunks(group, channels, levels):
    w = W.small(name=f"group_{group}_c{channels}", n_layers=2, n_tokens=100, chunk_len=48,
                n_channels=channels, level_mult=levels, group_size=group)
    run_all(w, 48)


def test_a_group_of_ten_in_shorter_chunks():
    """The chunks hold one group each; group size 10 keeps its own kernels."""
    run_all(W.small(name="chunks_of_7", n_tokens=20, chunk_len=7, n_channels=72), 7)

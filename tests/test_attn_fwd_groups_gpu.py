"""The forward's key groups: how many of them share a workgroup (one, two or four) follows from the extents of the call,
fewer the more workgroups there are, so the same sequence is run alone and inside larger batches to reach all three,
each against the oracle.  The count that every case is there for stands beside it; a test on the host holds the rule to
these tables, so that a change of the rule cannot leave a count untested."""
import numpy as np
import pytest
import torch

from oracle import ref_block as rb
from oracle import ref_numpy as rn
from paper_2604_27089_amd import binding as sp
from paper_2604_27089_amd import synth
from gpu_util import LSE_MAX_ABS, check_o, dev_bf16, host_f64

pytestmark = pytest.mark.gpu

# rows -> {batch entries of one head: key groups}: the edges of the classes, and counts between them
BATCHES = {
    1: {1: 1, 385: 1}, 31: {1: 1, 128: 1}, 33: {1: 1, 129: 1}, 64: {1: 1, 64: 1, 385: 1}, 65: {1: 1, 65: 1, 100: 1},
    127: {1: 4, 64: 4, 128: 4, 129: 2, 385: 2},
    129: {1: 4, 65: 4, 85: 4, 86: 2, 128: 2, 129: 1, 385: 1},
    255: {1: 4, 64: 4, 65: 2, 128: 2, 129: 1},
    256: {1: 4, 64: 4, 65: 2, 100: 2, 128: 2, 129: 1, 385: 1},
    257: {1: 4, 51: 4, 52: 2, 85: 2, 86: 1, 129: 2, 171: 1, 193: 1},
    300: {1: 4, 32: 4, 51: 4, 52: 2, 65: 2, 85: 2, 86: 1, 193: 1},
    512: {1: 4, 32: 4, 33: 2, 64: 2, 65: 1, 193: 1},
}
# (rows, keys, offset) -> the same
BLOCKS = {
    (1, 1, 0): {1: 1, 65: 1, 385: 1}, (1, 200, 199): {1: 4, 129: 4}, (40, 130, 90): {1: 4, 65: 4, 385: 4}, (300, 64, 7): {1: 1, 65: 1, 193: 1},
    (257, 500, 400): {1: 4, 51: 4, 52: 2, 85: 2, 86: 1, 193: 1}, (130, 129, 5000): {1: 4, 85: 4, 86: 2, 128: 2, 129: 1},
}
# document lengths -> {query heads: key groups}.  763 rows: three tiles, the last one ragged; 9000: walks of many tiles
SHORT, LONG = (70, 0, 1, 300, 63, 129, 200), (3100, 0, 2500, 3400)
PACKED = {SHORT: {4: 4, 20: 4, 22: 2, 42: 2, 44: 1, 60: 1, 140: 1}, LONG: {4: 2}}
# rows of one sequence of four heads
WALKS = {2048: 4, 12288: 2, 24832: 1}


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("S", sorted(BATCHES))
def test_batch_sizes_of_every_class(S, D):
    qb, kb, vb, _ = synth.attn_inputs(S + D, S, 1, 1, D)
    q, k, v = (dev_bf16(t) for t in (qb, kb, vb))
    o_ref, lse_ref = rn.attn_fwd(*(rn.widen_bf16(t[0]) for t in (qb, kb, vb)))
    for B in BATCHES[S]:
        o, lse = sp.sp_attn_fwd(*(t.expand(B, -1, -1, -1).contiguous() for t in (q, k, v)))
        assert torch.equal(o.view(torch.int16), o[:1].expand_as(o).contiguous().view(torch.int16))
        assert torch.equal(lse, lse[:1].expand_as(lse))
        check_o(host_f64(o[0]), o_ref, f"S={S} D={D} B={B}")
        assert np.abs(host_f64(lse[0]) - lse_ref).max() <= LSE_MAX_ABS


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Sq,Skv,off", sorted(BLOCKS))
def test_blocks_of_every_class(Sq, Skv, off, D):
    qb, _, _, _ = synth.attn_inputs(Sq, Sq, 1, 1, D)
    _, kb, vb, _ = synth.attn_inputs(Skv + 7, Skv, 1, 1, D)
    q, k, v = (dev_bf16(t) for t in (qb, kb, vb))
    o_ref, lse_ref = rb.block_attn_fwd(*(rn.widen_bf16(t[0]) for t in (qb, kb, vb)), 1.0 / np.sqrt(D), off)
    for B in BLOCKS[Sq, Skv, off]:
        o, lse = sp.sp_attn_block_fwd(*(t.expand(B, -1, -1, -1).contiguous() for t in (q, k, v)), off)
        check_o(host_f64(o[B - 1]), o_ref, f"Sq={Sq} Skv={Skv} off={off} D={D} B={B}")
        assert np.abs(host_f64(lse[B - 1]) - lse_ref).max() <= LSE_MAX_ABS


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("lengths,Hq", [(lengths, Hq) for lengths, heads in PACKED.items() for Hq in heads])
def test_packed_documents_of_every_class(lengths, Hq, D):
    cu_h = synth.cu_seqlens_from_lengths(lengths)
    qb, kb, vb, _ = synth.attn_inputs(Hq, sum(lengths), 2, 1, D)
    q, k, v = (dev_bf16(t[0]) for t in (qb, kb, vb))
    o_ref, lse_ref = rn.attn_varlen_fwd(*(rn.widen_bf16(t[0]) for t in (qb, kb, vb)), cu_h)
    rep = Hq // 2
    o, lse = sp.sp_attn_varlen_fwd(q.repeat(1, rep, 1), k.repeat(1, rep, 1), v.repeat(1, rep, 1), torch.from_numpy(cu_h).cuda())
    for h0 in (0, Hq - 2):
        check_o(host_f64(o[:, h0:h0 + 2]), o_ref, f"Hq={Hq} D={D} heads {h0}..")
        assert np.abs(host_f64(lse[h0:h0 + 2]) - lse_ref).max() <= LSE_MAX_ABS


@pytest.mark.parametrize("S", sorted(WALKS))
def test_longer_walks_of_every_class(S):
    """Many tiles per group; the last rows, whose walks are the longest, against the oracle."""
    qb, kb, vb, _ = synth.attn_inputs(S, S, 4, 1, 128)
    q, k, v = (dev_bf16(t) for t in (qb, kb, vb))
    o, lse = sp.sp_attn_fwd(q, k, v)
    n = 70
    kf, vf = (rn.widen_bf16(t[0]) for t in (kb, vb))
    o_ref, lse_ref = rb.block_attn_fwd(rn.widen_bf16(qb[0, S - n:]), kf, vf, 1.0 / np.sqrt(128), S - n)
    check_o(host_f64(o[0, S - n:]), o_ref, f"S={S}")
    assert np.abs(host_f64(lse[0, :, S - n:]) - lse_ref).max() <= LSE_MAX_ABS

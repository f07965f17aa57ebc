"""The backward's two matrix stages in one launch: whatever order the workgroups go out in, every one runs.  Heads are
copies of each other, so a workgroup left out or run twice shows as a head that differs; one head is held to the
oracle.  Sizes put the launch into every class of the order: alternation with either stage in front, dQ first and
dK/dV first, and single stages."""
import numpy as np
import pytest
import torch

from oracle import ref_block as rb
from oracle import ref_numpy as rn
from paper_2604_27089_amd import binding as sp
from paper_2604_27089_amd import synth
from gpu_util import GRAD_REL_L2, dev_bf16, grad_err, guarded, host_f64
from test_padded_build_gpu import run, same_bits
from paper_2604_27089_amd import build as spbuild

pytestmark = pytest.mark.gpu


def same_heads(t):
    return torch.equal(t.view(torch.int16), t[..., :1, :].expand_as(t).contiguous().view(torch.int16))


# (rows, copies of one query and one key/value head): up to 768 workgroups alternate, above that dQ goes first
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("S,heads", [(40, 1), (300, 3), (300, 191), (300, 260), (1100, 90)])
def test_full_attention(S, heads, D):
    bits = synth.attn_inputs(S + heads, S, 1, 1, D)
    q, k, v, do = (dev_bf16(t).expand(-1, -1, heads, -1).contiguous() for t in bits)
    o, lse = sp.sp_attn_fwd(q, k, v)
    ws = torch.empty(sp.sp_attn_bwd_workspace_bytes(1, S, heads, heads, D), dtype=torch.uint8, device="cuda")
    dq, dk, dv = sp.sp_attn_bwd(q, k, v, o, lse, do, workspace=ws)
    assert same_heads(dq) and same_heads(dk) and same_heads(dv)
    refs = rn.attn_bwd(*(rn.widen_bf16(t[0]) for t in bits), 0.0)[:3]
    for got, ref, name in zip((dq, dk, dv), refs, ("dq", "dk", "dv")):
        assert grad_err(host_f64(got[0, :, :1]), ref, name) <= GRAD_REL_L2
    # the stages one at a time give the same bits, and a stage writes its own outputs only
    parts = [torch.full_like(t, 7.0) for t in (dq, dk, dv)]
    for stage in (sp.SP_BWD_STAGE_DELTA, sp.SP_BWD_STAGE_DQ, sp.SP_BWD_STAGE_DKDV):
        sp.sp_attn_bwd_stages(q, k, v, o, lse, do, *parts, ws, stage)
        if stage != sp.SP_BWD_STAGE_DKDV:
            assert bool((parts[1] == 7.0).all()) and bool((parts[2] == 7.0).all())
            assert bool((parts[0] == 7.0).all()) == (stage == sp.SP_BWD_STAGE_DELTA)
    for a, b in zip(parts, (dq, dk, dv)):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))


# packed documents: alternation up to 1280 workgroups; above, dK/dV first when one document stands out (a long
# document among many short ones), else dQ first
@pytest.mark.parametrize("lengths,heads", [([70, 1, 200], 4), ([763], 240), ([600] + [3] * 60, 240), ([90] * 8, 260)])
def test_packed_documents(lengths, heads):
    D, T = 64, sum(lengths)
    cu_h = synth.cu_seqlens_from_lengths(lengths)
    cu = torch.from_numpy(cu_h).cuda()
    bits = synth.attn_inputs(T + heads, T, 1, 1, D)
    q, k, v, do = (dev_bf16(t[0]).expand(-1, heads, -1).contiguous() for t in bits)
    o, lse = sp.sp_attn_varlen_fwd(q, k, v, cu, max(lengths))
    grads = sp.sp_attn_varlen_bwd(q, k, v, o, lse, do, cu, max(lengths))
    assert all(same_heads(t) for t in grads)
    refs = rn.attn_varlen_bwd(*(rn.widen_bf16(t[0]) for t in bits), cu_h)[:3]
    for got, ref, name in zip(grads, refs, ("dq", "dk", "dv")):
        assert grad_err(host_f64(got[:, :1]), ref, name) <= GRAD_REL_L2


def check_block(Sq, Skv, off, Hq, Hkv, D):
    qb, _, _, dob = synth.attn_inputs(Sq, Sq, Hq, Hkv, D)
    _, kb, vb, _ = synth.attn_inputs(Skv + 3, Skv, Hq, Hkv, D)
    q, k, v, do = (dev_bf16(t) for t in (qb, kb, vb, dob))
    o, lse = sp.sp_attn_block_fwd(q, k, v, off)
    ws, check = guarded((sp.sp_attn_block_bwd_workspace_bytes(1, Sq, Skv, Hq, Hkv, D),), torch.uint8)
    dq, dk, dv = sp.sp_attn_block_bwd(q, k, v, o, lse, do, off, workspace=ws)
    check("workspace")
    q64, k64, v64, do64 = (rn.widen_bf16(t[0]) for t in (qb, kb, vb, dob))
    scale = 1.0 / np.sqrt(D)
    o_ref, lse_ref = rb.block_attn_fwd(q64, k64, v64, scale, off)
    refs = rb.block_attn_bwd(q64, k64, v64, lse_ref, np.einsum("shd,shd->hs", o_ref, do64), do64, scale, off)
    for got, ref, name in zip((dq, dk, dv), refs, ("dq", "dk", "dv")):
        assert grad_err(host_f64(got[0]), ref, name) <= GRAD_REL_L2, (name, Sq, Skv, off, Hq, Hkv, D)
    again = sp.sp_attn_block_bwd(q, k, v, o, lse, do, off)
    assert all(torch.equal(a.view(torch.int16), b.view(torch.int16)) for a, b in zip(again, (dq, dk, dv)))


# one-round launches: chunks of equal length, as many per key tile as its steps need; ragged last tiles, offsets, and
# shapes just past one round (unequal chunks).  The workspace has exactly the asked size, between canaries.
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Sq,Skv,off,Hq,Hkv", [(257, 257, 0, 4, 1), (513, 513, 0, 1, 1), (1030, 1030, 0, 3, 1), (900, 900, 0, 8, 2),
                                               (300, 1199, 900, 8, 1), (1500, 259, 0, 4, 1), (700, 800, 5000, 4, 2),
                                               (2047, 2047, 0, 2, 1), (1025, 1025, 0, 16, 8), (2050, 2050, 0, 10, 5)])
def test_equal_chunks(Sq, Skv, off, Hq, Hkv, D):
    check_block(Sq, Skv, off, Hq, Hkv, D)


# blocks that hide little, beyond one round of the chip: whole rounds of the longer stage, then the other
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Sq,Skv,off,Hq,Hkv", [(900, 900, 880, 32, 8), (700, 700, 699, 36, 9), (1025, 1025, 520, 40, 8), (1290, 1400, 1300, 24, 8)])
def test_even_walks(Sq, Skv, off, Hq, Hkv, D):
    check_block(Sq, Skv, off, Hq, Hkv, D)


# the hand-scheduled dQ program with two row blocks per wave runs above 128 tiles of 256 rows: there, too, the build
# with every wait spelled out must give the same bits
@pytest.mark.parametrize("B,S,Hq,Hkv,D", [(1, 777, 36, 9, 128), (3, 513, 20, 5, 64), (1, 5000, 8, 1, 128)])
def test_padded_build_two_row_blocks(B, S, Hq, Hkv, D):
    fast, padded = sp.lib(), sp.open_library(spbuild.LIB_PADDED)
    q, k, v, do = (dev_bf16(t) for t in synth.attn_inputs(S + D, S, Hq, Hkv, D, B))
    same_bits(run(fast, q, k, v, do), run(padded, q, k, v, do), f"B={B} S={S} {Hq}q/{Hkv}kv D={D}")


@pytest.mark.parametrize("D", [64, 128])
def test_padded_build_two_row_blocks_packed(D):
    fast, padded = sp.lib(), sp.open_library(spbuild.LIB_PADDED)
    lengths = [130, 0, 64, 1, 700, 63, 129, 2040, 8, 30, 2, 1500]
    cu = synth.cu_seqlens_from_lengths(lengths)
    q, k, v, do = (dev_bf16(t[0]) for t in synth.attn_inputs(78, int(cu[-1]), 9, 3, D))
    cud = torch.from_numpy(cu).cuda()
    same_bits(run(fast, q, k, v, do, cud), run(padded, q, k, v, do, cud), f"packed documents D={D}")

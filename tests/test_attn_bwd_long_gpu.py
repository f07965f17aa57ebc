"""The backward's programs of long launches (16x16x32 MFMAs) at their edges.  By rule they run where a reference takes
minutes, so a build of the library that sends every backward to them (LIB_LONG) is held to the oracle at small sizes, and
the regular library is shown to run the same programs, hazard-free, at sizes where the rule picks them."""
import numpy as np
import pytest
import torch

from oracle import ref_block as rb
from oracle import ref_numpy as rn
from paper_2604_27089_amd import binding as sp
from paper_2604_27089_amd import build as spbuild
from paper_2604_27089_amd import synth
from gpu_util import GRAD_REL_L2, dev_bf16, grad_err, host_f64
from test_padded_build_gpu import run, same_bits

pytestmark = pytest.mark.gpu


@pytest.fixture
def long_build(monkeypatch):
    L = sp.open_library(spbuild.LIB_LONG)
    monkeypatch.setattr(sp, "_lib", L)
    return L


def check_grads(got, refs, what):
    for t, ref, name in zip(got, refs, ("dQ", "dK", "dV")):
        assert grad_err(t, ref, f"{what} {name}") <= GRAD_REL_L2


# one row to several tiles; ragged ends; one and two row blocks of dQ; one chunk per key tile (the last three) and several,
# equal ones among them
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,S,Hq,Hkv", [(1, 1, 1, 1), (1, 31, 2, 1), (1, 33, 5, 5), (1, 65, 4, 2), (2, 257, 3, 1), (1, 513, 4, 1), (1, 1030, 3, 1),
                                        (1, 777, 36, 9), (33, 20, 4, 4), (3, 290, 48, 48), (1, 300, 200, 200)])
def test_dense_matches_oracle(long_build, B, S, Hq, Hkv, D):
    print(f"B={B} S={S} {Hq}/{Hkv} D={D}", flush=True)
    bits = synth.attn_inputs(S + D, S, Hq, Hkv, D, B)
    q, k, v, do = (dev_bf16(t) for t in bits)
    o, lse = sp.sp_attn_fwd(q, k, v)
    got = sp.sp_attn_bwd(q, k, v, o, lse, do)
    for b in sorted({0, B - 1}):
        refs = rn.attn_bwd(*(rn.widen_bf16(t[b]) for t in bits))[:3]
        check_grads([host_f64(t[b]) for t in got], refs, f"batch entry {b}")


# offsets: hidden keys beside whole rounds, rows that see every key, more keys than rows and the other way round
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Sq,Skv,off,Hq,Hkv", [(300, 1199, 900, 8, 1), (1500, 259, 0, 4, 1), (700, 700, 700, 36, 9), (1025, 1025, 520, 40, 8), (90, 95, 5, 2, 2)])
def test_blocks_match_oracle(long_build, Sq, Skv, off, Hq, Hkv, D):
    print(f"Sq={Sq} Skv={Skv} off={off} {Hq}/{Hkv} D={D}", flush=True)
    qb, _, _, dob = synth.attn_inputs(Sq, Sq, Hq, Hkv, D)
    _, kb, vb, _ = synth.attn_inputs(Skv + 3, Skv, Hq, Hkv, D)
    q, k, v, do = (dev_bf16(t) for t in (qb, kb, vb, dob))
    o, lse = sp.sp_attn_block_fwd(q, k, v, off)
    got = sp.sp_attn_block_bwd(q, k, v, o, lse, do, off)
    q64, k64, v64, do64 = (rn.widen_bf16(t[0]) for t in (qb, kb, vb, dob))
    scale = 1.0 / np.sqrt(D)
    o_ref, lse_ref = rb.block_attn_fwd(q64, k64, v64, scale, off)
    refs = rb.block_attn_bwd(q64, k64, v64, lse_ref, np.einsum("shd,shd->hs", o_ref, do64), do64, scale, off)
    check_grads([host_f64(t[0]) for t in got], refs, "block")


# Lanes hidden by a document's end stay hidden from step to step, until a step in which the next one ends.  Several ends
# inside one wave's 64 keys and rows, on and off the 32-row steps; documents that end with a tile; groups of heads, whose
# later heads start the walk again at the top; chunks that start in the middle of a head (several per tile: 32 to 96 steps
# of four to nine heads in up to eight chunks).  Two row blocks of dQ from 128 tiles on: 36 heads.
PACKED = {
    "many ends in a block": [5, 17, 10, 32, 64, 1, 31, 33, 96, 0, 128, 7, 9, 11, 200, 3, 3, 3, 60],
    "ends on steps": [32, 32, 64, 32, 96, 32, 256, 32, 32, 160],
    "ends one off a step": [33, 31, 65, 31, 95, 33, 255, 257, 1],
    "short ones behind a long one": [700, 1, 2, 29, 32, 16, 48, 20],
    "short ones before a long one": [20, 48, 16, 32, 29, 2, 1, 700],
    "long, short, long": [400, 30, 34, 2, 62, 510],
}


@pytest.mark.parametrize("Hq,Hkv,D", [(4, 1, 64), (4, 1, 128), (6, 2, 64), (9, 1, 128), (36, 9, 64), (36, 9, 128)])
@pytest.mark.parametrize("name", sorted(PACKED))
def test_packed_documents_match_oracle(long_build, name, Hq, Hkv, D):
    lengths = PACKED[name]
    print(f"{name}: {Hq}/{Hkv} D={D}", flush=True)
    cu = synth.cu_seqlens_from_lengths(lengths)
    T = int(cu[-1])
    bits = synth.attn_inputs(T + Hq, T, Hq, Hkv, D)
    q, k, v, do = (dev_bf16(t[0]) for t in bits)
    got = run(long_build, q, k, v, do, torch.from_numpy(cu).cuda())[2:]
    refs = rn.attn_varlen_bwd(*(rn.widen_bf16(t[0]) for t in bits), cu)[:3]
    check_grads([host_f64(t) for t in got], refs, name)


# Where the rule picks them: the regular library gives the bits of LIB_LONG (it runs these programs) and of the build with
# every wait spelled out (no register read early, no operand late).  One and two row blocks of dQ, one and several chunks.
def bits_of_three(q, k, v, do, cu, what):
    fast = run(sp.lib(), q, k, v, do, cu)
    same_bits(fast, run(sp.open_library(spbuild.LIB_LONG), q, k, v, do, cu), what + " (long build)")
    same_bits(fast, run(sp.open_library(spbuild.LIB_PADDED), q, k, v, do, cu), what + " (padded build)")
    return fast


@pytest.mark.parametrize("B,S,Hq,Hkv,D", [(1, 4096, 4, 1, 128), (1, 8190, 4, 1, 128), (1, 10300, 4, 1, 128), (40, 1100, 9, 9, 128), (1, 20001, 2, 1, 64), (1, 32700, 1, 1, 64), (3, 9001, 6, 2, 64)])
def test_rule_picks_these_programs_dense(B, S, Hq, Hkv, D):
    q, k, v, do = (dev_bf16(t) for t in synth.attn_inputs(S + D, S, Hq, Hkv, D, B))
    bits_of_three(q, k, v, do, None, f"B={B} S={S} {Hq}/{Hkv} D={D}")


@pytest.mark.parametrize("lengths,Hq,Hkv,D", [([9000, 33, 7000, 500], 4, 1, 128), ([30000, 700, 9000], 4, 1, 64)])
def test_rule_picks_these_programs_packed(lengths, Hq, Hkv, D):
    cu = synth.cu_seqlens_from_lengths(lengths)
    q, k, v, do = (dev_bf16(t[0]) for t in synth.attn_inputs(79, int(cu[-1]), Hq, Hkv, D))
    bits_of_three(q, k, v, do, torch.from_numpy(cu).cuda(), f"packed documents D={D}")


def test_one_long_document_equals_dense_bitwise():
    S, Hq, Hkv, D = 9001, 4, 1, 128
    q, k, v, do = (dev_bf16(t) for t in synth.attn_inputs(23, S, Hq, Hkv, D))
    dense = run(sp.lib(), q, k, v, do)
    packed = run(sp.lib(), q[0], k[0], v[0], do[0], torch.tensor([0, S], dtype=torch.int32, device="cuda"))
    same_bits([t[0] for t in dense], packed, "one packed document")

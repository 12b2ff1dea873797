"""The equal-share decode kernel where its cuts can go wrong: fewer pages than waves, pairs that end
exactly at a share's or a workgroup's boundary, one pair cut by many workgroups, many pairs per
share, a few short sequences that are not cut at all, kv-head counts that do not divide the grid, both plan forms (up to 64 sequences and more),
and workgroups of several kv-heads.  Each case goes through pearl_attn_decode_append (pools compared
byte for byte) and against the oracle.  Many sequences here hold only a few keys, so single weights
dominate their rows; the bound is the one gpu_helpers.peaked_bound derives for that from the bf16
roundings of the weights and the output (half an ulp of o, plus 2^-8 of the largest |v|, plus 1e-4
of fp32 rounding), with the mean at 1e-3."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_35158_amd as pa
from paper_2609_35158_amd import workloads
from gpu_helpers import assert_close, bits, gpu_append, oracle_sampled, say

pytestmark = pytest.mark.gpu

# name: (contexts, kv-heads, G, head_dim)
CASES = {
    "one-page": ([0], 1, 1, 64),
    "fewer-pages-than-waves": ([5, 16, 40], 1, 8, 128),
    "one-page-each-3-heads": ([0, 15, 14], 3, 2, 128),
    "65-sequences": ([(7 * i) % 50 for i in range(65)], 2, 4, 64),
    "64-sequences": ([(11 * i) % 70 for i in range(64)], 5, 1, 128),
    "cuts-at-pair-ends": ([16 * 16 - 1] * 48, 8, 4, 128),
    "cuts-at-pair-ends-d64": ([16 * 8 - 1] * 64, 4, 8, 64),
    "whole-pairs": ([300, 0, 17, 410, 1, 255, 256], 8, 4, 128),
    "whole-pairs-d64": ([50 * i for i in range(20)], 3, 8, 64),
    "one-too-long-for-whole-pairs": ([900, 100, 90], 2, 2, 128),
    "one-long": ([30011], 2, 8, 128),
    "long-beside-short": ([20000, 3, 17, 9000, 1], 4, 2, 64),
    "many-pairs-per-share": ([(37 * i) % 90 for i in range(520)], 8, 1, 64),
    "1024-sequences": ([(5 * i) % 33 for i in range(1024)], 3, 2, 64),
}


def _decode_append(case, max_kv):
    ctx = torch.from_numpy(case.ctx_lens.astype(np.int32)).cuda()
    out, lse = pa.decode_append(case.q, case.k_new, case.v_new, case.k_pool, case.v_pool, case.block_table, ctx, max_kv,
                                scale=case.scale, return_lse=True, out=torch.full_like(case.q, 7.0))
    torch.cuda.synchronize()
    return out, lse


@pytest.mark.parametrize("name", list(CASES))
def test_shares_against_oracle(name):
    ctx, H, G, d = CASES[name]
    say("case: decode shares %s" % name)
    case = workloads.build_case(name, 77, H * G, H, d, np.array(ctx), np.ones(len(ctx), np.int64), device="cuda",
                                extra_pages=2)
    kr, vr = oracle.kv_append(bits(case.k_pool), bits(case.v_pool), bits(case.k_new), bits(case.v_new),
                              case.block_table.cpu().numpy(), case.ctx_lens, None)
    out, lse = _decode_append(case, int(case.kv_lens.max()))
    assert np.array_equal(bits(case.k_pool), kr) and np.array_equal(bits(case.v_pool), vr)
    o, l = oracle.attention(bits(case.q), kr, vr, case.block_table.cpu().numpy(), case.ctx_lens, None, case.scale)
    assert_close(bits(out), o, lse.cpu().numpy(), l, what=name,
                 peaked_vmax=float(np.nanmax(np.abs(oracle.bf16_bits_to_f64(vr)))))
    again, lse2 = _decode_append(case, int(case.kv_lens.max()))
    assert torch.equal(out, again) and torch.equal(lse, lse2), "the same call differs"


@pytest.mark.parametrize("H,G,d", [(8, 2, 128), (4, 8, 128), (8, 1, 64)])
def test_several_heads_per_workgroup(H, G, d):
    """Shares of 64 pages or more per wave: H kv-heads in a workgroup, 8 / H shares of each."""
    say("case: decode shares, %d kv-heads per workgroup, d=%d" % (H, d))
    B = 130
    per_wave = 66 * (2 if d == 64 else 1)             # d = 64 runs two workgroups per compute unit
    pages = per_wave * (8 // H) * 256 // B + 1
    rng = np.random.default_rng(9)
    ctx = rng.integers(8 * pages, 24 * pages, size=B)
    case = workloads.build_case("heads", 78, H * G, H, d, ctx, np.ones(B, np.int64), device="cuda", sentinel_unused=False)
    out, lse = _decode_append(case, int(case.kv_lens.max()))
    seqs = [0, 1, 2, 37, 64, 65, 100, 128, 129]
    o, l = oracle_sampled(case, seqs)
    for b in seqs:
        assert_close(bits(out[b:b + 1]), o[b], lse[b:b + 1].cpu().numpy(), l[b], what="sequence %d" % b)


@pytest.mark.parametrize("batch", [2, 31, 33, 64])
def test_plan_of_one_wave(batch):
    """Up to 64 sequences each wave builds the page list alone, a lane per sequence, and then reads the
    other lanes' entries: a sequence's results must be the ones it gets in a batch of more, which is
    planned behind barriers."""
    say("case: decode shares, plan of one wave, %d sequences" % batch)
    rng = np.random.default_rng(70 + batch)
    ctx = rng.integers(0, 400, size=70)
    ctx[:batch] += 16 * rng.integers(0, 60, size=batch)
    case = workloads.build_case("one-wave", 79, 8, 2, 64, ctx, np.ones(70, np.int64), device="cuda", sentinel_unused=False)
    gpu_append(case)
    lens = torch.from_numpy(case.ctx_lens.astype(np.int32)).cuda()
    max_kv = int(case.kv_lens.max())
    args = lambda n: (case.q[:n], case.k_pool, case.v_pool, case.block_table[:n], lens[:n], max_kv)
    few, lse_few = pa.decode(*args(batch), scale=case.scale, return_lse=True)
    more, lse_more = pa.decode(*args(70), scale=case.scale, return_lse=True)
    torch.cuda.synchronize()
    # two cuts of the same sequence: each within the tolerance of the exact result
    assert (few.float() - more[:batch].float()).abs().max().item() <= 2e-2
    assert (lse_few - lse_more[:batch]).abs().max().item() <= 1e-3
    seqs = sorted({0, batch // 2, batch - 1})
    o, l = oracle_sampled(case, seqs)
    for b in seqs:
        assert_close(bits(few[b:b + 1]), o[b], lse_few[b:b + 1].cpu().numpy(), l[b], what="sequence %d" % b,
                     peaked_vmax=float(case.v_new.float().abs().max().clamp(min=5.6)))

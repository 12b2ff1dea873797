"""The equal-share decode kernel where its cuts can go wrong: fewer pages than waves, pairs that end
exactly at a share's or a workgroup's boundary, one pair cut by many workgroups, many pairs per
share, runs of whole sequences (one each and several), kv-head counts that do not divide the grid,
both plan forms (up to 64 sequences and more), and workgroups of several kv-heads.  The cut that a
case took is seen by the partials it leaves in the workspace.  Each case goes through pearl_attn_decode_append (pools compared
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
from gpu_helpers import assert_close, bits, decode_with_partials, gpu_append, oracle_sampled, say

pytestmark = pytest.mark.gpu

# name: (contexts, kv-heads, G, head_dim, whether the runs hold whole sequences)
CASES = {
    "one-page": ([0], 1, 1, 64, True),
    "fewer-pages-than-waves": ([5, 16, 40], 1, 8, 128, True),
    "one-page-each-3-heads": ([0, 15, 14], 3, 2, 128, True),
    "65-sequences": ([(7 * i) % 50 for i in range(65)], 2, 4, 64, True),
    "64-sequences": ([(11 * i) % 70 for i in range(64)], 5, 1, 128, True),
    "cuts-at-pair-ends": ([16 * 16 - 1] * 48 + [16 * 64 - 1], 8, 4, 128, False),
    "cuts-at-pair-ends-d64": ([16 * 8 - 1] * 64 + [16 * 64 - 1], 4, 8, 64, False),
    "whole-pairs": ([300, 0, 17, 410, 1, 255, 256], 8, 4, 128, True),
    "whole-pairs-d64": ([30 * i for i in range(20)], 3, 8, 64, True),
    "one-too-long-for-whole-pairs": ([900, 100, 90], 2, 2, 128, False),
    "one-long": ([30011], 2, 8, 128, False),
    "long-beside-short": ([20000, 3, 17, 9000, 1], 4, 2, 64, False),
    "many-pairs-per-share": ([(37 * i) % 90 for i in range(520)] + [2000], 8, 1, 64, False),
    "1024-sequences": ([(5 * i) % 33 for i in range(1023)] + [3000], 3, 2, 64, False),
    # more sequences than one wave plans, a workgroup each and several to a workgroup; as many or
    # more of them than the workspace (one slot per sequence) allows equal runs for
    "whole-130": ([20 + (13 * i) % 230 for i in range(130)], 1, 2, 128, True),
    "whole-130-one-longer": ([20 + (13 * i) % 230 for i in range(129)] + [1500], 1, 2, 128, False),
    "whole-700": ([(13 * i) % 200 for i in range(700)], 2, 1, 64, True),
    "whole-2-per-run": ([16 + (5 * i) % 48 for i in range(64)], 8, 4, 128, True),
    "whole-3-or-4-per-run": ([16 + (5 * i) % 48 for i in range(111)], 8, 1, 128, True),
    "whole-equal-lengths": ([16 * 20 - 1] * 128, 4, 1, 128, True),
    # more kv-heads than workgroups at a time
    "300-heads": ([40, 0, 100], 300, 1, 128, True),
    "300-heads-cut": ([3000], 300, 1, 128, False),
    "513-heads-d64": ([1500, 20], 513, 1, 64, False),
    "whole-1024-sequences": ([(5 * i) % 33 for i in range(1024)], 3, 2, 64, True),
}


def _decode_append(case, max_kv):
    ctx = torch.from_numpy(case.ctx_lens.astype(np.int32)).cuda()
    out, lse = pa.decode_append(case.q, case.k_new, case.v_new, case.k_pool, case.v_pool, case.block_table, ctx, max_kv,
                                scale=case.scale, return_lse=True, out=torch.full_like(case.q, 7.0))
    torch.cuda.synchronize()
    return out, lse


def _partials(ctx, runs, shares):
    """Partials per kv-head of a page list cut into runs of equal shares: one per run that holds pages of
    a sequence, for every sequence in more than one run."""
    end = np.cumsum(np.asarray(ctx) // 16 + 1)
    share, more = divmod(int(end[-1]), runs * shares)
    begin = np.array([shares * x * share + min(shares * x, more) for x in range(runs)])
    first = np.searchsorted(begin, np.concatenate([[0], end[:-1]]), side="right")
    last = np.searchsorted(begin, end - 1, side="right")
    return int((last - first + 1)[last > first].sum())


def _grid(d):
    """Workgroups of the decode grid: one per compute unit, two at head_dim 64."""
    return torch.cuda.get_device_properties(0).multi_processor_count * (2 if d == 64 else 1)


def _slot_runs(ctx, H, bound=0):
    """Runs that the workspace's partial slots allow: two slots each, or one more than one per sequence."""
    B, longest = len(ctx), max(int(np.max(ctx)) // 16 + 1, bound // 16)
    pps = min(512, -(-max(16, -(-B * H * longest // 4096)) // 16) * 16)
    slots = B * -(-longest // pps)
    return max(1, slots // 2, slots - B)


def _equal_runs(ctx, H, d):
    """Equal runs of one kv-head: a workgroup each, of at least 16 pages, as many as there are slots for."""
    total = int((np.asarray(ctx) // 16 + 1).sum())
    per_head = max(1, (_grid(d) if H <= _grid(d) else 4 * _grid(d)) // H)
    return max(1, min(per_head, _slot_runs(ctx, H), total // (16 + total // (64 * len(ctx)))))


@pytest.mark.parametrize("name", list(CASES))
def test_shares_against_oracle(name):
    ctx, H, G, d, whole = CASES[name]
    say("case: decode shares %s" % name)
    case = workloads.build_case(name, 77, H * G, H, d, np.array(ctx), np.ones(len(ctx), np.int64), device="cuda",
                                extra_pages=2)
    kr, vr = oracle.kv_append(bits(case.k_pool), bits(case.v_pool), bits(case.k_new), bits(case.v_new),
                              case.block_table.cpu().numpy(), case.ctx_lens, None)
    n, out, lse = decode_with_partials(case, int(case.kv_lens.max()))
    if whole:
        assert n == 0
    else:
        # (the quotient that gives the runs is an approximate one)
        runs = _equal_runs(ctx, H, d)
        assert n in {_partials(ctx, r, 8) for r in (runs - 1, runs, runs + 1) if r > 0}
    assert np.array_equal(bits(case.k_pool), kr) and np.array_equal(bits(case.v_pool), vr)
    o, l = oracle.attention(bits(case.q), kr, vr, case.block_table.cpu().numpy(), case.ctx_lens, None, case.scale)
    assert_close(bits(out), o, lse.cpu().numpy(), l, what=name,
                 peaked_vmax=float(np.nanmax(np.abs(oracle.bf16_bits_to_f64(vr)))))
    again, lse2 = _decode_append(case, int(case.kv_lens.max()))
    assert torch.equal(out, again) and torch.equal(lse, lse2), "the same call differs"


# (kv-heads, G, head_dim, sequences, shortest and longest context, host bound; kv-heads per workgroup)
HEAD_CASES = [
    # shares long for their sequences: 8 / heads shares of several kv-heads, one block of them and more
    (8, 2, 128, 130, 4000, 6000, 0, 8),
    (4, 8, 128, 130, 2000, 6000, 0, 4),
    (2, 4, 128, 256, 1000, 8000, 0, 2),
    (6, 1, 128, 300, 400, 1200, 0, 2),
    (10, 1, 128, 300, 400, 1200, 0, 2),
    (12, 2, 128, 150, 400, 1200, 0, 4),
    (24, 1, 128, 60, 400, 1200, 0, 8),
    (40, 1, 64, 100, 200, 900, 32768, 8),
    (64, 1, 128, 32, 400, 1600, 0, 8),
    # a last block of 8 kv-heads that overlaps the one before by 1, 7 and 5 of them
    (71, 1, 128, 28, 400, 1200, 0, 8),
    (129, 1, 64, 30, 500, 900, 32768, 8),
    (83, 2, 128, 20, 500, 900, 32768, 8),
    # more kv-heads than workgroups at a time
    (300, 1, 128, 6, 400, 1600, 0, 4),
    (257, 1, 128, 7, 400, 1600, 0, 8),
    # head_dim 64 runs two workgroups per compute unit: 512 runs need that many partial slots
    (4, 2, 64, 600, 1000, 1500, 0, 4),
    (8, 1, 64, 130, 2000, 6200, 65536, 8),
    (8, 1, 64, 130, 2000, 6200, 0, 1),
    # the longest sequence in too many pieces
    (8, 2, 128, 16, 2000, 30000, 0, 1),
    (16, 1, 128, 8, 4000, 16000, 0, 1),
    (8, 4, 128, 48, 2000, 6000, 0, 1),
]


@pytest.mark.parametrize("H,G,d,B,lo,hi,bound,heads", HEAD_CASES)
def test_several_heads_per_workgroup(H, G, d, B, lo, hi, bound, heads):
    """Workgroups of several kv-heads where their shares are long for the sequences, of one elsewhere
    (seen by the partials they leave); sampled sequences against the oracle, the pools byte for byte.  Slots of a last page past the new token hold NaN, which no result may show."""
    say("case: decode shares, H=%d G=%d d=%d, %d sequences" % (H, G, d, B))
    rng = np.random.default_rng(9)
    ctx = rng.integers(lo, hi, size=B, endpoint=True)
    ctx[0], ctx[-1] = hi, lo
    case = workloads.build_case("heads", 78, H * G, H, d, ctx, np.ones(B, np.int64), device="cuda")
    if bound:
        case.block_table = torch.nn.functional.pad(case.block_table, (0, bound // 16 - case.block_table.shape[1]))
    k, v = case.k_pool.clone(), case.v_pool.clone()
    last = torch.from_numpy(ctx).cuda()
    page = case.block_table.long().gather(1, (last // 16)[:, None])[:, 0]
    k[page, :, last % 16], v[page, :, last % 16] = case.k_new, case.v_new
    n, out, lse = decode_with_partials(case, bound or int(case.kv_lens.max()))
    runs = min(max(1, _grid(d) // -(-H // heads)), _slot_runs(ctx, H, bound))
    say("   partials per kv-head %d" % n)
    if heads > 1:
        assert n == _partials(ctx, runs, 8 // heads)
    else:
        assert n <= 2 * runs
    same = lambda x, y: torch.equal(x.view(torch.int16), y.view(torch.int16))
    assert same(case.k_pool, k) and same(case.v_pool, v)
    assert torch.isfinite(out.float()).all() and torch.isfinite(lse).all()
    seqs = sorted({0, 1, B // 4, B // 2, B - 2, B - 1} | {int(x) for x in rng.integers(0, B, size=3)})
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

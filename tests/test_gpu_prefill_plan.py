"""The planner's prefill entries where they can go wrong: key splits of tiles of very different
lengths in one sequence (short tiles have fewer splits), sequences with and without splits in one
launch, as many entries as one thread keeps and more, several chunks of sequences (with key splits
and without), and launches that never split; the header says whether tiles were split.  Every row's LSE (preset to NaN) must be written; rows are compared with the
oracle within the bf16 tolerance (1e-2 max, 1e-3 mean), rows of few keys within
gpu_helpers.peaked_bound."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_35158_amd as pa
from paper_2609_35158_amd import workloads
from gpu_helpers import assert_close, bits, bounds, dev_lengths, gpu_append, oracle_sampled, say, tile_edge_tokens

pytestmark = pytest.mark.gpu

# name: (contexts, new tokens, kv-heads, G, head_dim, sequences checked, whether prefill and mixed launches split tiles)
CASES = {
    "one-prompt-split": ([0], [1700], 2, 2, 64, [0], (True, True)),
    "prompt-beside-long-context": ([0, 9000, 40], [900, 70, 3], 2, 4, 128, [0, 1, 2], (True, True)),
    "equal-tiles-split": ([6000, 6010], [256, 250], 4, 8, 128, [0, 1], (True, True)),
    "no-split-below-1024-keys": ([700, 0, 300], [300, 1000, 1], 1, 1, 64, [0, 1, 2], (False, False)),
    "more-entries-than-kept": ([(13 * i) % 50 for i in range(200)], [180] * 200, 1, 8, 64, [0, 7, 99, 199], (False, False)),
    "two-chunks": ([(29 * i) % 400 for i in range(260)], [1 + (7 * i) % 90 for i in range(260)], 2, 4, 64, [0, 255, 256, 259],
                   (False, False)),
    # key splits where the planner goes over its sequences twice, more than 256 of them, with split tiles
    # in the first chunk and in the second; and as many splits as there are slots for
    "two-chunks-split": ([8000 if i in (3, 250, 258) else (29 * i) % 50 for i in range(262)], [1 + (7 * i) % 90 for i in range(262)],
                         1, 2, 128, [0, 3, 250, 255, 256, 258, 261], (True, False)),
    "chunks-beside-300-decodes": ([6500 if i == 100 else 9000 if i == 280 else (31 * i) % 400 for i in range(302)],
                                  [100 if i in (100, 280) else 1 for i in range(302)], 4, 8, 128, [0, 99, 100, 255, 256, 280, 301],
                                  (False, True)),
    "many-splits": ([5, 9000, 9100], [130, 500, 480], 1, 8, 64, [0, 1, 2], (True, True)),
}


@pytest.mark.parametrize("mode", ["prefill", "mixed"])
@pytest.mark.parametrize("name", list(CASES))
def test_prefill_entries(name, mode):
    from paper_2609_35158_amd import binding as bd
    ctx, ql, H, G, d, seqs, splits = CASES[name]
    say("case: prefill plan %s (%s)" % (name, mode))
    case = workloads.build_case(name, 91, H * G, H, d, np.array(ctx), np.array(ql), device="cuda", extra_pages=1)
    gpu_append(case)
    dctx, cu = dev_lengths(case)
    max_q, max_kv = bounds(case)
    lse = torch.full((case.total_q, case.num_q_heads), float("nan"), dtype=torch.float32, device="cuda")
    fn = {"prefill": pa.prefill_append, "mixed": pa.mixed}[mode]
    desc = bd.make_desc(case.block_table, dctx, cu, case.total_q, max_q, max_kv)
    ws = torch.empty(bd.workspace_bytes(case.num_q_heads, case.k_pool, desc), dtype=torch.uint8, device="cuda")
    out, lse = fn(case.q, case.k_pool, case.v_pool, case.block_table, dctx, cu, max_q, max_kv, scale=case.scale,
                  return_lse=True, lse=lse, workspace=ws)
    torch.cuda.synchronize()
    hdr = ws[:64 * 4].view(torch.int32).cpu().numpy()
    say("   entries %d, keys per split %d, split tiles %d" % (hdr[1], hdr[5], hdr[6]))
    assert hdr[3] == 0
    assert (hdr[5] > 0 and hdr[6] > 0) if splits[mode == "mixed"] else (hdr[5] == 0 and hdr[6] == 0)
    assert torch.isfinite(lse).all(), "rows left unwritten"
    rng = np.random.default_rng(3)
    toks = {b: tile_edge_tokens(ql[b], 256 // G, 8, rng) for b in seqs}
    o, l = oracle_sampled(case, seqs, toks)
    vmax = float(case.v_new.float().abs().max().clamp(min=5.6))
    for b in seqs:
        rows = case.cu_q_lens[b] + np.array(toks[b])
        assert_close(bits(out)[rows], o[b][toks[b]], lse.cpu().numpy()[rows], l[b][toks[b]],
                     what="sequence %d" % b, peaked_vmax=vmax)


@pytest.mark.parametrize("mode", ["prefill", "mixed"])
def test_refused_launch_leaves_no_stale_header(mode):
    """A length beyond the host bounds: nothing is computed, and every header word that the attention
    kernel reads is written, whatever the workspace held before."""
    from paper_2609_35158_amd import binding as bd
    say("case: refused %s launch" % mode)
    case = workloads.build_case("refused", 92, 8, 2, 64, np.array([100, 40, 7]), np.array([30, 1, 1]), device="cuda")
    gpu_append(case)
    dctx, cu = dev_lengths(case)
    max_q, _ = bounds(case)
    desc = bd.make_desc(case.block_table, dctx, cu, case.total_q, max_q, 64)   # the first sequence holds 130 keys
    ws = torch.full((bd.workspace_bytes(case.num_q_heads, case.k_pool, desc),), 0x7f, dtype=torch.uint8, device="cuda")
    out = torch.full_like(case.q, 7.0)
    fn = {"prefill": pa.prefill_append, "mixed": pa.mixed}[mode]
    fn(case.q, case.k_pool, case.v_pool, case.block_table, dctx, cu, max_q, 64, scale=case.scale, out=out, workspace=ws)
    torch.cuda.synchronize()
    hdr = ws[:64 * 4].view(torch.int32).cpu().numpy()
    assert hdr[3] == 1 and not hdr[[0, 1, 2, 4, 5, 6, 8]].any() and not hdr[16:24].any() and 0 < hdr[9] < 1 << 20
    assert torch.all(out == 7.0)

"""The parity tests ask for so few workers that their plans have no split for short contexts.  Here some of them run again with as many as the chip
has, as a caller asks for: the same inputs, oracle and bounds, on the kernels that take a call in one launch."""
import pytest

import paper_2503_23294_amd as ck

import test_gpu_parity as parity

pytestmark = pytest.mark.gpu

RUNS = [
    # appended tokens, as many as all sequences have: one part per row and several (their bounds by a reciprocal), a full buffer
    *[(parity.test_appended_decode_tokens, a) for a in [(2, 1, 1, 128), (1, 70, 70, 128), (1, 600, 67, 128), (4, 130, 67, 64), (3, 300, 66, 128), (8, 600, 66, 128), (16, 70, 66, 128)]],
    # a count per sequence, on the device
    *[(parity.test_sequences_that_stop_generating_at_different_steps, a) for a in [(1, 128, [40, 0, 700]), (4, 128, [3, 130, 66]), (4, 64, [700, 1, 64]), (8, 128, [5, 70, 0])]],
    # runs with room to grow, folds
    *[(parity.test_folding_appended_tokens_into_the_packed_cache, a) for a in [(1, 128, True), (4, 128, True), (4, 64, False), (8, 128, True), (1, 64, False)]],
    *[(parity.test_a_query_that_is_not_finite_stays_in_its_head, (*a, x)) for a in [(5, 128, 4), (16, 128, 9), (8, 64, 7)] for x in (float("nan"), float("inf"), float("-inf"))],
    *[(parity.test_logits_far_beyond_the_binary32_integers, (*a, bits, *x)) for a in [(1, 128), (4, 128), (4, 64), (8, 128), (8, 64)] for bits in (2, 4, 8, 16)
      for x in [(200.0, 100.0), (1.5e4, 1.5e4)]],
    *[(parity.test_value_ranges_from_tiny_to_near_the_fp16_limit, (rep, *x)) for rep in (1, 4, 8) for x in [(1.0, 2.0e4, 1.0), (3.0, 5.0e-5, 1.0), (1.0, 1.0, 1.0e-3)]],
    *[(parity.test_decode_calls_replayed_from_a_captured_graph, (rep,)) for rep in (1, 4, 8, 16)],
    *[(parity.test_grouped_queries_on_the_vector_alu_only, (*a, 2048)) for a in [(2, 128), (8, 128), (16, 64)]],
    *[(parity.test_eight_heads_per_wave_at_the_edges_of_its_tiles, a) for a in [(5, 128, 32), (8, 64, 32)]],
    (parity.test_runs_on_a_side_stream, ()),
    (parity.test_ragged_batch_with_empty_and_tail_only_sequences, ()),
    (parity.test_marked_call_equals_the_plain_call_and_records_its_event, ()),
]
# so few that a wave has more than one iteration, of several units each
FEW = [(parity.test_decode_calls_replayed_from_a_captured_graph, (4,))]


@pytest.mark.parametrize("test,args,workers", [(*r, 2048) for r in RUNS] + [(*r, 32) for r in FEW], ids=lambda x: x.__name__[5:] if callable(x) else str(x))
def test_on_the_kernels_for_short_contexts(test, args, workers, monkeypatch):
    plan, plans = ck.cocktail_plan, []

    def with_workers(shape, seq_lens, chunk_bits, num_workers, **options):
        plans.append(plan(shape, seq_lens, chunk_bits, workers, **options))
        return plans[-1]

    monkeypatch.setattr(ck, "cocktail_plan", with_workers)
    test(*args)
    assert plans and all(ck.cocktail_plan_field(p, "short_groups") > 0 for p in plans)
    assert all(ck.cocktail_plan_field(p, "short_units") == (workers == 2048) for p in plans)

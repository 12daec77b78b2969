"""The tests that are there for the maps, their construction, their failures' corrections and the slot compare,
once more with every call kept on slots: by expected time most of their instances are counted from bit rows,
which no map and no correction can reach."""
import pytest

import datagen

torch = pytest.importorskip("torch")
bm = pytest.importorskip("paper_1102_1003_amd")

from test_gpu_block import (test_block_family_is_the_default, test_chain_family_packed_fields,  # noqa: E402,F401
                            test_chain_family_still_exact, test_clustered_tids,
                            test_overflowing_block_falls_back_to_the_chain_family)
from test_gpu_cross import (test_cross_equals_definition, test_cross_of_a_family_with_itself,  # noqa: E402,F401
                            test_cross_with_caller_permutations)
from test_gpu_parity import (ctx, test_autotuned_batch, test_batch_graph_replays,  # noqa: E402,F401
                             test_batched_equals_each_instance, test_corrections_list_regrows, test_edge_shapes,
                             test_failures_past_the_first_failure_list, test_forced_failures_are_corrected,
                             test_more_than_2_32_slots, test_packed_field_lds_build, test_power_of_two_set_sizes,
                             test_pruned_build_frequent_pairs, test_random_instances, test_subset_queries,
                             test_tiny_config_all_pairs_and_filter,
                             test_transactions_path_with_repeats_and_shuffled_rows,
                             test_transactions_ragged_counts_and_repeats)
from test_gpu_serving import (data, test_concurrent_queries_equal_single_calls,  # noqa: E402,F401
                              test_server_right_after_a_build_with_a_second_corrections_pass,
                              test_tight_memory_admission)
from test_gpu_slots import test_wide_slot_cross_and_noalloc, test_wide_slots_all_pairs  # noqa: E402,F401
from test_gpu_triples import (test_transactions_path_order3, test_triples_among_the_largest_items,  # noqa: E402,F401
                              test_triples_equal_definition)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def slots(monkeypatch):
    monkeypatch.setenv("BM_BITMAP_ROUTE", "0")
    if not torch.cuda.is_available():
        yield
        return
    # every answer of all pairs names the compare's work: the route cannot drift unseen
    real = bm.Index.all_pair_supports

    def all_pair_supports(self, out=None):
        self.ctx.set_profiling(True)
        got = real(self, out)
        t = self.ctx.timings()
        self.ctx.set_profiling(False)
        assert self.n < 2 or t["compare_slot_pairs"] > 0
        return got
    monkeypatch.setattr(bm.Index, "all_pair_supports", all_pair_supports)
    # a context's own stream does not wait for the stream that the data is drawn on, and in a second run of the
    # same test no allocation does either
    drawn = datagen.bernoulli_sets_device

    def bernoulli_sets_device(*args, **kw):
        got = drawn(*args, **kw)
        torch.cuda.synchronize()
        return got
    monkeypatch.setattr(datagen, "bernoulli_sets_device", bernoulli_sets_device)
    yield

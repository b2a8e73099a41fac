"""The checkpoint walk's sums, queue and deferral on the geometries of the parity
tests: those use few orbits, whose launches otherwise cut the exposures over
several wavefronts; with the work counters on, every stack runs the checkpoint
walk, which the counters prove (the shared epoch leaves it no speed bound)."""
import pytest

from test_gpu_parity import (small, test_checkpoint_walk_edge_cases, test_exposure_order_does_not_matter,  # noqa: F401
                             test_fp16_images_match_oracle_on_the_same_values,
                             test_generate_and_stack_matches_stack_and_oracle, test_invalid_orbits_and_empty_sets,
                             test_pruned_stack_equals_exact_walk, test_sky_cone_edge_geometries,
                             test_stack_distant_objects_fp16, test_stack_survey_small, test_stack_tiny,
                             test_tiny_images_and_behind_the_plane, tiny)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def counted(monkeypatch, request):
    import paper_2503_08854_amd as dt
    made = []

    class Counting(dt.Context):
        predicted = 0

        def __init__(self, *args, **kwargs):
            super().__init__(*args, **kwargs)
            self.count_work(True)
            made.append(self)

        def close(self):
            if self.handle:
                self.predicted += self.work()["predicted"]
            super().close()

    monkeypatch.setattr(dt, "Context", Counting)
    yield
    walked = sum(c.predicted + (c.work()["predicted"] if c.handle else 0) for c in made)
    assert walked > 0 or "shared_epoch" in request.node.name

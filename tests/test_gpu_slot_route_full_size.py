"""The full-size steps and the full-size comparison with the bitmap product, with every call kept on slots (the
bitmap product's own call stays what it is)."""
import pytest

torch = pytest.importorskip("torch")
bm = pytest.importorskip("paper_1102_1003_amd")

from test_gpu_full_size import (stream_ctx, test_dense_comparator_full_size,  # noqa: E402,F401
                                test_transactions_step_full_size)
from test_gpu_slot_route import slots  # noqa: E402,F401

pytestmark = pytest.mark.gpu

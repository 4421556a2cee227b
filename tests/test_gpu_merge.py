"""The merge of per-chunk partials, at the chunk counts where it changes: groups of 16 and 32 partial rows, rounds of
64 chunks, and requests of fewer chunks beside longer ones."""
import pytest

from paper_2506_19830_amd import workloads as W
from test_gpu_attention import check_full

pytestmark = pytest.mark.gpu


# a request of 64 n tokens in splits of 64 has n chunks; 9 is the fewest that takes the wavefront-per-row merge
@pytest.mark.parametrize("chunks", [9, 16, 17, 32, 33, 64, 65, 97, 130])
@pytest.mark.parametrize("d", [64, 128, 256])
def test_chunk_counts(oracle, d, chunks):
    case = W.AttnCase(f"merge_{chunks}", (64 * chunks, 64, 64 * (chunks // 2) + 1, 0), 2, 3, 4, 2, d, "bf16", "bf16", "bf16",
                      "f32", seed=chunks + d)
    check_full(oracle, case, 1e-5 if d != 128 else 2e-2, 64, lse_tol=1e-5 if d != 128 else None)

"""top-p without top-k: the threshold search over the candidate segments, and the calls that fall back from it."""
import pytest

from paper_2506_19830_amd import workloads as W
from test_gpu_accept import check

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("accept_tables")]

CASES = [
    # vocabularies around a fine slice (2048) and a segment's group of four, aligned and odd rows
    *[W.AcceptCase(f"seg_v{v}_{dt}", 24, 3, v, dt, temperature=0.6, top_p=0.95, seed=500 + i)
      for i, (v, dt) in enumerate((v, dt) for v in (512, 2048, 2049, 8192, 8200, 16391) for dt in ("bf16", "f32"))],
    # nearly nothing and nearly everything kept; a flat row (its segments overflow), many ties of a low temperature
    W.AcceptCase("seg_p005", 8, 4, 32003, "bf16", temperature=1.0, top_p=0.05, seed=520),
    W.AcceptCase("seg_p999", 8, 4, 32003, "f32", temperature=1.0, top_p=0.999, seed=521),
    W.AcceptCase("seg_flat", 8, 4, 32000, "bf16", target_std=0.5, temperature=1.0, top_p=0.9, seed=522),
    W.AcceptCase("seg_cold", 8, 4, 32000, "bf16", temperature=0.05, top_p=0.95, seed=523),
    # long drafts: segments of 80 bytes (32 keys), which overflow; of 48 bytes, too small to be used at all
    W.AcceptCase("seg_long_draft", 2, 90, 4096, "bf16", temperature=0.6, top_p=0.95, seed=524),
    W.AcceptCase("seg_no_segment", 2, 150, 4096, "bf16", temperature=0.6, top_p=0.95, seed=526),
    W.AcceptCase("seg_no_segment_f32", 2, 200, 4100, "f32", temperature=0.6, top_p=0.95, seed=527),
    W.AcceptCase("seg_lookup", 6, 8, 152064, "bf16", temperature=0.6, top_p=0.95, point_mass=True, peak=14.0, seed=525),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: c.name)
def test_top_p(oracle, case):
    check(oracle, case)

"""The launch shape a batch plan starts with is the one the binding's calls
take without arguments, and the one the header states."""
import inspect
import re

from paper_1607_04245_amd import _native as N
from paper_1607_04245_amd import api


def test_one_default_shape():
    text = N.HEADER.read_text()
    doc = text[:text.index("fem_status fem_batch_plan_set_launch")]
    header = re.findall(r"Defaults (\d+) and (\d+)", doc)[-1]
    source = (N.HEADER.parents[1] / "paper_1607_04245_amd" / "csrc" / "batch.hip").read_text()
    plan = [re.search(rf"int {k} = (\d+);", source).group(1) for k in ("waves_per_block", "blocks_per_cu")]
    assert list(header) == plan
    for fn in (api.batch_run_noalloc, api.BatchPlan.set_launch):
        p = inspect.signature(fn).parameters
        assert [str(p[k].default) for k in ("waves_per_block", "blocks_per_cu")] == plan

"""Where the library's device memory comes from: the context's pool, which gives kept memory back before an allocation fails."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_09424_amd", "csrc")


def test_every_allocation_goes_through_the_pool():
    """hipMalloc is called in DevPool::alloc and nowhere else."""
    calls = []
    for path in sorted(glob.glob(os.path.join(CSRC, "**", "*.h*"), recursive=True)):
        where = None
        for line in open(path):
            m = re.match(r"\s*(?:inline )?hipError_t (?:DevPool::)?(\w+)\(", line)
            if m:
                where = m.group(1)
            if re.search(r"\bhipMalloc\(", line.split("//")[0]):
                calls.append((os.path.basename(path), where))
    assert calls and all(where == "alloc" for _, where in calls), calls

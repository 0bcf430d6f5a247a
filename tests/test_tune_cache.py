"""The shipped autotune entries were timed on the batched kernel as it is: their
keys carry the version that the tuner looks up (CPU only)."""
import json
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2504_10937_amd")


def test_entries_are_current():
    version = re.search(r'"(v\d+/)count="', open(os.path.join(LIB, "csrc", "tune.cpp")).read()).group(1)
    entries = json.load(open(os.path.join(LIB, "tune_cache.json")))["entries"]
    assert entries and all(e["key"].startswith(version) for e in entries)

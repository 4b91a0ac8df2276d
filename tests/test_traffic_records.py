"""What bench.py makes of the traffic records: those of an aggregation are scaled to the run's own algorithmic bytes."""
import json
import os

import pytest

import bench

RECORDS = os.path.join(bench.ROOT, "profiles", "hbm_traffic.json")


@pytest.mark.parametrize("workload", ["cfg4", "nn12"])
def test_aggregations_are_scaled(workload):
    with open(RECORDS) as f:
        entry = json.load(f)[workload]
    recorded, algorithmic = entry["bytes_per_launch"], entry["algorithmic_bytes_per_launch"]
    assert bench.load_traffic(workload, "encode", algorithmic) == (recorded, entry["source"])
    assert bench.load_traffic(workload, "encode", 2 * algorithmic)[0] == 2 * recorded
    assert 0.9 <= recorded / algorithmic <= 1.2


def test_other_records_stand_as_they_are():
    with open(RECORDS) as f:
        entry = json.load(f)["cfg5"]
    assert bench.load_traffic("cfg5", entry["split_signature"]) == (entry["bytes_per_launch"], entry["source"])
    assert bench.load_traffic("cfg5", "another")[0] is None

"""CPU check of bench.py's printed line: it stays short enough that the last
10000 characters of a log hold it whole, keeps every field of the contract as
it was, and names what it leaves to stderr."""
import json

import bench

CONTRACT = {
    "metric": bench.METRIC, "value": 10123456789.123456, "unit": "elements/s", "n_gpus": 1, "steps": 20, "warmup": 5,
    "ms_per_step": 13.123456789, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "int32",
    "data": "synthetic", "config": {"workload": "x" * 300, "tree_nodes": 1 << 24},
}


def _result(rows):
    detail = [{"ms": 0.123456789012345 * i, "rate": 1e9 / (i + 3)} for i in range(rows)]
    names = [n.split(".")[1] for n in bench.DETAILS if n.startswith("components.")]
    return dict(CONTRACT, components=dict({n: detail for n in names}, ms={"bridges": 2.7182818284}),
                kernels_ms_per_step={f"k_{i}": i / 7 for i in range(40)}, roofline={"frac": 0.123456789},
                kernel_rooflines={f"k_{i}": {"frac": i / 7} for i in range(rows)}, parity={"lca": True})


def test_long_result_fits():
    full = _result(80)
    assert len(json.dumps(full)) > 25000
    line = bench.result_line(full)
    assert len(line) <= bench.LINE_LIMIT < 10000 and "\n" not in line
    got = json.loads(line)
    for k, v in CONTRACT.items():
        assert got[k] == v, k
    assert got["components"]["ms"] == {"bridges": 2.71828} and got["roofline"] == {"frac": 0.123457}
    left = got["on_stderr"]
    assert left == list(bench.DETAILS[: len(left)])
    for name in bench.DETAILS[len(left):]:
        assert name.split(".")[-1] in (got["components"] if "." in name else got), name


def test_short_result_is_whole():
    got = json.loads(bench.result_line(_result(2)))
    assert "on_stderr" not in got and set(got) == set(_result(2))

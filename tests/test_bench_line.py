"""The line that bench.py prints: whole, valid JSON that a log's tail of a few thousand characters keeps."""
import json

import bench


def test_the_line_keeps_the_contract_and_stays_short():
    call = dict(kernel="k" * 300, bound="mfma", launches_per_step=32, ms=0.123456789, achieved=964.2380914244458, traffic=None)
    workload = dict(workload="w" * 30, ms_per_step=1 / 3, tokens_per_s=2e6 / 3, host_planned_ms_per_step=0.1, kernels={"cs_x" * 5: call},
                    roofline=call, serial_ms_per_step=2.0)
    head = dict(metric="m" * 150, value=2131252.6286388813, unit="tokens/s", n_gpus=1, steps=20, warmup=5, ms_per_step=10.69981084999938,
                higher_is_better=True, scaling="weak", vs_baseline=None, dtype="bf16", data="synthetic", config={"workload": "w", "streams": 64})
    record = dict(head, window_tokens_per_s=1 / 3, kernels={f"cs_{i}" * 5: call for i in range(5)}, roofline=dict(call, traffic_source="t" * 80),
                  workloads=[workload] * 5, mfma_probe={"curve": [1.0] * 500},
                  cpu_baseline=dict(value=111.487, unit="tokens/s", cores=16, kind="oracle", sample="s" * 300, parts_s={"x" * 2000: 1.0}))
    text = json.dumps(bench.short_line(record))
    line = json.loads(text)
    assert len(text) < 3700
    assert all(line[k] == v for k, v in head.items())
    assert line["cpu_baseline"]["value"] == 111.487 and "parts_s" not in line["cpu_baseline"]
    assert line["kernel_ms"]["cs_0" * 5] == [0.123457, 32] and line["roofline"]["achieved"] == 964.238
    assert [w["ms_per_step"] for w in line["workloads"]] == [0.333333] * 5

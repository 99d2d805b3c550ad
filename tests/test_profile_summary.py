"""The traffic summary of the overlap round from synthetic profiler output (no
GPU): every dispatch of a call is counted once, joined launches among them."""
import csv
import json

import pytest

from paper_2609_34388_amd import profile_summary as P

MAIN = "void rg::(anonymous namespace)::attn_fwd_kernel<128, 8, rg::AttnPlanT<rg::AttnReqBr, 64> >(rg::AttnArgs)"
JOINED = MAIN.replace("AttnReqBr, 64", "AttnReqBrPacked, 128")
MERGE = MAIN.replace("attn_fwd_kernel<128, 8", "attn_combine_kernel<128, 1")
PLAIN = MAIN.replace("AttnReqBr, 64", "AttnReq, 128")


def _csv(path, rows):
    path.parent.mkdir(parents=True)
    with open(path, "w", newline="") as f:
        w = csv.DictWriter(f, rows[0].keys())
        w.writeheader()
        w.writerows(rows)


@pytest.mark.parametrize("requests,launches,dispatches,kib", [
    (128, dict(launches=1, joined_launches=1, merge_launches=0), {JOINED: [1000.0, 1200.0]}, 1100.0),
    (129, dict(launches=2, joined_launches=1, merge_launches=0), {JOINED: [1000.0, 1000.0], MAIN: [10.0, 30.0]}, 1020.0),
    (128, dict(launches=2, joined_launches=0, merge_launches=2), {MAIN: [400.0, 600.0], MERGE: [40.0, 60.0]}, 1100.0),
    (16, dict(launches=1, joined_launches=0, merge_launches=0), {MAIN: [300.0]}, 300.0),
])
def test_overlap_traffic_counts_each_dispatch_once(tmp_path, requests, launches, dispatches, kib):
    mb = dict(bytes=int(3 * kib * 1024))
    ov = dict(requests=requests, branches=3, rows=9, kv_tokens=99, launches=launches, multibranch=mb)
    (tmp_path / "trace_overlap_w.log").write_text("noise\n" + json.dumps(dict(overlap=ov)) + "\n")
    names = {**dispatches, PLAIN: [7777.0]}  # the comparison's kernel is not the call's
    _csv(tmp_path / "trace_overlap_w" / "t_kernel_stats.csv",
         [dict(Name=k, Calls=len(v), AverageNs=1000.0) for k, v in names.items()])
    for c, factor in (("FETCH_SIZE", 2.0), ("WRITE_SIZE", 1.0)):
        _csv(tmp_path / f"copy_{c}" / "c_counter_collection.csv",
             [dict(Kernel_Name="__amd_rocclr_copyBuffer", Counter_Name=c, Counter_Value=262144.0 / factor)])
        _csv(tmp_path / f"pmc_{c}_overlap_w" / "p_counter_collection.csv",
             [dict(Kernel_Name=k, Counter_Name=c, Counter_Value=v) for k, vs in names.items() for v in vs])
    row = next(l for l in P.overlap_md(str(tmp_path), "w").splitlines() if l.startswith("| rg_multibranch_attention"))
    cells = [x.strip() for x in row.split("|")]
    assert cells[2:4] == [f"{kib:.0f}", f"{kib:.0f}"]
    assert cells[-2] == "1.000"  # (2 + 1) x kib over the algorithmic bytes

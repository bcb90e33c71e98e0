"""The benchmark's roofline describes the kernel that the timed rollouts run:
the one of the single launch where all bins go out together (chosen or asked
for), else the bin that takes longest."""
import csv
import json
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402
from paper_2502_11129_amd import sim as S  # noqa: E402
from paper_2502_11129_amd import traffic_record as TR  # noqa: E402
from paper_2502_11129_amd import workloads as W  # noqa: E402

TUNED = dict(min_body_slots=32, slots32_min_nvc=24, min_nv_capacity=16, ncr_by_nvc={16: 8, 20: 4})


@pytest.mark.parametrize("options,one", [
    ({}, True), (TUNED, True), (dict(streams=0, use_graph=True), True), (dict(min_body_slots=32, single_launch=True), True),
    (dict(streams=4), False), (dict(time_launches=True), False), (dict(ncr_by_nvc={28: 2}), False),
    (dict(min_body_slots=32, gpu_factorization="tree"), False)])
def test_handle_tells_whether_the_bins_go_out_together(options, one):
    h = S.Handle(W.random_trees(300), **options)
    assert h.one_launch() is one
    h.close()
    ball = S.Handle(W.box_and_ball(8))
    assert not ball.one_launch()
    ball.close()


def test_the_bins_alone_keep_their_contacts_in_registers():
    flat = W.chain(10, ["+x"] * 10, [W.AXIS_Z] * 10, root_type=W.ROOT_FREE)
    flat.half_ext[:] = W.BRICK_HALF                       # lies on every brick: its launch keeps 16 contacts, the snakes' too
    pop = W.concat([W.snake(20), flat, W.quadrupeds(2)])
    h = S.Handle(pop)
    o = bench.per_bin_options({}, h.one_launch(), h.bins())
    assert h.one_launch() and S.Handle(pop, **o).bins() == h.bins()
    assert S.Handle(pop, streams=1).bins() != h.bins()
    h.close()


@pytest.mark.parametrize("options,kernel", [
    ({}, "rollout_multi_kernel"), (dict(TUNED, steps_per_launch=250), "rollout_multi_kernel"),
    (dict(min_body_slots=32, single_launch=True), "rollout_multi_kernel"),
    (dict(streams=4), "rollout_kernel<28, 2, 8, false, false, false>"),
    (dict(min_body_slots=32, gpu_factorization="tree"), "rollout_kernel<24, 2, 8, false, false, true>")])
def test_kernel_and_time_of_the_timed_rollouts(options, kernel):
    pop, T, ms = W.random_trees(300), 1000, 50.0
    h = S.Handle(pop, **options)
    one, timed = h.one_launch(), h.bins()
    h.close()
    o = bench.per_bin_options(options, one, timed)
    t = S.Handle(pop, **o)
    assert t.one_launch() is bool(o.get("single_launch")) and o["time_launches"]
    if not one:
        assert {k: v for k, v in o.items() if k in options} == options   # the timed layout itself
    bins, facs, vb = t.bins(), t.bin_factorization(), t.variant_bins()
    t.close()
    assert [b[:3] for b in bins] == [b[:3] for b in S.Handle(pop, **options).bins()]
    slow = next(i for i, b in enumerate(bins) if kernel.startswith(f"rollout_kernel<{b[0]}, ")) if not one else 0
    times = [(30.0 if i == slow else 5.0, 3) for i in range(len(bins))]
    fl = np.arange(1.0, 301.0)
    n = -(-T // (options.get("steps_per_launch") or 1000))
    d = bench.dominant_kernel(one, bins, facs, vb, times, fl, ms, n, False, False)
    assert d["kernel"] == kernel
    if one:
        assert d["kernel_avg_launch_ms"] == ms / n and d["kernel_flops_per_launch"] == fl.sum() / n
        assert d["kernel_variants"] == 300 and d["kernel_launches_per_step"] == n
    else:
        assert d["kernel_avg_launch_ms"] == 10.0 and d["kernel_flops_per_launch"] == fl[vb == slow].sum() / 3


def test_traffic_of_the_one_launch_is_recorded_per_layout(tmp_path, monkeypatch):
    for counter in ("FETCH_SIZE", "WRITE_SIZE"):
        d = tmp_path / counter
        d.mkdir()
        with open(d / "c_counter_collection.csv", "w", newline="") as f:
            w = csv.writer(f)
            w.writerow(["Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value"])
            for i, (k, v) in enumerate([("void simk::rollout_multi_kernel<0>(simk::MultiArgs, simk::ModelParams)", 7), ("copy", 1 << 19),
                                        ("void simk::rollout_multi_kernel<0>(simk::MultiArgs, simk::ModelParams)", 90),
                                        ("void simk::rollout_kernel<28, 2, 8, false, false, false>(simk::BinArgs)", 3),
                                        ("void simk::rollout_kernel<28, 2, 8, false, false, false>(simk::BinArgs)", 40)]):
                w.writerow([i, k, counter, v])
    os.makedirs(tmp_path / "profiles")
    out = tmp_path / "profiles" / "rollout_traffic.json"
    TR.build([(1000, str(tmp_path / "FETCH_SIZE"), str(tmp_path / "WRITE_SIZE"), "28x2x8")], str(out), "w")
    rec = json.loads(out.read_text())
    assert rec["per_launch_kib_by_steps_per_launch"] == {"1000": {"rollout_kernel<28, 2, 8, false, false, false>": [40, 40]}}
    os.makedirs(tmp_path / os.path.dirname(rec["kernel_source"]))
    with open(os.path.join(ROOT, rec["kernel_source"]), "rb") as f:
        (tmp_path / rec["kernel_source"]).write_bytes(f.read())
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.recorded_traffic("rollout_multi_kernel 28x2x8", 1000) == (90 * 2 + 90 * 2) * 1024
    assert bench.recorded_traffic("rollout_multi_kernel 24x2x8+28x2x8", 1000) is None


def test_the_default_layout_of_the_benchmark_is_recorded():
    h = S.Handle(W.random_trees(8192))
    layout = "+".join(f"{b[0]}x{b[1] // 16}x{b[2]}" for b in sorted(h.bins()))
    assert h.one_launch() and bench.recorded_traffic(f"rollout_multi_kernel {layout}", 1000) is not None
    h.close()

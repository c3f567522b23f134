"""The measurement tools around the library: the instrumented build with time stamps in the kernels
(paper_2510_26577_amd/timeline.py), the few-rows comparison against a vector-ALU kernel
(paper_2510_26577_amd/small_rows.py) and the profile writers.  CPU part: shapes, names, the plain build's refusal
of the stamp read.  GPU part: the alternative kernel agrees with the library and with the oracle; the stamps of
the instrumented build are ordered and its outputs are the plain build's."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2510_26577_amd import binding, profile_kernels, small_rows, timeline, workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_cases_of_the_few_rows_comparison_have_the_rows_they_claim():
    rows = {}
    for name in small_rows.CASES:
        w, nq = small_rows.make_case(name)
        G = w.Hq // w.Hkv
        rows[name] = (nq if nq is not None else int(w.max_T)) * G
        assert w.max_T <= 128 and (nq is None or nq <= int(w.T.min()))
    assert rows == {"cfg1": 8, "decode_B64": 4, "draft_q12": 24}
    a = small_rows.AttnArgs()
    assert ctypes.sizeof(a) == 10 * 8 + 6 * 4 + 4 + 4 + 2 * 8      # ten pointers, six ints, the scale (+ padding), two pointers


def test_workload_names_and_profile_commands():
    for name in ("cfg1", "cfg2", "cfg2_B32", "cfg3_B16", "cfg4"):
        assert timeline.get_workload(name).B >= 1
    with pytest.raises(SystemExit):
        timeline.get_workload("nope")
    assert profile_kernels.bench_args("cfg3_B64+fp8") == ["--workload", "cfg3_B64", "--kv-fp8"]
    assert profile_kernels.bench_args("cfg2") == ["--workload", "cfg2"]
    for cs in profile_kernels.COUNTER_SETS:                      # what one rocprofv3 --pmc run can hold
        assert sum(c.startswith("SQ_") for c in cs) <= 8 and sum(c.startswith("GRBM_") for c in cs) <= 2


def test_plain_build_has_no_time_stamps():
    lib = binding.load_library()
    buf = (ctypes.c_uint64 * 8)()
    assert lib.tva_timeline_read(buf, 1) == -2                   # TVA_UNSUPPORTED: no GPU is touched


@pytest.mark.gpu
@pytest.mark.parametrize("name", small_rows.CASES)
def test_vector_alu_alternative_agrees_with_the_library(name):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    s = small_rows.Prepared(name, 0)
    st = torch.cuda.current_stream()
    s.run_mfma(st)
    s.run_valu(st)
    torch.cuda.synchronize()
    fin = torch.isfinite(s.lse_m)
    assert bool((torch.isfinite(s.lse_v) == fin).all())
    assert float((s.out_m - s.out_v).abs().max()) <= small_rows.TOL_O
    assert float((s.lse_m[fin] - s.lse_v[fin]).abs().max()) <= small_rows.TOL_LSE
    if name == "cfg1":                                           # the alternative against the oracle itself
        from oracle import tva_oracle
        ro, rl = tva_oracle.tree_verify_attn(s.w)
        assert np.abs(s.out_v.cpu().numpy().astype(np.float64) - ro).max() <= small_rows.TOL_O
        assert np.abs(s.lse_v.cpu().numpy().astype(np.float64) - rl).max() <= small_rows.TOL_LSE


@pytest.mark.gpu
def test_instrumented_build_stamps_are_ordered():
    """One process loads one build, so the instrumented one runs in a child: its summary must show every stage
    after the one before, for every workgroup (the minima of the stage differences are not negative)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if not os.path.exists(binding.TIMELINE_LIB_PATH):
        pytest.skip("libtva_timeline.so not built")
    r = subprocess.run([sys.executable, "-m", "paper_2510_26577_amd.timeline", "--workload", "cfg3_B4", "--copies", "4",
                        "--replays", "2"], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    stage_lines = [l for l in r.stdout.splitlines() if l.startswith("  + ")]
    assert len(stage_lines) == 6                                 # five attention stages + the merge block
    for l in stage_lines:
        assert float(l.split("min")[1].split()[0]) >= 0.0, l
    assert "merge kernel" in r.stdout and "gap between" in r.stdout


def test_counters_are_those_of_the_launches_they_are_said_to_be():
    """Launches of one kernel's name that merge their splits, leave them, or are followed by a merge: told apart by their order."""
    from paper_2510_26577_amd import profile_traffic
    attn, merge = "attn_kernel<1>(args)", "merge_kernel<2>(args)"
    launches = [["warm-up", 2], ["step", 2], ["kernel", 3], ["two calls", 1]]
    rows = ([("fill", 7.0), (attn, 9.0), (attn, 9.0), ("fill", 7.0)] + [(attn, 4.0), (merge, 1.0), (attn, 6.0), (merge, 2.0)] +
            [(attn, 1.0), (attn, 2.0), (attn, 3.0)] + [("anc_mask_kernel", 8.0), (attn, 5.0)])
    got = profile_traffic.by_region(rows, launches)
    assert got["step"] == {attn: 5.0, merge: 1.5} and got["kernel"] == {attn: 2.0} and got["two calls"] == {attn: 5.0}
    for wrong in (rows + [(attn, 1.0)], rows[:-1]):
        with pytest.raises(RuntimeError):
            profile_traffic.by_region(wrong, launches)


def test_timeline_tells_a_merge_in_the_launch_from_a_launch_of_its_own():
    """Synthetic stamps: four workgroups, the last without splits to merge or without rows, one call of each form; what is said does
    not follow from the times, which are the same in both."""
    t = np.arange(8, dtype=np.uint64) * np.uint64(100) + np.uint64(5000)         # a microsecond a stage
    buf = np.tile(t, (4, 1)) + np.arange(4, dtype=np.uint64)[:, None] * np.uint64(50)
    shared = buf.copy()
    shared[3, 6:] = 0
    own = buf.copy()
    own[3, :6] = 0
    own[:, 6:] |= timeline.MERGE_LAUNCH
    told = []
    around = np.where(shared, (shared + np.uint64((1 << 32) - 5555)) & np.uint64((1 << 32) - 1), 0)  # the clock's low words come round
    assert around.max() > 1 << 31 and 0 < around[around > 0].min() < 1000
    for x, y in zip(timeline.split_stamps(around, 4, 1), timeline.split_stamps(shared, 4, 1)):
        assert np.allclose(x - 0.01 * ((1 << 32) - 5555), y, equal_nan=True) if isinstance(x, np.ndarray) else x == y
    for stamps, n_merge in ((shared, 1), (own, 4)):
        attn, merge, apart = timeline.split_stamps(stamps, 4, n_merge)
        told.append(timeline.summarise("x", workloads.config1(), 0.0, 9.0, (64, 2, 64), attn, merge, apart, "cmd", "mode"))
        assert len(attn) == (3 if apart else 4) and len(merge) == 4
    assert "no merge kernel: merged in the attention launch, by 3 workgroups, no gap between launches" in told[0]
    assert "gap between the last" not in told[0] and told[0].count("\n  + ") == told[1].count("\n  + ") == 6
    assert "splits waited for and merged               min   2.00   median   2.00   max   2.00" in told[0]
    assert "until all of the row block have arrived min   1.00   median   1.00   max   1.00" in told[0]
    assert "to the last store: 8.00 us" in told[0]
    assert "merge kernel, same clock:" in told[1] and "no merge kernel" not in told[1]
    assert "gap between the last attention workgroup's stores and the first merge: 0.00 us" in told[1]
    assert "3 attention workgroups, 4 merge blocks" in told[1]

"""Jobs whose last stage writes the output to host memory, with no output copy behind
it, in the timeline tools: the per-job terms, the gap at a job's end and the output
side of the link, for the kernel sequences the library runs."""
import pytest

from paper_2606_05495_amd import trace

P = "void setrt::"
# [input copy, stages...] of one job, with its completion kernel where it has one
CHAINS = {
    "image": ["k_copy_in", "k_gauss_sobel_f32<false>"],
    "box": ["k_copy_in", "k_box_hist_u8", "k_copy_out_hist256"],
    "thermal, one launch": ["k_copy_in", "k_hotspot_steps_f32<4>"],
    "thermal, two launches, word": ["k_copy_in", "k_hotspot_steps_f32<3>", "k_hotspot_steps_f32<2>", "k_done_flag"],
    "scan, word": ["k_copy_in", "k_scan_down_i32_i64<0>", "k_done_flag"],
    "vector batch": ["k_copy_in", "k_vec_batch_tiles<256>", "k_vec_batch_final"],
    "image of two kernels": ["k_copy_in", "k_gauss5_win_f32<4, true>", "k_sobel_thresh_win_f32<4, true>", "k_copy_out_sobel"],
}


def _stream(chain, jobs):
    """Jobs of the chain one after another: 10 long kernels with gaps of 2 inside a
    job and 5 between jobs."""
    ks, ns, t = [], [], 0
    for _ in range(jobs):
        for i, n in enumerate(chain):
            t += 2 if i else 5
            ks.append((t, t + 10))
            ns.append(P + n + "(Args)")
            t += 10
    return ks, ns


@pytest.mark.parametrize("name", CHAINS)
def test_jobs_are_found(name):
    chain = CHAINS[name]
    ks, ns = _stream(chain, 4)
    stages = len(chain) - 1 - sum("done_flag" in n for n in chain)
    t = trace.eq_terms(ks + ks, ["A"] * len(ks) + ["B"] * len(ks), ns + ns)
    assert t["jobs"] == 8
    assert t["t_in"] == 10 and t["t_k"] == 10 * stages and t["t_in_k"] == 2 and t["delta_t_k"] == 2 * (stages - 1)
    assert t["t_out"] == 0 and t["t_k_out"] == 0
    g = trace.stream_gaps(ks, ["A"] * len(ks), ns)
    assert g["mean_job_boundary_gap"] == 5 and g["mean_intra_job_gap"] == 2


def test_a_cut_off_job_is_not_one_without_an_output_copy():
    ks, ns = _stream(["k_copy_in", "k_a", "k_b", "k_copy_out"], 3)
    t = trace.eq_terms(ks[:-1], ["A"] * (len(ks) - 1), ns[:-1])
    assert t["jobs"] == 2 and t["t_out"] == 10 and t["t_k"] == 20


def _csv(path, rows):
    with open(path / "run_kernel_trace.csv", "w") as fh:
        fh.write('"Kind","Stream_Id","Kernel_Name","Start_Timestamp","End_Timestamp"\n')
        for s, a, b, n in rows:
            fh.write('"KERNEL_DISPATCH",%d,"%s",%d,%d\n' % (s, P + n, a, b))


def test_outputs_of_the_last_stage_count_on_the_link(tmp_path):
    """Stream 1: in [0,10] image [10,14], in [20,30] image [30,34]; stream 2's input
    [12,18] is beside the first image for 2 of the 34 that either direction is busy."""
    _csv(tmp_path, [(1, 0, 10, "k_copy_in"), (1, 10, 14, "k_gauss_sobel_f32<true>"),
                    (2, 12, 18, "k_copy_in"), (2, 18, 20, "k_gauss_sobel_f32<true>"),
                    (1, 20, 30, "k_copy_in"), (1, 30, 34, "k_gauss_sobel_f32<true>")])
    m = trace.analyze_dir(str(tmp_path))
    assert m["eq_terms"]["jobs"] == 3
    assert m["h2d_d2h_overlap_fraction"] == pytest.approx(2 / 34)


@pytest.mark.parametrize("last", ["k_gauss_sobel_f32<true>", "k_copy_out_hist256"])
def test_batches_end_with_their_last_stage(tmp_path, last):
    """Two batches of two chains interleaved on one stream, the second starting 7
    after the first's last stage."""
    rows = []
    for t in (0, 41):
        rows += [(1, t, t + 10, "k_copy_in"), (1, t + 10, t + 20, "k_copy_in"), (1, t + 21, t + 27, last),
                 (1, t + 27, t + 34, last)]
    _csv(tmp_path, rows)
    assert trace.analyze_dir(str(tmp_path), batch=2)["mean_inter_batch_us"] == pytest.approx(7 / 1e3)


@pytest.mark.parametrize("final", ["k_sobel_final", "k_copy_out_sobel"])
def test_traffic_of_the_finaliser_under_both_names(tmp_path, final):
    for d, counter, kib in (("f", "FETCH_SIZE", 32768.0), ("w", "WRITE_SIZE", 65536.0)):
        (tmp_path / d).mkdir()
        with open(tmp_path / d / "pmc_counter_collection.csv", "w") as fh:
            fh.write("Dispatch_Id,Kernel_Name,Counter_Name,Counter_Value\n")
            fh.write('1,"setrt::%s(Args)",%s,8.0\n' % (final, counter))
            fh.write('2,"__amd_rocclr_copyBuffer",%s,%f\n' % (counter, kib))
    (tmp_path / "p.json").write_text('{"slots": 8, "reps": 1}\n')
    r = trace.traffic_file(str(tmp_path / "out.json"), {"x": (str(tmp_path / "f"), str(tmp_path / "w"), str(tmp_path / "p.json"))})
    k = r["workloads"]["x"]["kernels"]["sobel_final"]
    assert k["fetch"] == 2 * 8192 and k["write"] == 8192

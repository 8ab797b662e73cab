"""CPU-only checks of the rules that share work out over the chip, and of the build variants of the tile kernels."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run_host_check(tmp_path, name):
    exe = tmp_path / name
    subprocess.run(["g++", "-O2", "-std=c++17", "-o", str(exe), os.path.join(ROOT, "tests", "host", name + ".cpp")],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and "bad=0" in r.stdout, r.stdout + r.stderr


def test_tile_walk_is_balanced_over_the_xcds(tmp_path):
    _run_host_check(tmp_path, "tile_balance_check")


def test_split_of_dh_is_allowed_cheapest_and_within_its_scratch(tmp_path):
    _run_host_check(tmp_path, "dh_split_check")


def test_logits_edge_widens_with_the_slots_and_its_scratch_serves_fewer(tmp_path):
    _run_host_check(tmp_path, "logits_edge_check")


def test_the_gpu_tests_of_the_streaming_forward_take_it(tmp_path):
    from tests import test_gpu_shapes as shapes, test_gpu_stream as stream
    want = [(V, d, n, n <= 204) for d, V in stream.SIZES for n in (1, 130, 204, 205)]
    want += [(V, d, n, True) for d, V in stream.STEP_SIZES for n in (1, 204)]
    want += [(V, d, n, V >= 150000) for dtype, n, d, V in shapes.MASKED if dtype == "bf16"]
    _run_host_check(tmp_path, "logits_edge_check")
    r = subprocess.run([str(tmp_path / "logits_edge_check"), *(str(v) for w in want for v in w[:3])], capture_output=True, text=True)
    assert [bool(int(line)) for line in r.stdout.split()] == [w[3] for w in want]


def test_gradient_edges_follow_the_length_of_the_contraction(tmp_path):
    _run_host_check(tmp_path, "gradient_edge_check")


def test_k_major_operands_are_taken_in_pieces_of_a_window(tmp_path):
    _run_host_check(tmp_path, "window_check")


def test_kv_edge_is_the_faster_one_where_both_were_measured(tmp_path):
    _run_host_check(tmp_path, "kv_edge_check")


def test_kv_launches_are_merged_where_that_was_measured_to_be_faster(tmp_path):
    _run_host_check(tmp_path, "kv_launch_check")


def test_the_gpu_tests_of_the_kv_products_take_the_tiles_that_they_name(tmp_path):
    """The tables in the GPU tests say which tiles their sizes run on; the rule says which they really run on."""
    from tests import test_gpu_deep_tiles as deep, test_gpu_kmajor as kmajor
    want = [("bf16", 0, n, d, kind) for (n, d), kind in deep.SIZES.items()]
    want += [(dt, mode, n, d, kind) for (dt, n, d), kind in deep.MORE.items() for mode in (0, 2) if mode == 0 or kind == "256 ring"]
    for (n, d), edges in kmajor.EDGES.items():
        want += [(dt, mode, n, d, edge) for (dt, mode), edge in zip([("bf16", 0), ("bf16", 2), ("f32", 0), ("f32", 2)], edges)]
    _run_host_check(tmp_path, "kv_edge_check")
    r = subprocess.run([str(tmp_path / "kv_edge_check"), *(str(v) for w in want for v in w[:4])], capture_output=True, text=True)
    got = r.stdout.splitlines()
    assert len(got) == len(want)
    for w, line in zip(want, got):
        assert line == w[4] if isinstance(w[4], str) else line.startswith(f"{w[4]} "), (w, line)


@pytest.mark.parametrize("source", ["lmhead_gemm.hip", "dynakv_gemm.hip", "dynakv_gate.hip"])
def test_the_32x32x16_form_of_the_bf16_main_loop_still_compiles(source):
    from paper_2603_04411_amd import build
    r = subprocess.run([build._hipcc(), *build.FLAGS, "-DLMHEAD_BF16_BLOCK=32", "-fsyntax-only", "--cuda-device-only",
                        os.path.join(build.CSRC, source)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]


def test_the_tile_trace_reads_points_that_the_kernels_stamp():
    import re
    from paper_2603_04411_amd import build, tile_trace
    with open(os.path.join(build.CSRC, "lmhead_gemm.hip")) as src:
        stamped = {(int(p), int(k)) for p, k in re.findall(r"trace_stamp\((\d+), (\d)\)", src.read())}
    for kernel, kind in (("fwd", 1), ("dz", 2)):
        for _, a, b in tile_trace.EPILOGUE[kernel]:
            assert {(a, kind), (b, kind)} <= stamped, (kernel, a, b)

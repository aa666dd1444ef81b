"""Host-side checks of bench.py that need no GPU: the multi-GPU refusal and
the algorithmic byte model used by its roofline."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode != 0
    assert "one GPU" in r.stderr


class _Stats:
    n_rows, nnz, n_entries, n_hub_rows, n_hub_chunks = 1000, 50_000, 120, 3, 40


@pytest.mark.parametrize("F", [16, 128])
def test_kernel_bytes_model(F):
    st = _Stats()
    b7, b8 = bench.kernel_bytes(st, F, n_ref=900)
    nonhub = st.n_rows - st.n_hub_rows
    assert b7 == (8 * st.nnz + 16 * st.n_entries + 4 * nonhub + 4 * F * 900 + 4 * F * nonhub
                  + 4 * F * st.n_hub_chunks)
    assert b8 == 4 * F * st.n_hub_chunks + 4 * F * st.n_hub_rows + 8 * st.n_hub_rows
    w7, w8 = bench.kernel_bytes(st, F, n_ref=900, variant="warp_level")
    assert w7 == 8 * st.nnz + 16 * st.n_entries + 4 * F * 900 + 4 * F * st.n_rows
    assert w8 == 8 * st.n_rows


class _Graph:
    """A power-law plan of the default workload's size."""
    n_rows = n_cols = 230_000
    nnz, n_hub_rows, max_deg, max_wave_nzs = 11_386_022, 4_000, 3_391, 32
    n_hub_chunks, hub_chunk_nnz, hub_windows, flags = 9_000, 512, 0, 0


class _Uniform(_Graph):
    n_rows = n_cols = 1_000_000
    nnz, n_hub_rows, max_deg, n_hub_chunks = 20_000_000, 0, 50, 0


@pytest.mark.parametrize("st,F,cols,name", [
    (_Graph, 16, 16, "k_spmm<4, 4>"), (_Graph, 32, 32, "k_spmm<4, 8>"), (_Graph, 256, 32, "k_spmm<4, 8>"),
    (_Graph, 17, 17, "k_spmm<4, 0>"), (_Graph, 40, 40, "k_spmm<4, 0>"), (_Graph, 64, 32, "k_spmm<4, 8>"),
    (_Graph, 100, 100, "k_spmm<4, 0>"), (_Graph, 300, 152, "k_spmm<4, 0>"), (_Graph, 3, 3, "k_spmm<1, 0>"),
    (_Graph, 2, 2, "k_spmm<1, 2>"), (_Graph, 500, 252, "k_spmm<4, 0>"), (_Uniform, 64, 64, "k_spmm<4, 16>"),
    (_Uniform, 128, 64, "k_spmm<4, 16>"), (_Uniform, 256, 32, "k_spmm<4, 8>")])
def test_kernel_names_match_the_library_dispatch(st, F, cols, name):
    assert bench.slice_cols(st, F) == cols
    assert bench.spmm_kernel_name(F, "block", st) == name


def test_ablation_kernel_names():
    assert bench.spmm_kernel_name(64, "column_loop", _Graph) == "k_spmm_colloop"
    assert bench.spmm_kernel_name(64, "warp_level", _Graph) == "k_spmm_wl<4, 8>"


@pytest.mark.parametrize("n,fin,fout,name", [
    (230_000, 28, 128, "k_linear_rw<8>"), (230_000, 16, 32, "k_linear_rw<2>"), (230_000, 16, 60, "k_linear_rw<4>"),
    (230_000, 32, 16, "k_linear_split<1, 8>"), (230_000, 33, 17, "k_linear_split<2, 8>"),
    (230_000, 256, 40, "k_linear_split<3, 8>"), (230_000, 128, 64, "k_linear_split<4, 8>"),
    (230_000, 602, 256, "k_linear_split<8, 8>"), (30_000, 64, 64, "k_linear_split<4, 4>"),
    (3_000, 1000, 16, "k_linear_ksplit<1, 8>"), (12_000, 128, 64, "k_linear_ksplit<4, 4>")])
def test_linear_kernel_names_match_the_library_dispatch(n, fin, fout, name):
    assert bench.linear_kernel(n, fin, fout) == name
    # the tile shapes named are those the library's source launches
    src = open(os.path.join(ROOT, "paper_2308_11825_amd", "csrc", "agcn_linear.hip")).read()
    kind, args = name.split("<")
    launch = {"k_linear_rw": "launch_rw", "k_linear_split": "launch_split", "k_linear_ksplit": "launch_ksplit"}
    assert f"{launch[kind]}<{args}(" in src


def test_layer_order_matches_the_library():
    assert bench.aggregates_first(_Graph, 128, 256) and bench.aggregates_first(_Graph, 16, 32)
    assert not bench.aggregates_first(_Graph, 100, 128)
    assert not bench.aggregates_first(_Graph, 128, 128) and not bench.aggregates_first(_Graph, 256, 40)
    class Win(_Graph):
        hub_windows = 100
    assert not bench.aggregates_first(Win, 128, 256)


def test_small_path_kernel_name():
    class St(_Graph):
        n_hub_rows, max_deg, max_wave_nzs, nnz, n_rows, n_cols = 0, 21, 32, 36844, 4096, 4096
    assert bench.small_path(St)
    assert bench.spmm_kernel_name(16, "block", St) == "k_spmm_rows<4, 4>"
    assert bench.spmm_kernel_name(64, "block", St) == "k_spmm_rows<4, 8>"
    assert bench.spmm_kernel_name(17, "block", St) == "k_spmm_rows<4, 0>"
    St.max_deg = 33
    assert not bench.small_path(St)
    assert bench.spmm_kernel_name(16, "block", St) == "k_spmm<4, 4>"


def test_gather_requests_model():
    class St(_Graph):
        nnz = 1000
    assert bench.gather_requests(St, 16) == 1000
    assert bench.gather_requests(St, 32) == 1000
    assert bench.gather_requests(St, 256) == 8000
    assert bench.gather_requests(St, 40) == 2000        # 160 bytes from any multiple of 32
    assert bench.gather_requests(St, 41) == 1000 + 1250  # 164 bytes from any multiple of 4


class _WinStats:
    n_rows, nnz, n_hub_rows, hub_first_entry, deg_bound = 1_000_000, 111_640_508, 1000, 270_000, 512
    hub_windows = 1954


def test_window_shape_and_bytes_model():
    # skewed_hubs' shape: 1000 hub rows, 1954 windows of 512 columns; one row
    # batch; F = 64 is one slice, so about 512 workgroups means G = 4 windows
    # per group (489 groups); F = 256 has four slices, so G = 16 (123 groups).
    st = _WinStats()
    assert bench.win_shape(st, 64) == (1, 1, 4, 489)
    assert bench.win_shape(st, 256) == (4, 1, 16, 123)
    assert bench.win_shape(st, 96) == (2, 1, 8, 245)
    hub = {"hub_nnz": 107_144_212, "n_cols": 1_000_000, "low_nnz": 4_496_296,
           "low_entries": 270_000, "low_ref": 990_000}
    b_low, b_hub = bench.window_bytes(st, 64, hub)
    assert b_hub == (8 * hub["hub_nnz"] + 4 * 64 * hub["n_cols"] + 8 * 1000 * 1954
                     + 2 * (4 * 64 + 4) * 1000 * 489 + (4 * 64 + 4) * 1000)
    nonhub = st.n_rows - st.n_hub_rows
    assert b_low == (8 * hub["low_nnz"] + 16 * hub["low_entries"] + 4 * nonhub
                     + 4 * 64 * hub["low_ref"] + 4 * 64 * nonhub)
    # the windows serve F >= 64 on the float4 path of the block-level plan only
    assert bench.windows_used(st, 64) and bench.windows_used(st, 512)
    assert not bench.windows_used(st, 32) and not bench.windows_used(st, 66)
    assert not bench.windows_used(st, 64, "warp_level")
    st.hub_windows = 0
    assert not bench.windows_used(st, 64)

"""The benchmark's record of what the library runs: networks whose sums a kernel
ahead of the step takes are not counted as taking each unordered pair once."""
import bench
from paper_1612_01501_amd import inputs as I


class Sim:
    def __init__(self, paths):
        self.paths = paths

    def gap_path(self, k):
        return self.paths[k], False


def config(nets, paths, n_sym):
    info = dict(step_mode=2, n_tiles=4, n_tiles_wide=0, wide_threads=1024, n_bitmap=0, n_blocked=0, lanes_per_row=4,
                tile_rows=64, tuned=0, tune_cached=0, n_stream=0, tune_mode=-1, stream_round=0, n_sym=n_sym)
    return bench.tuned_config(info, Sim(paths), nets)


def test_grid_and_voltage_sums_are_not_unordered_pairs():
    big = I.Network(n=5000, conn="uniform", g=0.01)
    c = config([big], ["uniform_sym"], 1)
    assert c["gap_paths"] == ["uniform_grid_ahead"] and c["step_kernel"].startswith("infoli::k_grid_sums + ")
    assert c["unordered_pair_networks"] == 0 and c["sums_ahead_networks"] == 1
    sgj = I.Network(n=20000, conn="uniform", g=0.01, gap="sgj")
    c = config([sgj], ["uniform_sum"], 1)
    assert c["unordered_pair_networks"] == 0 and c["sums_ahead_networks"] == 1
    small = I.Network(n=600, conn="uniform", g=0.01)
    c = config([small, I.Network(n=8, conn="none")], ["uniform", "none"], 0)
    assert c["gap_paths"] == ["none", "uniform_grid"] and c["sums_ahead_networks"] == 0

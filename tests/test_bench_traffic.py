"""bench.py takes a recorded traffic figure only for the kernel that ran: the same
sources and the same variant."""
import bench


def test_recorded_traffic_matches_sources_and_variant(tmp_path):
    sha = bench.kernel_sources_sha("fp16split", 1)
    path = tmp_path / "traffic.txt"
    path.write_text("# a comment\n"
                    f"kernel=forward-c3-fp16split sources={sha} tuned=1 bytes_per_launch=3e9 variant=b\n"
                    f"kernel=forward-c3-fp16split sources={sha} tuned=0 bytes_per_launch=2e9 variant=a\n"
                    f"kernel=adjoint-c3-fp16split sources={sha} bytes_per_launch=4e9 variant=c\n"
                    "kernel=forward-c4-fp16split sources=0 tuned=0 bytes_per_launch=5e9 variant=d\n")
    get = lambda *a: bench.recorded_traffic(*a, path=str(path))
    assert get("forward", "c3", "fp16split", 1, 0) == 2e9
    assert get("forward", "c3", "fp16split", 1, 1) == 3e9
    assert get("forward", "c3", "fp16split", 1, 2) is None
    assert get("adjoint", "c3", "fp16split", 1, 0) is None      # no variant recorded
    assert get("forward", "c4", "fp16split", 2, 0) is None      # other sources

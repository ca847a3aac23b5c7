"""The seeded route shapes (tests/route_shapes.py) meet every GEMM kernel,
tile size and the split last round, as the library plans them without a
GPU (256 compute units, as on MI355X)."""
import paper_2604_06916_amd as sol
from route_shapes import SHAPES


def test_route_shapes_meet_every_kernel():
    nv = {(p["kernel"], p["tile"]) for p in (sol.gemm_plan(*s) for s in SHAPES)}
    assert {("nvfp4_gemm_wavek_kernel", 32), ("nvfp4_gemm_small_kernel", 64),
            ("nvfp4_gemm_lane_kernel", 128), ("nvfp4_gemm_lane_kernel", 256),
            ("nvfp4_gemm_kernel", 256)} <= nv
    assert any(sol.gemm_plan(*s)["splits"] == 2 for s in SHAPES)
    mx = {(p["kernel"], p["tile"]) for p in (sol.gemm_plan(M, N, K - K % 32, sol.FORMAT_MXFP4)
                                              for M, N, K in SHAPES if K >= 32)}
    assert mx == {("mxfp4_gemm_wavek_kernel", 32), ("mxfp4_gemm_kernel", 64),
                  ("mxfp4_gemm_kernel", 128), ("mxfp4_gemm_kernel", 256)}


def test_last_round_plan_boundaries():
    """Where the last round of 256 x 256 tiles runs as 128 x 128 quadrants
    (at most 64 tiles, a quarter of MI355X's 256 CUs), where those quadrants
    split in K halves (at most 32 tiles and at least 16 K stages of 128),
    and where whole tiles split instead (65 to 128 tiles).  The plan counts
    the workgroups of both launches; MXFP4 never splits K."""
    def plan(M, N, K, fmt=sol.FORMAT_NVFP4, ws=True):
        p = sol.gemm_plan(M, N, K, fmt, with_workspace=ws)
        assert p["tile"] == 256
        return p["workgroups"], p["splits"]
    # 288 tiles, 32 over: quadrants in K halves from 16 stages, whole below
    assert plan(4096, 4608, 2048) == (256 + 8 * 32, 2)
    assert plan(4096, 4608, 2048, ws=False) == (256 + 4 * 32, 1)
    assert plan(4096, 4608, 1920) == (256 + 4 * 32, 1)
    # 289 and 320 tiles: 33 and 64 over, whole quadrants
    assert plan(4352, 4352, 3072) == (256 + 4 * 33, 1)
    assert plan(4096, 5120, 3072) == (256 + 4 * 64, 1)
    # 321 tiles: 65 over, each of them in two K halves
    assert plan(768, 27392, 3072) == (256 + 2 * 65, 2)
    # whole rounds, and fewer tiles than CUs: one launch of whole tiles
    assert plan(4096, 4096, 3072) == (256, 1)
    assert plan(4096, 3840, 3072) == (240, 1)
    mx = sol.FORMAT_MXFP4
    assert plan(4096, 4608, 2048, mx) == (256 + 4 * 32, 1)
    assert plan(4096, 5120, 3072, mx) == (256 + 4 * 64, 1)
    assert plan(768, 27392, 3072, mx) == (321, 1)


def test_tiles_of_32_name_the_wavek_kernel():
    """32 x 32 tiles run on the wave-K kernel only, whatever the K: the plan
    names the kernel that is launched."""
    names = {sol.gemm_plan(M, N, K)["kernel"] for M, N, K in
             [(33, 40, 144), (1, 9, 656), (777, 1235, 1040), (128, 1152, 1152), (20000, 32, 3072)]}
    assert names == {"nvfp4_gemm_wavek_kernel"}
    assert all(sol.gemm_plan(*s)["kernel"] == "nvfp4_gemm_wavek_kernel"
               for s in SHAPES if sol.gemm_plan(*s)["tile"] == 32)


def test_whole_tiles_of_tokens_run_where_ragged_ones_do():
    """One token less does not change the kernel of few tokens: operands of
    whole 128 x 128 tiles take the wave-K kernel where it is the faster."""
    for N, K in [(1152, 1120), (3072, 1056), (256, 160), (128, 1120)]:
        assert sol.gemm_plan(128, N, K) == sol.gemm_plan(127, N, K)
        assert sol.gemm_plan(128, N, K)["kernel"] == "nvfp4_gemm_wavek_kernel"
        assert sol.gemm_plan(128, N, K, sol.FORMAT_MXFP4) == sol.gemm_plan(127, N, K, sol.FORMAT_MXFP4)
        assert sol.gemm_plan(128, N, K, sol.FORMAT_MXFP4)["kernel"] == "mxfp4_gemm_wavek_kernel"


def test_mx_sixteenths_at_any_depth():
    """A last round of at most 16 MXFP4 tiles runs as 64 x 64 sixteenths,
    short K or long; 17 tiles as quadrants."""
    for K in (32, 128, 1024, 1056, 4096):
        assert sol.gemm_plan(4352, 4096, K, sol.FORMAT_MXFP4)["workgroups"] == 256 + 16 * 16
        assert sol.gemm_plan(1792, 9984, K, sol.FORMAT_MXFP4)["workgroups"] == 256 + 4 * 17


def test_short_odd_block_counts_run_on_the_lane_kernel():
    """K % 32 == 16 below 160: the lane kernel on every tile size, but for K =
    16 and 48 on one round of 256 x 256 tiles; operands of fewer than 8 scale
    bytes stay on the workgroup-shared kernel."""
    def at(*s):
        p = sol.gemm_plan(*s)
        return p["kernel"], p["tile"]
    lane, shared = "nvfp4_gemm_lane_kernel", "nvfp4_gemm_kernel"
    for K in (16, 48, 80, 112):
        assert at(300, 300, K) == (lane, 128) and at(8192, 6720, K) == (lane, 256)
    assert at(8192, 6720, 144) == (lane, 256) and at(2930, 2235, 144) == (lane, 128)
    for K in (16, 48):
        assert at(4096, 4096, K) == (shared, 256)
    for K in (80, 112, 144):
        assert at(4096, 4096, K) == (lane, 256)
    assert at(7, 300, 16) == (shared, 256) and at(8, 300, 16) == (lane, 128)


def test_half_last_stages_on_whole_rounds():
    """K % 128 == 64 on unsplit 256 x 256 tiles: the lane kernel past K =
    1024, the workgroup-shared one below."""
    for M, N in [(4096, 4096), (8192, 5600)]:
        for K, name in [(64, "nvfp4_gemm_kernel"), (960, "nvfp4_gemm_kernel"),
                        (1088, "nvfp4_gemm_lane_kernel"), (2240, "nvfp4_gemm_lane_kernel")]:
            p = sol.gemm_plan(M, N, K)
            assert p["kernel"] == name and p["tile"] == 256 and p["splits"] == 1

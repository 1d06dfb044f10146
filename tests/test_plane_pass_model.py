"""The byte model of the plane pass (CPU): the benchmark's roofline point and
the traffic summary use the bytes of the kernel that runs at n <= 64."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def zl(n):
    K = n // 3
    return n * (2 * K + 1) * (K + 1)


def test_roofline_counts_the_plane_passes_own_bytes():
    sys.path.insert(0, ROOT)
    import bench
    from paper_2506_23712_amd import profiling as p
    ms = {"band": 0.0, "zinv": 0.02, "yinv": 0.0, "xpass": 0.3, "yfwd": 0.0, "zfwd_update": 0.12, "end_step": 0.01}
    res = {"name": "none", "prof": {(64, "fp32"): (ms, 47)}, "variants": {"zfwd_update:64:fp32": 1, "xpass:64:fp32": 5}}
    r = bench.roofline(res)
    assert r["kernel"] == "k_plane<float, 64>" and r["members_per_launch"] == 47
    assert r["bytes_per_launch"] == 47 * 8 * zl(64) * 8               # 5 fields of z-pencils read, 3 written
    assert abs(r["achieved"] - r["bytes_per_launch"] / 0.1e-3 / 1e9) < 0.1
    # the separate passes, and variant 5 where there is no plane pass
    res["variants"]["xpass:64:fp32"] = 2
    assert bench.roofline(res)["bytes_per_launch"] == int(47 * p.pass_bytes(64, "fp32")["xpass"])
    assert p.launch_bytes("xpass", 128, "fp64", 5) == p.pass_bytes(128, "fp64")["xpass"]
    assert p.launch_bytes("zfwd_update", 64, "fp32", 1) == sum(p.zfwd_stage_bytes(64, "fp32", 1, True))


def test_summary_has_the_plane_pass(tmp_path):
    """Row of the committed counters of the mixed set's 47 members of 64^3: the
    measured bytes are the model's but for the rows' partial lines."""
    from paper_2506_23712_amd import profiling as p
    out = tmp_path / "summary.md"
    p.write_summary(64, None, str(out), workloads=[("ens96_mixed_fp32", "fp32", 47)])
    rows = [[c.strip() for c in l.strip().strip("|").split("|")] for l in out.read_text().splitlines() if "`k_plane<" in l]
    assert len(rows) == 1 and rows[0][1] == "`k_plane<float, 64>`"
    r, w = (float(x) for x in rows[0][2].split("/"))
    assert abs(r - 47 * 5 * zl(64) * 8 / 1e9) < 1e-3 and abs(w - 47 * 3 * zl(64) * 8 / 1e9) < 1e-3
    assert 0.95 < float(rows[0][4]) < 1.2

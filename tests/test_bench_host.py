"""Host logic of bench.py that needs no GPU: which roofline a process is measured against, the
sweep's markdown table, and the refusal of more than one GPU."""
import bench


def test_roofline_bound_follows_the_machine_balance():
    # 78.6 TFLOP/s over 8 TB/s: about 9.8 flops per byte
    assert bench.roofline_bound(136, 4 * 300) == "hbm"          # e+e- -> mu+mu-: 4 helicities, ~300 flops each
    assert bench.roofline_bound(224, 64 * (26795 + 2401)) == "alu"   # gg -> tt~gg
    balance = bench.FP64_VALU_PEAK_TFLOPS * 1e12 / (bench.HBM_PEAK_GBS * 1e9)
    assert bench.roofline_bound(100, 0.99 * balance * 100) == "hbm"
    assert bench.roofline_bound(100, 1.01 * balance * 100) == "alu"


def test_sweep_markdown_table():
    res = {"gg_tt": [{"precision": "fp64", "n_evt": 256, "MEs_per_s": 1.0e8},
                     {"precision": "fp64", "n_evt": 1024, "MEs_per_s": 2.0e8},
                     {"precision": "mixed_fp16", "n_evt": 256, "MEs_per_s": 1.5e8}]}
    lines = bench.sweep_markdown(res).splitlines()
    assert lines[0] == "| process | form | 2^8 | 2^10 |"
    assert lines[2] == "| gg_tt | fp64 | 1e+08 | 2e+08 |"
    assert lines[3] == "| gg_tt | mixed_fp16 | 1.5e+08 | - |"


def test_more_than_one_gpu_is_refused():
    """the measurement covers one GPU; asked for more, bench.py says so and exits with status 2
    before touching a device"""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, timeout=120, cwd=root)
    assert r.returncode == 2
    assert "one GPU" in r.stderr and r.stdout == ""


def test_kernel_hash_covers_every_included_header(tmp_path):
    """committed HBM counters are dropped when any source of the amplitude kernels has changed, also one that is
    included through another; not for a source that the kernels do not include"""
    import os
    import shutil
    csrc = os.path.join(bench.ROOT, "paper_2210_11122_amd", "csrc")
    copy = str(tmp_path / "csrc")
    shutil.copytree(csrc, copy)
    used = {"gg_ttgg": ["generated/proc_gg_ttgg.hip", "rec_gg_ttgg.hip", "recursion.hpp", "flows.hpp", "helas.hpp",
                        "colorsum.hpp", "process.hpp", "generated/colour_blocks.hpp"],
            "gg_ttg": ["rec_gg_ttg.hip", "recursion.hpp", "colorsum.hpp", "process.hpp", "generated/channels.hpp"],
            "gg_ttggg": ["rec_gg_ttggg.hip", "recursion.hpp", "flows.hpp", "helas.hpp", "process.hpp"]}
    for process, names in used.items():
        want = bench.kernel_source_hash(process)
        assert bench.kernel_source_hash(process, copy) == want
        for name in names + ["rambo.hpp"]:
            path = os.path.join(copy, *name.split("/"))
            with open(path, "rb") as fh:
                text = fh.read()
            with open(path, "wb") as fh:
                fh.write(b"// another line\n" + text)
            assert (bench.kernel_source_hash(process, copy) == want) == (name == "rambo.hpp"), (process, name)
            with open(path, "wb") as fh:
                fh.write(text)

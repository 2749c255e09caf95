"""bench.py on the command line, without a GPU: the cases it must refuse."""
import os
import re
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode != 0
    assert "one GPU" in r.stderr
    assert r.stdout.strip() == ""  # no JSON line for a run that did not happen


def _library_kernel_names():
    with open(os.path.join(ROOT, "paper_2210_02574_amd", "csrc", "device.hip")) as fh:
        text = fh.read()
    return re.findall(r'"(k_\w+)"', re.search(r"kKernelNames\[KID_COUNT\] = \{(.*?)\};", text, re.S).group(1))


def test_counter_summary_is_read_for_every_kernel_of_the_step():
    """bench.py takes measured traffic and instruction counts per launch from the committed profile summary: every
    kernel of the benchmark step must be there with positive figures, none that the library does not report (its figures
    would belong to another kernel), and the summary must say where it comes from."""
    import bench

    table, source = bench.load_counter_summary()
    assert source and "Measured at commit" in source
    step = {"k_inner_fin", "k_inner_special", "k_inner_finished", "k_ntt_fwd_cols_modup", "k_ntt_fwd_blocks_fin", "k_ntt_fwd_cols_moddown",
            "k_ntt_fwd_cols_moddown_rescale", "k_ntt_inv_cols", "k_ntt_inv_blocks", "k_ntt_fwd_blocks", "k_ntt_fwd_cols"}
    assert step <= set(table)
    traced = {k for k in table if "<" not in k}
    assert traced <= set(_library_kernel_names()), traced - set(_library_kernel_names())
    for k in step:
        traffic, instr, alg = table[k]
        assert traffic > 0 and instr > 0 and alg > 0
        # measured traffic within a factor of two of the bytes the step has to move
        assert 0.5 < traffic / alg < 2.0, (k, traffic, alg)


def test_every_reported_kernel_is_one_the_library_has():
    """A reported name is a kernel's own, with the ring size dropped and the variant of a shared template added."""
    csrc = os.path.join(ROOT, "paper_2210_02574_amd", "csrc")
    defined = set()
    for name in os.listdir(csrc):
        if name.endswith((".h", ".hip")):
            with open(os.path.join(csrc, name)) as fh:
                defined |= set(re.findall(r"__global__[^;{]*?void (k_\w+)\(", fh.read()))
    for name in _library_kernel_names():
        base = re.sub(r"_(modup|moddown|moddown_rescale|rescale|fin)$", "", name) if name not in defined else name
        assert any(d == base or re.sub(r"1[267](_modup2)?$", "", d) == base for d in defined), name

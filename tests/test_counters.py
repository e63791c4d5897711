"""Counter summaries: which kernel and which sources a figure belongs to."""
import shutil

from paper_1202_6522_amd import counters


def test_kernels_are_told_apart():
    key = counters.kernel_key
    assert key("void shtn::k_legendre_analys<8, 1, 1>(shtn::LegArgs)") == ("legendre_analys", "legendre.hip")
    assert key("void shtn::k_legendre_analys_mf<4, 2, 1, false>(shtn::LegArgs)") == ("legendre_analys_mf", "analys_mf.hip")
    assert key("void shtn::k_legendre_synth<1, 1, false>(shtn::LegArgs)") == ("legendre_synth", "legendre.hip")
    assert key("shtn::k_vec_spread(shtn::DevPlan const*, double const*)") is None


def test_a_changed_header_outdates_a_summary(tmp_path):
    csrc = shutil.copytree(counters.os.path.join(counters.HERE, "csrc"), tmp_path / "csrc")
    before = {f: counters.source_hash(f, str(csrc)) for _, f in counters.KERNELS.values()}
    assert before["fft.hip"] == counters.source_hash("fft.hip")
    with open(csrc / "legendre_dev.h", "a") as f:
        f.write("// changed\n")
    assert all(counters.source_hash(f, str(csrc)) != h for f, h in before.items())

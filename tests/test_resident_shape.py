"""Waves and LDS of the resident search kernels, checked by the compiler on the
CPU: the kernels' own constants, asserted in a source that is only parsed.

launch_bounds does not see LDS: a kernel whose tables, candidates and stage
leave no room for the waves it is compiled for runs with fewer, silently."""
import subprocess
from pathlib import Path

CSRC = Path(__file__).resolve().parents[1] / "paper_2607_04415_amd" / "csrc"

HEAD = """
#include "launch.hpp"
using namespace gorio;
template <int KPL, class M, bool N2S>
constexpr bool fits() {
  return ResidentLds<KPL, M, VisitedLds16<M::ht_log2(KPL)>, N2S>::kFits &&
         ResidentLds<KPL, M, VisitedLds16<M::few_ht_log2(KPL)>, N2S>::kFits &&
         ResidentLds<KPL, M, ResidentHtLarge, N2S>::kFits;
}
template <class M>
constexpr bool all_fit() {
  return fits<1, M, false>() && fits<2, M, false>() && fits<4, M, false>() && fits<1, M, true>() &&
         fits<2, M, true>() && fits<4, M, true>();
}
// waves per SIMD that run with the 16-bit table
template <int KPL, class M>
constexpr int waves() {
  return M::grid_waves_per_simd(KPL, VisitedLds16<M::ht_log2(KPL)>::kWords);
}
"""


def holds(tmp_path, *conditions):
    """Every condition is a constant expression the compiler finds true."""
    from paper_2607_04415_amd import _build
    src = tmp_path / "shape.hip"
    src.write_text(HEAD + "".join(f"static_assert({c});\n" for c in conditions))
    r = subprocess.run([_build.HIPCC, *_build.FLAGS, "--cuda-host-only", "-fsyntax-only", "-w", f"-I{CSRC}",
                        f"-I{_build.INCLUDE}", str(src)], capture_output=True, text=True)
    assert r.returncode == 0, "\n".join(line for line in r.stderr.splitlines() if "error" in line)


def test_the_waves_of_every_kernel_fit_a_cu(tmp_path):
    lines = [f"all_fit<MetricF32Lines<{J}, {whole}>>()" for J in range(1, 9) for whole in ("false", "true")]
    rows = ["all_fit<MetricU8Rows<1, true>>()", "all_fit<MetricU8Rows<1, false>>()", "all_fit<MetricU8Rows<2, false>>()"]
    batches = ["all_fit<MetricU8<1, false>>()", "all_fit<MetricU8<16, false>>()", "all_fit<MetricU8<4, true, true>>()"]
    # two waves for rows of up to four lines and frontiers of up to 64, one with the 32-bit table
    two = [f"waves<1, MetricF32Lines<{J}>>() == 2" for J in (1, 2, 3, 4)]
    one = [f"MetricF32Lines<{J}>::waves_per_simd({k}, ResidentHtLarge::kWords) == 1" for J in (1, 4, 8) for k in (1, 2, 4)]
    holds(tmp_path, "all_fit<MetricF32Own>()", "waves<4, MetricF32Own>() == 2", *lines, *rows, *batches, *two, *one)


def test_short_float32_rows_keep_two_waves_at_any_frontier(tmp_path):
    # rows of one or two lines: 16 KB table, two waves; a batch of one wave per SIMD has 32 KB
    holds(tmp_path, *[f"waves<{k}, MetricF32Lines<{J}>>() == 2" for J in (1, 2) for k in (1, 2, 4)],
          *[f"MetricF32Lines<{J}>::few_ht_log2({k}) == 14" for J in (1, 2) for k in (2, 4)],
          *[f"waves<{k}, MetricF32Lines<{J}>>() == 1" for J in (3, 4, 8) for k in (2, 4)])


def test_a_batch_of_one_wave_per_simd_has_the_kernel_for_one(tmp_path):
    few = "VisitedLds16<MetricF32Lines<{J}, true>::few_ht_log2({k})>::kWords"
    holds(tmp_path, *[f"MetricF32Lines<{J}, true>::roomy({k}, {few.format(J=J, k=k)})" for J in (3, 4) for k in (1, 2, 4)],
          *[f"MetricF32Lines<3, true>::two_batches({k}, {few.format(J=3, k=k)})" for k in (1, 2)],
          "MetricF32Own::few_ht_log2(2) == 14")


def test_whole_lines_have_two_batches_in_flight_with_either_table(tmp_path):
    large = "ResidentHtLarge::kWords"
    holds(tmp_path, *[f"MetricF32Lines<3, true>::two_batches({k}, {large})" for k in (1, 2)],
          "MetricF32Lines<3, true>::two_batches(2, VisitedLds16<14>::kWords)")


def test_uint8_kernels_of_long_frontiers_are_scheduled_for_four_waves(tmp_path):
    # two run (16 KB table); the compiler must not see the table, or it schedules for two
    small = "VisitedLds16<13>"
    lds = [f"ResidentLds<{k}, {m}, {small}, {n}>" for m, k, n in (
        ("MetricU8<4, true, true>", 2, "false"), ("MetricU8<1, false>", 2, "true"), ("MetricU8<1, false>", 4, "false"))]
    holds(tmp_path, *[f"{x}::kCompiled == 4 && {x}::kGrid == 2 && {x}::kLaunchBytes == 16384" for x in lds],
          # nothing to gain where as many waves run as the registers leave room for
          f"ResidentLds<4, MetricU8<4, true, true>, {small}, false>::kLaunchBytes == 0",
          "ResidentLds<1, MetricU8<4, true, true>, VisitedLds16<12>, false>::kLaunchBytes == 0",
          *[f"ResidentLds<{k}, MetricU8Rows<1, true>, {small}, true>::kLaunchBytes == 0" for k in (1, 2, 4)],
          *[f"ResidentLds<{k}, MetricF32Lines<1>, {small}, true>::kLaunchBytes == 0" for k in (1, 2, 4)])


def test_a_team_is_as_wide_as_its_beam(tmp_path):
    # rows of up to 256 ids: a list fits the narrowest team that a beam of one gets
    holds(tmp_path, *[f"detail::team_width({ids}, {most}) == {min(t, most)}" for most in (4, 8)
                      for ids, t in ((1, 2), (64, 2), (128, 2), (129, 4), (256, 4), (257, most), (65536, most))],
          "MetricU8<4, true, true>::team_waves(1) == 4", "MetricU8<4, true, true>::team_waves(4) == 8")

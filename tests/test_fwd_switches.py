"""The forward's compile-time tuning switches (csrc/chunk_attn_fwd.hip), front end
only.  Only four waves of a 128-row item issue the tile DMA, so its DMA must be
laid out for four whichever way FASTVR_DMA_SPLIT is set: laid out for eight, half
of every K and V tile would never be loaded."""
import os
import subprocess

import pytest

from paper_2609_36757_amd import build

CHECK = """
#include "chunk_attn_fwd.hip"
namespace fastvr {
template <int D, bool NEG, bool RING>
constexpr bool issuers_match = HalfAttn<D, NEG, RING>::kDmaWaves == 4 &&
    HalfAttn<D, NEG, RING>::kDmaPer * 4 * 64 == kBK * D / 8;
static_assert(issuers_match<64, false, false> && issuers_match<64, true, true>, "DMA issuers");
static_assert(issuers_match<128, false, true> && issuers_match<128, true, false>, "DMA issuers");
static_assert(Attn<128, false, false>::kDmaWaves == (FASTVR_DMA_SPLIT ? 4 : 8), "256-row items");
}
"""


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
@pytest.mark.parametrize("switches", [[], ["-DFASTVR_DMA_SPLIT=0", "-DFASTVR_BK=64"]], ids=["default", "all_waves_bk64"])
def test_half_items_dma_issuers(tmp_path, switches):
    src = tmp_path / "check.hip"
    src.write_text(CHECK)
    r = subprocess.run([build.hipcc(), f"--offload-arch={build.ARCH}", "--offload-device-only", "-fsyntax-only",
                        "-std=c++17", "-w", "-I", build.INCLUDE, "-I", build.CSRC, *switches, str(src)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]

"""Host side of the kernels' launchers, without a GPU: arguments that no kernel applies are refused."""
import os
import subprocess

import pytest

from paper_2505_23317_amd import build

DRIVER = """
#include "kernels.h"
#include <cstdio>
using namespace cfdetr;
int main() {
  for (int bf16 = 0; bf16 < 2; ++bf16)
    for (Epilogue epi : {Epilogue::kBias, Epilogue::kBiasGelu, Epilogue::kBiasRelu, Epilogue::kBiasResidual})
      if (!(bf16 && epi == Epilogue::kBias))
        std::printf("scale %d\\n", (int)launch_gemm(nullptr, nullptr, nullptr, 64, 64, epi, nullptr, nullptr, bf16 != 0, nullptr,
                                                   64, 64, nullptr, 0.5f));
}
"""


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    """What the driver prints; it calls only what ends before a launch, and sees no GPU."""
    objects = [os.path.join(build.HERE, "_build", s.replace(".hip", ".o")) for s in build.SOURCES]
    if not all(os.path.exists(o) for o in objects):
        pytest.skip("the library has not been built here")
    at = tmp_path_factory.mktemp("rules")
    (at / "driver.hip").write_text(DRIVER)
    hipcc = [build._hipcc(), "--offload-arch=gfx950"]
    for cmd in ([*hipcc, "-std=c++17", "-I", build.CSRC, "-c", str(at / "driver.hip"), "-o", str(at / "driver.o")],
                [*hipcc, str(at / "driver.o"), *objects, "-o", str(at / "driver")]):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
    got = subprocess.run([str(at / "driver")], capture_output=True, text=True, check=True,
                         env={**os.environ, "HIP_VISIBLE_DEVICES": "-1"}).stdout
    return [line.split() for line in got.splitlines()]


def test_a_factor_that_nothing_applies_is_refused(lines):
    """The activations, the residual form and the fp32 path have no factor: 1 is hipErrorInvalidValue."""
    assert [v for k, *v in lines if k == "scale"] == [["1"]] * 7

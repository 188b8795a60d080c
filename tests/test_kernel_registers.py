"""No kernel keeps a lane's values in scratch memory: what the compiler says of each when it is built for gfx950.  CPU only."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2408_08490_amd.build import CSRC, FLAGS, hipcc_path


@pytest.mark.parametrize("source", ["kernels_attn.hip", "kernels_gemm.hip", "kernels_gemm_direct.hip", "kernels_mem.hip", "kernels_spmm.hip"])
def test_no_scratch_memory(source):
    if shutil.which(hipcc_path()) is None:
        pytest.skip("no hipcc")
    cmd = [hipcc_path()] + FLAGS + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(CSRC, source), "-o", os.devnull]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    kernels = re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+)", res.stderr, re.S)
    assert kernels and [k for k in kernels if int(k[1])] == []

"""The flow schedule hands particles and weighing state to wavefronts on other
XCDs without writing an L2 cache back, so every store of its kernel has to be
an agent-scope one: read from the kernel's own instructions (no GPU)."""
import glob
import re
import subprocess

import pytest

from paper_1606_08281_amd import lik
from paper_1606_08281_amd import workloads as W

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.parametrize("precision", [lik.FP64, lik.FP32_MIXED])
@pytest.mark.parametrize("model", ["telegraph", "lacgfp", "both"])
def test_every_store_of_the_flow_kernel_is_agent_scope(monkeypatch, tmp_path, model, precision):
    monkeypatch.setenv("LIK_KERNEL_CACHE", str(tmp_path))
    nets = [lik.Network(n.orders, n.stoich) for n in (W.telegraph(), W.lacgfp())]
    if model == "both":
        lik.precompile_requests(nets, precision)
    else:
        nets[model == "lacgfp"].precompile(precision)
    code, = glob.glob(str(tmp_path / "*.co"))
    text = subprocess.run([OBJDUMP, "-d", code], check=True, capture_output=True, text=True).stdout
    kernel, stores = None, []
    for line in text.splitlines():
        name = re.match(r"[0-9a-f]+ <(\w+)>:", line)
        kernel = name[1] if name else kernel
        if kernel and "flow" in kernel and re.search(r"\b(global|flat|buffer|scratch)_store", line):
            stores.append(line.split("//")[0].strip())
    assert len(stores) > 20
    assert not [s for s in stores if "sc1" not in s.split()]

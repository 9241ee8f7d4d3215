"""The scratch bytes behind the benchmark's training_scratch_gbps, from what the fused training step
stores (flow_train.hip): the operands of both hidden layers and a gradient per workgroup."""
import os
import re

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_fused_step_bytes():
    with open(os.path.join(ROOT, "paper_2302_05730_amd", "csrc", "flow_train.hip")) as f:
        source = f.read()
    with open(os.path.join(ROOT, "paper_2302_05730_amd", "csrc", "flow_mfma.h")) as f:
        layout = f.read()
    assert re.search(r"constexpr int H_OPS = G2K \+ G3K;", source)
    assert re.search(r"keep\[ks \* 64\] = h1\[ks\];", source)
    assert re.search(r"keep\[\(G2K \+ ks\) \* 64\] = h2\[ks\];", source)
    g2k, g3k = (int(re.search(rf"\b{n} = (\d+)", layout).group(1)) for n in ("G2K", "G3K"))
    blocks = int(re.search(r"kMaxBlocks = (\d+);", source).group(1))
    # an operand is 16 bytes in each of 64 lanes, of 32 samples
    per_layer = (g2k + g3k) * 16 * 64 // 32
    step, layers, params = 65536, 4, 67212
    assert bench.FLOW_FUSED_BYTES == 2 * layers * per_layer + 2 * blocks * params * 4 / step

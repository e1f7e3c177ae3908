"""Launch rules, on the CPU."""
from launch_rules import ask


def test_quantization_streams_large_inputs_only():
    # inputs that the kernel before has left in the caches lose by it below 64 MB
    short = [(64, 14336), (512, 8192), (2048, 3072), (16384, 256), (65535, 256)]
    assert ask(*(("quant_streams", m, k) for m, k in short)) == [[0]] * len(short)
    assert ask(("quant_streams", 65536, 256), ("quant_streams", 8192, 4096)) == [[1], [1]]

"""Launch rules, on the CPU."""
from launch_rules import ask


def test_quantization_streams_large_inputs_only():
    # inputs that the kernel before has left in the caches lose by it below 64 MB
    short = [(64, 14336), (512, 8192), (2048, 3072), (16384, 256), (65535, 256)]
    assert ask(*(("quant_streams", m, k) for m, k in short)) == [[0]] * len(short)
    assert ask(("quant_streams", 65536, 256), ("quant_streams", 8192, 4096)) == [[1], [1]]


def test_quantization_workgroups_cover_rows_and_fit_the_grid():
    # a grid holds 2^32 - 1 threads; one long matrix among many short rows must
    # not push a grouped launch past it that 256 threads per row keep
    rows = [1, 64, (1 << 23) - 1, 1 << 23, (1 << 23) + 1, (1 << 24) - 1]
    ks = [4, 2048, 2052, 4096, 4100, 8192, 8196, 16384, 16388, 32768, 32772, 174720]
    cases = [(m, k) for m in rows for k in ks]
    for (m, k), (threads, pieces) in zip(cases, ask(*(("quant_shape", m, k) for m, k in cases))):
        assert m * threads < 1 << 32, (m, k)
        assert pieces == 0 or 4 * threads * pieces >= k, (m, k)
        assert threads == (256 if k <= 8192 or m >= 1 << 23 else 512), (m, k)

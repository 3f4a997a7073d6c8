"""Device memory of gd_create: host code only, the HIP calls recorded in place
of made (no GPU)."""
import hip_stub


def test_memory_per_element_and_tensor(tmp_path):
    # what gd.h states, on either side of the direct form's limit (6,291,456
    # elements) and for numbers of tensors that keep one or several histogram copies;
    # 16 bytes an element, sample keys up to 2 more, tile descriptors and sums a tenth
    hip_stub.run("""
for n in (1, 600_000, 6_291_456, 6_291_457, 20_000_000):
    for tensors in (1, 30, 1024, 1025, 20_000):
        got, _ = create([n * t // tensors for t in range(tensors + 1)])
        assert got <= 18.2 * n + 135_700 * tensors + 65_536, (n, tensors, got)
""", tmp_path)

"""The build refuses a kernel that reserves scratch memory (no GPU needed)."""
import pytest

from paper_2401_11504_amd import build

PLAIN = "#include <hip/hip_runtime.h>\n__global__ void plain(float* p) { p[threadIdx.x] += 1.f; }\n"
INDEXED = """__global__ void indexed(float* p, int n) {
    float t[64];
    for (int i = 0; i < n; ++i) t[(int)p[i] & 63] = p[i];
    p[0] = t[n & 63];
}
"""


def test_no_kernel_reserves_scratch_memory(tmp_path, monkeypatch):
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "OUT", str(tmp_path / "lib.so"))
    build.build()


@pytest.mark.parametrize("source", [PLAIN, PLAIN + INDEXED])
def test_a_kernel_with_scratch_memory_fails_the_build(tmp_path, monkeypatch, source):
    (tmp_path / "k.hip").write_text(source)
    monkeypatch.setattr(build, "CSRC", str(tmp_path))
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "OUT", str(tmp_path / "k.so"))
    monkeypatch.setattr(build, "SOURCES", ["k.hip"])
    if source == PLAIN:
        build.build()
        return
    with pytest.raises(RuntimeError, match="indexed"):
        build.build()

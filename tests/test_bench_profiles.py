"""bench.py quotes a profile's HBM traffic only for the kernel source it was taken on."""
import os
import shutil

import bench


def test_a_profile_belongs_to_the_source_of_its_kernel(tmp_path, monkeypatch):
    kernels = ("k_gemm_rows", "k_gemm_batch_col", "k_gemm_mx", "k_gemm_split", "k_gemm_tile")
    base = {k: bench.source_hash(k) for k in kernels}
    csrc = tmp_path / "csrc"
    shutil.copytree(bench.CSRC, csrc)
    monkeypatch.setattr(bench, "CSRC", str(csrc))

    def changed(name, old, new):
        text = (csrc / name).read_text()
        assert old in text
        (csrc / name).write_text(text.replace(old, new, 1))
        diff = {k for k in kernels if bench.source_hash(k) != base[k]}
        (csrc / name).write_text(text)
        return diff

    assert changed("gemm_mx.hip", "constexpr int kPieces = 4;", "constexpr int kPieces = 3;") == {
        "k_gemm_mx"}
    assert changed("gemm_mfma.hip", "constexpr int kTileWaves = 4;",
                   "constexpr int kTileWaves = 8;") == {"k_gemm_split", "k_gemm_tile"}
    assert changed("shiftadd.hip", "constexpr int kThreads = 256;",
                   "constexpr int kThreads = 512;") == {"k_gemm_rows", "k_gemm_batch_col"}
    # comments and the host code that chooses a kernel do not change what it moves
    assert changed("shiftadd.hip", "double best = 0.93 *", "double best = 0.5 *") == set()
    assert changed("shiftadd.hip", "// ", "// other words: ") == set()


def test_the_headline_has_a_profile():
    assert os.path.exists(os.path.join(bench.PROFILES, "k_gemm_rows_llama2_7b_attn_l0_b1.md"))
    assert bench.measured_traffic("k_gemm_rows", "llama2_7b_attn", 0, 1)

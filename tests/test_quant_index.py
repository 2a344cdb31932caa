"""Sizes at which the MXFP8 quantiser's 32-bit thread index no longer covers its
byte offsets: the offset helpers and the launch rule of the kernel source,
compiled for the host, and on the GPU a Q^ of more than 4 GiB, whose last batch
must hold what the same rows give when they are quantised alone."""
import os
import re
import subprocess

import pytest
import torch

SRC = os.path.join(os.path.dirname(__file__), "..", "paper_2609_09721_amd", "csrc", "efq_attn.hip")


def _function(src, head):
    m = re.search(re.escape(head) + r"[^{]*\{.*?\}\n?", src, flags=re.S)
    assert m, head
    return m.group(0)


def test_offsets_and_launch_rule(tmp_path):
    src = open(SRC).read()
    code = _function(src, "__host__ __device__ __forceinline__ size_t q8_code_at(")
    scale = _function(src, "__host__ __device__ __forceinline__ size_t q8_scale_at(")
    fits = _function(src, "bool fits_launch(")
    # the kernel stores through the helpers, the merged launch asks the rule
    assert "y + q8_code_at(block, threadIdx.x)" in src and "y[a.soff + q8_scale_at(block, threadIdx.x)]" in src
    assert "!fits_launch(nv + nq + nk)" in src
    prog = tmp_path / "q8.cpp"
    prog.write_text("#include <cstddef>\n#include <initializer_list>\n"
                    "#define __host__\n#define __device__\n#define __forceinline__ inline\n"
                    + code + scale + fits + """
int main() {
  typedef unsigned long long u64;
  for (int D : {64, 128})   // thread n holds part n % (D / 8) of row n / (D / 8)
    for (unsigned block : {0u, 1u, 0x000fffffu, 0x001fffffu, 0x00200000u, 0x00200001u, 0x00fffffeu, 0x01ffffffu})
      for (unsigned t = 0; t < 256; ++t) {
        const u64 n = (u64)block * 256 + t, row = n / (D / 8), part = n % (D / 8);
        if (q8_code_at(block, t) != row * D + 8 * part) return 1;
        if (q8_scale_at(block, t) != row * (D / 32) + part / 4) return 2;
      }
  for (long n : {1L, 16384L, (1L << 24) - 1, 1L << 24, 1L << 25, 0x7fffffffL})
    if (fits_launch(n) != (n * 256 < (1L << 32))) return 3;
  return 0;
}
""")
    exe = tmp_path / "q8"
    subprocess.run(["g++", "-O1", "-o", str(exe), str(prog)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0


@pytest.mark.gpu
def test_codes_past_4_gib():
    from paper_2609_09721_amd import binding as B
    b, s, hq, D = 2, 131072, 160, 128                     # Q^ codes: 5 GiB
    print(f"[quant index] {(b, s, hq, D)}", flush=True)
    q = torch.empty((b, s, hq, D), dtype=torch.bfloat16, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(3)
    for i in range(b):
        for j in range(0, s, 16384):
            q[i, j: j + 16384] = torch.randn((16384, hq, D), generator=g, device="cuda", dtype=torch.bfloat16)
    k = torch.randn((b, s, 1, D), generator=g, device="cuda", dtype=torch.bfloat16)
    qh, _ = B.quant_qk(q, k)
    n = s * hq                                            # rows of one batch (s is a whole number of tiles)
    assert b * n * D > 1 << 32
    for i in range(b):
        one, _ = B.quant_qk(q[i: i + 1], k[i: i + 1])
        assert torch.equal(qh[i * n * D: (i + 1) * n * D], one[: n * D]), i
        at = b * n * D + i * n * (D // 32)                # the scales follow the codes, 256-byte aligned
        assert torch.equal(qh[at: at + n * (D // 32)], one[n * D: n * D + n * (D // 32)]), i
        del one

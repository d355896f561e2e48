"""The table region of the bin scheme's workspace holds what the fast transforms write there, at every length (CPU): the
plan and the table size of csrc/bins_fft.h, compiled for the host, against the counts of the kernels that fill the tables (m
phases, then L twiddles, or L / 4 twiddles and L / 2 + 1 points in Bluestein's form, all complex), and the workspace sizes
that callers have been given."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2307_12041_amd", "csrc")

PROGRAM = """
#include <cstdio>
#include "bins_fft.h"
int main() {
    for (int m = 1; m <= 16384; ++m) {
        const pp::BinFft f = pp::bin_fft_plan(m);
        printf("%d %d %d %zu\\n", m, f.L, (int)f.chirp, f.L > 0 ? pp::bin_fft_table_doubles(f) : (size_t)0);
    }
}
"""


def test_tables_fit_their_region(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    src, exe = tmp_path / "plan.hip", str(tmp_path / "plan")
    src.write_text(PROGRAM)
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", exe], check=True)
    for line in subprocess.run([exe], capture_output=True, text=True, check=True).stdout.splitlines():
        m, L, chirp, doubles = map(int, line.split())
        if L == 0:
            assert m > 4096 and m != 8192
            continue
        assert L & (L - 1) == 0 and (L >= max(8, 2 * m - 1) if chirp else L == m)
        assert doubles == 2 * (m + (L // 4 + L // 2 + 1 if chirp else L))
        assert m <= 2 or doubles <= 8 * m


@pytest.mark.parametrize("m", [1, 2, 3, 4, 31, 64, 100, 4095, 4097])
def test_workspace_sizes_stay(m):
    """256-byte regions of 8 m doubles of tables (the 16 and 18 of m = 1 and 2 fit the first 256 bytes), max(m Mp, 2 Mu m) of
    intermediates and n + 1 ints."""
    import paper_2307_12041_amd as pp

    def al(v):
        return (v + 255) // 256 * 256
    for n, Mu, Mp in ((0, 1, 1), (1000, m, max(1, m // 2)), (63, 1, m)):
        want = al(64 * m) + al(8 * max(m * Mp, 2 * Mu * m)) + al(4 * (n + 1))
        assert pp.bin_workspace_size(3.0, 2.0, n, m, Mu, Mp) == want


@pytest.mark.gpu
@pytest.mark.parametrize("m", [1, 2])
def test_one_and_two_bins(m):
    """The smallest lengths: sums of one and two terms per axis, written out.  Bar 1e-14: a handful of FP64 operations."""
    import numpy as np
    import torch

    import paper_2307_12041_amd as pp
    W, H = 3.0, 2.0
    rng = np.random.default_rng(m)
    P, a = rng.uniform(0.5, 1.5, (m, m)), rng.standard_normal((m, m))
    s, f = np.arange(m)[:, None], np.arange(m)[None, :]
    C, S = np.cos(f * (2 * s + 1) * np.pi / (2 * m)), np.sin(f * (2 * s + 1) * np.pi / (2 * m))   # [bin, frequency]
    got = pp.bin_coeffs(torch.as_tensor(P, device="cuda:0"), W=W, H=H, Mu=m, Mp=m).cpu().numpy()
    ref = np.zeros((m, m))
    if m == 2:
        u = np.pi / W, np.pi / H
        b = (W / 2, 2 * np.sin(u[0] * W / 4) / u[0]), (H / 2, 2 * np.sin(u[1] * H / 4) / u[1])   # a bin's cosine integrals
        R = C.T @ P @ C
        for i, j in ((0, 1), (1, 0), (1, 1)):
            e = (2 if i else 1) * (2 if j else 1) / (W * H * ((i * u[0]) ** 2 + (j * u[1]) ** 2))
            ref[i, j] = e * R[i, j] * b[0][i] * b[1][j]
    assert np.abs(got - ref).max() <= 1e-14 * max(1.0, np.abs(ref).max())
    fields = [t.cpu().numpy() for t in pp.bin_field(torch.as_tensor(a, device="cuda:0"), W=W, H=H, m=m)]
    wu, vp = np.arange(m) * np.pi / W, np.arange(m) * np.pi / H
    for g, r in zip(fields, (C @ a @ C.T, (S * wu) @ a @ C.T, C @ a @ (S * vp).T)):
        assert np.abs(g - r).max() <= 1e-14 * max(1.0, np.abs(r).max())

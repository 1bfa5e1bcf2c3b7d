"""The convolution background's LDS reads against what its launches ask for.

The vertical pass's sums run here on the host, compiled from the kernels' own
header, over buffers of exactly the launch's bytes that end at an inaccessible
page: any read past the allocation ends the program."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCE = r"""
#include <cstdio>
#include <sys/mman.h>
#include "k_convsum.h"
using namespace gpk;

// n bytes that end at an inaccessible page
static unsigned char* guarded(size_t n) {
    const size_t page = 4096, all = (n + page - 1) / page * page;
    unsigned char* p = (unsigned char*)mmap(nullptr, all + page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (p == MAP_FAILED || mprotect(p + all, page, PROT_NONE) != 0) abort();
    return p + all - n;
}

// 1: the sums of the last wavefront of a full tile stay inside the band (the
// data part of the allocation) and are those of the plain loop
template <typename Real>
static void vertical(int ly) {
    const int rows = kCvRows + cv_pad(ly);
    const size_t band_bytes = (size_t)rows * kCvCols * sizeof(Real);
    if (band_bytes > conv_v_data_bytes(ly, sizeof(Real) == 8) || band_bytes > conv_v_lds(ly, sizeof(Real) == 8)) abort();
    Real* band = (Real*)guarded(band_bytes);
    for (int i = 0; i < rows * kCvCols; ++i) band[i] = (Real)((i * 37) % 1009);
    double k[kConvTapsPad] = {0.0};
    for (int b = 0; b < ly; ++b) k[b] = 0.25 + (b * 7) % 13;
    for (int rb = 0; rb < kCvRows; rb += kCvN)
        for (int c = 0; c < kCvCols; c += 21) {
            double acc[kCvN];
            cv_sum16<false>(band + rb * kCvCols + c, k, ly, acc);
            for (int j = 0; j < kCvN; ++j) {
                double want = 0.0;
                for (int b = 0; b < ly; ++b) want = fma(k[b], (double)band[(rb + j + b) * kCvCols + c], want);
                if (want != acc[j]) { printf("vertical %d %d %d\n", ly, rb, j); exit(1); }
            }
        }
}

// 2: the same for a row segment
template <typename Real>
static void horizontal(int lx) {
    const size_t bytes = conv_h_lds<Real>();
    Real* row = (Real*)guarded(bytes);
    for (size_t i = 0; i < bytes / sizeof(Real); ++i) row[i] = (Real)(i % 911);
    double k[kConvTapsPad] = {0.0};
    for (int b = 0; b < lx; ++b) k[b] = 0.5 + (b * 5) % 11;
    for (int i0 = 0; i0 < kCvSeg; i0 += kCvN) {
        double acc[kCvN];
        cv_sum16<true>(row + cv_hpos<Real>(i0), k, lx, acc);
        for (int j = 0; j < kCvN; ++j) {
            double want = 0.0;
            for (int b = 0; b < lx; ++b) want = fma(k[b], (double)row[cv_hpos<Real>(i0 + j + b)], want);
            if (want != acc[j]) { printf("horizontal %d %d %d\n", lx, i0, j); exit(1); }
        }
    }
}

int main() {
    for (int t = 1; t <= 129; t += 2) {
        printf("taps %d\n", t);
        fflush(stdout);
        vertical<float>(t);
        vertical<double>(t);
        horizontal<float>(t);
        horizontal<double>(t);
    }
    printf("in bounds\n");
    return 0;
}
"""


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="needs hipcc to build the host program")
def test_convolution_sums_stay_in_their_lds(tmp_path):
    src, exe = tmp_path / "bounds.cpp", tmp_path / "bounds"
    src.write_text(SOURCE)
    hipcc = HIPCC if os.path.exists(HIPCC) else "hipcc"
    # -O0: no load whose value is unused is dropped
    cmd = [hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O0", "-ffp-contract=off",
           "-I", os.path.join(ROOT, "paper_2609_32375_amd", "csrc"), str(src), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and "in bounds" in r.stdout, (r.returncode, r.stdout[-200:])

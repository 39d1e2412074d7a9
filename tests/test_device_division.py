"""What the device compiler makes of a division by floats whose dividend is half of a 64-bit load: one conversion to floating
point, from 32 bits.  No kernel is launched."""
import os
import subprocess

import pytest

from paper_1711_01912_amd import build

KERNEL = """
#include <hip/hip_runtime.h>
#include "device_math.hpp"
using namespace cpeval;
// as the lane-window sweep does: entries are loaded ahead of the iteration that divides them
template <typename Word, typename Tab>
__global__ void probe(const uint2 *entries, const Tab *tab, Word *out, uint32_t *plain, int n) {
    const Tab up = round_up(Tab());
    __shared__ uint2 lds[4096];
    uint2 e[2];
    auto ask = [&](int at) {
        const uint2 *p = lds + at + threadIdx.x;
        e[0] = p[0];
        e[1] = p[64];
    };
    Word best = 0;
    uint32_t sum = 0;
    ask(0);
    for (int t = 0; t < n; ++t) {
        __syncthreads();
        const int items = plain[t];
        int i = threadIdx.x >> 6;
        if (i >= items) ask(t & 1023);
        while (i < items) {
            const uint2 now = e[0];
            const uint32_t x = e[1].y;
            const Word v = (Word)lds[e[1].x].x;
            i += 4;
            ask(i < items ? i : t & 1023);
            const Word q = add_quotient(v, x, tab[v & 63], up);
            sum += inverse_div(word_for<Tab>(now.y), tab[now.x], up);
            best = q > best ? q : best;
        }
    }
    out[threadIdx.x] = best;
    plain[threadIdx.x] = sum;
}
template __global__ void probe<uint32_t, float>(const uint2 *, const float *, uint32_t *, uint32_t *, int);
template __global__ void probe<unsigned long long, float>(const uint2 *, const float *, unsigned long long *, uint32_t *, int);
"""


def test_no_conversion_from_64_bits(tmp_path):
    source, listing = tmp_path / "probe.hip", tmp_path / "probe.s"
    source.write_text(KERNEL)
    r = subprocess.run([build._hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-I", build.CSRC, "-Xclang", "-target-feature",
                        "-Xclang", "-packed-fp32-ops", "-S", "--cuda-device-only", str(source), "-o", str(listing)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    text = listing.read_text()
    assert text.count(".amdhsa_kernel") == 2
    assert "v_cvt_f32_u32" in text
    assert "v_ldexp" not in text

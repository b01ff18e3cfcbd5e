"""The drafter's sigmoid and tanh (lstm_gate in fv_lstm_chain.hpp), compiled for the host from the header's own text and compared with
64-bit values.  The reciprocal, the one operation that a GPU rounds in its own way, is taken exactly rounded and one unit off either way."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2412_12639_amd import build

HARNESS = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#define __device__
#define __forceinline__ inline
static int off;
static float recip(float d) {
    float r = (float)(1.0 / (double)d);
    for (int i = 0; i < off; ++i) r = nextafterf(r, INFINITY);
    for (int i = 0; i > off; --i) r = nextafterf(r, 0.f);
    return r;
}
#define __builtin_amdgcn_rcpf recip
%s
static float f32(uint32_t b) { float f; memcpy(&f, &b, 4); return f; }
static uint32_t bits(float f) { uint32_t b; memcpy(&b, &f, 4); return b; }
static double worst[2][2];
static float place[2][2];
static long bad, n;
static void one(float x) {
    for (int th = 0; th < 2; ++th) {
        const double ref = th ? tanh((double)x) : 1.0 / (1.0 + exp(-(double)x));
        const float got = lstm_gate(x, th);
        const double err[2] = {fabs(got - ref), fabs(ref) >= 0x1p-126 ? fabs(got - ref) / fabs(ref) : 0.0};
        for (int k = 0; k < 2; ++k) if (!(err[k] <= worst[th][k])) { worst[th][k] = err[k]; place[th][k] = x; }
        if (!(fabsf(got) <= 1.f) || (th && x != 0.f && std::signbit(got) != std::signbit(x)) || (!th && got < 0.f)) ++bad;
        ++n;
    }
}
int main() {
    for (off = -1; off <= 1; ++off) {
        for (uint32_t b = 0; b < bits(INFINITY); b += b < bits(1e-6f) || b > bits(128.f) ? 65521 : 61) { one(f32(b)); one(-f32(b)); }
        for (float c : {0.5f, 0.55667f, 8.f, 9.0109f, 16.f, 17.3287f, 52.f, 87.3365f, 88.f, 103.28f, 104.f})   // the ends of the series, of the saturation and of the exponential
            for (uint32_t b = bits(c) - 40000; b < bits(c) + 40000; ++b) { one(f32(b)); one(-f32(b)); }
        for (uint32_t b = 0; b < 5000; ++b) { one(f32(b)); one(-f32(b)); }                                     // denormals
        if (lstm_gate(INFINITY, true) != 1.f || lstm_gate(-INFINITY, true) != -1.f || lstm_gate(INFINITY, false) != 1.f || lstm_gate(-INFINITY, false) != 0.f) ++bad;
        if (lstm_gate(NAN, true) == lstm_gate(NAN, true) || lstm_gate(NAN, false) == lstm_gate(NAN, false)) ++bad;
        if (lstm_gate(0.f, true) != 0.f || lstm_gate(0.f, false) != 0.5f) ++bad;
    }
    printf("%%ld %%ld %%.9e %%.9e %%.9e %%.9e %%.9g %%.9g %%.9g %%.9g\n", n, bad, worst[0][0], worst[0][1], worst[1][0], worst[1][1], place[0][0], place[0][1], place[1][0], place[1][1]);
}
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="no host compiler")
def test_gates_against_64_bits(tmp_path):
    """Results lie in [-1, 1] whatever comes in (the exchange of the hidden state relies on it), signs and specials are kept, and the errors
    stay below those of functions that err by 1.2 units: half a unit for the last rounding, and 0.7 for exponential and quotient together."""
    header = open(os.path.join(build.CSRC, "fv_lstm_chain.hpp")).read()
    function = re.search(r"^__device__ __forceinline__ float lstm_gate\(.*?^}\n", header, re.S | re.M).group(0)
    src, exe = tmp_path / "gate.cpp", tmp_path / "gate"
    src.write_text(HARNESS % function)
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()
    print(out)
    n, bad = int(out[0]), int(out[1])
    sig_abs, sig_rel, tanh_abs, tanh_rel = map(float, out[2:6])
    assert n > 10_000_000 and bad == 0
    unit = 2.0 ** -23
    assert sig_abs <= 0.6 * unit and tanh_abs <= 0.6 * unit     # below 1, a unit of the result is at most half of this
    assert sig_rel <= 1.2 * unit and tanh_rel <= 1.2 * unit

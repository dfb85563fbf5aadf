"""The double-double operations of csrc/dd.h, built for the host, against
113-bit arithmetic and against the forms with every operation renormalised
(accurate sums, three quotients): over random operands no operation may have a
larger mean error than those, and none a worst case above a few units of
2^-106 of the magnitudes that enter.  Sums must not depend on the order of
their two operands (partners of a wavefront reduction add the same two
values), or its lanes would hold different bits.
"""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1404_0812_amd", "csrc")

SOURCE = r"""
#include <cmath>
#include <cstdio>
#include <random>
#define __device__
#define __forceinline__ inline
// a hardware reciprocal has some 26 bits
static double dd_rcp(double q) { return (double)(1.0f / (float)q); }
#include "dd.h"
typedef __float128 Q;
static std::mt19937_64 rng(11);
static double uni() { return std::uniform_real_distribution<double>(-1, 1)(rng); }
static dd rnd() { const double h = uni(); return quick_two_sum(h, uni() * std::ldexp(std::fabs(h), -54)); }
static Q q(dd a) { return (Q)a.hi + (Q)a.lo; }
static Q ab(Q x) { return x < 0 ? -x : x; }
static dd full_dvd(dd a, dd b) {
    const double q1 = a.hi / b.hi;
    dd r = sub(a, mul_d(b, q1));
    const double q2 = r.hi / b.hi;
    r = sub(r, mul_d(b, q2));
    return add(quick_two_sum(q1, q2), mk(r.hi / b.hi));
}
struct Err {
    double sum = 0, top = 0;
    long n = 0;
    void put(Q got, Q want, Q mag) {
        const double e = (double)(ab(got - want) / mag) * std::ldexp(1.0, 106);
        sum += e; top = std::fmax(top, e); ++n;
    }
    void show(const char* name) const { std::printf("%s %.17g %.17g\n", name, sum / n, top); }
};
int main() {
    Err dn, df, mn, mf, sn, sf, tn, tf;
    int asym = 0;
    for (int i = 0; i < 400000; ++i) {
        const dd s = rnd(), a = rnd(), b = rnd(), c = rnd(), d = rnd();
        const double x = uni();
        if (std::fabs(b.hi) < 1e-3) continue;
        dn.put(q(dvd(a, b)), q(a) / q(b), ab(q(a) / q(b)));
        df.put(q(full_dvd(a, b)), q(a) / q(b), ab(q(a) / q(b)));
        const Q v = q(s) + q(a) * q(b) + q(c) * q(d), m = ab(q(s)) + ab(q(a) * q(b)) + ab(q(c) * q(d));
        mn.put(q(mac2(s, a, b, c, d)), v, m);
        mf.put(q(add(add(s, mul(a, b)), mul(c, d))), v, m);
        sn.put(q(sub_q(s, x, a)), (q(s) - (Q)x) - q(a), ab(q(s)) + ab((Q)x) + ab(q(a)));
        sf.put(q(sub(sub(s, mk(x)), a)), (q(s) - (Q)x) - q(a), ab(q(s)) + ab((Q)x) + ab(q(a)));
        const dd p = add(a, b), r = add(b, a);
        asym += p.hi != r.hi || p.lo != r.lo;
    }
    for (int i = 0; i < 40000; ++i) {
        dd n = mk(0.0), n2 = mk(0.0), f = mk(0.0);
        Q v = 0, m = 0;
        for (int k = 0; k < 16; ++k) {
            const dd a = rnd(), b = rnd(), c = rnd(), d = rnd();
            (k & 1 ? n2 : n) = mac2(k & 1 ? n2 : n, a, b, c, d);
            f = add(add(f, mul(a, b)), mul(c, d));
            v += q(a) * q(b) + q(c) * q(d);
            m += ab(q(a) * q(b)) + ab(q(c) * q(d));
        }
        tn.put(q(add(n, n2)), v, m);
        tf.put(q(f), v, m);
    }
    dn.show("dvd"); df.show("dvd_full");
    mn.show("mac2"); mf.show("mac2_full");
    sn.show("sub_q"); sf.show("sub_q_full");
    tn.show("dot"); tf.show("dot_full");
    std::printf("asym %d 0\n", asym);
}
"""


@pytest.fixture(scope="module")
def errors(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("dd")
    (d / "t.cpp").write_text(SOURCE)
    subprocess.run([cxx, "-O2", "-std=gnu++17", "-mfma", "-ffp-contract=off", "-w", "-I", CSRC, str(d / "t.cpp"), "-o",
                    str(d / "t")], check=True)
    out = subprocess.run([str(d / "t")], check=True, capture_output=True, text=True).stdout
    return {f[0]: (float(f[1]), float(f[2])) for f in (l.split() for l in out.splitlines())}


# worst cases: the rounding errors of each form added up, in units of 2^-106 of the magnitudes
@pytest.mark.parametrize("op,worst", [("dvd", 2.5), ("mac2", 5.0), ("sub_q", 4.0), ("dot", 5.0)])
def test_no_less_accurate_than_renormalised_forms(errors, op, worst):
    mean, top = errors[op]
    assert mean <= errors[op + "_full"][0], (op, mean, errors[op + "_full"])
    assert top <= worst, (op, top)


def test_sums_do_not_depend_on_order(errors):
    assert errors["asym"][0] == 0

"""The multiply-high divisions of the passes (MDiv of csrc/geo.hpp) against integer division, on
the CPU: the header and the transforms' radix table are compiled for the host.

div is exact while n d <= 2^24; every quotient that a pass forms with it is listed below with the
largest divisor and dividend that an accepted plan or tile gives.  The small grid's y' lines of one
to three points are dealt by div_any, which has to be exact for everything an LDS buffer
holds: there can be thousands of them (a decimated grid of 3 x 192 in blocks of 32 x').
"""
import os
import subprocess

import pytest

from paper_2503_13802_amd import build

SRC = r"""
#include "lines.hpp"
#include <algorithm>
#include <cstdio>
#include <vector>
using namespace mh3d;
static int pad_odd(int n) { return n | 1; }
static long bad = 0;
static void exact(const char* what, long d, long n) {   // [0, n) by div
  const MDiv v = make_mdiv((int)d);
  for (long i = 0; i < n; ++i)
    if (v.div((int)i) != i / d) { printf("%s: %ld / %ld = %d\n", what, i, d, v.div((int)i)); ++bad; return; }
}
static void exact_any(const char* what, long d, long n) {   // [0, n) by div_any
  const MDiv v = make_mdiv((int)d);
  for (long i = 0; i < n; ++i) {
    int r;
    const int q = v.div_any((int)i, r);
    if (q != i / d || r != i % d) { printf("%s: %ld / %ld = %d rem %d\n", what, i, d, q, r); ++bad; return; }
  }
}
// the dealing of nl lines of n points: butterflies of compiled stages, elements otherwise
static void lines(const char* what, int n, long nl, bool many = false) {
  const int r0 = line_radix(n, 0, false);
  if (n < 4 || !r0) {
    if (many) exact_any(what, nl, nl * n);
    else exact(what, nl, nl * n);
    return;
  }
  for (bool few : {false, true})
    for (int s = 0; s < 3; ++s)
      if (const int r = line_radix(n, s, few)) exact(what, nl, nl * (n / r));
}
int main() {
  std::vector<int> len;   // 2^a 3^b up to 256
  for (int n = 1; n <= 256; ++n) {
    int t = n;
    while (t % 2 == 0) t /= 2;
    while (t % 3 == 0) t /= 3;
    if (t == 1) len.push_back(n);
  }
  const long kLds = 160 * 1024 / 16;   // complex values of one of two buffers
  // small-grid passes: every decimated plane and x'-block that fits
  long small = 0, beyond = 0;
  for (int my : len)
    for (int mz : len)
      for (int xb = 1; xb <= 64; ++xb) {
        if (mz % 2 || !std::count(len.begin(), len.end(), xb)) continue;
        const long mzh = mz / 2 + 1, sp = (xb * my + 1) / 2;
        if (my + mz + 2 * std::max(sp * pad_odd(mz), xb * mzh * pad_odd(my)) > 2 * kLds) continue;
        ++small;
        const MDiv v = make_mdiv((int)(xb * mzh));
        bool ok = true;
        for (long i = 0; i < xb * mzh * my; ++i) ok = ok && v.div((int)i) == i / (xb * mzh);
        beyond += !ok;
        lines("y' lines", my, xb * mzh, true);
        lines("z' lines", mz, sp);
        const int mv = mz / (mz % 4 ? 2 : 4);
        exact("mz", mz, xb * my * mz);
        exact("vectors of mz", mv, xb * my * mv);
        exact("my", my, xb * my + 1);
        exact("xb", xb, my * mzh * xb);
        exact("mzh", mzh, std::max<long>(my, xb) * mzh);
      }
  // plane passes: ny x nz of up to three components at once, the rows of y residues
  for (int ny : len)
    for (int nz : len) {
      const long np = (ny + 1) / 2, nzh = nz / 2 + 1;
      if (nz % 2 || std::max(np * pad_odd(nz), nzh * pad_odd(ny)) > kLds) continue;
      const int nv = nz / (nz % 4 ? 2 : 4);
      for (int c = 1; c <= 3; ++c) {
        if (c * std::max(np * pad_odd(nz), nzh * pad_odd(ny)) > kLds) continue;
        lines("z lines", nz, c * np);
        lines("y lines", ny, c * nzh);
        exact("row vectors", nv, c * np * nv);
        exact("row pairs", np, c * np);
        for (int ps = 2; ps <= 4 && c == 1; ++ps)
          for (int more = 0; more < 2; ++more) {
            if (nzh / ps) lines("columns of a share", ny, nzh / ps + more);
            if (np / ps) lines("row pairs of a share", nz, np / ps + more);
          }
      }
      exact("nzh", nzh, ny * nzh);
      for (int mz : len)
        if (mz <= nz) { exact("mz of nz", mz, nzh); exact("mzh of classes", mz / 2 + 1, (long)ny * (mz / 2 + 1)); }
    }
  for (int sy = 1; sy <= 128; ++sy) exact("sy", sy, 256 * sy);
  // column passes: K harmonics in groups of any size that the LDS holds
  for (int mx : len) {
    if (mx < 2) continue;
    int cpc = 4;
    while (cpc * mx < 64 && cpc < 16) cpc *= 2;
    while (cpc * mx > 256 && cpc > 2) cpc /= 2;
    for (int kg = 1; kg <= 32 && kg * cpc * pad_odd(mx) <= kLds; ++kg) {
      lines("x' lines", mx, kg * cpc);
      exact("columns of harmonics", cpc * mx, (long)kg * cpc * mx);
      exact("q'x", mx, kg * cpc * mx);
      for (int xb : len)
        if (mx % xb == 0) { exact("runs of G", cpc * xb, cpc * mx); exact("x' of a run", xb, cpc * xb); }
    }
    for (int nx : len)
      if (nx % mx == 0) { lines("x lines", nx, cpc); exact("columns", cpc, cpc * nx); }
    exact("threads", mx, 1024);
    exact("threads per frequency", cpc * mx, 1025);
    for (int xb : len)
      if (mx % xb == 0) exact("x'-blocks", mx / xb, 32 * (mx / xb));
  }
  // class passes: 64 KiB (4096 complex values in one of two buffers)
  for (int W = 1; W <= 4096; ++W) {
    const int ls = 4096 / W;   // the longest line that W of them leave room for
    for (int n : len)
      if (n <= ls) {
        lines("lines of a class block", n, W);
        exact("elements of a class block", W, (long)W * n);
        exact("lines of a component", n, (long)W * n);
      }
  }
  printf("small-grid blocks %ld, %ld of them beyond div\n", small, beyond);
  if (!beyond) { printf("no block needs div_any: the list is incomplete\n"); ++bad; }
  return bad != 0;
}
"""


def test_every_divisor_over_its_range(tmp_path):
    src, exe = tmp_path / "divisors.hip", tmp_path / "divisors"
    src.write_text(SRC)
    csrc = os.path.join(build.PKG, "csrc")
    subprocess.run([build.HIPCC, "--cuda-host-only", "-O2", "-std=c++17", "-I" + csrc, str(src), "-o", str(exe)], check=True,
                   stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=300)
    run = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True, timeout=300)
    print(run.stdout)
    assert run.returncode == 0, run.stdout

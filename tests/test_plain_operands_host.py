"""The set-up's fast quotients and roots (csrc/lfdpr_device.h, compiled for the
host) are exact for operands and results in the middle of the binary32 range:
wherever plain_operands lets the view loop use them, every operand and result
lies there, for rigs and triangles across the whole range of scales."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

PROGRAM = r'''
#include "lfdpr_device.h"
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
using namespace lfdpr;
static long bad = 0;
static bool mid(float x, float lo, float hi) { return x >= lo && x <= hi; }
static void expect(bool ok, const char* what, float a, float b) {
  if (!ok && bad++ < 8) std::printf("%s: %g %g\n", what, a, b);
}
static void quotients(float a, float b, const char* what) {  // a >= 0
  expect((a == 0.0f || mid(a, 0x1p-100f, 0x1p100f)) && mid(b, 0x1p-100f, 0x1p100f) &&
             (a == 0.0f || mid(a / b, 0x1p-100f, 0x1p100f)), what, a, b);
}
int main() {
  std::mt19937_64 rng(11);
  auto U = [&](double lo, double hi) { return lo + (hi - lo) * (double)(rng() >> 11) * 0x1p-53; };
  long tris = 0, plain = 0, views = 0;
  for (int it = 0; it < 3000000; ++it) {
    Rig rg{};
    rg.W = 1 + (int)(rng() % 4096);
    rg.H = 1 + (int)(rng() % 4096);
    const double D = std::exp2(U(-33, 31)), fy = rg.H / 2.0 / std::tan(std::exp2(U(-30, 0.6)));
    rg.fy = (float)fy;
    rg.fx = (float)(fy * std::exp2((rng() & 1) ? 0.0 : U(-12, 12)));
    rg.fxfy = rg.fx * rg.fy;
    rg.cx = rg.W / 2.0f;
    rg.cy = rg.H / 2.0f;
    rg.rD = (float)(1.0 / D);
    const float b = (float)(D * std::exp2(U(-12, 10)) * ((rng() & 1) ? 1 : -1) * (rng() % 8 ? 1 : 0));
    rg.eye_lo = std::min(b, 0.0f);
    rg.eye_hi = std::max(b, 0.0f);
    // vertices in or around the view of eye b: x = cx + fx (X / Z) - b fx (1 / Z - 1 / D)
    float P[3][3];
    const double z0 = D * std::exp2(U(-8, 2)), size = std::exp2(U(-8, 14)), dz = std::exp2(U(-20, 1)), px0 = U(0, rg.W), py0 = U(0, rg.H);
    for (int k = 0; k < 3; ++k) {
      const double z = z0 * (1.0 + dz * U(0, 1));
      P[k][0] = (float)((px0 + size * U(-1, 1) - rg.cx) / rg.fx * z + b * (1.0 - z / D));
      P[k][1] = (float)((py0 + size * U(-1, 1) - rg.cy) / rg.fy * z);
      P[k][2] = (float)z;
    }
    F3 P0{P[0][0], P[0][1], P[0][2]}, P1{P[1][0], P[1][1], P[1][2]}, P2{P[2][0], P[2][1], P[2][2]};
    rg.znear = std::min(P0.z, std::min(P1.z, P2.z));
    F3 e1 = sub3(P1, P0), e2 = sub3(P2, P0);
    F3 n{e1.y * e2.z - e1.z * e2.y, e1.z * e2.x - e1.x * e2.z, e1.x * e2.y - e1.y * e2.x};
    const float nl = sqrtf((n.x * n.x + n.y * n.y) + n.z * n.z);
    if (!(nl > 0.0f) || std::isinf(nl)) continue;
    TriRec R{};
    R.nx = n.x / nl; R.ny = n.y / nl; R.nz = n.z / nl;
    R.p0x = P0.x; R.p0y = P0.y; R.p0z = P0.z;
    R.h = (R.nx * P0.x + R.ny * P0.y) + R.nz * P0.z;
    vertex_proj(rg, P0.x, P0.y, P0.z, R.a0, R.c0, R.y0);
    vertex_proj(rg, P1.x, P1.y, P1.z, R.a1, R.c1, R.y1);
    vertex_proj(rg, P2.x, P2.y, P2.z, R.a2, R.c2, R.y2);
    if (!may_be_seen(rg, R)) continue;
    ++tris;
    float far = fabsf(b);
    for (auto& v : P)
      for (float c : v) far = fmaxf(far, fabsf(c));
    if (!plain_operands(rg, rg.znear, far)) continue;
    ++plain;
    int32_t qx[3], qy[3];
    if (!view_active(rg, R, b, qx, qy)) continue;
    ++views;
    uint32_t odd = 0;
    const F3 e{b, 0.0f, 0.0f}, Ps = nearest_on_triangle<true>(e, P0, P1, P2, &odd), d = sub3(Ps, e);
    if (odd) continue;  // taken again with the plain operators
    const float delta = R.h - R.nx * b, ad = fabsf(delta), Zs = Ps.z;
    for (int axis = 0; axis < 2; ++axis) {
      const float c = axis ? R.ny : R.nx, g = c / delta;
      expect(mid(ad, 0x1p-100f, 0x1p100f), "delta", delta, 0.0f);
      if (fabsf(c) >= 0x1p-100f && fabsf(g) >= 0x1p-60f) quotients(fabsf(c), ad, "normal / delta");
      else expect(fabsf(g) * 0x1p32f <= 0x1p-26f, "small normal", c, g);  // far below one beside d, 2^32 at most
      const float vx = (axis ? 0.0f : 1.0f) - d.x * g, vy = (axis ? 1.0f : 0.0f) - d.y * g, vz = 0.0f - d.z * g;
      expect(mid((vx * vx + vy * vy) + vz * vz, 0x1p-90f, 0x1p90f), "root", vx, vz);
    }
    quotients(Zs, rg.fx, "depth / fx");
    quotients(Zs, rg.fy, "depth / fy");
    quotients((Zs * Zs) * Zs, rg.fxfy * ad, "depth^3 / (fx fy delta)");
  }
  std::printf("triangles %ld, plain %ld, views %ld, bad %ld\n", tris, plain, views, bad);
  return bad != 0 || views < 100000 || plain > tris * 95 / 100;
}
'''


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_plain_operands_bound_every_operand(tmp_path):
    src, exe = str(tmp_path / "plain.hip"), str(tmp_path / "plain")
    open(src, "w").write(PROGRAM)
    cmd = [HIPCC, "--offload-arch=gfx950", "-O2", "-std=c++17", "-ffp-contract=off", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2601_19901_amd", "csrc"), "-o", exe, src]
    subprocess.run(cmd, check=True, capture_output=True, timeout=600)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    print(out.stdout)
    assert out.returncode == 0, out.stdout + out.stderr

// Lays out the SVD's work areas of every shape as the library does and checks them: inside the doubles that
// svd_work_doubles asks for, apart from each other, and the ones accessed in 16-byte pairs aligned to that,
// whatever 8-byte boundary the block starts on.  Exit status 0 when all hold.
#include <cstdio>

#include "internal.h"

int main() {
  int bad = 0;
  long seen = 0;
  alignas(16) static double base[2];  // addresses only: nothing is read or written through them
  for (int m : {1, 2, 15, 31, 32, 33, 64, 65, 127, 130, 200, 255, 256, 257, 300, 331, 517, 1025, 4095, 4096})
    for (int n : {1, 2, 17, 32, 63, 64, 65, 97, 130, 201, 256, 259, 300, 331, 512, 1024, 4096})
      for (int batch : {1, 3, 64})
        for (int off = 0; off < 2; ++off) {
          tna::SvdMat a;
          if (tna::svd_plan_mat(m, n, TNA_F64, batch, &a, 0) != TNA_OK) return 2;
          double *const dw = base + off;
          int idum = 0;
          tna::svd_bind_work(&a, dw, &idum);
          const size_t pairs = a.nb / 2, R = a.R, C = a.C, qws = 2048 + 64 * C + 2 * R + 8 * 32 * C;
          struct Area {
            const char *name;
            double *p;
            size_t n;
            bool paired;
          } area[] = {{"gram", a.gram, pairs * a.ksplit * 4096, true}, {"qt", a.qt, pairs * 4096, true},
                      {"qws", a.qws, a.precond ? qws : 0, true},      {"qv", a.qv, a.precond ? R * R : 0, false},
                      {"bw", a.bw, R * C, false},                     {"jt", a.jt, R * R, false},
                      {"sig", a.sig, R, false},                       {"fro2", a.fro2, 2, false}};
          const uintptr_t lo = (uintptr_t)dw, hi = lo + sizeof(double) * tna::svd_work_doubles(a);
          for (const Area &x : area) {
            if (x.n == 0) continue;
            ++seen;
            const uintptr_t b = (uintptr_t)x.p, e = b + sizeof(double) * x.n;
            bool ok = b >= lo && e <= hi && b % (x.paired ? 16 : 8) == 0;
            for (const Area &y : area)
              if (&y != &x && y.n) ok = ok && (e <= (uintptr_t)y.p || (uintptr_t)(y.p + y.n) <= b);
            if (!ok && bad++ < 10) std::printf("%d x %d, batch %d, offset %d: %s\n", m, n, batch, off, x.name);
          }
        }
  std::printf("%ld areas, %d bad\n", seen, bad);
  return bad != 0;
}

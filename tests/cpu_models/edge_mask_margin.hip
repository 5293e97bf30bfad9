// edge_mask_margin.hip -- CPU check of the mesh fine pass's edge masks, with
// the kernel's own edge_mask (csrc/device.hpp) compiled for the host.
//
// A mask must keep every pixel that lies within the plain radius (sqrt(blur)
// and the exact test's own margin, edge_radius without slack) of the inner
// side of all three edge lines, evaluated in long double.  The hardware's
// reciprocal and root are modelled with an error of one unit in the last place
// either way, at random.  Triangles of many shapes and sizes over many image
// sizes; half of them have an edge line placed at the radius from one of the
// tile's pixels, to the resolution of their FP32 vertices.
//
//   edge_mask_margin TRIALS SHARE   the radius has SHARE of the slack that
//                                   edge_radius adds (1: the kernel's)
// Prints the pixels that had to be kept and the lost ones; exit status 1 if
// any was lost.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "../../paper_2007_08501_amd/csrc/device.hpp"

static std::mt19937_64 rng(20240807);
static double U() { return (double)(rng() >> 11) * 0x1p-53; }
static double Z() { return std::sqrt(-2.0 * std::log(U() + 1e-300)) * std::cos(6.283185307179586 * U()); }

struct HostMath {
    static float jitter(float v) {
        const int k = (int)(rng() % 3) - 1;
        return k == 0 ? v : std::nextafterf(v, k > 0 ? INFINITY : -INFINITY);
    }
    static float rcp(float x) { return jitter(1.0f / x); }
    static float sqrt(float x) { return jitter(sqrtf(x)); }
    static float med3(float x, float lo, float hi) { return fminf(fmaxf(x, lo), hi); }
};

int main(int argc, char** argv) {
    const long trials = argc > 1 ? atol(argv[1]) : 200000;
    const double share = argc > 2 ? atof(argv[2]) : 1.0;
    const int sizes[] = {1, 2, 3, 8, 17, 64, 130, 512, 1024, 4096};
    const float blurs[] = {0.0f, 1e-8f, 1e-6f, 1e-5f, 1e-4f, 1e-3f, 1e-2f, 0.3f};
    long must = 0, kept = 0, all = 0, lost = 0;
    for (long it = 0; it < trials; ++it) {
        const int W = sizes[rng() % 10], H = rng() % 2 ? W : sizes[rng() % 10];
        const float blur = blurs[rng() % 8];
        const float plain = rast::edge_radius(blur, H, W, 0.0f);
        const float full = rast::edge_radius(blur, H, W);
        const float rg = (float)((double)plain + share * ((double)full - (double)plain));
        const int x0 = 8 * (int)(U() * ((W + 7) / 8)), y0 = 8 * (int)(U() * ((H + 7) / 8));
        const double px = 1.0 - (double)(2 * x0 + 1) / W, py = 1.0 - (double)(2 * y0 + 1) / H;
        const int pr = (int)(8 * U()), pc = (int)(8 * U());
        const double qx = px - pc * 2.0 / W, qy = py - pr * 2.0 / H;  // a pixel of the tile
        const double size = std::pow(10.0, -4.0 + 5.0 * U()), th = 6.283185307179586 * U();
        float v[6];
        if (rng() % 2) {
            // an edge along th, the pixel `plain` outside it
            const int ax = (int)(rng() % 8);
            const double t = ax == 0 ? 0.0 : (ax == 1 ? 1.5707963267948966 : th);
            const double ux = std::cos(t), uy = std::sin(t), nx = -uy, ny = ux;
            const double back = size * U(), on = size * U(), in = size * std::pow(10.0, -2.0 * U());
            const double d = plain * (1.0 - 1e-7 * (U() - 0.5));
            v[0] = (float)(qx - back * ux + d * nx), v[1] = (float)(qy - back * uy + d * ny);
            v[2] = (float)(qx + on * ux + d * nx), v[3] = (float)(qy + on * uy + d * ny);
            const double s = size * (2.0 * U() - 1.0);
            v[4] = (float)(qx + s * ux + (d + in) * nx), v[5] = (float)(qy + s * uy + (d + in) * ny);
        } else {
            const double ax = qx + size * Z(), ay = qy + size * Z();
            v[0] = (float)ax, v[1] = (float)ay;
            switch (rng() % 4) {
                case 0:  // a sliver
                    v[2] = (float)(ax + size * std::cos(th)), v[3] = (float)(ay + size * std::sin(th));
                    v[4] = (float)(ax + 2 * size * std::cos(th) + 1e-4 * size * Z());
                    v[5] = (float)(ay + 2 * size * std::sin(th) + 1e-4 * size * Z());
                    break;
                case 1: {  // a short edge
                    const double t = std::pow(10.0, -6.0 + 4.0 * U());
                    v[2] = (float)(ax + t * Z()), v[3] = (float)(ay + t * Z());
                    v[4] = (float)(ax + size * Z()), v[5] = (float)(ay + size * Z());
                    break;
                }
                default:
                    for (int i = 2; i < 6; ++i) v[i] = (float)((i & 1 ? ay : ax) + size * Z());
            }
        }
        if (rng() % 2) std::swap(v[2], v[4]), std::swap(v[3], v[5]);  // the other orientation
        rast::EdgeGeo G;
        G.pa = make_double2(v[0], v[1]);
        G.ab = make_double2((double)v[2] - v[0], (double)v[3] - v[1]);
        G.ac = make_double2((double)v[4] - v[0], (double)v[5] - v[1]);
        G.E = G.ab.x * G.ac.y - G.ab.y * G.ac.x;
        if (std::fabs(G.E) < rast::kEpsArea) continue;
        const uint64_t m = rast::edge_mask<HostMath>(G, rg, px, py, 2.0f / (float)W, 2.0f / (float)H);
        const long double abx = G.ab.x, aby = G.ab.y, acx = G.ac.x, acy = G.ac.y, E = abx * acy - aby * acx;
        const long double sg = E > 0 ? 1 : -1, bcx = acx - abx, bcy = acy - aby;
        const long double l0 = sqrtl(bcx * bcx + bcy * bcy), l1 = sqrtl(acx * acx + acy * acy),
                          l2 = sqrtl(abx * abx + aby * aby);
        for (int r = 0; r < 8 && y0 + r < H; ++r)
            for (int c = 0; c < 8 && x0 + c < W; ++c) {
                const long double dx = 1.0L - (long double)(2 * (x0 + c) + 1) / W - G.pa.x;
                const long double dy = 1.0L - (long double)(2 * (y0 + r) + 1) / H - G.pa.y;
                const long double e1 = dx * acy - dy * acx, e2 = abx * dy - aby * dx, e0 = E - e1 - e2;
                const bool need = sg * e0 > -plain * l0 && sg * e1 > -plain * l1 && sg * e2 > -plain * l2;
                const bool k = (m >> (8 * r + c)) & 1;
                ++all;
                must += need;
                kept += k;
                if (need && !k && lost++ == 0)
                    std::printf("lost: %d x %d blur %g row %d column %d size %g\n", H, W, blur, r, c, size);
            }
    }
    std::printf("pixels %ld to keep %ld kept %ld lost %ld\n", all, must, kept, lost);
    return lost != 0;
}

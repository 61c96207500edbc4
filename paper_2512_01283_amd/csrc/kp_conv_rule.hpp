// kp_conv_rule.hpp -- the tile that a convolution takes (kp_conv.hip), without HIP,
// so that the rule can be checked on its own.
#pragma once
#include <cmath>
#include <initializer_list>

namespace kp {
namespace dn {

constexpr int CT_E = 18;  // halo columns (16 + 2)
constexpr int CT_CUS = 256;

// The tile (rows 32, 16 or 8; nt x 16 channels) with the least estimated time
// of its busiest CU: a step of 32 input channels costs 0.45 us whatever its
// size (its loads' latency, shared by the workgroups resident on a CU) and
// rows (0.004 + 0.0165 nt) us of MFMAs.  Fitted to 25 x 43 x 2 images, 192 ->
// 192 (us by rows 32 / 16 / 8: nt 4 18.1 / 12.3 / 8.7, nt 2 11.8 / 8.1 / 6.5,
// nt 1 8.9 / 6.9 / 6.9); 256^2 x 8, 144 -> 48, nt 3 67 / 73 / 85; 100 x 172 x 2,
// 144 -> 48, nt 3 14.6 / 12.0 / 11.5, nt 1 15.3 / 10.6 / 12.0.
inline void conv_tile_shape(int B, int H, int W, int cin, int nout, int& rows, int& nt) {
  double best = 1e30;
  const int t16 = nout / 16, nb = (cin + 31) / 32;
  for (int r : {32, 16, 8})
    for (int n : {4, 3, 2, 1}) {
      if (t16 % n) continue;
      const double items = (double)B * ((H + r - 1) / r) * ((W + 15) / 16) * (t16 / n);
      const int lds = 2 * 1024 * (((r + 2) * CT_E + 15) / 16 + 9 * n) + 2048, res = 160 * 1024 / lds;
      const double t = nb * (0.45 * std::ceil(items / (CT_CUS * res)) +
                             std::ceil(items / CT_CUS) * r * (0.004 + 0.0165 * n));
      if (t < best) {
        best = t;
        rows = r;
        nt = n;
      }
    }
}

}  // namespace dn
}  // namespace kp

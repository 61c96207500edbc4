// kp_rules.hpp -- the arithmetic of the run's host-side decisions, without HIP, so
// that it can be checked on its own.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace kp {

// Bytes that a buffer of `have` elements must find free before it can hold
// `need`: nothing, or, as it is replaced, all of the new one.
constexpr size_t grow_bytes(size_t need, size_t have, size_t elem) { return need > have ? need * elem : 0; }

// Near a point source every packet adds to the same few cells, and the L2 takes
// one addition to a line about every 37 ns: 1e6 packets leaving a grid vertex
// spend 4.6 ms on the eight cells around it.  The cells of an 8 x 8 x 8 box around
// the source (HOT_SIDE^3) are therefore tallied in HOT_COPIES copies behind the
// tally, one per group of wavefronts, and summed into it after the launch
// (k_hot_sum).  Transport: aligned slab, 3e6 packets 33.3 -> 17.7 ms; 45^3 disk,
// 1.9e6: 8.9 -> 2.7; 100^3 sphere, 3e6: 20.4 -> 15.6 (its 2.4e10 lines/s are the
// L2's limit); the 256^3 disk, whose hole surrounds the star, +1 %.
constexpr int HOT_SIDE = 8;
constexpr int HOT_CELLS = HOT_SIDE * HOT_SIDE * HOT_SIDE;
constexpr int HOT_COPIES = 32;                    // at most
constexpr size_t HOT_BYTES = size_t(16) << 20;    // of all copies and wavelengths together
constexpr uint64_t HOT_MIN_PACKETS = 1u << 15;    // fewer packets queue for less than the sum costs

// a cell's index along one axis of the box whose lowest cell is `low`; HOT_SIDE or
// more outside it, and for every cell where low is HOT_NONE (in unsigned numbers:
// the signed difference would overflow there)
constexpr int HOT_NONE = INT32_MIN;
constexpr uint32_t hot_index(int cell, int low) { return (uint32_t)cell - (uint32_t)low; }

// Copies of the cells around the source (HOT_COPIES) that a run takes: those it
// wants, or none where the tally of `tally` doubles would fit but not with
// `per_copy` more for each.  have: doubles allocated; other: bytes that the
// run's other buffers still need.  The copies only save time: they must
// never be why a run is refused, nor why a tally that is held is replaced
// without room for its successor.
constexpr int copies_that_fit(int copies, size_t tally, size_t per_copy, size_t have, size_t other, size_t free_b) {
  return grow_bytes(tally + (size_t)copies * per_copy, have, sizeof(double)) + other <= free_b ? copies : 0;
}

// Packets a wavefront holds: all lanes, or, of a run that does not fill the chip, an
// equal share of it for every wavefront of the blocks that run at a time (further
// blocks find nothing left to do: 3e5 packets in a 32^3 sphere with 64 blocks per CU
// asked for and 3 running took 4.6 ms with a share for each, 1.6 so).
constexpr int packets_per_wave(uint64_t total, uint64_t running_blocks, int waves_per_block) {
  const uint64_t waves = running_blocks * (uint64_t)waves_per_block, share = (total + waves - 1) / waves;
  return share < 64 ? (int)share : 64;
}

// Parked lanes from which a wavefront of `lanes` packets (`nactive` still under way,
// no ids left if `exhausted`) runs their scattering events together: that share of
// a full wavefront's setting.  With peel-off an event marches to every camera,
// once for all the lanes that run it together, and the setting stays as it is:
// aligned grains in a 32^3 sphere, one camera, 3e4 packets 2.9 ms, 4.7 with the
// share; 8 cameras, 17 and 38 ms; spheres, 3e4 packets, 1.6 and 2.7 ms.
constexpr int events_together(int batch, int lanes, int nactive, bool exhausted, bool peel) {
  return peel ? batch : batch * (exhausted ? nactive : lanes) >> 6;
}

// Pixel p of an npx x npy image in the order that the imaging wavefronts take them:
// bands of 16 rows, in them groups of 16 columns, in them 8 rows and 8 columns at a
// time, each row by row.  64 consecutive pixels are an 8 x 8 tile and 256 a 16 x 16
// one where the image has room for them, and no pixel is missing where not.
constexpr void image_pixel(uint32_t p, uint32_t npx, uint32_t npy, int& ix, int& iy) {
  const uint32_t band = p / (16u * npx);
  p -= band * 16u * npx;
  const uint32_t h = npy - 16u * band < 16u ? npy - 16u * band : 16u;
  const uint32_t group = p / (16u * h);
  p -= group * 16u * h;
  const uint32_t w = npx - 16u * group < 16u ? npx - 16u * group : 16u;
  const uint32_t row = p / (8u * w);
  p -= row * 8u * w;
  const uint32_t h8 = h - 8u * row < 8u ? h - 8u * row : 8u;
  const uint32_t col = p / (8u * h8);
  p -= col * 8u * h8;
  const uint32_t w8 = w - 8u * col < 8u ? w - 8u * col : 8u;
  iy = (int)(16u * band + 8u * row + p / w8);
  ix = (int)(16u * group + 8u * col + p % w8);
}

// A wavefront takes 64 pixels of one (wavelength, view) map, so that its camera and
// grain constants are scalars; where a map leaves more than 0.3 of its wavefronts'
// lanes without a pixel, it takes 64 pixels of any maps.  64^3 sphere / aligned
// grains, one map's pixels and any (us): 256 views x 32 wavelengths of 4 x 4 pixels
// 435 / 994 and 193 / 465, of 5 x 5 474 / 1015 and 322 / 832, of 9 x 9 859 / 1825 and
// 676 / 1809, of 8 x 8 591 / 1308 and 562 / 1490; 64 x 32 of 12 x 12 400 / 899 and 408 /
// 1015.
constexpr bool image_multi(uint64_t npix) { return 10u * npix < 7u * ((npix + 63u) / 64u * 64u); }
constexpr uint64_t image_waves(uint64_t npix, uint64_t maps) {
  return image_multi(npix) ? (maps * npix + 63u) / 64u : maps * ((npix + 63u) / 64u);
}

}  // namespace kp

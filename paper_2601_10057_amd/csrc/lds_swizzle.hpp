// Generated by gen_lds_swizzle.py; do not edit by hand.
//
// XOR layouts of the LDS lines of the transform kernels: element x of a
// buffer of lines lives at x ^ T(x >> B), T(h) = XOR of col[b] over the set
// bits b of h (B = 5 for 8-byte, 4 for 16-byte elements). Per table: the
// modelled LDS cycles per lane group over the class's accesses, with this
// layout and with the plain layout (ideal 1.0).
#pragma once

namespace ccm {

enum SwzClass { SWZ_ROW = 0, SWZ_LINE = 1, SWZ_GRAM = 2 };

template <int ESZ, int N, int CLS> struct SwzTab {
  static constexpr int NC = 0;
  static constexpr int col[1] = {0};
};

// 8-byte elements, N = 16, SWZ_ROW: 1.000 cycles/group (plain 3.022)
template <> struct SwzTab<8, 16, SWZ_ROW> {
  static constexpr int NC = 3;
  static constexpr int col[3] = {14, 1, 29};
};
// 8-byte elements, N = 32, SWZ_ROW: 1.000 cycles/group (plain 4.573)
template <> struct SwzTab<8, 32, SWZ_ROW> {
  static constexpr int NC = 4;
  static constexpr int col[4] = {31, 2, 17, 20};
};
// 8-byte elements, N = 64, SWZ_ROW: 1.061 cycles/group (plain 5.939)
template <> struct SwzTab<8, 64, SWZ_ROW> {
  static constexpr int NC = 5;
  static constexpr int col[5] = {11, 25, 7, 31, 21};
};
// 8-byte elements, N = 64, SWZ_LINE: 1.000 cycles/group (plain 1.773)
template <> struct SwzTab<8, 64, SWZ_LINE> {
  static constexpr int NC = 1;
  static constexpr int col[1] = {10};
};
// 8-byte elements, N = 64, SWZ_GRAM: 1.071 cycles/group (plain 1.786)
template <> struct SwzTab<8, 64, SWZ_GRAM> {
  static constexpr int NC = 1;
  static constexpr int col[1] = {31};
};
// 8-byte elements, N = 128, SWZ_ROW: 1.043 cycles/group (plain 7.234)
template <> struct SwzTab<8, 128, SWZ_ROW> {
  static constexpr int NC = 6;
  static constexpr int col[6] = {29, 27, 17, 2, 12, 12};
};
// 8-byte elements, N = 128, SWZ_LINE: 1.036 cycles/group (plain 2.929)
template <> struct SwzTab<8, 128, SWZ_LINE> {
  static constexpr int NC = 2;
  static constexpr int col[2] = {22, 26};
};
// 8-byte elements, N = 128, SWZ_GRAM: 1.031 cycles/group (plain 1.812)
template <> struct SwzTab<8, 128, SWZ_GRAM> {
  static constexpr int NC = 2;
  static constexpr int col[2] = {31, 17};
};
// 8-byte elements, N = 256, SWZ_ROW: 1.043 cycles/group (plain 9.522)
template <> struct SwzTab<8, 256, SWZ_ROW> {
  static constexpr int NC = 7;
  static constexpr int col[7] = {9, 20, 19, 17, 9, 2, 2};
};
// 8-byte elements, N = 256, SWZ_LINE: 1.050 cycles/group (plain 4.500)
template <> struct SwzTab<8, 256, SWZ_LINE> {
  static constexpr int NC = 3;
  static constexpr int col[3] = {11, 22, 19};
};
// 8-byte elements, N = 256, SWZ_GRAM: 1.050 cycles/group (plain 3.100)
template <> struct SwzTab<8, 256, SWZ_GRAM> {
  static constexpr int NC = 3;
  static constexpr int col[3] = {11, 22, 19};
};
// 8-byte elements, N = 512, SWZ_ROW: 1.034 cycles/group (plain 7.644)
template <> struct SwzTab<8, 512, SWZ_ROW> {
  static constexpr int NC = 8;
  static constexpr int col[8] = {23, 8, 3, 17, 4, 23, 1, 1};
};
// 8-byte elements, N = 512, SWZ_LINE: 1.062 cycles/group (plain 6.375)
template <> struct SwzTab<8, 512, SWZ_LINE> {
  static constexpr int NC = 4;
  static constexpr int col[4] = {4, 17, 2, 26};
};
// 8-byte elements, N = 512, SWZ_GRAM: 1.047 cycles/group (plain 4.375)
template <> struct SwzTab<8, 512, SWZ_GRAM> {
  static constexpr int NC = 4;
  static constexpr int col[4] = {1, 19, 12, 29};
};
// 8-byte elements, N = 1024, SWZ_ROW: 1.028 cycles/group (plain 7.644)
template <> struct SwzTab<8, 1024, SWZ_ROW> {
  static constexpr int NC = 9;
  static constexpr int col[9] = {27, 18, 3, 22, 23, 5, 27, 3, 3};
};
// 8-byte elements, N = 1024, SWZ_LINE: 1.055 cycles/group (plain 6.375)
template <> struct SwzTab<8, 1024, SWZ_LINE> {
  static constexpr int NC = 5;
  static constexpr int col[5] = {30, 3, 1, 20, 1};
};
// 8-byte elements, N = 1024, SWZ_GRAM: 1.044 cycles/group (plain 4.500)
template <> struct SwzTab<8, 1024, SWZ_GRAM> {
  static constexpr int NC = 5;
  static constexpr int col[5] = {17, 20, 11, 17, 21};
};
// 8-byte elements, N = 2048, SWZ_ROW: 1.032 cycles/group (plain 7.438)
template <> struct SwzTab<8, 2048, SWZ_ROW> {
  static constexpr int NC = 9;
  static constexpr int col[9] = {11, 7, 6, 20, 30, 8, 12, 7, 7};
};
// 8-byte elements, N = 2048, SWZ_LINE: 1.059 cycles/group (plain 6.375)
template <> struct SwzTab<8, 2048, SWZ_LINE> {
  static constexpr int NC = 6;
  static constexpr int col[6] = {13, 7, 6, 18, 12, 20};
};
// 8-byte elements, N = 2048, SWZ_GRAM: 1.047 cycles/group (plain 6.050)
template <> struct SwzTab<8, 2048, SWZ_GRAM> {
  static constexpr int NC = 6;
  static constexpr int col[6] = {25, 26, 23, 6, 16, 2};
};
// 8-byte elements, N = 4096, SWZ_ROW: 1.045 cycles/group (plain 7.324)
template <> struct SwzTab<8, 4096, SWZ_ROW> {
  static constexpr int NC = 9;
  static constexpr int col[9] = {21, 15, 27, 19, 24, 15, 1, 21, 21};
};
// 8-byte elements, N = 4096, SWZ_LINE: 1.060 cycles/group (plain 6.875)
template <> struct SwzTab<8, 4096, SWZ_LINE> {
  static constexpr int NC = 7;
  static constexpr int col[7] = {7, 19, 21, 26, 27, 29, 19};
};
// 8-byte elements, N = 4096, SWZ_GRAM: 1.023 cycles/group (plain 6.075)
template <> struct SwzTab<8, 4096, SWZ_GRAM> {
  static constexpr int NC = 7;
  static constexpr int col[7] = {27, 15, 30, 0, 24, 1, 27};
};
// 8-byte elements, N = 8192, SWZ_ROW: 1.043 cycles/group (plain 7.578)
template <> struct SwzTab<8, 8192, SWZ_ROW> {
  static constexpr int NC = 9;
  static constexpr int col[9] = {21, 29, 9, 19, 2, 9, 5, 29, 16};
};
// 8-byte elements, N = 8192, SWZ_LINE: 1.049 cycles/group (plain 6.475)
template <> struct SwzTab<8, 8192, SWZ_LINE> {
  static constexpr int NC = 8;
  static constexpr int col[8] = {2, 10, 31, 17, 6, 22, 2, 25};
};
// 8-byte elements, N = 8192, SWZ_GRAM: 1.048 cycles/group (plain 7.250)
template <> struct SwzTab<8, 8192, SWZ_GRAM> {
  static constexpr int NC = 8;
  static constexpr int col[8] = {15, 26, 4, 19, 5, 30, 4, 17};
};
// 16-byte elements, N = 16, SWZ_ROW: 1.000 cycles/group (plain 2.575)
template <> struct SwzTab<16, 16, SWZ_ROW> {
  static constexpr int NC = 3;
  static constexpr int col[3] = {10, 14, 9};
};
// 16-byte elements, N = 32, SWZ_ROW: 1.120 cycles/group (plain 3.580)
template <> struct SwzTab<16, 32, SWZ_ROW> {
  static constexpr int NC = 4;
  static constexpr int col[4] = {5, 9, 11, 8};
};
// 16-byte elements, N = 32, SWZ_LINE: 1.000 cycles/group (plain 1.643)
template <> struct SwzTab<16, 32, SWZ_LINE> {
  static constexpr int NC = 1;
  static constexpr int col[1] = {4};
};
// 16-byte elements, N = 32, SWZ_GRAM: 1.083 cycles/group (plain 1.750)
template <> struct SwzTab<16, 32, SWZ_GRAM> {
  static constexpr int NC = 1;
  static constexpr int col[1] = {15};
};
// 16-byte elements, N = 64, SWZ_ROW: 1.052 cycles/group (plain 4.583)
template <> struct SwzTab<16, 64, SWZ_ROW> {
  static constexpr int NC = 5;
  static constexpr int col[5] = {11, 14, 9, 0, 2};
};
// 16-byte elements, N = 64, SWZ_LINE: 1.050 cycles/group (plain 2.500)
template <> struct SwzTab<16, 64, SWZ_LINE> {
  static constexpr int NC = 2;
  static constexpr int col[2] = {5, 3};
};
// 16-byte elements, N = 64, SWZ_GRAM: 1.036 cycles/group (plain 1.786)
template <> struct SwzTab<16, 64, SWZ_GRAM> {
  static constexpr int NC = 2;
  static constexpr int col[2] = {15, 9};
};
// 16-byte elements, N = 128, SWZ_ROW: 1.042 cycles/group (plain 3.949)
template <> struct SwzTab<16, 128, SWZ_ROW> {
  static constexpr int NC = 6;
  static constexpr int col[6] = {7, 13, 9, 5, 9, 1};
};
// 16-byte elements, N = 128, SWZ_LINE: 1.062 cycles/group (plain 3.625)
template <> struct SwzTab<16, 128, SWZ_LINE> {
  static constexpr int NC = 3;
  static constexpr int col[3] = {6, 13, 9};
};
// 16-byte elements, N = 128, SWZ_GRAM: 1.031 cycles/group (plain 1.938)
template <> struct SwzTab<16, 128, SWZ_GRAM> {
  static constexpr int NC = 3;
  static constexpr int col[3] = {15, 1, 10};
};
// 16-byte elements, N = 256, SWZ_ROW: 1.038 cycles/group (plain 4.220)
template <> struct SwzTab<16, 256, SWZ_ROW> {
  static constexpr int NC = 7;
  static constexpr int col[7] = {1, 3, 12, 15, 3, 9, 3};
};
// 16-byte elements, N = 256, SWZ_LINE: 1.055 cycles/group (plain 3.625)
template <> struct SwzTab<16, 256, SWZ_LINE> {
  static constexpr int NC = 4;
  static constexpr int col[4] = {1, 3, 14, 12};
};
// 16-byte elements, N = 256, SWZ_GRAM: 1.050 cycles/group (plain 3.650)
template <> struct SwzTab<16, 256, SWZ_GRAM> {
  static constexpr int NC = 4;
  static constexpr int col[4] = {9, 14, 15, 13};
};
// 16-byte elements, N = 512, SWZ_ROW: 1.034 cycles/group (plain 4.254)
template <> struct SwzTab<16, 512, SWZ_ROW> {
  static constexpr int NC = 8;
  static constexpr int col[8] = {5, 1, 14, 3, 9, 15, 0, 5};
};
// 16-byte elements, N = 512, SWZ_LINE: 1.059 cycles/group (plain 3.875)
template <> struct SwzTab<16, 512, SWZ_LINE> {
  static constexpr int NC = 5;
  static constexpr int col[5] = {5, 2, 9, 14, 2};
};
// 16-byte elements, N = 512, SWZ_GRAM: 1.055 cycles/group (plain 3.875)
template <> struct SwzTab<16, 512, SWZ_GRAM> {
  static constexpr int NC = 5;
  static constexpr int col[5] = {7, 4, 9, 12, 2};
};
// 16-byte elements, N = 1024, SWZ_ROW: 1.031 cycles/group (plain 4.500)
template <> struct SwzTab<16, 1024, SWZ_ROW> {
  static constexpr int NC = 9;
  static constexpr int col[9] = {3, 2, 14, 15, 2, 5, 10, 11, 8};
};
// 16-byte elements, N = 1024, SWZ_LINE: 1.047 cycles/group (plain 3.675)
template <> struct SwzTab<16, 1024, SWZ_LINE> {
  static constexpr int NC = 6;
  static constexpr int col[6] = {11, 2, 13, 11, 15, 3};
};
// 16-byte elements, N = 1024, SWZ_GRAM: 1.047 cycles/group (plain 4.050)
template <> struct SwzTab<16, 1024, SWZ_GRAM> {
  static constexpr int NC = 6;
  static constexpr int col[6] = {3, 10, 12, 4, 15, 14};
};
// 16-byte elements, N = 2048, SWZ_ROW: 1.034 cycles/group (plain 4.808)
template <> struct SwzTab<16, 2048, SWZ_ROW> {
  static constexpr int NC = 9;
  static constexpr int col[9] = {9, 4, 11, 6, 1, 1, 2, 9, 1};
};
// 16-byte elements, N = 2048, SWZ_LINE: 1.036 cycles/group (plain 3.688)
template <> struct SwzTab<16, 2048, SWZ_LINE> {
  static constexpr int NC = 7;
  static constexpr int col[7] = {4, 13, 14, 13, 0, 10, 2};
};
// 16-byte elements, N = 2048, SWZ_GRAM: 1.023 cycles/group (plain 4.075)
template <> struct SwzTab<16, 2048, SWZ_GRAM> {
  static constexpr int NC = 7;
  static constexpr int col[7] = {4, 15, 13, 8, 0, 11, 2};
};
// 16-byte elements, N = 4096, SWZ_ROW: 1.033 cycles/group (plain 4.583)
template <> struct SwzTab<16, 4096, SWZ_ROW> {
  static constexpr int NC = 9;
  static constexpr int col[9] = {11, 13, 9, 7, 0, 11, 3, 1, 7};
};
// 16-byte elements, N = 4096, SWZ_LINE: 1.030 cycles/group (plain 3.694)
template <> struct SwzTab<16, 4096, SWZ_LINE> {
  static constexpr int NC = 8;
  static constexpr int col[8] = {15, 4, 9, 0, 0, 5, 7, 1};
};
// 16-byte elements, N = 4096, SWZ_GRAM: 1.012 cycles/group (plain 4.088)
template <> struct SwzTab<16, 4096, SWZ_GRAM> {
  static constexpr int NC = 8;
  static constexpr int col[8] = {10, 1, 13, 0, 0, 2, 4, 1};
};
// 16-byte elements, N = 8192, SWZ_ROW: 1.042 cycles/group (plain 3.894)
template <> struct SwzTab<16, 8192, SWZ_ROW> {
  static constexpr int NC = 9;
  static constexpr int col[9] = {11, 12, 14, 9, 9, 8, 11, 1, 14};
};
// 16-byte elements, N = 8192, SWZ_LINE: 1.034 cycles/group (plain 3.247)
template <> struct SwzTab<16, 8192, SWZ_LINE> {
  static constexpr int NC = 9;
  static constexpr int col[9] = {5, 10, 11, 11, 0, 15, 2, 6, 1};
};
// 16-byte elements, N = 8192, SWZ_GRAM: 1.026 cycles/group (plain 3.578)
template <> struct SwzTab<16, 8192, SWZ_GRAM> {
  static constexpr int NC = 9;
  static constexpr int col[9] = {2, 9, 14, 14, 0, 14, 2, 6, 1};
};

}  // namespace ccm

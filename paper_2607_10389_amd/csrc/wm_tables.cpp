// wm_tables.cpp -- host construction of the GF(2) shift tables.
//
// Everything here is derived from the polynomial: the one-bit register step
// Z (and its inverse), composed into byte shifts F^m by square-and-multiply
// over 32x32 GF(2) matrices stored as columns.
#include <cstring>

#include "wm_internal.h"

namespace wm {

namespace {

struct Mat {
  uint32_t c[32];
};

uint32_t apply(const Mat &m, uint32_t v) {
  uint32_t r = 0;
  for (int i = 0; i < 32; ++i)
    if ((v >> i) & 1u) r ^= m.c[i];
  return r;
}

// a after b
Mat compose(const Mat &a, const Mat &b) {
  Mat r;
  for (int i = 0; i < 32; ++i) r.c[i] = apply(a, b.c[i]);
  return r;
}

Mat identity() {
  Mat r;
  for (int i = 0; i < 32; ++i) r.c[i] = 1u << i;
  return r;
}

// One zero bit: Z(c) = (c >> 1) ^ (P & -(c & 1)).
Mat zero_bit(uint32_t poly) {
  Mat r;
  for (int i = 0; i < 32; ++i) {
    uint32_t c = 1u << i;
    r.c[i] = (c >> 1) ^ (poly & (0u - (c & 1u)));
  }
  return r;
}

// Inverse of Z.  Bit 31 of Z(c) equals bit 0 of c (P has bit 31 set and
// c >> 1 has it clear), so c = ((z ^ (P if bit) ) << 1) | bit.
Mat zero_bit_inverse(uint32_t poly) {
  Mat r;
  for (int i = 0; i < 32; ++i) {
    uint32_t z = 1u << i;
    uint32_t b0 = z >> 31;
    r.c[i] = ((z ^ (poly & (0u - b0))) << 1) | b0;
  }
  return r;
}

Mat power(Mat base, uint64_t e) {
  Mat r = identity();
  while (e) {
    if (e & 1) r = compose(base, r);
    base = compose(base, base);
    e >>= 1;
  }
  return r;
}

Mat byte_shift(uint32_t poly, int64_t m) {
  if (m >= 0) return power(power(zero_bit(poly), 8), (uint64_t)m);
  return power(power(zero_bit_inverse(poly), 8), (uint64_t)(-m));
}

void byte_tables(const Mat &m, uint32_t out[4][256]) {
  for (int j = 0; j < 4; ++j)
    for (uint32_t b = 0; b < 256; ++b) out[j][b] = apply(m, b << (8 * j));
}

// Tables of the matrix-core CRC.  A wave's row of 1 KiB is the A operand of
// four 32x32x64 products, one per bit plane: lane l holds 16 bytes, 32
// nibbles, and nibble e (dword e / 8) contributes its bit p.  The 32 rows of
// the product are the streams s = l % 32; the two halves l / 32, 512 bytes
// apart, and the nibbles are the 64 terms contracted with B, whose column n
// is bit n of the 32-bit CRC register.
void build_mc_tables(uint32_t poly, CrcTables *t) {
  // fp4 (e2m1) codes of the weights that make every product 0 or 1 (planes
  // 0..2, data elements 0.5, 1, 2) or +-0.5 (plane 3, data elements +-1)
  const uint32_t code[4] = {4u, 2u, 1u, 1u};  // 2, 1, 0.5, 0.5
  int k3[32] = {0};  // ones of plane 3's column n
  for (int h = 0; h < kRows; ++h)
    for (int half = 0; half < 2; ++half)
      for (int j = 0; j < 4; ++j) {
        const Mat m = byte_shift(poly, (int64_t)kRow * (kRows - 1 - h) + 512 * (1 - half) +
                                           4 * (3 - j) + 4);
        for (int b = 0; b < 32; ++b)
          for (int n = 0; n < 32; ++n)
            if ((m.c[b] >> n) & 1u) {
              t->mc_b[4 * h + (b & 3)][32 * half + n][j] |= code[b & 3] << (4 * (b >> 2));
              if ((b & 3) == 3) ++k3[n];
            }
      }
  for (int l = 0; l < 64; ++l) {
    // product register i of lane l: stream 8 (i / 4) + 4 (l / 32) + i % 4
    for (int i = 0; i < 16; ++i) {
      const int s = 8 * (i / 4) + 4 * (l / 32) + i % 4;
      t->mc_lane[i / 4][l][i % 4] = apply(byte_shift(poly, 16 * (31 - s)), 1u << (l % 32));
    }
    // starting at 1.5 * 2^22 keeps the sums in [2^22, 2^23), where a float's last bit is
    // one half and the bit above it the parity of the count; plane 3's
    // constant half-sum is taken off
    const float bias = 6291456.0f - 0.5f * (float)k3[l % 32];
    std::memcpy(&t->mc_bias[l], &bias, 4);
  }
  for (int l = 0; l < 64; ++l)  // bits 2l, 2l + 1: of word l / 16
    for (int i = 0; i < 2; ++i)
      t->mc_msg[l][i] = apply(byte_shift(poly, 16 - 4 * (l / 16)), 1u << (2 * (l % 16) + i));
  t->k_msg16 = apply(byte_shift(poly, 16), 0xFFFFFFFFu) ^ 0xFFFFFFFFu;
  t->k_msg12 = apply(byte_shift(poly, 12), 0xFFFFFFFFu) ^ 0xFFFFFFFFu;
  for (int w = 0; w < kWaves; ++w)
    std::memcpy(t->mc_wave[w], byte_shift(poly, (int64_t)kSub * (kWaves - 1 - w)).c,
                sizeof(t->mc_wave[w]));
}

}  // namespace

uint32_t poly_of(uint32_t crc_kind) {
  return crc_kind == 1 ? 0x82F63B78u : 0xEDB88320u;
}

void shift_matrix(uint32_t poly, int64_t m, uint32_t cols[32]) {
  Mat s = byte_shift(poly, m);
  std::memcpy(cols, s.c, sizeof(s.c));
}

uint32_t shift_apply(uint32_t poly, int64_t m, uint32_t v) {
  return apply(byte_shift(poly, m), v);
}

void build_crc_tables(uint32_t poly, CrcTables *t) {
  std::memset(t, 0, sizeof(*t));
  byte_tables(byte_shift(poly, kRow), t->row);
  byte_tables(byte_shift(poly, 4), t->f4);
  byte_tables(byte_shift(poly, 8), t->f8);
  byte_tables(byte_shift(poly, 12), t->f12);
  for (int l = 0; l < 64; ++l) {
    const Mat m = byte_shift(poly, 16 * (63 - l) + 4);
    for (int i = 0; i < 32; ++i) t->lane_mat[i / 4][l][i % 4] = m.c[i];
  }
  byte_tables(byte_shift(poly, kSub), t->wave_step);
  Mat one = byte_shift(poly, 1);
  for (uint32_t b = 0; b < 256; ++b) t->byte1[b] = apply(one, b);
  Mat p = byte_shift(poly, 1);
  for (int i = 0; i < 48; ++i) {
    std::memcpy(t->pow2[i], p.c, sizeof(p.c));
    p = compose(p, p);
  }
  t->k_full = apply(byte_shift(poly, kChunk), 0xFFFFFFFFu) ^ 0xFFFFFFFFu;
  build_mc_tables(poly, t);
}

WsLayout ws_layout(uint32_t n_chunks) {
  WsLayout L;
  uint64_t n = n_chunks ? n_chunks : 1;
  L.ctl = 0;
  L.status = 256;
  L.table = L.status + ((8 * n + 255) & ~255ull);
  L.entry_crc = L.table + ((16 * n + 255) & ~255ull);
  L.flags = L.entry_crc + ((4 * n + 255) & ~255ull);
  L.total = L.flags + ((4 * n + 255) & ~255ull);
  return L;
}

}  // namespace wm

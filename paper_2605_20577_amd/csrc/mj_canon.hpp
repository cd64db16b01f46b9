// Conversion between the packed structure-of-arrays state and the canonical
// per-environment record of include/mj.h, the hand query records, and the observations.
#pragma once
#include <cstddef>
#include "../../include/mj.h"
#include "mj_engine.hpp"
#include "mj_layout.hpp"

namespace mj {

// ------------------------------------------------------------------- records
// A canonical record is 250 words.  It is written and read in eight parts, so that the kernels can give each part of a
// group of games to a wavefront of its own; what a part holds is fixed here, once, for the kernels and for export_env /
// import_env, which go through the parts one after the other.  All loads of a part are issued before its stores.
constexpr int kRecParts = 8;
constexpr int kRecWords = (int)(sizeof(MjEnvCanon) / 4);
constexpr int kRecMeld = offsetof(MjEnvCanon, meld) / 4, kRecHist = offsetof(MjEnvCanon, hist) / 4, kRecWall = offsetof(MjEnvCanon, wall) / 4,
              kRecHand = offsetof(MjEnvCanon, hand), kRecRiver = offsetof(MjEnvCanon, river), kRecSeat = offsetof(MjEnvCanon, hand_red),
              kRecResult = offsetof(MjEnvCanon, han), kRecGlob = offsetof(MjEnvCanon, kyoku) / 4;
static_assert(offsetof(MjEnvCanon, waits) == 32 && offsetof(MjEnvCanon, mask) == 64 && offsetof(MjEnvCanon, yaku) == 128 &&
              offsetof(MjEnvCanon, score) == 160 && offsetof(MjEnvCanon, delta) == 176 && offsetof(MjEnvCanon, gain) == 192 &&
              offsetof(MjEnvCanon, episode) == 208 && offsetof(MjEnvCanon, kyoku_serial) == 212 && kRecMeld == 54 && kRecHist == 62 &&
              kRecWall == 126 && kRecSeat + 44 == kRecResult && kRecResult + 24 == 4 * kRecGlob && kRecGlob + 7 == kRecWords &&
              offsetof(MjEnvCanon, n_hist) == 999 && offsetof(MjEnvCanon, dora_pending) == 998, "record layout in words");
// array of the state behind row r of the record's leading 8-byte fields: discarded_kinds, waits, mask (arrays 0..15), yaku
MJ_HD int rec_u64_array(int r) { return r < 16 ? r : kHotU64 + (r - 16); }
// ... and behind row r of its 4-byte fields: score, delta (arrays 0..7), gain, episode, serial
MJ_HD int rec_u32_array(int r) { return r < 8 ? r : r < 12 ? kHotU32 + (r - 8) : r - 4; }

// part g of the record of a game whose every field is in HBM (make_env); the history is apart (record_hist_out)
MJ_HD void record_part_out(const Env &e, int g, uint32_t *rec)
{
  uint8_t *const bytes = (uint8_t *)rec;
  const int64_t n = e.n;
  const uint32_t last = e.glob[6 * n];                                   // ... wall_sel, hist_len
  const int s = g & 3;
  const uint32_t sw = e.seatw[s * n];
  const int nriv = (int)sw_get(sw, SW_NRIVER, 6);
  const uint64_t *q = e.dk;                                              // array 0, this game
  const uint32_t *w = (const uint32_t *)e.score;
  uint64_t v64[3];
  uint32_t v32[2], wall[5], hw[2], riv[16], gl = 0;
#pragma unroll
  for (int k = 0; k < 3; k++) { const int r = g + kRecParts * k; v64[k] = r < 20 ? q[(int64_t)rec_u64_array(r) * n] : 0ull; }
#pragma unroll
  for (int k = 0; k < 2; k++) { const int r = g + kRecParts * k; v32[k] = r < 14 ? w[(int64_t)rec_u32_array(r) * n] : 0u; }
  const uint64_t seat64 = g < 4 ? e.meld[s * n] : e.resw[s * n];
#pragma unroll
  for (int k = 0; k < 2; k++) hw[k] = e.hand[(int64_t)(s * 4 + 2 * (g >> 2) + k) * n];
  if (g < 7) gl = e.glob[g * n];
  const uint32_t gl3 = e.glob[3 * n];
#pragma unroll
  for (int k = 0; k < 16; k++) riv[k] = e.river[(int64_t)(s * 32 + 16 * (g >> 2) + k) * n];
  const uint32_t *wl = e.wallw + (int64_t)((last >> 16 & 1u) * 34) * n;
#pragma unroll
  for (int k = 0; k < 5; k++) { const int r = g + kRecParts * k; wall[k] = r < 34 ? wl[(int64_t)r * n] : 0u; }
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const int r = g + kRecParts * k;
    if (r >= 4 && r < 8) v64[k] &= K_ALL;                                // waits without the facts that ride in the upper bits
    if (r < 20) { rec[2 * r] = (uint32_t)v64[k]; rec[2 * r + 1] = (uint32_t)(v64[k] >> 32); }
  }
#pragma unroll
  for (int k = 0; k < 2; k++) { const int r = g + kRecParts * k; if (r < 14) rec[40 + r] = v32[k]; }
#pragma unroll
  for (int k = 0; k < 5; k++) { const int r = g + kRecParts * k; if (r < 34) rec[kRecWall + r] = wall[k]; }
  if (g < 4) {
    rec[kRecMeld + 2 * s] = (uint32_t)seat64; rec[kRecMeld + 2 * s + 1] = (uint32_t)(seat64 >> 32);
    uint8_t *b = bytes + kRecSeat + s;
    b[0] = (uint8_t)sw_get(sw, SW_RED, 3); b[4] = (uint8_t)sw_get(sw, SW_NMELD, 3); b[8] = (uint8_t)nriv;
    b[12] = (uint8_t)sw_get(sw, SW_RIDX, 8); b[16] = (uint8_t)sw_get(sw, SW_RIICHI, 2); b[20] = (uint8_t)sw_get(sw, SW_IPPATSU, 1);
    b[24] = (uint8_t)sw_get(sw, SW_FIRST, 1); b[28] = (uint8_t)sw_get(sw, SW_FTEMP, 1); b[32] = (uint8_t)sw_get(sw, SW_FRIICHI, 1);
    b[36] = (uint8_t)sw_get(sw, SW_KANBY, 3); b[40] = (uint8_t)sw_get(sw, SW_RANK, 2);
  } else {
#pragma unroll
    for (int j = 0; j < 6; j++) bytes[kRecResult + 4 * j + s] = (uint8_t)(seat64 >> (8 * j));
  }
  if (g < 7) {
    if (g == 3) gl = (gl & ~0xFE00u);                                    // kanflags: only "replacement tile" here ...
    if (g == 6) gl = (gl & 0xFF00FFFFu) | (gl3 >> 9 & 1u) << 16;         // ... and the waiting indicator in wall_sel's place
    rec[kRecGlob + g] = gl;
  }
  uint8_t *hb = bytes + kRecHand + 34 * s + 18 * (g >> 2);
#pragma unroll
  for (int r = 0; r < 18; r++) if (r < 16 || g < 4) hb[r] = (uint8_t)cnt3(hw[r / 9], r % 9);
  uint8_t *rb = bytes + kRecRiver + 32 * s + 16 * (g >> 2);
#pragma unroll
  for (int k = 0; k < 16; k++) rb[k] = 16 * (g >> 2) + k < nriv ? (uint8_t)riv[k] : (uint8_t)0;
}
// word i (entries 2 i and 2 i + 1) of the record's history
MJ_HD uint32_t record_hist_out(const Env &e, int i)
{
  const int nh = (int)(e.glob[6 * e.n] >> 24);
  const uint32_t x = row_word(e.hist, i);
  return (2 * i < nh ? x & 0xFFFFu : 0u) | (2 * i + 1 < nh ? x & 0xFFFF0000u : 0u);
}

MJ_HD void record_part_in(const Env &e, int g, const uint32_t *rec)
{
  const uint8_t *const bytes = (const uint8_t *)rec;
  const int64_t n = e.n;
  const int s = g & 3;
  uint64_t *q = e.dk;
  uint32_t *w = (uint32_t *)e.score;
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const int r = g + kRecParts * k;
    if (r < 20) q[(int64_t)rec_u64_array(r) * n] = (uint64_t)rec[2 * r] | (uint64_t)rec[2 * r + 1] << 32;
  }
#pragma unroll
  for (int k = 0; k < 2; k++) { const int r = g + kRecParts * k; if (r < 14) w[(int64_t)rec_u32_array(r) * n] = rec[40 + r]; }
#pragma unroll
  for (int k = 0; k < 5; k++) { const int r = g + kRecParts * k; if (r < 34) e.wallw[(int64_t)r * n] = rec[kRecWall + r]; }      // buffer 0
  if (g < 4) {
    e.meld[s * n] = (uint64_t)rec[kRecMeld + 2 * s] | (uint64_t)rec[kRecMeld + 2 * s + 1] << 32;
    const uint8_t *b = bytes + kRecSeat + s;
    uint32_t sw = 0;
    sw = sw_set(sw, SW_RED, 3, b[0] & 7u); sw = sw_set(sw, SW_NMELD, 3, b[4] & 7u); sw = sw_set(sw, SW_NRIVER, 6, b[8] & 63u);
    sw = sw_set(sw, SW_RIDX, 8, b[12]); sw = sw_set(sw, SW_RIICHI, 2, b[16] & 3u); sw = sw_set(sw, SW_IPPATSU, 1, b[20] & 1u);
    sw = sw_set(sw, SW_FIRST, 1, b[24] & 1u); sw = sw_set(sw, SW_FTEMP, 1, b[28] & 1u); sw = sw_set(sw, SW_FRIICHI, 1, b[32] & 1u);
    sw = sw_set(sw, SW_KANBY, 3, b[36] & 7u); sw = sw_set(sw, SW_RANK, 2, b[40] & 3u);
    e.seatw[s * n] = sw;
  } else {
    uint64_t rw = 0;
#pragma unroll
    for (int j = 0; j < 6; j++) rw |= (uint64_t)bytes[kRecResult + 4 * j + s] << (8 * j);
    e.resw[s * n] = rw;
  }
  if (g < 7) {
    uint32_t gl = rec[kRecGlob + g];
    if (g == 3) gl = (gl & ~0xFF00u) | (gl >> 8 & 1u) << 8 | (rec[kRecGlob + 6] >> 16 & 1u) << 9;
    if (g == 6) { const uint32_t nh = gl >> 24; gl = (gl & 0xFFFFu) | (nh > 128u ? 128u : nh) << 24; }      // wall_sel 0
    e.glob[g * n] = gl;
  } else {
    e.nserial[0] = 0xFFFFFFFFu;                      // whatever was made ahead of time is gone
    e.tdisc[0] = 0;                                  // ... and so is the cache of tenpai-keeping discards
  }
  const uint8_t *hb = bytes + kRecHand + 34 * s + 18 * (g >> 2);
  uint32_t hw[2] = {0, 0};
#pragma unroll
  for (int r = 0; r < 18; r++) if (r < 16 || g < 4) hw[r / 9] |= (uint32_t)(hb[r] & 7) << (3 * (r % 9));
#pragma unroll
  for (int k = 0; k < 2; k++) e.hand[(int64_t)(s * 4 + 2 * (g >> 2) + k) * n] = hw[k];
  const uint8_t *rb = bytes + kRecRiver + 32 * s + 16 * (g >> 2);
#pragma unroll
  for (int k = 0; k < 16; k++) e.river[(int64_t)(s * 32 + 16 * (g >> 2) + k) * n] = rb[k];
}
MJ_HD void record_hist_in(const Env &e, int i, uint32_t word) { set_row_word(e.hist, i, word); }

MJ_HD void export_env(const Env &e, MjEnvCanon &o)
{
  uint32_t rec[kRecWords];
  for (int g = 0; g < kRecParts; g++) record_part_out(e, g, rec);
  for (int i = 0; i < 64; i++) rec[kRecHist + i] = record_hist_out(e, i);
  __builtin_memcpy(&o, rec, sizeof o);
}
MJ_HD void import_env(const Env &e, const MjEnvCanon &o)
{
  uint32_t rec[kRecWords];
  __builtin_memcpy(rec, &o, sizeof o);
  for (int g = 0; g < kRecParts; g++) record_part_in(e, g, rec);
  for (int i = 0; i < 64; i++) record_hist_in(e, i, rec[kRecHist + i]);
}

// -------------------------------------------------------------- hand queries
// a query record as sixteen words, which stay in registers: every byte is read at a constant place
MJ_HD void read_query(const uint32_t w[16], HandIn &hi)
{
  static_assert(sizeof(MjHandQuery) == 64 && offsetof(MjHandQuery, meld) % 2 == 0 && sizeof(MjHandQuery::meld) == 8 &&
                sizeof(MjHandQuery::hand) == 34, "query record layout");
#define MJ_Q(at) (w[(at) >> 2] >> (8 * ((at) & 3)) & 255u)
#define MJ_QF(field) (int)MJ_Q(offsetof(MjHandQuery, field))
#pragma unroll
  for (int su = 0; su < 4; su++) {
    uint32_t hw = 0;
#pragma unroll
    for (int r = 0; r < (su == 3 ? 7 : 9); r++) {
      const uint32_t cnt = MJ_Q(offsetof(MjHandQuery, hand) + 9 * su + r);
      hw |= (cnt > 7 ? 7u : cnt) << (3 * r);
    }
    hi.h[su] = hw;
  }
  hi.meldw = 0;
#pragma unroll
  for (int j = 0; j < 8; j++) hi.meldw |= (uint64_t)MJ_Q(offsetof(MjHandQuery, meld) + j) << (8 * j);
  hi.n_meld = MJ_QF(n_meld); hi.win = MJ_QF(win_kind); hi.flags = MJ_QF(flags); hi.riichi = MJ_QF(riichi);
  hi.seat_wind = MJ_QF(seat_wind); hi.round_wind = MJ_QF(round_wind); hi.n_ind = MJ_QF(n_ind); hi.n_aka = MJ_QF(n_aka);
  hi.kuitan = MJ_QF(kuitan);
#pragma unroll
  for (int j = 0; j < 5; j++) {
    hi.ind[j] = (uint8_t)MJ_Q(offsetof(MjHandQuery, ind) + j); hi.ura[j] = (uint8_t)MJ_Q(offsetof(MjHandQuery, ura) + j);
  }
#undef MJ_QF
#undef MJ_Q
}
MJ_HD void hand_result(const HandOut &ho, MjHandResult &r)
{
  r.yaku = ho.yaku; r.points = ho.points; r.han = (uint8_t)ho.han; r.fu = (uint8_t)ho.fu;
  r.yakuman_units = (uint8_t)ho.units; r.shape_ok = (uint8_t)ho.shape_ok; r.yaku_ok = (uint8_t)ho.yaku_ok;
  r.n_dora = (uint8_t)ho.n_dora; r.n_ura = (uint8_t)ho.n_ura; r.n_aka = (uint8_t)ho.n_aka;
  r.pad_[0] = r.pad_[1] = r.pad_[2] = r.pad_[3] = 0;
}

// ---------------------------------------------------------------- observation
// 56 planes of 34 bits per viewer.  Per absolute seat: 14 masks (hand >= 1..4, river >= 1..4, meld >= 1..4,
// score thermometer, riichi plane); per environment: 9 masks (indicator >= 1..4, red visible, round wind,
// scalars, responded tile, dealer seat as a number).
enum { OB_HAND = 0, OB_RIVER = 4, OB_MELD = 8, OB_SCORE = 12, OB_RIICHI = 13, OB_SEAT_WORDS = 14 };
enum { OG_IND = 0, OG_REDVIS = 4, OG_ROUND = 5, OG_SCALARS = 6, OG_RESP = 7, OG_MISC = 8, OG_WORDS = 9 };

MJ_HD uint64_t ge_mask(const uint32_t w[4], int c)      // kinds whose packed count is >= c
{
  uint64_t m = 0;
#pragma unroll
  for (int su = 0; su < 4; su++) {
    uint32_t b0 = w[su] & O111, b1 = (w[su] >> 1) & O111, b2 = (w[su] >> 2) & O111, f;
    if (c == 1) f = b0 | b1 | b2;
    else if (c == 2) f = b1 | b2;
    else if (c == 3) f = (b0 & b1) | b2;
    else f = b2;
    m |= (uint64_t)squeeze9(f) << (9 * su);
  }
  return m & K_ALL;
}
MJ_HD void bump(uint32_t w[4], int k, int d) { int su = suit_of(k); w[su] += (uint32_t)d << (3 * rank_of(k, su)); }

// masks of absolute seat s; returns the red-five kinds this seat shows in river and melds
MJ_HD uint64_t obs_seat_masks(const Env &e, int s, uint64_t out[OB_SEAT_WORDS])
{
  const int64_t n = e.n;
  uint32_t sw = e.seatw[s * n];
  uint32_t h[4] = {e.hand[(s * 4) * n], e.hand[(s * 4 + 1) * n], e.hand[(s * 4 + 2) * n], e.hand[(s * 4 + 3) * n]};
  uint32_t rv[4] = {0, 0, 0, 0}, ml[4] = {0, 0, 0, 0};
  uint64_t redvis = 0;
  int nriv = (int)sw_get(sw, SW_NRIVER, 6);
  // the river bytes are one load each from rows B apart: issue them in groups of eight before using them
  for (int i0 = 0; i0 < nriv; i0 += 8) {
    int t[8];
#pragma unroll
    for (int j = 0; j < 8; j++) t[j] = (i0 + j < nriv) ? e.river[(s * 32 + i0 + j) * n] : 255;
#pragma unroll
    for (int j = 0; j < 8; j++) {
      if (t[j] == 255) continue;
      bump(rv, t[j] & 63, 1);
      if (t[j] & 64) redvis |= kbit(t[j] & 63);
    }
  }
  uint64_t mw = e.meld[s * n];
  int nm = (int)sw_get(sw, SW_NMELD, 3);
  for (int j = 0; j < nm; j++) {
    uint32_t m = meld_at(mw, j);
    int t = m_type(m), k = m_kind(m);
    if (t == MT_CHI) { bump(ml, k, 1); bump(ml, k + 1, 1); bump(ml, k + 2, 1); }
    else bump(ml, k, t == MT_PON ? 3 : 4);
    if (m >> 13 & 1) redvis |= kbit((k / 9) * 9 + 4);
  }
#pragma unroll
  for (int c = 1; c <= 4; c++) {
    out[OB_HAND + c - 1] = ge_mask(h, c);
    out[OB_RIVER + c - 1] = ge_mask(rv, c);
    out[OB_MELD + c - 1] = ge_mask(ml, c);
  }
  int32_t sc = e.score[s * n];
  int steps = sc < 2000 ? 0 : sc / 2000;
  out[OB_SCORE] = steps >= 34 ? K_ALL : (1ull << steps) - 1;
  out[OB_RIICHI] = sw_get(sw, SW_RIICHI, 2) ? K_ALL : 0;
  return redvis;
}

// the two words of the current wall that hold the dora indicators (wall positions 124..131; the indicators are 126..130)
MJ_HD void dora_words(const Env &e, int wall_sel, uint32_t dw[2])
{
  dw[0] = e.wallw[(int64_t)(wall_sel * 34 + 31) * e.n];
  dw[1] = e.wallw[(int64_t)(wall_sel * 34 + 32) * e.n];
}
MJ_HD void obs_env_masks(const Glob &g, uint32_t rule_flags, uint64_t seat_red, const uint32_t dw[2], uint64_t out[OG_WORDS])
{
  uint32_t ind[4] = {0, 0, 0, 0};
  uint64_t redvis = seat_red;
  for (int i = 0; i < g.n_dora; i++) {
    int id = (int)(dw[(i + 2) >> 2] >> (8 * ((i + 2) & 3)) & 255u);
    bump(ind, id >> 2, 1);
    if ((rule_flags & F_RED) && (id == 16 || id == 52 || id == 88)) redvis |= kbit(id >> 2);
  }
#pragma unroll
  for (int c = 1; c <= 4; c++) out[OG_IND + c - 1] = ge_mask(ind, c);
  out[OG_REDVIS] = redvis;
  out[OG_ROUND] = kbit(27 + (g.kyoku >> 2));
  int a = g.live_left / 4, hb = g.honba > 8 ? 8 : g.honba, ky = g.kyotaku > 8 ? 8 : g.kyotaku;
  out[OG_SCALARS] = ((1ull << a) - 1) | (((1ull << hb) - 1) << 18) | (((1ull << ky) - 1) << 26);
  uint64_t resp = 0;
  if (g.phase == PH_RESPOND) resp = kbit(code_kind(g.last_discard));
  if (g.phase == PH_RESPOND_KAKAN) resp = kbit(code_kind(g.kakan_tile));
  out[OG_RESP] = resp;
  uint64_t drawn = (g.phase == PH_TURN && g.drawn != 255) ? kbit(code_kind(g.drawn)) : 0;
  out[OG_MISC] = (uint64_t)(g.kyoku & 3) | (uint64_t)g.cur << 2 | drawn << 8;     // dealer, cur, drawn-kind bit
}

// plane p (0..55) as seen by `me`, from the per-seat masks S[4][OB_SEAT_WORDS], own red bits and the env masks
MJ_HD uint64_t obs_plane(int p, int me, const uint64_t *S, uint32_t own_red, const uint64_t *G)
{
  if (p < 4) return S[me * OB_SEAT_WORDS + OB_HAND + p];
  if (p == 4) return (own_red & 1 ? kbit(4) : 0) | (own_red & 2 ? kbit(13) : 0) | (own_red & 4 ? kbit(22) : 0);
  if (p < 21) { int q = p - 5; return S[((me + (q >> 2)) & 3) * OB_SEAT_WORDS + OB_RIVER + (q & 3)]; }
  if (p < 37) { int q = p - 21; return S[((me + (q >> 2)) & 3) * OB_SEAT_WORDS + OB_MELD + (q & 3)]; }
  if (p < 41) return G[OG_IND + p - 37];
  if (p == 41) return G[OG_REDVIS];
  if (p < 46) return S[((me + p - 42) & 3) * OB_SEAT_WORDS + OB_RIICHI];
  if (p == 46) return G[OG_ROUND];
  int dealer = (int)(G[OG_MISC] & 3), cur = (int)(G[OG_MISC] >> 2 & 3);
  if (p == 47) return kbit(27 + ((me - dealer) & 3));
  if (p == 48) return kbit((dealer - me) & 3);
  if (p < 53) return S[((me + p - 49) & 3) * OB_SEAT_WORDS + OB_SCORE];
  if (p == 53) return G[OG_SCALARS];
  if (p == 54) return G[OG_RESP];
  return cur == me ? (G[OG_MISC] >> 8) : 0;
}

// ------------------------------------------------------- token observation
// The record of a viewer (see MjTokenObs) is put together from four pieces, so that the kernel can compute what the
// four viewers of a game share only once: the viewer's own hand, the game's scalars, the seats' public words
// rotated to the viewer, and the rivers (token bytes by absolute seat, picked by relative seat on the way out).
MJ_HD uint8_t tile_token(int kind, int red) { return (uint8_t)(red ? 34 + (kind >= 9) + (kind >= 18) : kind); }
MJ_HD uint8_t river_token(int t) { return (uint8_t)(tile_token(t & 63, t >> 6 & 1) | (t & 0x80)); }
// own hand: tokens in ascending order (the red five first among the fives) and the shanten number
MJ_HD void tok_own(const Env &e, int me, const uint32_t *sh_suit, const uint32_t *sh_honor, MjTokenObs &o)
{
  const int64_t n = e.n;
  const uint32_t swm = e.seatw[me * n];
  uint32_t h[4];
  for (int su = 0; su < 4; su++) h[su] = e.hand[(me * 4 + su) * n];
  // fourteen slots in turn, every lane in step: k = the kind at hand, c = copies of it still to be written
  uint64_t left = 0;
  int tiles = 0;
  for (int su = 0; su < 4; su++) {
    const uint32_t w = h[su] & (su == 3 ? 0x1FFFFFu : 0x7FFFFFFu);
    left |= (uint64_t)squeeze9(fields_nonzero(w)) << (9 * su);
    tiles += tiles_in(w);
  }
  int k = 0, c = 0, red = 0;
#pragma unroll 1
  for (int i = 0; i < 14; i++) {
    if (c == 0 && left) {
      k = ctz64(left);
      left &= left - 1;
      c = hand_count(h, k);
      red = is_five(k) ? (int)(swm >> (k / 9) & 1u) : 0;
    }
    o.hand[i] = c ? tile_token(k, red) : (uint8_t)255;
    red = 0;
    c -= c ? 1 : 0;
  }
  o.n_hand = (uint8_t)tiles;
  o.shanten = (int8_t)shanten_of(sh_suit, sh_honor, h[0], h[1], h[2], h[3], (int)sw_get(swm, SW_NMELD, 3));
}
// the game's scalars as the viewer sees them
MJ_HD void tok_env(const Env &e, const Glob &g, int me, uint32_t rule_flags, MjTokenObs &o)
{
  o.drawn = (g.phase == PH_TURN && g.cur == me && g.drawn != 255) ? tile_token(code_kind(g.drawn), code_red(g.drawn)) : 255;
  o.phase = g.phase;
  o.cur = g.phase == PH_TURN ? (uint8_t)((g.cur - me) & 3) : 255;
  o.last_discarder = g.last_discarder == 255 ? 255 : (uint8_t)((g.last_discarder - me) & 3);
  o.last_discard = g.last_discard == 255 ? 255 : tile_token(code_kind(g.last_discard), code_red(g.last_discard));
  o.kyoku = g.kyoku; o.honba = g.honba; o.kyotaku = g.kyotaku;
  o.dealer = (uint8_t)(((g.kyoku & 3) - me) & 3);
  o.live_left = g.live_left; o.n_dora = g.n_dora;
  for (int i = 0; i < 5; i++) {
    const int id = wall_at(e, g.wall_sel, 126 + i);
    const bool red = (rule_flags & F_RED) && (id == 16 || id == 52 || id == 88);
    o.dora[i] = i < g.n_dora ? tile_token(id >> 2, red) : 255;
  }
}
// the four seats' public words (control word, points, melds; by absolute seat) rotated to the viewer
MJ_HD void tok_seats(const uint32_t sw[4], const int32_t score[4], const uint64_t meld[4], int me, MjTokenObs &o)
{
  for (int rel = 0; rel < 4; rel++) {
    const int s = (me + rel) & 3;
    const int nm = (int)sw_get(sw[s], SW_NMELD, 3);
    o.n_meld[rel] = (uint8_t)nm; o.n_river[rel] = (uint8_t)sw_get(sw[s], SW_NRIVER, 6);
    o.riichi[rel] = (uint8_t)sw_get(sw[s], SW_RIICHI, 2); o.riichi_idx[rel] = (uint8_t)sw_get(sw[s], SW_RIDX, 8);
    o.score[rel] = score[s];
    for (int j = 0; j < 4; j++) o.meld[rel][j] = j < nm ? (uint16_t)(meld[s] >> (16 * j)) : (uint16_t)0;
  }
}
// one seat's river as 32 token bytes
MJ_HD void tok_river(const Env &e, int s, uint8_t out[32])
{
  const int nriv = (int)sw_get(e.seatw[s * e.n], SW_NRIVER, 6);
  uint8_t t[32];
#pragma unroll
  for (int i = 0; i < 32; i++) t[i] = e.river[(int64_t)(s * 32 + i) * e.n];      // all 32 loads in flight together
#pragma unroll
  for (int i = 0; i < 32; i++) out[i] = i < nriv ? river_token(t[i]) : (uint8_t)255;
}
// one entry of the action history as viewer `me` sees it
MJ_HD uint16_t hist_token(uint32_t ev, int me) { return (uint16_t)((ev & 0xFFu) | (((ev >> 8) - (uint32_t)me) & 3u) << 8); }
// the whole record of viewer `me` (the plain composition; every field of the record is written)
MJ_HD void token_obs(const Env &e, const Glob &g, int me, uint32_t rule_flags, const uint32_t *sh_suit, const uint32_t *sh_honor,
                     MjTokenObs &o)
{
  uint32_t sw[4];
  int32_t score[4];
  uint64_t meld[4];
  for (int s = 0; s < 4; s++) { sw[s] = e.seatw[s * e.n]; score[s] = e.score[s * e.n]; meld[s] = e.meld[s * e.n]; }
  tok_own(e, me, sh_suit, sh_honor, o);
  tok_env(e, g, me, rule_flags, o);
  tok_seats(sw, score, meld, me, o);
  for (int rel = 0; rel < 4; rel++) tok_river(e, (me + rel) & 3, o.river[rel]);
  o.n_hist = g.hist_len;
  for (int i = 0; i < 15; i++) o.zero_[i] = 0;
  for (int i = 0; i < 128; i++)
    o.hist[i] = i < g.hist_len ? hist_token(e.hist[i], me) : (uint16_t)0xFFFF;
}

}  // namespace mj

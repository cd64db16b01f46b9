// Sanitizer driver of the TEST-ONLY host build of the kernels' per-environment code: rollouts of every game mode
// under three rule sets (the last one with every rule flag on), both observations, the record code of the export and
// import kernels, and all forms of the hand evaluator on the hands of the games and on arbitrary counts.  Built by
// tests/test_sanitizers.py with AddressSanitizer + UndefinedBehaviorSanitizer and, where clang offers it, with
// MemorySanitizer (uninitialised reads), once with every function inlined as in the kernels and once with every
// function out of line (-DSAN_OUT_OF_LINE).
#ifdef SAN_OUT_OF_LINE
#define MJ_HD inline __attribute__((noinline))
#endif
#include "../hostsim/hostsim.cpp"
#include <cstdio>
int main(int argc, char **argv)
{
  const int B = argc > 1 ? atoi(argv[1]) : 64, steps = argc > 2 ? atoi(argv[2]) : 1200;
  unsigned flagsets[3] = {1u | 2u | 4u | 8u, 4u | 8u, 511u};
  for (int f = 0; f < 3; f++)
    for (int mode = 0; mode < 3; mode++) {
      MjRules r;
      memset(&r, 0, sizeof r);
      r.flags = flagsets[f]; r.start_score = 25000; r.illegal_penalty = -1.0f; r.mode = (uint8_t)mode;
      Sim *h = hs_create(B, 5, &r);
      hs_step_random(h, steps, 1);
      std::vector<MjTokenObs> t((size_t)B * 4);
      std::vector<uint8_t> obs((size_t)B * 4 * 56 * 34);
      std::vector<MjEnvCanon> ex(B);
      hs_observe_tokens(h, t.data()); hs_observe(h, obs.data()); hs_export(h, 0, B, ex.data());
      hs_import(h, 0, B, ex.data());
      std::vector<MjHandQuery> q((size_t)B * 8);
      std::vector<MjHandResult> res(q.size());
      uint32_t x = 12345u + (uint32_t)f;
      for (size_t i = 0; i < q.size(); i++) {
        for (size_t k = 0; k < sizeof(MjHandQuery); k++) { x = x * 1664525u + 1013904223u; ((uint8_t *)&q[i])[k] = (uint8_t)(x >> 24); }
        for (int k = 0; k < 5; k++) { q[i].ind[k] %= 34; q[i].ura[k] %= 34; }
        q[i].seat_wind &= 3; q[i].round_wind &= 3; q[i].riichi %= 3;
        // every other one has any counts, any winning kind and no melds; the rest a seat's hand and melds, its lowest kind wins
        if (i & 1) { q[i].n_meld = 0; memset(q[i].meld, 0, 8); continue; }
        const MjEnvCanon &c = ex[i / 8];
        const int s = (int)(i / 2 & 3);
        memcpy(q[i].hand, c.hand[s], 34);
        memcpy(q[i].meld, c.meld[s], 8);
        q[i].n_meld = c.n_meld[s];
        q[i].win_kind = 0;
        while (q[i].win_kind < 33 && !q[i].hand[q[i].win_kind]) q[i].win_kind++;
        int total = 3 * q[i].n_meld;
        for (int k = 0; k < 34; k++) total += q[i].hand[k];
        if (total == 13) q[i].hand[q[i].win_kind]++;
      }
      for (int form = EVAL_STEP; form <= EVAL_BATCH; form++) hs_eval_hands(h, (int64_t)q.size(), q.data(), res.data(), form);
      hs_step_random(h, 200, 1);
      printf("host build flags %u mode %d ok, n_hist[0]=%d\n", r.flags, mode, t[0].n_hist);
      hs_destroy(h);
    }
  return 0;
}

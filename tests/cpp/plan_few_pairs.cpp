// The planner's checks (plan_check.cpp) on rounds of at most 4 (request, KV
// head) pairs, which have 64 or 128 state slots: every history call of the
// scenarios covers every token once, writes dense slots below the round's
// count and stays inside its chunks, through both ways of starting a round.
// Then the workgroup count of short shares: one per CU, or two where they span
// requests or all run the VALU body, and one of 128 tokens for each share of six
// to eight tiles where one spans requests.
#define main plan_check_main
#include "plan_check.cpp"
#undef main

int main() {
  std::mt19937 rng(5);
  for (int layout : {SS_KV_TOKEN_MAJOR, SS_KV_HEAD_MAJOR_KV}) {
    // 256 / Hkv workgroups per KV head while a share keeps 512 tokens
    scenario("1 x 131072, 2 KV heads (128 slots)", 1, 8, 2, {8}, {131072}, 8192, 0, layout, 16, 0, 0, 0, 128);
    scenario("1 x 32768, 4 KV heads (64 slots)", 1, 32, 4, {6}, {32768}, 4096, 0, layout, 8, 0, 0, 0, 64);
    scenario("1 x 20000, 4 KV heads (39 shares)", 1, 32, 4, {4}, {20000}, 4096, 0, layout, 8, 0, 0, 0, 39);
    scenario("1 x 16384, 4 KV heads (32 slots)", 1, 32, 4, {4}, {16384}, 4096, 0, layout, 8, 0, 0, 0, 32);
    // never fewer workgroups than 32 slots a request allow: two per CU for row-split units, shares of 128 tokens
    scenario("4 x 4400, 64 rows", 4, 8, 1, {8, 8, 8, 8}, {4400, 4400, 4400, 4400}, 4400, 0, layout, 1, 0, 0, 0, 69);
    scenario("4 x 4400, 24 rows", 4, 4, 1, {6, 6, 6, 6}, {4400, 4400, 4400, 4400}, 4400, 0, layout, 1, 0, 0, 0, 69);
    scenario("3 x 6000, 48 rows", 3, 8, 1, {6, 6, 6}, {6000, 6000, 6000}, 6000, 0, layout, 1, 0, 0, 0, 70);
    scenario("4 x 8192, 64 rows", 4, 8, 1, {8, 8, 8, 8}, {8192, 8192, 8192, 8192}, 4096, 0, layout, 2, 0, 0, 0, 128);
    scenario("4 x 32768, 64 rows", 4, 8, 1, {8, 8, 8, 8}, std::vector<int>(4, 32768), 8192, 0, layout, 4, 0, 0, 0, 256);
    scenario("4 x 70000, 1 KV head", 4, 8, 1, {8, 1, 3, 5}, {70000, 1, 40000, 33}, 9000, 0, layout, 8);
    scenario("1 x 400000, 1 KV head", 1, 8, 1, {8}, {400000}, 20000, 0, layout, 20);
    scenario("per-chunk calls", 1, 32, 4, {8}, {100000}, 40000, 0, layout, 1);
    scenario("caller's shares keep 32 slots", 1, 8, 2, {5}, {65536}, 4096, 512, layout, 16, 0, 0, -1, 32);
    scenario("8 x 4096 (1024 tokens a share)", 8, 32, 8, std::vector<int>(8, 6), std::vector<int>(8, 4096), 4096, 0, layout, 1, 0, 0, 0, 32);
    scenario("16 x 1000 (500 tokens a share)", 16, 32, 8, std::vector<int>(16, 6), std::vector<int>(16, 1000), 4096, 0, layout, 1, 0, 0, 0, 64);
    scenario("16 x 1024 (512 tokens a share)", 16, 32, 8, std::vector<int>(16, 6), std::vector<int>(16, 1024), 4096, 0, layout, 1, 0, 0, 0, 32);
    scenario("17 x 2000 (over half the shares span requests)", 17, 32, 8, std::vector<int>(17, 6), std::vector<int>(17, 2000), 4096, 0, layout, 1, 0, 0, 0, 64);
    scenario("8 x 8191, one row per KV head (VALU)", 8, 8, 8, std::vector<int>(8, 1), std::vector<int>(8, 8191), 8192, 0, layout, 1, 0, 0, 0, 64);
    scenario("8 x 8192, one row per KV head", 8, 8, 8, std::vector<int>(8, 1), std::vector<int>(8, 8192), 8192, 0, layout, 1, 0, 0, 0, 32);
    scenario("8 x 4096, one request on the VALU body", 8, 8, 8, {1, 6, 6, 6, 6, 6, 6, 6}, std::vector<int>(8, 4096), 4096, 0, layout, 1, 0, 0, 0, 32);
    scenario("8 x 4096, VALU but for a request without tokens", 8, 8, 8, {1, 1, 1, 1, 1, 1, 1, 8}, {4096, 4096, 4096, 4096, 4096, 4096, 4096, 0}, 4096, 0, layout, 1, 0, 0, 0, 64);
    scenario("3 x 2048 (192 tokens a share, some span requests)", 3, 32, 8, std::vector<int>(3, 6), std::vector<int>(3, 2048), 2048, 0, layout, 1, 0, 0, 0, 48);
    scenario("3 x 2037 (190 tokens a share)", 3, 32, 8, std::vector<int>(3, 6), std::vector<int>(3, 2037), 2048, 0, layout, 1, 0, 0, 0, 32);
    scenario("7 x 1165 (254 tokens a share, some span requests)", 7, 32, 8, std::vector<int>(7, 6), std::vector<int>(7, 1165), 2048, 0, layout, 1, 0, 0, 0, 63);
    scenario("3 x 2731 (256 tokens a share)", 3, 32, 8, std::vector<int>(3, 6), std::vector<int>(3, 2731), 4096, 0, layout, 1, 0, 0, 0, 32);
    scenario("4 x 1536 (192 tokens a share, none spans requests)", 4, 32, 8, std::vector<int>(4, 6), std::vector<int>(4, 1536), 2048, 0, layout, 1, 0, 0, 0, 32);
    scenario("2 x 3100, one without tokens between (none spans)", 3, 32, 8, std::vector<int>(3, 6), {3100, 0, 3100}, 4096, 0, layout, 1, 0, 0, 0, 32);
    scenario("2000 and 5000 tokens (one share spans requests)", 2, 32, 8, {6, 6}, {2000, 5000}, 8192, 0, layout, 1, 0, 0, 0, 28);
    scenario("4 x 4096, 64 rows (512 tokens a share)", 4, 64, 8, std::vector<int>(4, 8), std::vector<int>(4, 4096), 4096, 0, layout, 1, 0, 0, 0, 32);
    scenario("4 x 16383, 64 rows (2047 tokens a share)", 4, 64, 8, std::vector<int>(4, 8), std::vector<int>(4, 16383), 16384, 0, layout, 1, 0, 0, 0, 32);
    scenario("4 x 16384, 64 rows (2048 tokens a share)", 4, 64, 8, std::vector<int>(4, 8), std::vector<int>(4, 16384), 16384, 0, layout, 1, 0, 0, 0, 64);
    scenario("12 x 1000, 48 rows (375 tokens a share)", 12, 48, 8, std::vector<int>(12, 8), std::vector<int>(12, 1000), 1000, 0, layout, 1, 0, 0, 0, 32);
    scenario("17 x 1000, 48 rows (over half the shares span requests)", 17, 48, 8, std::vector<int>(17, 8), std::vector<int>(17, 1000), 1000, 0, layout, 1, 0, 0, 0, 64);
    // A workspace allocated for a larger cohort serves a smaller one, which asks for more slots than it holds.
    auto bytes_of = [](int B, int Hq, int Hkv, int n) {
      const std::vector<int> nc(B, n);
      ss_round_desc d{};
      d.num_requests = B; d.num_q_heads = Hq; d.num_kv_heads = Hkv; d.head_dim = 128; d.softmax_scale = 0.088f;
      d.num_cand = nc.data(); d.max_chunk_tokens = 1;
      return ss_round_workspace_bytes(&d);
    };
    g_ws_bytes = bytes_of(3, 16, 2, 8);
    CHECK(g_ws_bytes < bytes_of(2, 16, 2, 8) && g_ws_bytes < bytes_of(1, 16, 2, 8), "the smaller cohorts ask for more");
    scenario("2 x 65536, workspace of 3 requests (32 slots)", 2, 16, 2, {8, 8}, {65536, 65536}, 8192, 0, layout, 8, 0, 0, -1);
    scenario("1 x 65536, workspace of 3 requests (64 slots)", 1, 16, 2, {8}, {65536}, 8192, 0, layout, 8, 0, 0, 0, 64);
    scenario("1 x 65536 by chunk, workspace of 3 requests", 1, 16, 2, {8}, {65536}, 32768, 0, layout, 1);
    g_ws_bytes = bytes_of(5, 16, 2, 8);
    scenario("1 x 65536, workspace of 5 requests (128 slots)", 1, 16, 2, {8}, {65536}, 8192, 0, layout, 8, 0, 0, 0, 128);
    // One zero-filled workspace serves cohorts of other sizes and slot counts in turn: the counter block stays where
    // it is, outside every round's states (the calls have a balancing tail).
    g_ws_bytes = bytes_of(40, 32, 4, 4) + 100;
    scenario("16 x 65536, workspace of 40 requests", 16, 32, 4, std::vector<int>(16, 3), std::vector<int>(16, 65536), 4096, 0, layout, 32, 0, 0, 1);
    scenario("40 x 40000, workspace of 40 requests", 40, 32, 4, std::vector<int>(40, 4), std::vector<int>(40, 40000), 4096, 0, layout, 32, 0, 0, 1);
    scenario("5 x 400000, workspace of 40 requests", 5, 32, 4, {4, 1, 2, 3, 4}, std::vector<int>(5, 400000), 16384, 0, layout, 32, 0, 0, 1);
    g_ws_bytes = 0;
    for (int rep = 0; rep < 60; ++rep) {
      const int hkv = 1 + rng() % 4, B = 1 + rng() % (4 / hkv), G = 1 + rng() % 8;
      std::vector<int> nc(B), h(B);
      for (int b = 0; b < B; ++b) { nc[b] = 1 + rng() % 8; h[b] = (int)(rng() % (rep % 3 ? 90000 : 700)); }
      const int S = 32 * (1 + rng() % 512);
      int nch = 0;
      for (int x : h) nch = std::max(nch, (x + S - 1) / S);
      if (nch == 0 || nch > 2000) continue;
      scenario("random", B, G * hkv, hkv, nc, h, S, rng() % 4 ? 0 : 32 * (1 + rng() % 64), layout, 1 + rng() % 32);
    }
  }
  printf("%s\n", fails ? "FAILURES" : "all ok");
  return fails ? 1 : 0;
}

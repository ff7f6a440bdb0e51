// Driver of the dispatch rules on the host: the test splices the rules' source in front of this file.  One question a line on the
// standard input, one answer a line.
int main() {
  using namespace aqt;
  char what[64];
  while (scanf("%63s", what) == 1) {
    long v[6] = {};
    if (!strncmp(what, "attention", 9)) {   // utterances, frames, heads, head width, left, right
      for (long &x : v)
        if (scanf("%ld", &x) != 1) return 1;
      const AttnShape g{v[0], v[2] * v[3], (int)v[1], (int)v[2], (int)v[3], (int)v[4], (int)v[5], 0, 0.0f, 0.0f};
      printf("%d\n", !strcmp(what, "attention_few") ? attention_few_ok(g) : attention_bwd_few_ok(g));
    } else {   // rows, fan-in, columns; rows, width, whether in pieces of 16 bytes
      for (int i = 0; i < 3; ++i)
        if (scanf("%ld", v + i) != 1) return 1;
      printf("%d\n", !strcmp(what, "layernorm_blocks") ? layernorm_blocks(v[0], v[1], v[2]) : dense_fwd_rows_ok(v[0], v[1], v[2]));
    }
  }
  return 0;
}

"""Host-side checks of the index arithmetic in csrc/des_index.h: every element that a kernel requests, also the ones it then leaves
out, lies inside the array it was given.  No device is involved."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def walk(tmp_path, body):
    """Compiles and runs `body` (statements that call need(condition, values...))."""
    src = tmp_path / "walk.cpp"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include <initializer_list>\n#include "des_index.h"\nusing namespace des;\n'
                   "static void need(bool ok, long long a, long long b = 0, long long c = 0, long long d = 0) {\n"
                   '  if (!ok) { std::printf("%lld %lld %lld %lld\\n", a, b, c, d); std::exit(1); }\n}\n'
                   "int main() {\n" + body + "\n  return 0;\n}\n")
    exe = tmp_path / "walk"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-Wall", "-Wextra", "-Werror",
                           "-I", os.path.join(ROOT, "paper_1909_04823_amd", "csrc"), str(src), "-o", str(exe)])
    run = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert run.returncode == 0, run.stdout


def test_aggregation_requests_whole_aligned_columns(tmp_path):
    """P_sum[K][B][D] down to one sample of one shard: four floats from a multiple of four, inside the array, for all eight lanes."""
    walk(tmp_path, """
  for (int D = 4; D <= 256; D += 4)
    for (long long K = 1; K <= 5; ++K)
      for (long long B = 1; B <= 9; ++B)
        for (long long s = 0; s < K; ++s)
          for (long long b = 0; b < B; ++b)
            for (int sub = 0; sub < 8; ++sub) {
              const long long at = s * (B * D) + ahead_column(b, D, sub);
              need(at % 4 == 0 && at >= (s * B + b) * D && at + 4 <= (s * B + b + 1) * D, D, K, B, sub);
              if (sub < D / 4) need(at == (s * B + b) * D + sub * 4, D, K, B, sub);
            }""")


def test_entries_ahead_stay_in_the_batch(tmp_path):
    """Up to the largest batch, 2^31 - 2 entries: what lies ahead of an entry is the entry there or the last one, also where the sum
    does not fit 32 signed bits; and a loop over batches of entries ends."""
    walk(tmp_path, """
  const uint32_t most = 2147483646u;
  for (uint32_t n : {1u, 2u, 600u, 4097u, most - 1, most})
    for (uint32_t back = 1; back <= 1100 && back <= n; ++back) {
      const uint32_t i = n - back, last = n - 1;
      for (uint32_t ahead = 0; ahead <= 1024; ahead += ahead < 8 ? 1 : 31) {
        const long long want = (long long)i + ahead < last ? (long long)i + ahead : last;
        need(entry_ahead(i, ahead, last) == want, n, i, ahead, entry_ahead(i, ahead, last));
      }
    }""")

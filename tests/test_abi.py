"""The C-ABI library builds, loads, exports every symbol include/gptaq.h declares, and
rejects bad arguments on the host before anything is launched (no GPU needed)."""
import ctypes
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "gptaq.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(gptaq_[a-z0-9_]+)\s*\(", text)))


@pytest.fixture(scope="module")
def lib():
    from paper_2504_02692_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2504_02692_amd import build
        build.build(verbose=False)
    return binding.load()


def test_header_symbols_are_exported(lib):
    from paper_2504_02692_amd import binding
    names = declared_symbols()
    assert len(names) >= 9
    for name in names:
        assert hasattr(lib, name), name
    assert sorted(binding.EXPORTS) == names


def test_missing_library_fails_loudly(monkeypatch):
    from paper_2504_02692_amd import binding
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "LIB_PATH", "/nonexistent/libgptaq.so")
    with pytest.raises(binding.GptaqError):
        binding.load()


def test_workspace_queries(lib):
    assert lib.gptaq_accumulate_workspace_bytes(4096, 512) == 3 * 512 * 4096 * 2
    assert lib.gptaq_accumulate_workspace_bytes(262144, 4096) == 3 * 4096 * 32768 * 2
    assert lib.gptaq_accumulate_workspace_bytes(0, 512) == 0
    assert lib.gptaq_prepare_workspace_bytes(512) > 512 * 512 * 8
    # two sets of (-E / V of a super-block of 1024 columns, left operands of the updates inside it), the right operands
    # of one super-block for the block-by-block path, and the far right operands of every super-block that has columns
    # after it: 3072 + 2048 + 1024 rows and a 256-row tile of padding each at n = 4096, none at n = 512
    sets = lambda m: 2 * (4 * m * 1024 + 4 * (1024 // 16) * 1024 * 16) * 2
    assert lib.gptaq_quantize_workspace_bytes(512, 512) == sets(512) + 4 * (512 + 256) * 1024 * 2
    assert lib.gptaq_quantize_workspace_bytes(512, 4096) == sets(512) + 4 * (4096 + 256) * 1024 * 2 + 4 * (6144 + 3 * 256) * 1024 * 2
    assert lib.gptaq_status_string(0) == b"ok"


def test_a_workspace_for_more_tokens_has_room_for_fewer(lib):
    """Sums taken in parts of the tokens need room for the parts: more of it only with more tokens, so that the workspace of a series' largest
    call serves the others.  And where the rule's measurements lie: parts of 1024 columns and 2048 tokens and of 1280 columns from 4096 to
    16384, none where one form of the call is the slower for it."""
    size = lib.gptaq_accumulate_workspace_bytes
    operands = lambda tokens, n: 6 * -(-n // 128) * 128 * tokens
    for n in [8, 400, 512, 520, *range(576, 2060, 8)]:
        sizes = [size(tokens, n) for tokens in range(64, 32769, 64)]
        assert sizes == sorted(sizes), n
        assert all(s >= operands(64 * (i + 1), n) for i, s in enumerate(sizes))
    for n, tokens in [(1024, 2048), (1280, 4096), (1280, 8192), (1280, 12288), (640, 2048)]:
        assert size(tokens, n) > operands(tokens, n), (n, tokens)
    for n, tokens in [(1408, 6144), (1408, 8192), (1664, 6144), (1664, 8128), (1536, 16384), (1920, 32768), (640, 1024)]:
        assert size(tokens, n) == operands(tokens, n), (n, tokens)


def test_argument_errors_are_reported_before_any_launch(lib):
    one = ctypes.c_void_p(256)      # a non-null, aligned, never dereferenced address
    null = ctypes.c_void_p(0)
    for f in (lib.gptaq_accumulate, lib.gptaq_accumulate_upper):
        assert f(null, one, 64, 64, 64, one, one, 64, one, 1 << 20, null) == -1
        assert f(one, one, 64, 60, 64, one, one, 64, one, 1 << 20, null) == -2          # n % 8
        assert f(one, one, 64, 64, 32, one, one, 64, one, 1 << 20, null) == -2          # ldx < n
        assert f(one, one, 64, 64, 64, one, one, 64, one, 16, null) == -4               # workspace
        assert f(one, one, 64, 64, 64, one, one, 64, ctypes.c_void_p(264), 1 << 20, null) == -4
        assert f(one, one, 0, 64, 64, one, one, 64, one, 1 << 20, null) == 0            # empty chunk: no-op
    assert lib.gptaq_accumulate_upper_permuted(one, one, 64, 64, 64, null, one, one, 64, one, 1 << 20, null) == -1   # inv_perm
    assert lib.gptaq_accumulate_upper_permuted(one, one, 64, 60, 64, one, one, one, 64, one, 1 << 20, null) == -2
    assert lib.gptaq_accumulate_diag(null, 64, 64, 64, one, null) == -1
    assert lib.gptaq_accumulate_diag(one, 64, 64, 32, one, null) == -2                  # ldx < n
    assert lib.gptaq_accumulate_diag(one, 0, 64, 64, one, null) == 0
    assert lib.gptaq_invert_permutation(one, 0, one, null) == -2
    assert lib.gptaq_act_order(one, 64, 32, one, null) == -2                            # 0 < ldh < n
    big = 6 * 256 * 32768
    for g in (lib.gptaq_accumulate_staged, lib.gptaq_accumulate_staged_upper):
        pend = ctypes.c_int64(0)
        assert g(one, one, 64, 64, 64, one, one, 64, one, big, None, 0, null) == -1     # pending required
        assert g(one, one, 100, 64, 64, one, one, 64, one, big, ctypes.byref(pend), 0, null) == -2   # ragged, no flush
        assert g(one, one, 64, 64, 64, one, one, 64, one, 1 << 20, ctypes.byref(pend), 0, null) == -4
        pend.value = 32
        assert g(one, one, 64, 64, 64, one, one, 64, one, big, ctypes.byref(pend), 0, null) == -2    # pending % 64
        pend.value = 0
        assert g(null, null, 0, 64, 64, one, one, 64, one, big, ctypes.byref(pend), 1, null) == 0    # empty flush: no-op
        assert pend.value == 0
    p = lib.gptaq_prepare
    assert p(one, one, 64, 64, 0.01, null, null, one, 1 << 30, null) == -1          # info required
    assert p(one, one, 64, 32, 0.01, null, one, one, 1 << 30, null) == -2
    assert p(one, one, 64, 64, 0.01, null, one, one, 1024, null) == -4
    q = lib.gptaq_quantize_layer
    ok = (one, 64, 64, 64, one, one, 64, null)
    assert q(*ok, 1, 0, 0, 128, one, one, one, one, 1 << 30, null) == -3            # bits
    assert q(*ok, 4, 48, 0, 128, one, one, one, one, 1 << 30, null) == -3           # n % group
    assert q(*ok, 4, 32, 0, 48, one, one, one, one, 1 << 30, null) == -3            # blocksize % group
    assert q(*ok, 4, 0, 0, 256, one, one, one, one, 1 << 30, null) == -3            # blocksize > 128
    assert q(*ok, 4, 0, 0, 128, one, one, one, one, 16, null) == -4
    assert b"workspace" in lib.gptaq_status_string(-4)


def test_events_between_the_streams_release_what_they_order():
    """Results cross from one stream to the other through the L2s of eight XCDs, so an event that orders the two must be recorded
    with a release.  hipEventDisableSystemFence leaves it out (hip_runtime_api.h: for events that only take times)."""
    csrc = os.path.join(ROOT, "paper_2504_02692_amd", "csrc")
    flags = []
    for f in sorted(os.listdir(csrc)):
        if f.endswith((".hip", ".h")):
            code = re.sub(r"//[^\n]*", "", open(os.path.join(csrc, f)).read())
            flags += re.findall(r"hipEventCreateWithFlags\([^,]*,([^)]*)\)", code)
    assert [x.strip() for x in flags] == ["hipEventDisableTiming"]


def test_row_halves_have_rows(tmp_path):
    """Where the column loop takes a matrix as two row halves, the first is whole tiles of 256 rows and the second has rows: for every
    number of rows and super-blocks around the rule's lines, up to the most super-blocks that the column loop accepts."""
    src = tmp_path / "check.cpp"
    src.write_text("""#include "row_halves.h"
#include <cstdio>
int main() {
  long taken = 0, bad = 0;
  auto check = [&](int64_t m, int64_t nsb) {
    for (int terms = 0; terms < 4; ++terms)
      for (int clip = 0; clip < 2; ++clip) {
        const int64_t first = gptaq::first_row_half(m, nsb, terms, clip != 0);
        if (first == 0) continue;
        ++taken;
        if ((first < 1 || first >= m || first % 256 != 0) && bad++ == 0)
          std::printf("m %lld, super-blocks %lld: first half %lld rows\\n", (long long)m, (long long)nsb, (long long)first);
      }
  };
  for (int64_t m = 1; m <= 20000; ++m)
    for (int64_t nsb = 1; nsb <= 64; ++nsb) check(m, nsb);
  for (int64_t m = 1; m <= 2100; ++m)
    for (int64_t nsb = 65; nsb <= 16384; nsb = nsb * 9 / 8) check(m, nsb);
  if (!bad) std::printf("%ld\\n", taken);
  return bad != 0;
}
""")
    exe = tmp_path / "check"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2504_02692_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) > 1000000


def test_waits_end_and_wait_for_those_that_have_not_started(tmp_path):
    """A workgroup that waits for others of its launch does not give up while some of them have no place on the GPU yet, gives up when all
    have been running for a while, and ends in any case; what it reports then is no pivot's and no row's code."""
    from paper_2504_02692_amd import binding
    src = tmp_path / "check.cpp"
    src.write_text("""#include "gptaq.h"
#include "patience.h"
#include <cstdio>
using gptaq::Patience;
// spells until a wait ends whose team has started by the end of spell `from`
static int spells(int from) {
  Patience p;
  for (long polls = 1;; ++polls)
    if (p.over([&]() { return polls / Patience::kPolls >= from; })) return polls % Patience::kPolls ? -1 : (int)(polls / Patience::kPolls);
}
int main() {
  static_assert(Patience::kPolls >= 1 << 20 && Patience::kLongest >= 32, "a minute of other streams' kernels");
  Patience gap;                                    // (a counter that something else clears meanwhile)
  int flips = 0, asked = 0;
  while (!gap.over([&]() { ++asked; return flips++ % 2 == 0; })) {}
  std::printf("%d %d %d %d %d\\n", spells(1), spells(7), spells(1 << 20), asked, GPTAQ_INFO_STALLED);
}
""")
    exe = tmp_path / "check"
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2504_02692_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    str(src), "-o", str(exe)], check=True)
    longest = 64
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split() == [
        "2", "8", str(longest), str(longest), str(binding.INFO_STALLED)]
    assert not -65280 - 1 <= binding.INFO_STALLED <= 65280


def test_row_halves_where_they_are_the_faster(tmp_path):
    """The lines of the rule, both terms, no search: what has been measured on either side of them (against one chain up to 1024 rows and from 4097 on,
    against two between)."""
    src = tmp_path / "check.cpp"
    src.write_text("""#include "row_halves.h"
#include <cstdio>
#include <cstdlib>
int main(int argc, char** argv) {
  for (int i = 1; i + 1 < argc; i += 2) {
    const int64_t m = atoll(argv[i]), n = atoll(argv[i + 1]);
    std::printf("%d\\n", gptaq::first_row_half(m, (n + 1023) / 1024, 3, false) > 0);
  }
}
""")
    exe = tmp_path / "check"
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2504_02692_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    faster = [(9216, 3072), (4352, 4096), (6144, 4096), (5120, 5120), (900, 11008), (1024, 11008), (586, 14336), (1024, 14336), (513, 16384), (1024, 28672),
              (512, 53248), (1100, 9216), (1536, 9216), (1100, 11008), (1536, 11008), (1536, 14336), (1536, 16384)]
    slower = [(4096, 4096), (4096, 5120), (3584, 5248), (2048, 6144), (4096, 6144), (512, 8192), (1024, 8192), (1536, 8192), (3584, 8192), (4096, 8192), (1024, 9216),
              (1792, 9216), (820, 10240), (1792, 10240), (512, 11008), (2048, 11008), (3584, 11008), (4096, 11008), (400, 14336), (1664, 14336), (4096, 14336), (384, 16384),
              (2048, 16384), (2048, 28672)]
    out = subprocess.run([str(exe), *(str(x) for mn in faster + slower for x in mn)], check=True, capture_output=True, text=True).stdout.split()
    assert out == ["1"] * len(faster) + ["0"] * len(slower)

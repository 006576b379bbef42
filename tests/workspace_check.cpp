// Host check of the context's workspace (dst_workspace.h) with a counting
// allocator: prints "ok", or what failed.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>

#include "dst_workspace.h"

namespace {
std::map<void*, size_t> live;
size_t room = 1 << 20;  // bytes the allocator has
size_t used() {
  size_t n = 0;
  for (auto& kv : live) n += kv.second;
  return n;
}
bool take(void** p, size_t bytes) {
  if (used() + bytes > room) return false;
  *p = std::malloc(bytes);
  live[*p] = bytes;
  return true;
}
void give(void* p) {
  if (!live.erase(p)) std::abort();  // freed twice, or never allocated
  std::free(p);
}
int fail(const char* what) {
  std::printf("%s\n", what);
  return 1;
}
}  // namespace

int graph() {
  dst::Workspace w(take, give);
  w.begin(false);
  void* a = w.get("a", 1000);
  void* b = w.get("b", 1000);
  w.begin(true);  // the call under capture finds "a" and uses it
  if (w.get("a", 900) != a) return fail("a captured call moved a buffer that was large enough");
  w.begin(false);  // longer calls after it
  void* a2 = w.get("a", 5000);
  void* a3 = w.get("a", 9000);
  void* b2 = w.get("b", 5000);
  if (!live.count(a) || a2 == a || a3 == a) return fail("a buffer that a graph holds was freed or handed out again");
  if (live.size() != 3 || live.count(b2) != 1) return fail("buffers that no graph holds are freed when outgrown");
  w.begin(true);  // a second capture, of the longer call
  w.get("a", 9000);
  w.begin(false);
  void* a4 = w.get("a", 20000);
  if (!live.count(a) || !live.count(a3) || !live.count(a4)) return fail("each graph keeps its own buffer");
  if (w.held("a") != 20000 || w.held("none") != 0) return fail("held");
  // no room: a buffer in a graph stays as it was
  w.begin(true);
  if (w.get("a", 2 << 20) != nullptr || w.get("a", 20000) != a4) return fail("a growth that failed lost a graph's buffer");
  w.clear();
  if (!live.empty()) return fail("clear left something");
  (void)b;
  return 0;
}

int give_back() {
  dst::Workspace w(take, give);
  room = 10000;
  w.begin(false);
  w.get("records", 6000);
  w.get("small", 256);
  w.begin(true);
  w.get("graph", 1000);
  w.begin(false);  // a call that needs the records' room
  void* a = w.get("a", 2000);
  void* small = w.get("small", 256);
  void* b = w.get("b", 6000);
  if (!b) return fail("a buffer of an earlier call was not given back");
  if (!live.count(a) || !live.count(small) || w.held("graph") != 1000) return fail("a buffer in use was given back");
  if (w.held("records") != 0) return fail("a freed buffer is still held");
  if (w.get("c", 9000) != nullptr) return fail("no room: nullptr");
  if (!live.count(a) || !live.count(b)) return fail("the present call's buffers were given back");
  w.begin(false);
  if (!w.get("records", 6000) || w.held("b") != 0) return fail("and the other way round");
  w.begin(true);  // under capture nothing is freed
  if (w.get("d", 6000) != nullptr || w.held("records") != 6000) return fail("a captured call freed a buffer");
  w.clear();
  return live.empty() ? 0 : fail("clear left something");
}

int main(int argc, char** argv) {
  int rc = 1;
  if (argc == 2 && !std::strcmp(argv[1], "graph")) rc = graph();
  if (argc == 2 && !std::strcmp(argv[1], "give_back")) rc = give_back();
  if (rc == 0) std::printf("ok\n");
  return rc;
}

// Named device buffers of a context: grown on demand, kept from call to call.
// Host code only (the allocator is the caller's).
//
// A call made while its stream is captured leaves the addresses it was given in
// the caller's graph, and a replay writes there whenever it comes.  Such a
// buffer is never freed or moved before the context ends: when a later call
// needs more, it gets another one.
//
// What a call leaves in a buffer no later call reads, so buffers that the
// present call has not asked for are given back when memory runs out: a context
// that has binned a long timeline holds a gigabyte of records, and a solve after
// it may need that.
#pragma once

#include <cstddef>
#include <cstdint>
#include <string>
#include <unordered_map>
#include <vector>

namespace dst {

class Workspace {
 public:
  using Alloc = bool (*)(void** ptr, size_t bytes);
  using Free = void (*)(void* ptr);

  Workspace(Alloc alloc, Free release) : alloc_(alloc), free_(release) {}
  Workspace(const Workspace&) = delete;
  Workspace& operator=(const Workspace&) = delete;

  // Start of a call; captured: what it gets ends up in a graph.
  void begin(bool captured) {
    captured_ = captured;
    ++call_;
  }
  bool captured() const { return captured_; }
  // Times that memory ran out and buffers were given back.
  uint64_t given_back() const { return given_back_; }

  // Buffer `name` of at least `bytes`; nullptr, with nothing held under the
  // name, when it cannot be had (a buffer in a graph stays).
  void* get(const std::string& name, size_t bytes) {
    Buf& b = bufs_[name];
    if (b.bytes < bytes) {
      void* p = nullptr;
      if (captured_) {
        if (!alloc_(&p, bytes)) return nullptr;
        if (b.ptr) retired_.push_back(b.ptr);
      } else if (b.in_graph) {
        if (!alloc_(&p, bytes) && !(give_back() && alloc_(&p, bytes))) return nullptr;
        if (b.ptr) retired_.push_back(b.ptr);
      } else {
        drop(b);  // first, so that both need not fit
        if (!alloc_(&p, bytes) && !(give_back() && alloc_(&p, bytes))) return nullptr;
      }
      b = Buf{p, bytes, 0, false};
    }
    b.in_graph |= captured_;
    b.call = call_;
    return b.ptr;
  }

  // Bytes held under `name`.
  size_t held(const std::string& name) const {
    const auto it = bufs_.find(name);
    return it == bufs_.end() ? 0 : it->second.bytes;
  }

  // Frees buffer `name`, unless a graph holds it.
  void release(const std::string& name) {
    const auto it = bufs_.find(name);
    if (it != bufs_.end() && !it->second.in_graph) drop(it->second);
  }

  // End of the context: frees everything.
  void clear() {
    for (auto& kv : bufs_)
      if (kv.second.ptr) free_(kv.second.ptr);
    for (void* p : retired_) free_(p);
    bufs_.clear();
    retired_.clear();
  }

 private:
  struct Buf {
    void* ptr = nullptr;
    size_t bytes = 0;
    uint64_t call = 0;  // the last call that asked for it
    bool in_graph = false;
  };
  // Frees the buffers that no graph holds and the present call has not asked
  // for; whether there were any.
  bool give_back() {
    bool any = false;
    for (auto& kv : bufs_) {
      Buf& b = kv.second;
      if (!b.ptr || b.in_graph || b.call == call_) continue;
      drop(b);
      any = true;
    }
    given_back_ += any;
    return any;
  }
  void drop(Buf& b) {
    if (b.ptr) free_(b.ptr);
    b = Buf{};
  }

  Alloc alloc_;
  Free free_;
  bool captured_ = false;
  uint64_t call_ = 0, given_back_ = 0;
  std::unordered_map<std::string, Buf> bufs_;
  std::vector<void*> retired_;  // outgrown buffers that a graph holds
};

}  // namespace dst

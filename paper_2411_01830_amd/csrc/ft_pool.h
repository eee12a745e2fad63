// Host bookkeeping of the pooled GPU store (Sec. 7.1): segments of caller-owned
// device memory cut into slabs, first-fit runs, no device calls.
#pragma once
#include <stdint.h>
#include <deque>
#include <map>
#include <memory>
#include <vector>

namespace ft {

struct Segment {
  char *base;           // device pointer
  uint64_t bytes;
  uint64_t first_slab;  // index of its first slab in the logical space
  uint64_t nslabs;
};

struct Allocation {
  uint64_t nslabs;
  uint32_t busy;    // references by jobs not yet waited for
  uint64_t serial;  // tells this allocation from an earlier one in the same record; 0: the record is free
};

// A job's reference to an allocation. Records outlive their allocations (the pool hands them out again), so it may be looked at at
// any time: the serial says whether it is still that allocation.
struct Held {
  Allocation *al;
  uint64_t serial;
};

class SlabPool {
 public:
  // Argument rules of ft_pool_create; returns an FT_* code.
  static int check_segment(const void *base, uint64_t bytes, uint64_t slab_bytes);

  SlabPool(uint64_t slab_bytes) : slab_(slab_bytes) {}
  SlabPool(const SlabPool &) = delete;  // its records are pointed at
  SlabPool &operator=(const SlabPool &) = delete;
  int add_segment(void *base, uint64_t bytes);
  // Drops the last segment if no allocation lies in it (FT_EBUSY otherwise; FT_EINVAL if
  // it is the only one): the pool never shrinks below its first segment.
  int drop_last_segment(void **base_out, uint64_t *bytes_out);
  uint64_t live_bytes() const;
  int alloc(uint64_t nbytes, uint64_t *off_out);
  // FT_EBUSY while a job that has not been waited for refers to the allocation, unless `ordered`:
  // then the caller vouches that whatever reuses the slabs is ordered after those jobs on the device.
  int free(uint64_t off, bool ordered = false);
  Allocation *at(uint64_t start);
  // A live allocation: its bytes [start, end) of the pool, and the device address of its first one.
  struct Entry {
    uint64_t start, end, dev;
    Allocation *al;
  };
  // Where in the index an answer lay; valid while nothing is allocated or freed.
  struct Place {
    uint32_t block = 0, pos = 0;
  };
  Place begin() const { return Place(); }
  // The live allocation containing [off, off + extent), or nullptr. For callers that ask for one allocation after another, mostly in
  // ascending order: `near` is where the last answer lay (begin() at first), and the one behind it is looked at before the
  // index is searched.
  const Entry *find(uint64_t off, uint64_t extent, Place *near) const {
    const Entry *e = entry(*near);
    if (e != nullptr && off >= e->end) {
      const Place next = near->pos + 1 < blocks_[near->block]->n ? Place{near->block, near->pos + 1} : Place{near->block + 1, 0};
      e = entry(next);
      if (e != nullptr && holds(*e, off)) *near = next;
    }
    if (e == nullptr || !holds(*e, off)) {
      if (!last_at_or_before(off, near)) return nullptr;
      e = entry(*near);
      if (!holds(*e, off)) return nullptr;
    }
    return extent <= e->end - off ? e : nullptr;  // allocations do not overlap: no other one holds `off`
  }
  // The allocation behind the one at `near`, which then is the one at `near`; nullptr: none.
  const Entry *step(Place *near) const {
    if (near->block >= blocks_.size()) return nullptr;
    *near = near->pos + 1 < blocks_[near->block]->n ? Place{near->block, near->pos + 1} : Place{near->block + 1, 0};
    return entry(*near);
  }
  static bool holds(const Entry &e, uint64_t off) { return off >= e.start && off < e.end; }
  void *ptr(uint64_t off) const;
  uint64_t slab_bytes() const { return slab_; }
  uint64_t total_bytes() const { return total_slabs_ * slab_; }

 private:
  uint64_t slab_;
  uint64_t total_slabs_ = 0;
  uint64_t next_serial_ = 1;
  std::vector<Segment> segs_;
  std::map<uint64_t, uint64_t> free_runs_;   // first slab -> length; runs never cross a segment edge
  // The live allocations in ascending order, in blocks of up to kBlock: neighbours lie next to each other in memory, which is
  // what a submit of a thousand tensors walks over (a tree's nodes, each found through the one before, took 16 ns an answer), and
  // one comes or goes at the cost of moving a block.
  static constexpr uint32_t kBlock = 64;
  struct Block {
    uint32_t n = 0;
    Entry e[kBlock];
  };
  std::vector<std::unique_ptr<Block>> blocks_;
  std::deque<Allocation> records_;
  std::vector<Allocation *> free_records_;
  const Entry *entry(const Place &p) const { return p.block < blocks_.size() && p.pos < blocks_[p.block]->n ? &blocks_[p.block]->e[p.pos] : nullptr; }
  bool last_at_or_before(uint64_t off, Place *p) const;
  void insert(const Entry &e);
  void erase(const Place &p);
  const Segment *segment_of_slab(uint64_t slab) const;
};

}  // namespace ft

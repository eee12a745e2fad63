#include "ft_pool.h"

#include <algorithm>
#include <cstddef>

#include "../../include/faastube.h"

namespace ft {

int SlabPool::check_segment(const void *base, uint64_t bytes, uint64_t slab_bytes) {
  if (base == nullptr) return FT_EINVAL;
  if (slab_bytes == 0 || slab_bytes % 256 != 0) return FT_EINVAL;
  if (bytes == 0 || bytes % slab_bytes != 0) return FT_EINVAL;
  if (reinterpret_cast<uintptr_t>(base) % 256 != 0) return FT_EINVAL;
  return FT_OK;
}

int SlabPool::add_segment(void *base, uint64_t bytes) {
  int rc = check_segment(base, bytes, slab_);
  if (rc != FT_OK) return rc;
  Segment s;
  s.base = static_cast<char *>(base);
  s.bytes = bytes;
  s.first_slab = total_slabs_;
  s.nslabs = bytes / slab_;
  segs_.push_back(s);
  free_runs_[s.first_slab] = s.nslabs;  // kept apart from the previous segment's tail run
  total_slabs_ += s.nslabs;
  return FT_OK;
}

int SlabPool::drop_last_segment(void **base_out, uint64_t *bytes_out) {
  if (segs_.size() < 2) return FT_EINVAL;
  const Segment s = segs_.back();
  // a segment without allocations is exactly one free run
  auto it = free_runs_.find(s.first_slab);
  if (it == free_runs_.end() || it->second != s.nslabs) return FT_EBUSY;
  free_runs_.erase(it);
  segs_.pop_back();
  total_slabs_ -= s.nslabs;
  if (base_out) *base_out = s.base;
  if (bytes_out) *bytes_out = s.bytes;
  return FT_OK;
}

uint64_t SlabPool::live_bytes() const {
  uint64_t n = 0;
  for (const auto &b : blocks_)
    for (uint32_t i = 0; i < b->n; ++i) n += b->e[i].al->nslabs;
  return n * slab_;
}

const Segment *SlabPool::segment_of_slab(uint64_t slab) const {
  size_t lo = 0, hi = segs_.size();
  if (hi == 0 || slab >= total_slabs_) return nullptr;
  while (hi - lo > 1) {
    size_t mid = (lo + hi) / 2;
    if (segs_[mid].first_slab <= slab) lo = mid; else hi = mid;
  }
  return &segs_[lo];
}

int SlabPool::alloc(uint64_t nbytes, uint64_t *off_out) {
  if (nbytes == 0 || off_out == nullptr) return FT_EINVAL;
  uint64_t need = nbytes / slab_ + (nbytes % slab_ != 0);
  // free runs are keyed by first slab, so the first run that is long enough is the
  // lowest-indexed fit
  for (auto it = free_runs_.begin(); it != free_runs_.end(); ++it) {
    if (it->second < need) continue;
    uint64_t start = it->first, len = it->second;
    free_runs_.erase(it);
    if (len > need) free_runs_[start + need] = len - need;
    if (free_records_.empty()) {
      records_.emplace_back();
      free_records_.push_back(&records_.back());
    }
    Allocation *a = free_records_.back();
    free_records_.pop_back();
    a->nslabs = need;
    a->busy = 0;
    a->serial = next_serial_++;
    insert(Entry{start * slab_, (start + need) * slab_, reinterpret_cast<uint64_t>(ptr(start * slab_)), a});
    *off_out = start * slab_;
    return FT_OK;
  }
  return FT_ENOMEM;
}

int SlabPool::free(uint64_t off, bool ordered) {
  Place at;
  if (!last_at_or_before(off, &at) || entry(at)->start != off) return FT_EINVAL;
  Allocation *al = entry(at)->al;
  if (al->busy != 0 && !ordered) return FT_EBUSY;
  uint64_t start = off / slab_, len = al->nslabs;
  erase(at);
  al->serial = 0;
  free_records_.push_back(al);
  const Segment *seg = segment_of_slab(start);
  // merge with the free neighbours that lie in the same segment
  auto next = free_runs_.find(start + len);
  if (next != free_runs_.end() && start + len < seg->first_slab + seg->nslabs) {
    len += next->second;
    free_runs_.erase(next);
  }
  auto after = free_runs_.lower_bound(start);
  if (after != free_runs_.begin()) {
    auto prev = std::prev(after);
    if (prev->first + prev->second == start && start > seg->first_slab) {
      prev->second += len;
      return FT_OK;
    }
  }
  free_runs_[start] = len;
  return FT_OK;
}

// The last allocation that starts at or before `off`.
bool SlabPool::last_at_or_before(uint64_t off, Place *p) const {
  uint32_t lo = 0, hi = (uint32_t)blocks_.size();  // blocks that start at or before off
  while (lo < hi) {
    const uint32_t mid = (lo + hi) / 2;
    if (blocks_[mid]->e[0].start <= off) lo = mid + 1; else hi = mid;
  }
  if (lo == 0) return false;
  const Block &b = *blocks_[lo - 1];
  uint32_t i = 1, n = b.n;
  while (i < n) {
    const uint32_t mid = (i + n) / 2;
    if (b.e[mid].start <= off) i = mid + 1; else n = mid;
  }
  p->block = lo - 1;
  p->pos = i - 1;
  return true;
}

void SlabPool::insert(const Entry &e) {
  Place at;
  if (last_at_or_before(e.start, &at)) at.pos += 1;  // else: in front of the first
  else if (blocks_.empty()) blocks_.push_back(std::make_unique<Block>());
  Block *b = blocks_[at.block].get();
  if (b->n == kBlock) {
    // A full block is halved; where allocations come in ascending order the new one is begun with the newcomer alone.
    auto next = std::make_unique<Block>();
    const uint32_t keep = at.pos == kBlock ? kBlock : kBlock / 2;
    next->n = kBlock - keep;
    std::copy(b->e + keep, b->e + kBlock, next->e);
    b->n = keep;
    Block *n = next.get();
    blocks_.insert(blocks_.begin() + at.block + 1, std::move(next));
    if (at.pos > keep || keep == kBlock) {
      at.pos -= keep;
      b = n;
    }
  }
  std::copy_backward(b->e + at.pos, b->e + b->n, b->e + b->n + 1);
  b->e[at.pos] = e;
  b->n += 1;
}

void SlabPool::erase(const Place &p) {
  Block &b = *blocks_[p.block];
  std::copy(b.e + p.pos + 1, b.e + b.n, b.e + p.pos);
  b.n -= 1;
  if (b.n == 0) blocks_.erase(blocks_.begin() + p.block);
}

Allocation *SlabPool::at(uint64_t start) {
  Place p;
  return last_at_or_before(start, &p) && entry(p)->start == start ? entry(p)->al : nullptr;
}

void *SlabPool::ptr(uint64_t off) const {
  const Segment *seg = segment_of_slab(off / slab_);
  if (!seg) return nullptr;
  return seg->base + (off - seg->first_slab * slab_);
}

}  // namespace ft

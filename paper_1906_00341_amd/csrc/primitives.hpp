// Scans, reductions, compaction and a radix sort of 64-bit keys (host launchers).
#pragma once

#include <vector>

#include "common.hpp"

namespace dsd {

// Device memory beyond what a call was admitted with (a server's budget).
// take: bytes, or nothing and false where they do not fit; safe with several
// threads.  What was taken goes back with the call's end.
class MemoryGrant {
public:
    virtual bool take(size_t bytes) = 0;

protected:
    ~MemoryGrant() = default;
};

// Bump allocator over device chunks; reset() recycles everything (stream-ordered reuse).
// Device scratch: a bump allocator over chunks of at least min_chunk bytes
// (64 MiB unless given).  A new
// chunk comes from a process-wide pool of recycled chunks (per device, at
// most 16 GiB kept) before hipMalloc is asked; recycle() hands the chunks to
// that pool, and the caller promises that no work still uses them (its
// stream is idle).  Chunks not recycled are freed with the scratch.
class Scratch {
public:
    explicit Scratch(size_t min_chunk = (size_t)64 << 20) : min_chunk_(min_chunk) {}
    // a scratch over a caller-owned device buffer: it never allocates, frees
    // or recycles the buffer; a request beyond it throws DSD_ENOMEM
    Scratch(void *buf, size_t bytes) : min_chunk_(0), external_(true) { chunks_.push_back({(char *)buf, bytes}); }
    Scratch(const Scratch &) = delete;
    Scratch &operator=(const Scratch &) = delete;
    ~Scratch();
    void *get(size_t bytes);
    void recycle();
    template <typename T> T *get_n(int64_t n) { return (T *)get((size_t)(n > 0 ? n : 1) * sizeof(T)); }
    void reset() { cur_ = 0; off_ = 0; }
    size_t capacity() const;
    bool external() const { return external_; }
    // what a user of the scratch asks before it takes memory that its call
    // could do without (nullptr: nobody to ask)
    void set_grant(MemoryGrant *g) { grant_ = g; }
    MemoryGrant *grant() const { return grant_; }
    bool may_take(size_t bytes) { return !grant_ || grant_->take(bytes); }

private:
    std::vector<std::pair<char *, size_t>> chunks_;
    size_t cur_ = 0, off_ = 0;
    size_t min_chunk_;
    bool external_ = false;
    MemoryGrant *grant_ = nullptr;
};

// out[i] = sum_{j<i} in[j]; returns nothing, total = out[n-1] + in[n-1].  in == out allowed.
void scan_exclusive_i64(const int64_t *in, int64_t *out, int64_t n, hipStream_t s, Scratch &sc);
void scan_exclusive_u32(const uint32_t *in, uint32_t *out, int64_t n, hipStream_t s, Scratch &sc);

// Sort n 64-bit keys ascending on their low `bits` bits (higher bits must be 0).
// The result is in *keys; tmp has room for n keys.
void radix_sort_u64(u64 *keys, u64 *tmp, int64_t n, int bits, hipStream_t s, Scratch &sc);

// One stable counting pass: keys[0, n) grouped into out by the 8-bit digit at
// shift.  start (256 * radix_tiles(n) counters): group q begins at
// start[q * radix_tiles(n)].
int64_t radix_tiles(int64_t n);
void radix_pass_u64(const u64 *keys, u64 *out, int64_t n, int shift, uint32_t *start, hipStream_t s, Scratch &sc);

// sum of a u64 array as a 128-bit (lo, hi) pair written to out[0], out[1] (device)
void sum_u64_128(const u64 *in, int64_t n, u64 *out2, hipStream_t s, Scratch &sc);

// free every recycled chunk of every device
void release_chunk_pool();

// Small values read back in one trip: a kernel gathers the pieces into a pinned
// buffer of the calling thread, then one synchronisation.  (A copy into ordinary
// host memory is a trip of its own, 10 to 12 us each.)  A piece too large for the
// buffer, and every piece of a caller-owned scratch (sc), is copied as it is.
class Readback {
public:
    explicit Readback(const Scratch &sc) : plain_(sc.external()) {}
    // n values at dev, 4-byte aligned or single bytes
    template <typename T> Readback &add(T *host, const T *dev, int64_t n = 1) {
        piece(host, dev, (size_t)n * sizeof(T));
        return *this;
    }
    // waits for the stream; the values are in place when it returns
    void run(hipStream_t s);

private:
    static constexpr int PIECES = 8;
    void piece(void *host, const void *dev, size_t bytes);
    bool plain_;
    int np_ = 0;
    void *host_[PIECES];
    const void *dev_[PIECES];
    size_t bytes_[PIECES];
};

// fill helpers (kernels, usable under stream capture)
void fill_u64(u64 *p, u64 v, int64_t n, hipStream_t s);
void fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s);
void fill_u8(uint8_t *p, uint8_t v, int64_t n, hipStream_t s);

}  // namespace dsd

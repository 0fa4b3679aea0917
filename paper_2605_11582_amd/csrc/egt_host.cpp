// Host side of the SparseGemv library: shape rules, N:4 magnitude pruning, the
// group-wise INT4 quantiser and the 2bit-CSR encoder / decoder (Sec. 3.2 and
// Sec. 3.3 "Sparse Index Structure" of the paper).  Plain C++, no GPU calls.
#include "egt.h"

#include "egt_host_simd.h"
#include "egt_host_simd512.h"

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <new>
#include <thread>
#include <type_traits>

#if defined(__unix__)
#include <pthread.h>
#define EGT_HOST_ATFORK 1
#endif

namespace {

// ---------------------------------------------------------------- binary16
inline double half_to_double(uint16_t h) {
  const int sign = h >> 15, e = (h >> 10) & 31, m = h & 1023;
  double v;
  if (e == 0) v = (double)m * 0x1p-24;
  else if (e == 31) v = m ? NAN : INFINITY;
  else {
    const uint64_t u = ((uint64_t)(e + 1008) << 52) | ((uint64_t)m << 42);
    std::memcpy(&v, &u, 8);
  }
  return sign ? -v : v;
}

// One rounding, nearest-even, straight from binary64 (never through binary32).
inline uint16_t double_to_half(double v) {
  const uint16_t sign = std::signbit(v) ? 0x8000u : 0u;
  if (std::isnan(v)) return sign | 0x7E00u;
  double a = std::fabs(v);
  if (a >= 65520.0) return sign | 0x7C00u;          // rounds to infinity
  if (a < 0x1p-14) {                                 // subnormal range: units of 2^-24
    const double q = std::nearbyint(a * 0x1p24);
    return sign | (uint16_t)q;                       // q == 1024 is the smallest normal
  }
  uint64_t u;                                        // 42 of the 52 mantissa bits go, to nearest even
  std::memcpy(&u, &a, 8);
  u = (u + 0x1FFFFFFFFFFull + ((u >> 42) & 1)) >> 42;    // (a carry moves on into the exponent)
  return sign | (uint16_t)(u - (1008u << 10));
}

inline bool half_is_finite(uint16_t h) { return ((h >> 10) & 31) != 31; }

// ---------------------------------------------------------------- threading
// Worker threads of the host functions.  Starting 15 threads takes 300 us, longer than they
// then need for a matrix of four million weights, so they stay for the next call - and leave
// by themselves when none has come for a fifth of a second.  At most MAX of them live at a
// time, whatever calls there are; a call that finds them at work for another thread's call
// does its work alone.  The calling thread takes part itself: a job is finished even if no
// worker could be started.  A library that is unloaded (or a process that ends) first stops
// and joins them: no thread may be left in code that is no longer mapped.
class Workers {
 public:
  static constexpr int MAX = 15;

  // job(0), ..., job(parts - 1), each once, in any order and on any of up to `helpers` + 1 threads.  A part does not
  // throw - on a worker it would have nowhere to throw to - and so allocates nothing.
  template <class F>
  static void run(int parts, int helpers, F &&job) {
    static_assert(noexcept(job(0)), "a part does not throw");
    Workers *w = helpers > 0 ? &instance() : nullptr;
    if (!w || !w->begin(parts, helpers, [](void *f, int k) noexcept { (*(std::remove_reference_t<F> *)f)(k); }, (void *)&job)) {
      for (int k = 0; k < parts; ++k) job(k);
      return;
    }
    w->work();
    w->finish();
  }

  // No worker is started from here on, and none is left when this returns.
  void stop() {
    std::thread last;
    {
      std::unique_lock<std::mutex> lock(mu_);
      stopping_ = true;
      epoch_.fetch_add(1);
      wake_.notify_all();
      done_.wait(lock, [&] { return alive_ == 0; });
      last = std::move(left_);
    }
    if (last.joinable()) last.join();
  }

  // One object for the process, in memory of the library's own: it is stopped, but never destroyed (at the end of
  // a process other threads may still be in a call).  A child process starts with a fresh one: threads do not
  // survive fork, and a lock of another thread would stay locked.
  static Workers &instance() { return *reinterpret_cast<Workers *>(memory_); }
  static void start_afresh() { new (memory_) Workers; }

 private:
  typedef void (*Part)(void *, int) noexcept;
  static unsigned char memory_[];
  std::mutex mu_;
  std::condition_variable wake_, done_;
  std::atomic<uint32_t> epoch_{0};                   // counts jobs: idle workers watch it before they go to sleep
  std::thread thread_[MAX];                          // joinable: a worker that has not left
  std::thread left_;                                 // the worker that left last; it has joined the one before it
  int alive_ = 0, inside_ = 0, seats_ = 0;           // workers; workers in the current job; how many more may join it
  bool busy_ = false, stopping_ = false;
  Part part_ = nullptr;
  void *arg_ = nullptr;
  int parts_ = 0;
  std::atomic<int> next_{0};

  bool begin(int parts, int helpers, Part part, void *arg) {
    std::lock_guard<std::mutex> lock(mu_);
    if (busy_ || stopping_) return false;
    busy_ = true;
    part_ = part; arg_ = arg; parts_ = parts;
    next_.store(0);
    seats_ = std::min(helpers, MAX);
    for (int k = 0; k < MAX && alive_ < seats_; ++k) {
      if (thread_[k].joinable()) continue;
      try {
        thread_[k] = std::thread([this, k] { serve(k); });
      } catch (const std::exception &) {              // (no thread or no memory for one)
        break;
      }
      ++alive_;
    }
    epoch_.fetch_add(1);
    wake_.notify_all();
    return true;
  }
  void work() {
    for (int k; (k = next_.fetch_add(1)) < parts_;) part_(arg_, k);
  }
  void finish() {
    std::unique_lock<std::mutex> lock(mu_);
    seats_ = 0;                                       // who has not come by now is not needed
    done_.wait(lock, [&] { return inside_ == 0; });
    busy_ = false;
  }
  void serve(int k) {
    std::unique_lock<std::mutex> lock(mu_);
    for (;;) {
      const bool called = wake_.wait_for(lock, std::chrono::milliseconds(200), [&] { return seats_ > 0 || stopping_; });
      if (!called || seats_ == 0) break;              // (a job that has begun is finished first)
      --seats_;
      ++inside_;
      const uint32_t seen = epoch_.load();
      lock.unlock();
      work();
      lock.lock();
      if (--inside_ == 0) done_.notify_all();
      lock.unlock();
      // the next pass over the same matrix usually follows at once: worth 20 us of looking
      const auto until = std::chrono::steady_clock::now() + std::chrono::microseconds(20);
      while (epoch_.load(std::memory_order_relaxed) == seen && std::chrono::steady_clock::now() < until) {}
      lock.lock();
    }
    // a thread cannot join itself: it leaves its handle to the next one that leaves, or to stop()
    std::thread before = std::move(left_);
    left_ = std::move(thread_[k]);
    if (--alive_ == 0) done_.notify_all();
    lock.unlock();
    if (before.joinable()) before.join();
  }
};
alignas(Workers) unsigned char Workers::memory_[sizeof(Workers)];

// Runs when the library is loaded, and when it is unloaded or the process ends.
struct WorkersOfTheLibrary {
  WorkersOfTheLibrary() {
    Workers::start_afresh();
#ifdef EGT_HOST_ATFORK
    pthread_atfork(nullptr, nullptr, [] { Workers::start_afresh(); });     // (given back when the library is unloaded)
#endif
  }
  ~WorkersOfTheLibrary() { Workers::instance().stop(); }
} workers_of_the_library;

// body(r0, r1) over all rows in blocks; a thread pays from about 64 Ki columns' work on
template <class F>
void parallel_rows(int rows, int cols, F &&body) {
  const unsigned hw = std::thread::hardware_concurrency();
  const int64_t by_work = ((int64_t)rows * (int64_t)std::max(cols, 1)) >> 16;
  const int nt = (int)std::max<int64_t>(1, std::min<int64_t>({(int64_t)(hw ? hw : 1u), (int64_t)Workers::MAX + 1, (int64_t)rows / 8, by_work}));
  if (nt <= 1) { body(0, rows); return; }
  const int parts = std::min(rows, 4 * nt);           // (a thread that is held up leaves its share to the others)
  Workers::run(parts, nt - 1, [&](int k) noexcept { body((int)((int64_t)rows * k / parts), (int)((int64_t)rows * (k + 1) / parts)); });
}

// INT4 values in either nibble order
inline bool is_int4(int val_kind) { return val_kind == EGT_VAL_INT4 || val_kind == EGT_VAL_INT4_PAIRED; }
// Where the code of global slot t lives: byte and shift.  Canonical order: slot j of a word
// of eight slots in nibble j.  Paired order: in nibble (j >> 1) + 4 (j & 1), i.e. the
// nibbles of a word hold the slots 0, 2, 4, 6, 1, 3, 5, 7.
inline int64_t nibble_byte(int64_t t, int val_kind, int &shift) {
  const int j = (int)(t & 7);
  const int pos = val_kind == EGT_VAL_INT4_PAIRED ? (j >> 1) + 4 * (j & 1) : j;
  shift = 4 * (pos & 1);
  return (t >> 3) * 4 + (pos >> 1);
}

// ---------------------------------------------------------------- shape rules
egt_status check_shape(int rows, int cols, int n_keep, int group, int val_kind) {
  if (rows < 0 || cols < 0) return EGT_ERR_SHAPE;
  if (cols % 32 != 0) return EGT_ERR_SHAPE;
  if (n_keep < 1 || n_keep > 4) return EGT_ERR_SHAPE;
  if (is_int4(val_kind)) {
    if (group <= 0 || group % 4 != 0 || cols % group != 0) return EGT_ERR_SHAPE;
  } else if (val_kind == EGT_VAL_FP16) {
    if (group != 0) return EGT_ERR_SHAPE;
  } else {
    return EGT_ERR_SHAPE;
  }
  const uint64_t slots = (uint64_t)rows * (uint64_t)n_keep * (uint64_t)(cols / 4);
  if (slots >= (1ull << 32)) return EGT_ERR_SHAPE;   // row_ptr is uint32
  return EGT_OK;
}

// Shape rules of a matrix whose rows keep row_n_keep[r] (1..4) entries per 4-group each;
// `slots`: the total number of slots.
egt_status check_rows(int rows, int cols, const int32_t *row_n_keep, int group, int val_kind, uint64_t &slots) {
  const egt_status st = check_shape(rows, cols, 1, group, val_kind);
  if (st != EGT_OK) return st;
  slots = 0;
  for (int r = 0; r < rows; ++r) {
    if (row_n_keep[r] < 1 || row_n_keep[r] > 4) return EGT_ERR_SHAPE;
    slots += (uint64_t)row_n_keep[r] * (uint64_t)(cols / 4);
  }
  if (slots >= (1ull << 32)) return EGT_ERR_SHAPE;
  return EGT_OK;
}

void fill_sizes(int rows, int cols, uint64_t slots, int group, int val_kind, size_t bytes[4]) {
  bytes[0] = sizeof(uint32_t) * ((size_t)rows + 1);
  bytes[1] = is_int4(val_kind) ? (size_t)(slots / 2) : (size_t)(slots * 2);
  bytes[2] = (size_t)(slots / 8) * sizeof(uint16_t);
  bytes[3] = is_int4(val_kind) ? sizeof(uint16_t) * 2 * (size_t)rows * (size_t)(cols / group) : 0;
}

egt_status pack_rows(const uint16_t *w, int64_t ldw, const uint8_t *mask, int64_t ldm, int rows, int cols,
                     int n_keep, const int32_t *row_n_keep, int group, int val_kind, const int32_t *row_group,
                     egt_2bitcsr *out);

// Scale and zero point of one group from the extrema of its kept values.
struct QParam { uint16_t s_bits; double s; int z; };
inline QParam make_qparam(double vmin, double vmax) {
  const double xmin = std::min(0.0, vmin), xmax = std::max(0.0, vmax);
  uint16_t sb = double_to_half((xmax - xmin) / 15.0);
  if ((sb & 0x7FFF) == 0) sb = 0x3C00;               // s == 0 -> 1.0
  const double s = half_to_double(sb);
  double z = std::nearbyint(-xmin / s);
  z = std::min(15.0, std::max(0.0, z));
  return {sb, s, (int)z};
}
#ifdef EGT_HOST_SIMD
// the same from extrema that hold 0
inline QParam make_qparam_simd(float lo, float hi) {
  uint16_t sb = double_to_half(((double)hi - (double)lo) / 15.0);
  if ((sb & 0x7FFF) == 0) sb = 0x3C00;
  const float s = egt_simd::half_to_float(sb);
  return {sb, s, egt_simd::zero_point(lo, s)};
}
#endif
// FP16 bits of a zero point
inline uint16_t zero_bits(int z) {
  static const uint16_t bits[16] = {0x0000, 0x3C00, 0x4000, 0x4200, 0x4400, 0x4500, 0x4600, 0x4700,
                                    0x4800, 0x4880, 0x4900, 0x4980, 0x4A00, 0x4A80, 0x4B00, 0x4B80};
  return bits[z];
}
// ... and back from the two halves a group is stored as
inline QParam stored_qparam(const uint16_t *p) { return {p[0], half_to_double(p[0]), (int)half_to_double(p[1])}; }
inline int make_code(double v, const QParam &p) {
  double q = std::nearbyint(v / p.s) + (double)p.z;
  q = std::min(15.0, std::max(0.0, q));
  return (int)q;
}

// Chosen in-group offsets of one 4-group: the kept ones plus, if fewer than n,
// the smallest unused offsets.  Returns a 4-bit set, or -1 when over-full.
inline int choose4(const uint8_t *m, int n) {
  int set = 0, cnt = 0;
  for (int j = 0; j < 4; ++j) if (m[j]) { set |= 1 << j; ++cnt; }
  if (cnt > n) return -1;
  for (int j = 0; j < 4 && cnt < n; ++j) if (!(set >> j & 1)) { set |= 1 << j; ++cnt; }
  return set;
}

}  // namespace

extern "C" {

const char *egt_status_str(egt_status status) {
  switch (status) {
    case EGT_OK: return "ok";
    case EGT_ERR_NULL: return "null pointer";
    case EGT_ERR_SHAPE: return "bad shape";
    case EGT_ERR_MASK: return "mask keeps more than n_keep entries in a 4-group";
    case EGT_ERR_NONFINITE: return "non-finite kept weight";
    case EGT_ERR_BUFFER: return "inconsistent buffer contents";
    case EGT_ERR_UNSUPPORTED: return "unsupported configuration";
    case EGT_ERR_HIP: return "HIP runtime error";
    default: return "unknown status";
  }
}

egt_status egt_2bitcsr_sizes(int rows, int cols, int n_keep, int group, int val_kind,
                             size_t bytes[4]) {
  if (!bytes) return EGT_ERR_NULL;
  const egt_status st = check_shape(rows, cols, n_keep, group, val_kind);
  if (st != EGT_OK) return st;
  const size_t slots = (size_t)rows * (size_t)n_keep * (size_t)(cols / 4);
  bytes[0] = 4 * ((size_t)rows + 1);
  bytes[1] = is_int4(val_kind) ? slots / 2 : slots * 2;
  bytes[2] = 2 * (slots / 8);
  bytes[3] = is_int4(val_kind) ? 4 * (size_t)rows * (size_t)(cols / group) : 0;
  return EGT_OK;
}

egt_status egt_prune_n4(const uint16_t *w, int64_t ldw, int rows, int cols, int n_keep,
                        uint8_t *mask, int64_t ldm) {
  if (!w || !mask) return EGT_ERR_NULL;
  if (rows < 0 || cols < 0 || cols % 4 != 0 || n_keep < 1 || n_keep > 4 || ldw < cols || ldm < cols)
    return EGT_ERR_SHAPE;
#ifdef EGT_HOST_SIMD512
  const bool wide = egt_simd512::available() && cols % 64 == 0;
#endif
  parallel_rows(rows, cols, [=](int r0, int r1) {
    for (int r = r0; r < r1; ++r) {
      const uint16_t *wr = w + (int64_t)r * ldw;
      uint8_t *mr = mask + (int64_t)r * ldm;
#ifdef EGT_HOST_SIMD
#ifdef EGT_HOST_SIMD512
      if (wide) {
        egt_simd::with_n(n_keep, [&](auto c) { egt_simd512::prune_row<decltype(c)::n>(wr, cols, mr); });
        continue;
      }
#endif
      if (egt_simd::available()) { egt_simd::prune_row(wr, cols, n_keep, mr); continue; }
#endif
      for (int c = 0; c < cols; c += 4) {
        // |w| ordering of finite binary16 numbers = ordering of the low 15 bits
        int mag[4];
        for (int j = 0; j < 4; ++j) mag[j] = wr[c + j] & 0x7FFF;
        for (int j = 0; j < 4; ++j) {
          int beats = 0;
          for (int i = 0; i < 4; ++i) {
            if (i == j) continue;
            beats += i < j ? (mag[i] >= mag[j]) : (mag[i] > mag[j]);
          }
          mr[c + j] = beats < n_keep ? 1 : 0;
        }
      }
    }
  });
  return EGT_OK;
}

egt_status egt_prune_n4_importance(const uint16_t *w, int64_t ldw, const float *act_norm,
                                   const float *grad_abs, int64_t ldg, int rows, int cols,
                                   int n_keep, uint8_t *mask, int64_t ldm) {
  if (!w || !act_norm || !mask) return EGT_ERR_NULL;
  if (rows < 0 || cols < 0 || cols % 4 != 0 || n_keep < 1 || n_keep > 4 || ldw < cols || ldm < cols ||
      (grad_abs && ldg < cols))
    return EGT_ERR_SHAPE;
  for (int c = 0; c < cols; ++c)
    if (!(act_norm[c] >= 0.0f) || std::isinf(act_norm[c])) return EGT_ERR_NONFINITE;
  std::atomic<int> err(EGT_OK);
  parallel_rows(rows, cols, [&](int r0, int r1) {
    for (int r = r0; r < r1; ++r) {
      for (int c = 0; c < cols; ++c) {
        if ((w[(int64_t)r * ldw + c] & 0x7C00) == 0x7C00) err.store(EGT_ERR_NONFINITE);
        if (grad_abs) {
          const float gv = grad_abs[(int64_t)r * ldg + c];
          if (!(gv >= 0.0f) || std::isinf(gv)) err.store(EGT_ERR_NONFINITE);
        }
      }
    }
  });
  if (err.load() != EGT_OK) return (egt_status)err.load();
  parallel_rows(rows, cols, [=](int r0, int r1) {
#pragma clang fp contract(off)
    for (int r = r0; r < r1; ++r) {
      const uint16_t *wr = w + (int64_t)r * ldw;
      uint8_t *mr = mask + (int64_t)r * ldm;
      for (int c = 0; c < cols; c += 4) {
        double score[4];
        for (int j = 0; j < 4; ++j) {
          const double a = std::fabs(half_to_double(wr[c + j]));
          const double p1 = a * (double)act_norm[c + j];
          const double p2 = grad_abs ? a * (double)grad_abs[(int64_t)r * ldg + c + j] : 0.0;
          score[j] = p1 + p2;
        }
        for (int j = 0; j < 4; ++j) {
          int beats = 0;
          for (int i = 0; i < 4; ++i) {
            if (i == j) continue;
            beats += i < j ? (score[i] >= score[j]) : (score[i] > score[j]);
          }
          mr[c + j] = beats < n_keep ? 1 : 0;
        }
      }
    }
  });
  return EGT_OK;
}

egt_status egt_pack_2bitcsr(const uint16_t *w, int64_t ldw, const uint8_t *mask, int64_t ldm,
                            int rows, int cols, int n_keep, int group, int val_kind,
                            egt_2bitcsr *out) {
  return pack_rows(w, ldw, mask, ldm, rows, cols, n_keep, nullptr, group, val_kind, nullptr, out);
}

egt_status egt_pack_2bitcsr_rowgroups(const uint16_t *w, int64_t ldw, const uint8_t *mask, int64_t ldm,
                                      int rows, int cols, int n_keep, int group, int val_kind,
                                      const int32_t *row_group, egt_2bitcsr *out) {
  return pack_rows(w, ldw, mask, ldm, rows, cols, n_keep, nullptr, group, val_kind, row_group, out);
}

egt_status egt_pack_2bitcsr_rows(const uint16_t *w, int64_t ldw, const uint8_t *mask, int64_t ldm,
                                 int rows, int cols, const int32_t *row_n_keep, int group, int val_kind,
                                 egt_2bitcsr *out) {
  if (!row_n_keep) return EGT_ERR_NULL;
  return pack_rows(w, ldw, mask, ldm, rows, cols, 0, row_n_keep, group, val_kind, nullptr, out);
}

egt_status egt_2bitcsr_sizes_rows(int rows, int cols, const int32_t *row_n_keep, int group, int val_kind,
                                  size_t bytes[4]) {
  if (!bytes || !row_n_keep) return EGT_ERR_NULL;
  uint64_t slots = 0;
  const egt_status st = check_rows(rows, cols, row_n_keep, group, val_kind, slots);
  if (st != EGT_OK) return st;
  fill_sizes(rows, cols, slots, group, val_kind, bytes);
  return EGT_OK;
}

}  // extern "C"

namespace {

// The encoder.  row_n_keep == nullptr: n_keep entries per 4-group in every row; else row r
// keeps row_n_keep[r] (rows of different lengths, row_ptr a true prefix sum, n_keep = 0
// in the view).
egt_status pack_rows(const uint16_t *w, int64_t ldw, const uint8_t *mask, int64_t ldm, int rows, int cols,
                     int n_keep, const int32_t *row_n_keep, int group, int val_kind, const int32_t *row_group,
                     egt_2bitcsr *out) {
  if (!w || !mask || !out) return EGT_ERR_NULL;
  uint64_t total_slots = 0;
  egt_status st = row_n_keep ? check_rows(rows, cols, row_n_keep, group, val_kind, total_slots)
                             : check_shape(rows, cols, n_keep, group, val_kind);
  if (st != EGT_OK) return st;
  auto n_of = [=](int r) { return row_n_keep ? (int)row_n_keep[r] : n_keep; };
#ifdef EGT_HOST_SIMD512
  // (whole registers only: a matrix with a ragged end takes the 256-bit loops for all of it)
  const bool wide = egt_simd512::available() && cols % 64 == 0 && (!is_int4(val_kind) || group % 32 == 0);
#endif
  if (ldw < cols || ldm < cols) return EGT_ERR_SHAPE;
  if (!out->row_ptr || !out->values || !out->idx) return EGT_ERR_NULL;
  if (is_int4(val_kind) && !out->qparams) return EGT_ERR_NULL;
  if (row_group) {
    if (!is_int4(val_kind)) return EGT_ERR_SHAPE;
    for (int r = 0; r < rows; ++r)
      if (row_group[r] <= 0 || row_group[r] % group != 0 || cols % row_group[r] != 0) return EGT_ERR_SHAPE;
  }

  // pass 1: validate everything before a single output byte is written.  The error reported
  // is that of the first offending 4-group in row-major order, whatever the thread timing; a
  // group that is both over-full and holds a non-finite kept weight reports the mask.
  std::atomic<int64_t> first(INT64_MAX);             // (index of the 4-group in the matrix) * 8 + code
  const int64_t gpr = cols / 4;
  auto validate = [&](int r0, int r1) {
    for (int r = r0; r < r1; ++r) {
      if ((int64_t)r * gpr * 8 > first.load(std::memory_order_relaxed)) break;
      const uint16_t *wr = w + (int64_t)r * ldw;
      const uint8_t *mr = mask + (int64_t)r * ldm;
      const int n_row = n_of(r);
#ifdef EGT_HOST_SIMD
#ifdef EGT_HOST_SIMD512
      if (wide && egt_simd512::row_valid(wr, mr, cols, n_row)) continue;
#endif
      if (egt_simd::available() && egt_simd::row_valid(wr, mr, cols, n_row)) continue;
#endif
      for (int c = 0; c < cols; c += 4) {
        int cnt = 0;
        bool nonfinite = false;
        for (int j = 0; j < 4; ++j) {
          if (!mr[c + j]) continue;
          ++cnt;
          nonfinite |= !half_is_finite(wr[c + j]);
        }
        if (cnt <= n_row && !nonfinite) continue;
        const int64_t key = ((int64_t)r * gpr + (c >> 2)) * 8 + (cnt > n_row ? EGT_ERR_MASK : EGT_ERR_NONFINITE);
        int64_t seen = first.load();
        while (key < seen && !first.compare_exchange_weak(seen, key)) {}
        r = r1;                                         // later rows of this range cannot come first
        break;
      }
    }
  };

  parallel_rows(rows, cols, validate);
  if (first.load() != INT64_MAX) return (egt_status)(first.load() & 7);

  const int G = is_int4(val_kind) ? cols / group : 0;
  // first slot of every row (uniform rows: r * S)
  for (int64_t r = 0, t = 0; r <= rows; ++r) {
    out->row_ptr[r] = (uint32_t)t;
    if (r < rows) t += (int64_t)n_of((int)r) * (cols / 4);
  }
  uint8_t *vals8 = (uint8_t *)out->values;
  uint16_t *vals16 = (uint16_t *)out->values;
  const uint32_t *row_ptr = out->row_ptr;
  uint16_t *idx = out->idx, *qparams = out->qparams;
#ifdef EGT_HOST_SIMD
  const bool simd = egt_simd::available() && (!is_int4(val_kind) || group % 8 == 0);
#else
  const bool simd = false;
#endif

  auto encode = [=](int r0, int r1) {
    for (int r = r0; r < r1; ++r) {
      const uint16_t *wr = w + (int64_t)r * ldw;
      const uint8_t *mr = mask + (int64_t)r * ldm;
      const int n_row = n_of(r);
      uint16_t *qr = is_int4(val_kind) ? qparams + (int64_t)r * G * 2 : nullptr;     // the row's {scale, zero} pairs
      if (is_int4(val_kind)) {
        // the row's own group size; its parameters are stored once per `group` columns
        const int gr = row_group ? row_group[r] : group, rep = gr / group;
        for (int g0 = 0; g0 < G; g0 += rep) {
          QParam p;
#ifdef EGT_HOST_SIMD
          if (simd) {
            float lo, hi;
#ifdef EGT_HOST_SIMD512
            if (wide) egt_simd512::extrema(wr + g0 * group, mr + g0 * group, gr, lo, hi);
            else
#endif
            egt_simd::extrema(wr + g0 * group, mr + g0 * group, gr, lo, hi);
            p = make_qparam_simd(lo, hi);
          } else
#endif
          {
            double vmin = INFINITY, vmax = -INFINITY;
            for (int c = g0 * group; c < g0 * group + gr; ++c) {
              if (!mr[c]) continue;
              const double v = half_to_double(wr[c]);
              vmin = std::min(vmin, v);
              vmax = std::max(vmax, v);
            }
            if (vmin > vmax) { vmin = 0.0; vmax = 0.0; }        // nothing kept
            p = make_qparam(vmin, vmax);
          }
          for (int g = g0; g < g0 + rep; ++g) {
            qr[2 * g] = p.s_bits;
            qr[2 * g + 1] = zero_bits(p.z);
          }
        }
      }
      int64_t t = (int64_t)row_ptr[r];                            // global slot id
#ifdef EGT_HOST_SIMD
      if (simd) {
        // (a row starts on a whole index word and a whole byte of values)
        egt_simd::with_n(n_row, [&](auto c) {
          constexpr int n = decltype(c)::n;
#ifdef EGT_HOST_SIMD512
          if (wide && val_kind == EGT_VAL_FP16) egt_simd512::pack_row_fp16<n>(wr, mr, cols, (uint8_t *)(vals16 + t), (uint8_t *)(idx + (t >> 3)));
          else if (wide) egt_simd512::pack_row_int4<n>(wr, mr, cols, group, qr, val_kind == EGT_VAL_INT4_PAIRED, vals8 + (t >> 1),
                                                       (uint8_t *)(idx + (t >> 3)));
          else
#endif
          if (val_kind == EGT_VAL_FP16) egt_simd::pack_row_fp16<n>(wr, mr, cols, (uint8_t *)(vals16 + t), (uint8_t *)(idx + (t >> 3)));
          else egt_simd::pack_row_int4<n>(wr, mr, cols, group, qr, val_kind == EGT_VAL_INT4_PAIRED, vals8 + (t >> 1),
                                          (uint8_t *)(idx + (t >> 3)));
        });
        continue;
      }
#endif
      uint32_t word = 0;
      for (int c = 0; c < cols; c += 4) {
        const int set = choose4(mr + c, n_row);
        const QParam p = qr ? stored_qparam(qr + 2 * (c / group)) : QParam{};       // (group % 4 == 0)
        for (int j = 0; j < 4; ++j) {
          if (!(set >> j & 1)) continue;
          word |= (uint32_t)j << (2 * (t & 7));
          const bool kept = mr[c + j] != 0;
          if (val_kind == EGT_VAL_FP16) {
            vals16[t] = kept ? wr[c + j] : (uint16_t)0;
          } else {
            const int q = kept ? make_code(half_to_double(wr[c + j]), p) : p.z;
            // (a row is a whole number of 4-byte words and no other row shares them: the
            //  first nibble of a byte sets it, the second is or-ed in)
            int shift;
            const int64_t b = nibble_byte(t, val_kind, shift);
            vals8[b] = shift ? (uint8_t)(vals8[b] | (q << 4)) : (uint8_t)q;
          }
          if ((t & 7) == 7) { idx[t >> 3] = (uint16_t)word; word = 0; }
          ++t;
        }
      }
    }
  };
  parallel_rows(rows, cols, encode);
  out->rows = rows; out->cols = cols; out->n_keep = row_n_keep ? 0 : n_keep;
  out->group_size = group; out->val_kind = val_kind;
  out->total_slots = row_ptr[rows];
  return EGT_OK;
}

}  // namespace

extern "C" {

egt_status egt_unpack_2bitcsr(const egt_2bitcsr *in, uint16_t *w_dense, int64_t ldw,
                              uint8_t *mask, int64_t ldm) {
  if (!in) return EGT_ERR_NULL;
  const int rows = in->rows, cols = in->cols, group = in->group_size;
  const bool mixed = in->n_keep == 0;                  // rows of different lengths
  egt_status st = check_shape(rows, cols, mixed ? 1 : in->n_keep, group, in->val_kind);
  if (st != EGT_OK) return st;
  if (!in->row_ptr || !in->values || !in->idx) return EGT_ERR_NULL;
  if (is_int4(in->val_kind) && !in->qparams) return EGT_ERR_NULL;
  if ((w_dense && ldw < cols) || (mask && ldm < cols)) return EGT_ERR_SHAPE;
  // row_ptr: the uniform progression, or a running sum of whole rows that ends at total_slots
  const int64_t quarter = cols / 4;
  for (int r = 0; r < rows; ++r) {
    const int64_t len = (int64_t)in->row_ptr[r + 1] - (int64_t)in->row_ptr[r];
    if (mixed) {
      if (quarter == 0 || len % quarter != 0 || len / quarter < 1 || len / quarter > 4) return EGT_ERR_BUFFER;
    } else if (in->row_ptr[r] != (uint32_t)((int64_t)r * in->n_keep * quarter) || len != in->n_keep * quarter) {
      return EGT_ERR_BUFFER;
    }
  }
  auto n_of = [=](int r) { return mixed ? (int)((int64_t)(in->row_ptr[r + 1] - in->row_ptr[r]) / quarter) : in->n_keep; };
  if (rows > 0 && in->row_ptr[0] != 0) return EGT_ERR_BUFFER;
  if (mixed && in->row_ptr[rows] != in->total_slots) return EGT_ERR_BUFFER;
  // offsets of a 4-group must ascend strictly
  std::atomic<int> err(EGT_OK);
  const uint16_t *idx = in->idx;
  const uint32_t *row_ptr = in->row_ptr;
  auto ascending = [&](int r0, int r1) {
    for (int r = r0; r < r1; ++r) {
      int64_t t = (int64_t)row_ptr[r];
      const int n_row = n_of(r);
#ifdef EGT_HOST_SIMD
      if (egt_simd::available()) {
        const uint8_t *ix = (const uint8_t *)(idx + (t >> 3));
        if (!egt_simd::with_n(n_row, [&](auto c) { return egt_simd::offsets_ascend<decltype(c)::n>(ix, cols); })) err.store(EGT_ERR_BUFFER);
        continue;
      }
#endif
      for (int c = 0; c < cols; c += 4) {
        int prev = -1;
        for (int k = 0; k < n_row; ++k, ++t) {
          const int off = (idx[t >> 3] >> (2 * (t & 7))) & 3;
          if (off <= prev) err.store(EGT_ERR_BUFFER);
          prev = off;
        }
      }
    }
  };
  parallel_rows(rows, cols, ascending);
  if (err.load() != EGT_OK) return (egt_status)err.load();

  const uint8_t *vals8 = (const uint8_t *)in->values;
  const uint16_t *vals16 = (const uint16_t *)in->values;
  const uint16_t *qparams = in->qparams;
  const int val_kind = in->val_kind;
  const int G = is_int4(val_kind) ? cols / group : 0;
  auto decode = [=](int r0, int r1) {
#ifdef EGT_HOST_SIMD
    const bool simd = egt_simd::available() && (!is_int4(val_kind) || group % 8 == 0);
#endif
    for (int r = r0; r < r1; ++r) {
      const int n_row = n_of(r);
#ifdef EGT_HOST_SIMD
      bool plain = simd;                               // zero points are integers in 0..15 and scales finite (of any encoder)
      for (int g = 0; g < G && plain; ++g) {
        const uint16_t *p = qparams + ((int64_t)r * G + g) * 2;
        const float z = egt_simd::half_to_float(p[1]);
        plain = half_is_finite(p[0]) && z >= 0.0f && z <= 15.0f && z == (float)(int)z;
      }
      if (plain) {
        const int64_t t = (int64_t)row_ptr[r];
        egt_simd::with_n(n_row, [&](auto c) {
          egt_simd::unpack_row<decltype(c)::n>(val_kind == EGT_VAL_FP16 ? (const uint8_t *)(vals16 + t) : vals8 + (t >> 1),
                                               (const uint8_t *)(idx + (t >> 3)), cols, group, is_int4(val_kind) ? qparams + (int64_t)r * G * 2 : nullptr,
                                               val_kind == EGT_VAL_INT4_PAIRED, w_dense ? w_dense + (int64_t)r * ldw : nullptr,
                                               mask ? mask + (int64_t)r * ldm : nullptr);
        });
        continue;
      }
#endif
      if (w_dense) std::memset(w_dense + (int64_t)r * ldw, 0, sizeof(uint16_t) * (size_t)cols);
      if (mask) std::memset(mask + (int64_t)r * ldm, 0, (size_t)cols);
      int64_t t = (int64_t)row_ptr[r];
      for (int c = 0; c < cols; c += 4) {
        for (int k = 0; k < n_row; ++k, ++t) {
          const int col = c + ((idx[t >> 3] >> (2 * (t & 7))) & 3);
          if (mask) mask[(int64_t)r * ldm + col] = 1;
          if (!w_dense) continue;
          uint16_t bits;
          if (val_kind == EGT_VAL_FP16) {
            bits = vals16[t];
          } else {
            int shift;
            const int64_t b = nibble_byte(t, val_kind, shift);
            const int q = (vals8[b] >> shift) & 15;
            const uint16_t *p = qparams + ((int64_t)r * G + col / group) * 2;
            bits = double_to_half(half_to_double(p[0]) * ((double)q - half_to_double(p[1])));
          }
          w_dense[(int64_t)r * ldw + col] = bits;
        }
      }
    }
  };
  parallel_rows(rows, cols, decode);
  return EGT_OK;
}

egt_status egt_quant_int4(const uint16_t *w, int64_t ldw, int rows, int cols, int group,
                          uint8_t *q, uint16_t *qparams) {
  if (!w || !q || !qparams) return EGT_ERR_NULL;
  if (rows < 0 || cols < 0 || group <= 0 || group % 4 != 0 || cols % group != 0 || ldw < cols)
    return EGT_ERR_SHAPE;
  std::atomic<int> err(EGT_OK);
  auto finite = [&](int r0, int r1) {
    for (int r = r0; r < r1; ++r) {
#ifdef EGT_HOST_SIMD
      if (egt_simd::available() && egt_simd::all_finite(w + (int64_t)r * ldw, cols)) continue;
#endif
      for (int c = 0; c < cols; ++c)
        if (!half_is_finite(w[(int64_t)r * ldw + c])) err.store(EGT_ERR_NONFINITE);
    }
  };
  parallel_rows(rows, cols, finite);
  if (err.load() != EGT_OK) return (egt_status)err.load();
  const int G = cols / group;
  auto quantise = [=](int r0, int r1) {
#ifdef EGT_HOST_SIMD
    const bool simd = egt_simd::available() && group % 8 == 0;
#endif
#ifdef EGT_HOST_SIMD512
    const bool wide = simd && egt_simd512::available() && group % 64 == 0;
#endif
    for (int r = r0; r < r1; ++r) {
      const uint16_t *wr = w + (int64_t)r * ldw;
      for (int g = 0; g < G; ++g) {
#ifdef EGT_HOST_SIMD
        if (simd) {
          float lo, hi;
#ifdef EGT_HOST_SIMD512
          if (wide) egt_simd512::extrema(wr + g * group, nullptr, group, lo, hi);
          else
#endif
          egt_simd::extrema(wr + g * group, nullptr, group, lo, hi);
          const QParam p = make_qparam_simd(lo, hi);
          uint16_t *o = qparams + ((int64_t)r * G + g) * 2;
          o[0] = p.s_bits;
          o[1] = zero_bits(p.z);
          uint8_t *to = q + (int64_t)r * (cols / 2) + g * group / 2;
#ifdef EGT_HOST_SIMD512
          if (wide) egt_simd512::quant_group(wr + g * group, group, (float)p.s, p.z, to);
          else
#endif
          egt_simd::quant_group(wr + g * group, group, (float)p.s, p.z, to);
          continue;
        }
#endif
        double vmin = INFINITY, vmax = -INFINITY;
        for (int c = g * group; c < (g + 1) * group; ++c) {
          const double v = half_to_double(wr[c]);
          vmin = std::min(vmin, v);
          vmax = std::max(vmax, v);
        }
        const QParam p = make_qparam(vmin, vmax);
        uint16_t *o = qparams + ((int64_t)r * G + g) * 2;
        o[0] = p.s_bits;
        o[1] = zero_bits(p.z);
        for (int c = g * group; c < (g + 1) * group; c += 2) {
          const int q0 = make_code(half_to_double(wr[c]), p);
          const int q1 = make_code(half_to_double(wr[c + 1]), p);
          q[(int64_t)r * (cols / 2) + c / 2] = (uint8_t)(q0 | (q1 << 4));
        }
      }
    }
  };
  parallel_rows(rows, cols, quantise);
  return EGT_OK;
}

egt_status egt_fit_verify_cost(const int *m, const double *t, int n, double *a, double *b) {
  if (!m || !t || !a || !b) return EGT_ERR_NULL;
  if (n < 2) return EGT_ERR_SHAPE;
  double sm = 0, st = 0, smm = 0, smt = 0;
  for (int i = 0; i < n; ++i) {
    if (m[i] < 1 || !std::isfinite(t[i])) return EGT_ERR_SHAPE;
    sm += m[i]; st += t[i]; smm += (double)m[i] * m[i]; smt += (double)m[i] * t[i];
  }
  const double den = n * smm - sm * sm;
  if (den == 0.0) return EGT_ERR_SHAPE;               // all M equal: no slope
  *b = (n * smt - sm * st) / den;
  *a = (st - *b * sm) / n;
  return EGT_OK;
}

egt_status egt_trigger_depth(double t_ar, double a, double b, const int *cand, const int *remaining,
                             int depth, int *best, double *benefit) {
  if (!cand || !remaining || !best || !benefit) return EGT_ERR_NULL;
  if (depth < 1) return EGT_ERR_SHAPE;
  int arg = -1;
  double top = 0.0;
  for (int d = 0; d < depth; ++d) {
    if (cand[d] < 0 || remaining[d] < 0) return EGT_ERR_SHAPE;
    const double gain = remaining[d] * t_ar - (a + b * cand[d]);
    if (gain > top) { top = gain; arg = d; }          // first depth wins among equal gains
  }
  *best = arg;
  *benefit = top;
  return EGT_OK;
}

}  // extern "C"

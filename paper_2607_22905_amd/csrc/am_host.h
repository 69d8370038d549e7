// Host-side structure of AlgMortar: validation, partitioners, permutation,
// interface edge sets and mortar numbering (paper Sec. 3.1-3.2), and the
// device-oriented layout plan derived from them.  Plain C++17, no HIP.
#pragma once

#include <algorithm>

#include <atomic>
#include <condition_variable>
#include <cstdint>
#include <functional>
#include <mutex>
#include <string>
#include <system_error>
#include <thread>
#include <vector>

#include "algmortar.h"

namespace am {

// Host threads for the set-up loops: ALGMORTAR_HOST_THREADS if set, else the
// hardware threads, at most 16.
int host_threads();

// The threads of one set-up call: made at its first parallel loop, waiting
// between the loops, joined with the call.  (A set-up has a dozen loops of
// 0.1-0.5 ms; 15 new threads for each of them took about as long again.)  The
// object lives on the caller's stack and belongs to the calling thread, so
// set-ups on several threads have a team each; a loop inside a loop, or
// without a team, makes its own threads.
class HostTeam {
 public:
  HostTeam() : prev_(current()) { current() = this; }
  ~HostTeam() {
    current() = prev_;
    {
      std::lock_guard<std::mutex> l(m_);
      stop_ = true;
    }
    wake_.notify_all();
    for (auto& th : pool_) th.join();
  }
  HostTeam(const HostTeam&) = delete;
  HostTeam& operator=(const HostTeam&) = delete;
  static HostTeam*& current() {
    static thread_local HostTeam* t = nullptr;
    return t;
  }
  // work() on the caller and up to nt - 1 of the team's threads; returns when
  // every call of it has returned (false: not run, a loop is under way)
  bool run(const std::function<void()>& work, int nt) {
    {
      std::lock_guard<std::mutex> l(m_);
      if (job_) return false;
      job_ = &work;
      seats_ = nt - 1;
      ++epoch_;
    }
    struct Finish {  // also where work() throws here: the others still use it
      HostTeam* t;
      ~Finish() {
        std::unique_lock<std::mutex> l(t->m_);
        t->job_ = nullptr;  // a thread that wakes from now on finds nothing to do
        t->done_.wait(l, [this] { return t->active_ == 0; });
      }
    } finish{this};
    try {
      while ((int)pool_.size() < nt - 1) pool_.emplace_back([this] { serve(); });
    } catch (const std::system_error&) {  // no more threads: with those there are
    }
    wake_.notify_all();
    work();
    return true;
  }

 private:
  void serve() {
    uint64_t seen = 0;
    std::unique_lock<std::mutex> l(m_);
    for (;;) {
      wake_.wait(l, [&] { return stop_ || (job_ && epoch_ != seen && seats_ > 0); });
      if (stop_) return;
      seen = epoch_;
      --seats_;
      ++active_;
      const std::function<void()>* w = job_;
      l.unlock();
      (*w)();
      l.lock();
      if (--active_ == 0) done_.notify_one();
    }
  }
  std::mutex m_;
  std::condition_variable wake_, done_;
  std::vector<std::thread> pool_;
  const std::function<void()>* job_ = nullptr;
  uint64_t epoch_ = 0;
  int seats_ = 0, active_ = 0;
  bool stop_ = false;
  HostTeam* prev_;
};

// Runs f(i) for every i in [0, n) on up to host_threads() threads (the
// caller's included), handing out chunks of `grain` indices in increasing
// order.  f must write only data that belongs to its own index; results are
// then independent of the thread count and the schedule.
template <typename F>
void parallel_for(int64_t n, int64_t grain, F&& f) {
  const int nt = (int)std::min<int64_t>(host_threads(), (n + grain - 1) / grain);
  if (nt <= 1) {
    for (int64_t i = 0; i < n; ++i) f(i);
    return;
  }
  std::atomic<int64_t> next{0};
  auto work = [&]() {
    for (;;) {
      const int64_t lo = next.fetch_add(grain);
      if (lo >= n) return;
      const int64_t hi = std::min(n, lo + grain);
      for (int64_t i = lo; i < hi; ++i) f(i);
    }
  };
  if (HostTeam* t = HostTeam::current(); t && t->run(work, nt)) return;
  std::vector<std::thread> pool;
  pool.reserve(nt - 1);
  for (int t = 1; t < nt; ++t) pool.emplace_back(work);
  work();
  for (auto& th : pool) th.join();
}

struct HostCSR {
  int64_t n = 0, nnz = 0;
  const int64_t* rp = nullptr;
  const int32_t* ci = nullptr;
  const double* v = nullptr;
};

// Validates pattern (monotone row_ptr, strictly ascending in-range columns),
// finiteness, bitwise symmetry of values (a missing transpose counts as 0)
// and the sign of every off-diagonal (< 0 or an explicit zero).
am_status validate_csr(const HostCSR& A, std::string& err);
am_status validate_partition(int64_t n, const int32_t* part, int32_t nparts, std::string& err);

struct Structure {
  int64_t n = 0;
  int32_t m = 0;
  std::vector<int32_t> part;      // [n]
  std::vector<int32_t> perm;      // [n] perm[new] = old (ascending inside a part)
  std::vector<int64_t> sub_ptr;   // [m+1]
  std::vector<int32_t> edge_k, edge_l;  // [|E|] original indices, k in the lower part
  std::vector<double> edge_a;           // [|E|] a_kl
  std::vector<int64_t> iface_ptr;       // [NL+1]
  std::vector<int32_t> iface_ij;        // [2 NL]
  std::vector<int64_t> isub_ptr;        // [m+1]   I_i as CSR
  std::vector<int32_t> isub_list;       // [2 NL]  ascending basis ids per part
  int64_t n_iface() const { return (int64_t)iface_ptr.size() - 1; }
  int64_t n_edges() const { return (int64_t)edge_k.size(); }
};

am_status build_structure(const HostCSR& A, const int32_t* part, int32_t nparts, int mortar,
                          Structure& st, std::string& err);

am_status partition_blocks(int32_t nx, int32_t ny, int32_t nz, int32_t bx, int32_t by,
                           int32_t bz, int32_t* part, int32_t* nparts, std::string& err);
am_status partition_bisect(const HostCSR& A, int32_t lo, int32_t hi, uint64_t seed,
                           int32_t* part, int32_t* nparts, std::string& err);

uint64_t splitmix64(uint64_t x);

// Band layout of the local factors.  Inside every subdomain the device uses
// an ordering (identity or reverse Cuthill-McKee, whichever has the smaller
// bandwidth) and a window width Wp = 64 * ceil(bandwidth / 64).
// Whether the block-inverse kernels (window 64) take a subdomain of np padded
// rows, kc couplings of a row per side and ni basis functions: they index its
// couplings, basis functions and 16 columns of a vector with 32 bits.
inline bool tri_indexable(int64_t np, int64_t kc, int64_t ni) {
  constexpr int64_t lim = INT32_MAX;
  return np <= lim / 16 && kc <= lim / (2 * std::max<int64_t>(np, 1)) &&
         ni <= lim / std::max<int64_t>(np, 1);
}

struct LocalPlan {
  std::vector<int32_t> dperm;      // [n] device order: dperm[new] = old
  std::vector<int32_t> dpos;       // [n] inverse: dpos[old] = new
  std::vector<int32_t> wp;         // [m] window width per subdomain
  std::vector<int64_t> roff;       // [m+1] padded row offsets (rows padded to a multiple of 64)
  // [m+1] element offsets of the factors: 2048 per 64-row block (window 64,
  // packed block inverses), 128 per row (window 128, band)
  std::vector<int64_t> fac_off;
  std::vector<int64_t> band_off;   // [m+1] element offsets of the band factors = padded rows * wp
  // window 64: most couplings of a row to the block before or after its own
  // (window 128: 0), and [m+1] element offsets of the coupling lists (2 * cpl_k * padded rows)
  std::vector<int32_t> cpl_k;
  std::vector<int64_t> cpl_off;
  int32_t max_wp = 64;
  int32_t max_ni = 0;              // max |I_i|
  int32_t max_sub = 0;             // max subdomain size
};

am_status plan_local(const HostCSR& A, const Structure& st, LocalPlan& lp, std::string& err);

// Nested-dissection layout of the interface system (iface_nd.cpp): the basis
// functions in an order where the first nrows form nblk mutually uncoupled
// diagonal blocks of S and the last ntop are the separators above them.
struct IfaceND {
  int32_t depth = 0;              // dissection levels above the blocks
  int32_t nblk = 0;
  int64_t nrows = 0;              // rows in blocks
  int64_t ntop = 0;               // separator ("top") rows
  std::vector<int32_t> order;     // [NL] ND position -> basis function
  std::vector<int64_t> blk_off;   // [nblk+1] ND positions of the blocks
  std::vector<int64_t> pad_off;   // [nblk+1] positions with every block padded to 64 rows;
                                  // pad_off[nblk] is where the top rows start
  int64_t ld = 0;                 // padded dimension, a multiple of 64
  std::vector<int64_t> t_ptr;     // [ntop+1] per top row ..
  std::vector<int64_t> t_pos;     // .. the ND positions (< nrows) of the block rows it couples to
  std::vector<int64_t> b_ptr;     // [nrows+1] per block row ..
  std::vector<int64_t> b_top;     // .. the top indices (ND position - nrows) it couples to
};

// Builds the layout from the interface structure; blocks have at most
// max_rows rows and the padded dimension is at most max_growth times that of
// S (the depth minimises the bytes of one solve under these limits).
// AM_ERR_UNSUPPORTED when no depth meets the limits.
am_status build_iface_nd(const Structure& st, int64_t max_rows, double max_growth, IfaceND& nd,
                         std::string& err);

}  // namespace am

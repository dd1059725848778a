// Matrix-free solver of the projected Kernel-SHAP normal equations (Sec. 3.5:
// large systems are fitted iteratively instead of being factored).
#pragma once

#include <memory>

#include "common.h"

namespace gnnshap {

// Device state of one iterative solve.
struct CgState {
  double rr0;      // squared norm of the initial residual
  int32_t last;    // passes of iterations beyond this one do nothing: set by the pass that stops
  int32_t iters;   // iterations run
  int32_t status;  // 0 converged, 1 iteration limit, 2 lost positive curvature
  int32_t pad;
};

// Buffers of the iterative solver, carved from the solve workspace.
struct CgWs {
  double* x;       // M: psi
  double* r;       // M + 1: residual, then a zero
  double* p;       // M: search direction
  double* s;       // M: A p
  double* us;      // rs: R r of the sparse rows
  double* qd;      // parts x (4 words_per_row + 5) x 256: digit sums of R^T u by part (parts > 1)
  char* rdig;      // digits of r, MFMA operands over the players
  char* udig;      // digits of R r of the bit rows, MFMA operands over these rows
  double* uu;      // (2 nbits + rbd0) x 2: partial |u|^2 and |m|.u
  double* rr;      // 3 x 2 words_per_row: partial r.r of iterations t mod 3
  double* mx;      // 2 x 2 x 2 words_per_row: largest |r| and |s|, by iteration parity
  double* hist;    // 2: step lengths of even and odd iterations
  int32_t* ex;     // 3: fixed-point exponents of r (even and odd iterations) and u
  int32_t* sz;     // kr: sizes of the random representative rows
  uint64_t* blocked;  // nrb x words_per_row x 64: the random rows in row blocks
  CgState* st;
  // sparse rows (random rows [0, rs), the smallest coalitions): their players
  int64_t* ell_ptr;   // rbd0 + 1: entries per row of the blocks of 64 sparse rows before each
  int32_t* ell_idx;   // nell: players of the sparse rows, ascending, padded with M; entry i of a block's rows contiguous
  int64_t* csc_ptr;   // M + 1: rows of each player, ascending
  int32_t* csc_row;   // nnz
  int32_t* segcnt;    // 8 x max(rs, M): per-segment list lengths while the lists are built
};

// Launch shape of the iterative solver for M players and kr random
// representative rows (words_per_row mask words per row).
struct CgShape {
  int64_t M, wpr, kr, nrb;
  int64_t rs, nnz;         // sparse rows [0, rs) (whole row blocks), their players
  int64_t rbd0;            // first row block of the bit products (rs / 64)
  int64_t nbits;           // row blocks of the bit products
  int64_t parts;           // parts of them in pass B (1: its own workgroups take all)
  int64_t nell;            // room for the padded entries of the sparse rows' lists
};
// The split of the random rows [rb0, rb0 + kr) of a class table into sparse
// rows (coalition size at most M / kSparseDiv, whole blocks of 64 rows) and
// bit rows; the shape of the solver for that split.
CgShape cg_shape(int64_t M, int64_t wpr, int64_t kr, int64_t rb0, const gnnshap_class* classes, int64_t ncls);
CgWs cg_carve(Carver& c, const CgShape& sh);

// The problem handed over by the solve entry point: the bit-transposed random
// rows T (word rb of the 64 players of block w contiguous, block after block:
// T[(w nrb + rb) 64 + j % 64], zero beyond M), the same rows in row blocks (word w of the 64 rows of
// block rb contiguous, rows beyond kr zero),
// the summed right-hand side dv (M, before centring) with its per-block sums
// bsum (nb of them), the class table (device) and the enumerated part alpha.
struct CgProblem {
  const uint64_t* T;
  const uint64_t* blocked;
  const double* dv;
  const double* bsum;
  int64_t nb;
  const gnnshap_class* classes;
  int64_t ncls;
  int64_t rb0;          // first random representative row
  double alpha;         // enumerated classes: their projected Gram is alpha P
  double wr;            // weight of every random row
  const float* fef;     // f(empty), f(full)
  float* phi;
  int32_t* info;
};

// Several iterative solves advanced together on one stream.  Every chunk of
// iterations is one launch per pass for all members (one flat grid over the
// members' workgroups), so the members share the GPU inside each launch and
// the short passes of all members cost one launch latency instead of one
// each.  add() queues a new member's set-up on the stream (at most
// kCgGroupMax members at once); step() first waits for the chunk before the
// last one queued and reads the members' stop flags, queues phi and info of
// every member that has stopped and releases it, then queues the next chunk
// of iterations for the members left (each at its own iteration count), so
// at most two chunks are in flight; ready() says whether step() would return
// without waiting on the device.  Once empty() every member's phi and info
// are queued on the stream.  Each member holds a mapped stop flag; at most
// 16 are held per host thread at once.
constexpr int kCgGroupMax = 6;

class CgGroup {
 public:
  CgGroup();
  ~CgGroup();
  CgGroup(const CgGroup&) = delete;
  CgGroup& operator=(const CgGroup&) = delete;
  void set_stream(hipStream_t s) { s_ = s; }
  hipStream_t stream() const { return s_; }
  int add(const CgProblem& pr, const CgShape& sh, const CgWs& w);
  int size() const;
  bool empty() const { return size() == 0; }
  bool full() const { return size() >= kCgGroupMax; }
  bool ready() const;
  int step();
  // iterations of the member released last (-1 before any)
  int64_t last_iters() const { return last_iters_; }

 private:
  struct State;
  std::unique_ptr<State> st_;
  hipStream_t s_ = nullptr;
  int64_t last_iters_ = -1;
};

// Conjugate gradients on 1-perp for one system; returns once its phi and
// info are queued on `s` (the host waits on the stream for the stopping
// test).  *iters_out (may be null) receives the iterations run.
int cg_solve(const CgProblem& pr, const CgShape& sh, const CgWs& w, hipStream_t s, int64_t* iters_out);

// Largest number of players a plan's system is solved by factorisation for;
// larger systems are solved iteratively (Sec. 3.5 switches at 5000, the
// default when the plan's field is 0 or negative).
inline int64_t iterative_threshold(const gnnshap_sample_plan* p) {
  return p->iterative_threshold > 0 ? p->iterative_threshold : 5000;
}

}  // namespace gnnshap

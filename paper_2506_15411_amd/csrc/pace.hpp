// How many iterations a blocking solve enqueues ahead of the device.
#pragma once

#include <algorithm>
#include <cmath>

namespace cbs {

// Two quanta of check_every iterations in flight keep the device at work while the
// host reads the state of the one before, but what is enqueued past the iteration
// that meets tol still runs to its stop test, and a pass that looks at the flag behind
// its loads reads its field for that: with whole quanta of 20, 1.4 to 2 ms at 189 x
// 189 x 121 and 121 x 189 x 100, 0.6 at 128^3; a warm start that converges at once
// took 2.88 ms at 189 x 189 x 121.  So the quanta are sized by the residual: its rate
// over the last two that were read says how many iterations are left, and no more
// than those are enqueued.  Until two have been read one quantum is in flight, a short
// one after a warm start, which may converge at any iteration.  With tol = 0, or a
// residual that does not fall, nothing is ever left out.  What stays behind then: 0 to
// 0.3 ms and 0.06, and the warm start takes 0.61 ms.
class Pace {
 public:
  // long_iter: an iteration takes longer than the host's reading of one
  Pace(double tol, int check_every, bool warm, bool long_iter)
      : tol_(tol), every_(check_every), quarter_(std::max(1, check_every / 4)),
        least_(long_iter ? 1 : quarter_), warm_(warm) {
    if (!(tol > 0.0)) left_ = INFINITY;
  }
  // the residual eta after iteration iter, as the host reads it
  void read(int iter, double eta) {
    if (tol_ > 0.0 && iter > iter_) {
      if (iter_ > 0)
        left_ = eta < eta_ ? std::log(eta / tol_) * (iter - iter_) / std::log(eta_ / eta) : INFINITY;
      iter_ = iter;
      eta_ = eta;
    }
  }
  // iterations to enqueue next when `ahead` of them are in flight past the last that
  // was read (none: something has to be enqueued); 0: wait.  Where iterations are as
  // short as a reading, less than a quarter of a quantum is not worth one.
  int next(int ahead) const {
    if (left_ < 0.0) return ahead ? 0 : warm_ ? quarter_ : every_;
    const double q = std::min((double)every_, std::ceil(left_) - ahead);
    if (q >= least_) return (int)q;
    return ahead ? 0 : least_;
  }

 private:
  double tol_;
  int every_, quarter_, least_;
  bool warm_;
  int iter_ = 0;
  double eta_ = 0.0;
  double left_ = -1.0;   // iterations left after iter_; -1: not known yet
};

}  // namespace cbs

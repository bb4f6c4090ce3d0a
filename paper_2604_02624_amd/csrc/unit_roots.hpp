// Roots of unity of one transform length on the host, in double precision, from which every table of the
// length is taken.  An eighth of the circle is evaluated and mirrored: creating a plan spends most of its
// own time on these (512 x 512, padded: 108 us with a sine and a cosine per table entry, 48 this way).
#pragma once

#include <cmath>
#include <vector>

namespace dpx {

class UnitRoots {
 public:
  // M: a multiple of eight
  explicit UnitRoots(int M) : m_(M), c_(M), s_(M) {
    for (int k = 0; k <= M / 8; ++k) {
      const double ang = 6.283185307179586476925286766559 * k / M;
      const double c = std::cos(ang), s = std::sin(ang);
      set(k, c, s);
      set(M / 4 - k, s, c);
      set(M / 4 + k, -s, c);
      set(M / 2 - k, -c, s);
      set(M / 2 + k, -c, -s);
      set(3 * M / 4 - k, -s, -c);
      set(3 * M / 4 + k, s, -c);
      if (k > 0) set(M - k, c, -s);
    }
  }
  // index of num / den of a turn; den divides M
  int index(long long num, long long den) const { return static_cast<int>(num % den * (m_ / den)); }
  int length() const { return m_; }
  // cosine and sine of k / M of a turn, 0 <= k < M
  double cos(int k) const { return c_[k]; }
  double sin(int k) const { return s_[k]; }

 private:
  void set(int k, double c, double s) {
    c_[k] = c;
    s_[k] = s;
  }
  int m_;
  std::vector<double> c_, s_;
};

}  // namespace dpx

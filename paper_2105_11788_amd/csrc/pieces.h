// Which pieces of one region are in use: places only, no memory of its own.
#pragma once

#include <stddef.h>

#include <vector>

namespace bisim {

// Pieces are cut one behind the other.  A piece given back makes room once all
// that were cut after it have been given back too (temporaries are, in some
// order, before anything that stays is cut), so nothing is searched and a
// caller that cuts and gives back the same pieces again and again takes the
// same places.
class Pieces {
 public:
  explicit Pieces(size_t capacity) : capacity_(capacity) {}

  // the place of a new piece; false if the rest of the region is too small
  bool cut(size_t bytes, size_t* at) {
    if (bytes > capacity_ - used_) return false;
    pieces_.push_back({used_, false});
    *at = used_;
    used_ += bytes;
    return true;
  }
  void give_back(size_t at) {
    for (size_t i = pieces_.size(); i-- > 0;)
      if (pieces_[i].at == at) {
        pieces_[i].free = true;
        break;
      }
    while (!pieces_.empty() && pieces_.back().free) {
      used_ = pieces_.back().at;
      pieces_.pop_back();
    }
  }
  size_t used() const { return used_; }

 private:
  struct Piece {
    size_t at;
    bool free;
  };
  size_t capacity_, used_ = 0;
  std::vector<Piece> pieces_;
};

}  // namespace bisim

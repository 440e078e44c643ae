// Host-only logic of the C interface (see host_logic.cpp): no HIP types here.
#pragma once
#include <stdint.h>
#include <string>
#include <vector>
#include "actionstudio.h"

// one run of tokens of the packed stream: destination offset, source offset in turn_tokens (-1: pad), mask bit
struct Piece { int32_t dst, src; uint8_t mask; };

// Every function returns AS_OK or a negative as_status and, on failure, a message in *err.
int check_config(const as_model_config* c, std::string* err);
// Validation, row assignment (policy), piece list, segment table and loss-free-segment flags of as_pack / as_pack_policy.
int pack_plan(int vocab, const int32_t* turn_tokens, const int32_t* turn_offsets,
              const uint8_t* turn_roles, const int32_t* traj_offsets, int32_t n_traj,
              int32_t T, int32_t max_rows, int32_t truncate, int32_t policy, std::vector<Piece>& pieces,
              std::vector<int32_t>& cu, std::vector<uint8_t>& skip, int32_t* n_rows, int32_t* n_consumed,
              int32_t* traj_row, std::string* err);
// cu[0..S] is a partition of [0, N) into segments none of which crosses a multiple of T; *max_seg = longest segment
int check_cu(const int32_t* cu, int32_t S, int64_t N, int32_t T, int* max_seg, std::string* err);

// Launches over many items, as many at a time as a kernel argument holds (Batch: m[CAP], n, n_tiles; an item's first_tile is set here).
// add() launches the collected items first when one more would exceed CAP or max_tiles.  Once a launch has failed nothing is
// collected any more; finish() launches the rest and returns the first status that was not AS_OK.
template <typename Batch, int CAP, typename Launch> class BatchedLaunches {
 public:
  BatchedLaunches(int64_t max_tiles, Launch launch) : max_tiles_(max_tiles), launch_(launch) { b_.n = 0; b_.n_tiles = 0; }
  template <typename Item> void add(const Item& item, int64_t tiles) {
    if (!rc_ && b_.n > 0 && (b_.n == CAP || b_.n_tiles + tiles > max_tiles_)) send();
    if (rc_) return;
    b_.m[b_.n] = item; b_.m[b_.n].first_tile = b_.n_tiles;
    b_.n++; b_.n_tiles += (int)tiles;
  }
  int finish() { if (!rc_ && b_.n > 0) send(); return rc_; }
 private:
  void send() { rc_ = launch_(b_); b_.n = 0; b_.n_tiles = 0; }
  Batch b_; int64_t max_tiles_; Launch launch_; int rc_ = AS_OK;
};

// Internal definitions shared by the host planner, the launchers and the kernels.
#pragma once
#include <cstddef>
#include <cstdint>
#include <memory>
#include <string>
#include <vector>

#include "ca_attention.h"

namespace ca {

// Tile geometry.  Every document's sorted query rows occupy a run of "slots" padded to the plan's slot alignment
// (at most SLOT_ALIGN), so that forward tiles and backward q blocks (BWD_BQ slots) both tile the same arrays.
constexpr int SLOT_ALIGN = 256;
constexpr int FWD_BM = 256;  // query rows per forward work unit (8 row groups x 32)
constexpr int FWD_BN = 64;   // keys per forward inner step
constexpr int BWD_BN = 128;  // keys owned by one backward work unit (4 waves x 32)
constexpr int BWD_BQ = 64;   // query rows per backward inner step

// One workgroup of the forward / dQ kernels, or two (halves; always in the joint backward launch): 8 row groups of 32 slots, one or
// two to a wave.  A full tile of a document is 256 slots of one query head (hp = 1).  The slots a document has left over
// after its full tiles are covered by head-packed units instead: 256 / hp slots of hp consecutive query heads of one KV
// group (they read the same K/V), row group w taking slots slot0 + 32 (w / hp) .. of head  head + w % hp  - so that
// short documents keep all waves busy too.
struct FwdUnit {
  int32_t slot0;    // first slot of the unit
  int32_t kv_row0;  // packed KV row of the document's token 0
  int32_t n_keys;   // keys the unit needs: max position + 1
  int32_t head;     // first query head
  int32_t hp;       // query heads per unit: 1, 2, 4 or 8
  // Pieces (see CombineUnit).  A unit that attends a window of its keys: kv_row0 and n_keys are the window's, and key0
  // is the document position of its first key (a multiple of FWD_BN).  Its results go, as they stand in the
  // accumulators, to block `part` of the workspace's partial results; -1 in a unit that attends all its keys.
  int32_t key0;
  int32_t part;
  int32_t rows;  // slots of the unit that hold rows (padding is behind them)
};
constexpr int FWD_UNIT_INTS = 5;  // leading fields reported by ca_plan_fwd_units

struct BwdUnit {  // one (KV tile, KV head)
  int32_t slot_begin;  // first slot of the first q block that sees this KV tile
  int32_t slot_end;    // end of the document's slots
  int32_t slot_full;   // first q block (slot index) from which every slot sees all keys of the tile
  int32_t kv_row;      // packed KV row of the tile's first key
  int32_t n_valid;     // valid keys in the tile
  int32_t key_pos0;    // document position of the tile's first key
  int32_t kv_head;
  // Chains.  The first n_bwd_workgroups units of the list are one workgroup each; a workgroup goes on with the
  // `count - 1` units stored from index `follow` on (behind the workgroups' own units; same KV head, no longer than
  // its first).  Long units run alone (count 1); short ones are chained: fewer workgroups to hand out, of more nearly
  // equal length.
  int32_t follow;
  int32_t count;  // units of this workgroup including this one; 0 in a unit that follows another
  // (block, head) tiles per query block: the heads of the KV group, or fewer where a document of at most 32 rows has
  // the rows of 2 or 4 heads packed into each 64-row tile (the heads of a group add into the same dK and dV)
  int32_t heads;
};
// A piece of a unit's query blocks (see CombineUnit) runs alone, and its `follow` is -1 - (block of partial results).

// Batches with few long units leave most of the 256 CUs idle: a lone 256-row shard with a 16K context is 32 workgroups of
// 256 tiles each, a 4K-token batch has dK/dV workgroups of up to 200 steps at an average of 88 per CU.  For those the
// planner makes a second list of units, in which long ones are cut into pieces along the loop they run (the keys of a
// forward / dQ unit, the query blocks of a dK/dV unit).  A piece writes its fp32 accumulators to the workspace, and
// ca_combine_* add the pieces of a unit up, in order (no atomics: bit-reproducible), and store the results.  Measured,
// whole units against pieces: forward of that lone shard (32/8 heads, head_dim 128) 271 -> 81 us; forward + backward of
// 1000 rows with a 130K context 9.8 -> 7.3 ms; of the 4K-token batch 597 -> 395 us; of documents of 512 and 1024 tokens
// (4/2 heads, head_dim 64) 85 -> 34 us.
struct CombineUnit {
  int32_t part0, n_parts;  // blocks of partial results of the unit
  // forward / dQ unit: first slot, first query head, hp.   dK/dV unit: first packed KV row, valid keys, KV head.
  int32_t a, b, c, reserved;
};
// a block of partial results: FWD_BM x head_dim fp32 (a forward / dQ unit's rows, or dK and then dV of BWD_BN keys), in
// the order of the accumulators: [wave and row group][32-column block][4 quads][64 lanes][4]; behind all blocks, for
// forward, {running maximum, the lane's share of the row sum} as [block][8 row groups][64 lanes][2] fp32
inline size_t part_bytes(int d) { return size_t(FWD_BM) * d * 4; }
constexpr size_t FWD_STAT_BYTES = 8 * 64 * 2 * 4;

constexpr int N_CU = 256, N_XCD = 8;
constexpr int FUSED_BQ = 32;                                        // query rows per step of the one-pass backward
constexpr size_t FUSED_CTRL_BYTES = 256;                          // per queue: its XCD + 1, and, 128 bytes on, the units taken
constexpr int fused_waves(int d) { return d == 128 ? 8 : 4; }  // its workgroups, each wave with 32 keys
// How the forward kernel runs a list of units (the planner chooses, see there)
struct FwdForm {
  bool halves = false;  // workgroups are halves of units (of 128 rows)
  bool turns = false;   // workgroups that share a CU take turns at having priority
};

}  // namespace ca

struct ca_plan {
  // descriptor copy
  int32_t n_docs = 0, n_tasks = 0, hq = 0, hkv = 0, d = 0;
  int64_t total_q = 0, total_kv = 0;
  float scale = 0.f;
  std::vector<int64_t> doc_kv_start, doc_kv_len, task_q_start, task_q_len, task_q_pos, task_kv_len;
  std::vector<int32_t> task_doc;
  // schedule (host)
  std::vector<int32_t> slot_row, slot_pos;
  // for the dK/dV kernel: rows per head in the packed tiles of a 64-slot block (16 or 32; 0 = one head per tile), and
  // the position of every row of its tiles (= slot_pos except in packed blocks)
  std::vector<int32_t> block_rpk, pos_kv;
  std::vector<ca::FwdUnit> fwd_units;
  std::vector<ca::BwdUnit> bwd_units;
  int32_t bwd_workgroups = 0;  // workgroups of the dK/dV kernel: the leading units of bwd_units
  int64_t fwd_steps = 0, bwd_steps = 0;
  // the lists with long units cut into pieces; empty where that gains nothing
  std::vector<ca::FwdUnit> fwd_pieces;
  std::vector<ca::BwdUnit> bwd_pieces;
  std::vector<ca::CombineUnit> fwd_combine, bwd_combine;
  int32_t bwd_piece_workgroups = 0;
  int32_t n_fwd_parts = 0, n_bwd_parts = 0;
  ca::FwdForm fwd_form, fwd_piece_form;
  // workspace with which the piece lists are used: forward, and backward, where the parts lie behind ws_bwd
  size_t ws_fwd_split = 0, ws_bwd_split = 0, ws_off_parts_kv = 0, ws_off_parts_dq = 0;
  // dK, dV and dQ in one pass (ca_bwd_fused.hip): whole units by queue, where each queue begins, and what the pass needs behind ws_bwd
  bool fused = false;
  std::vector<ca::BwdUnit> fused_units;
  int32_t fused_queue[ca::N_XCD + 1] = {};
  size_t ws_off_dq_sums = 0, ws_off_flags = 0, ws_off_ctrl = 0, ws_bwd_fused = 0;
  const ca::BwdUnit *d_fused_units = nullptr;
  bool joint = false;  // backward runs dK/dV and dQ units in one launch: dK/dV workgroups, then dQ halves 1, then 0, or,
  // if not empty, in this order: i >= 0: dK/dV workgroup i; below: -1 - (half * dQ units + unit)
  std::vector<int32_t> joint_order;
  bool joint_lost = false;  // one launch looked better, but the parts are shared
  bool pieces_lost = false;  // shorter forward pieces looked better, but their parts are beyond the static workspace
  bool shared_parts = false;  // the dQ parts take the place of the dK/dV parts once those have been added up
  // simulated time of the cut forward units (0: nothing to cut) and of the backward units and their partial results (0: not simulated)
  double us_fwd = 0, us_bwd = 0;
  // where the partial results take the backward workspace beyond the static one, which whole units fit: the plan of the same batch
  // that stays within it, for calls with less workspace than this plan's lists need
  std::unique_ptr<ca_plan> within_static;
  // workspace layout for backward: [Delta fp32 hq*padded_slots][log2e*LSE fp32 hq*padded_slots]
  int slot_align = ca::SLOT_ALIGN, heads_packed = 1;  // padding of a document's slots; hp of the packed units
  size_t ws_fwd = 0, ws_bwd = 0, ws_off_l2 = 0, ws_off_qs = 0, ws_off_dos = 0;
  size_t ws_off_stats_kv = 0;  // the row statistics once more: [block][head][half of 32 rows of the dK/dV tile][log2e*LSE, -Delta][32]
  bool q_covered = false, kv_covered = false;  // every packed Q row / KV row belongs to some unit
  // device copies
  int device = -1;
  void *d_blob = nullptr;  // one allocation that holds all of the arrays below
  std::vector<char> blob;  // host copies of the small ones, which go up together
  const int32_t *d_slot_row = nullptr, *d_slot_pos = nullptr, *d_block_rpk = nullptr, *d_pos_kv = nullptr;
  const int32_t *d_joint_order = nullptr;
  const ca::FwdUnit *d_fwd_units = nullptr, *d_fwd_pieces = nullptr;
  const ca::BwdUnit *d_bwd_units = nullptr, *d_bwd_pieces = nullptr;
  const ca::CombineUnit *d_fwd_combine = nullptr, *d_bwd_combine = nullptr;
  // optional timing events (hipEvent_t, kept as void* so that host-only code needs no HIP header)
  bool profile = false;
  void *ev[7] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
  bool ev_fwd = false, ev_bwd = false;
};

namespace ca {
void set_error(const std::string &msg);
int build_plan(const ca_batch_desc *desc, ca_plan_t **out);  // host only
}  // namespace ca

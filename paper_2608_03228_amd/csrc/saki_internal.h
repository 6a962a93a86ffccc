// Internal layout and launch planning shared by the host helpers and the HIP
// launchers of libsaki.  Not part of the public ABI.
#pragma once

#include <cstddef>
#include <cstdint>

namespace saki {

constexpr int kHeadDim = 128;  // d on the GPU path
constexpr int kMaxK = 64;      // top-k lists hold 64 entries, one per wave lane
constexpr int kTile = 64;      // keys per index tile
constexpr int kChunkBytes = 16;
constexpr int kScanWaves = 1;          // waves per work-group of the one-pass MFMA scoring kernel
constexpr int kScanMinKeys = 16384;    // rows at least this long take it
constexpr int kBatchMaxChunk = 4096;   // keys per chunk of the two-pass MFMA scoring kernel
constexpr size_t kMaxChunk = 0x7fff0000;  // keys per chunk of any kernel: steps past its end fit an int
constexpr int kBatchWaves = 1;         // its waves per work-group (16 rows each)

inline bool rank_supported(int r) { return r == 16 || r == 32 || r == 64 || r == 128; }
// bytes per code element: float32 (0), bf16 (1), fp8 E4M3 (2)
inline int elem_bytes(int dtype) { return dtype == 2 ? 1 : dtype == 1 ? 2 : 4; }
constexpr size_t n_tiles(int N) { return ((size_t)N + kTile - 1) / kTile; }
inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Index layout, per (sequence b, query head h): tiles of 64 keys; inside a
// tile, the code of key t is cut into 16-byte pieces and piece p of all 64
// keys is stored contiguously:
//   byte offset = ((b*H_q + h)*n_tiles + tile)*64*r*es + p*64*16 + t*16 + e*es
// so a wave that reads piece p of 64 consecutive keys reads 1 KiB contiguously.
inline size_t tile_bytes(int r, int dtype) { return (size_t)kTile * r * elem_bytes(dtype); }
inline size_t index_bytes(int B, int H_q, int N_cap, int r, int dtype) {
  return (size_t)B * H_q * n_tiles(N_cap) * tile_bytes(r, dtype);
}

// How saki_score_topk / saki_recall split the work.  Each wave owns `rows`
// consecutive query rows of one (b, h) and one key chunk; when a row's keys
// are split over several chunks each chunk writes a partial top-64 to the
// workspace and a merge pass reduces them.
struct Plan {
  bool mfma = false;   // 16-row MFMA kernels (Q >= 16) or the streaming kernels
  int rows = 1;        // query rows per wave
  int waves = 1;       // waves per workgroup
  int row_blocks = 0;  // workgroups along the query axis
  bool scan = false;   // MFMA rows scored in one pass (row_blocks: 16-row blocks, one per wave;
                       // with a split key axis z_off: chunk gates, flag_off: rows to redo)
  int chunk = kTile;   // keys per chunk (multiple of 64)
  int n_chunks = 1;
  size_t z_off = 0, b_off = 0, part_off = 0, flag_off = 0, ws_bytes = 0;
  size_t flag_count = 0;  // flags per tier (recall path)
};

// `heads` groups of `Q` rows each (the rows of one group read the same codes).
inline Plan make_plan(int B, int heads, int Q, int N_valid, int part_entry_bytes, bool mfma) {
  Plan p;
  p.mfma = mfma;
  p.rows = p.mfma ? 16 : (Q >= 4 ? 4 : 1);
  const int wave_rows = (Q + p.rows - 1) / p.rows;
  const int H_q = heads;
  const int max_waves = p.mfma ? 2 : 4;  // workgroup size of the kernels
  p.waves = wave_rows < max_waves ? (wave_rows < 1 ? 1 : wave_rows) : max_waves;
  p.row_blocks = (Q + p.rows * p.waves - 1) / (p.rows * p.waves);
  const size_t total_waves = (size_t)B * H_q * wave_rows;
  const size_t n = N_valid > 0 ? (size_t)N_valid : 1;
  size_t chunk = round_up(n, kTile);
  // waves wanted over the whole GPU before the key axis is split too
  const size_t target = p.mfma ? 2048 : 8192;
  if (total_waves > 0 && total_waves < target) {
    const size_t want = (target + total_waves - 1) / total_waves;
    size_t c = round_up((n + want - 1) / want, kTile);
    if (c < 2048) c = 2048;
    if (c < chunk) chunk = c;
  }
  if (chunk > kMaxChunk) chunk = kMaxChunk;
  p.chunk = (int)chunk;
  p.n_chunks = (int)((n + chunk - 1) / chunk);
  const size_t rows_total = (size_t)B * H_q * Q;
  size_t off = 0;
  if (p.n_chunks > 1) {
    p.part_off = off;
    off = round_up(off + rows_total * p.n_chunks * kMaxK * part_entry_bytes, 256);
  }
  p.ws_bytes = off;
  return p;
}

// Score path: the workspace holds the partial lists of a split key axis
// (float score + int index), at least 256 bytes so that a size of 0 keeps
// meaning invalid arguments.  The MFMA kernels take 16 queries of one head per
// wave (the one-pass kernel when the rows are long); the decode kernel takes the
// rows of one code set: the H_q / index_heads heads sharing it, times Q, and its
// launch makes the chunks longer, never more.  The two-pass MFMA kernel reads the query sketches z (r values per
// row: bf16 for bf16 and fp8 codes (dtype 1, 2), float32 for float32 codes)
// at z_off and b = q . mu (one float per row) at b_off, written by a kernel
// before it; the other kernels form the sketch themselves.
inline Plan score_plan(int B, int H_q, int index_heads, int Q, int N_valid, int r, int dtype) {
  const bool mfma = Q >= 16;
  Plan p = mfma ? make_plan(B, H_q, Q, N_valid, 8, true)
                : make_plan(B, index_heads, (H_q / index_heads) * Q, N_valid, 8, false);
  if (mfma && N_valid >= kScanMinKeys) {
    p.scan = true;
    p.waves = kScanWaves;
    p.row_blocks = (Q + 15) / 16;
    if (p.n_chunks > 1) {  // per (row, chunk) gate of a chunk that kept too few keys; per-row redo flags
      const size_t rows_total = (size_t)B * H_q * Q;
      p.z_off = round_up(p.ws_bytes, 256);
      p.flag_off = round_up(p.z_off + rows_total * p.n_chunks * sizeof(float), 256);
      p.flag_count = rows_total;
      p.ws_bytes = round_up(p.flag_off + rows_total * sizeof(int), 256);
    }
  }
  if (mfma && !p.scan) {  // the two-pass kernel: chunks of at most kBatchMaxChunk keys
    p.waves = kBatchWaves;
    p.row_blocks = ((Q + 15) / 16 + kBatchWaves - 1) / kBatchWaves;
    const size_t n = N_valid > 0 ? (size_t)N_valid : 1;
    if ((size_t)p.chunk > (size_t)kBatchMaxChunk) {
      p.chunk = kBatchMaxChunk;
      p.n_chunks = (int)((n + kBatchMaxChunk - 1) / kBatchMaxChunk);
    }
    const size_t rows_total = (size_t)B * H_q * Q;
    p.part_off = 0;
    p.z_off = p.n_chunks > 1 ? round_up(rows_total * p.n_chunks * kMaxK * 8, 256) : 0;
    p.b_off = round_up(p.z_off + rows_total * r * (dtype == 0 ? 4 : 2), 256);
    p.ws_bytes = round_up(p.b_off + rows_total * sizeof(float), 256);
  }
  if (p.ws_bytes < 256) p.ws_bytes = 256;
  return p;
}

// Recall path: partial lists hold a double score and an int index (16 bytes
// with padding).  The MFMA path also keeps the keys split into bf16 hi and lo
// parts in tile layout (z_off), the key norm bounds in rows of n_tiles * 64
// (b_off) and two arrays of one flag per wave (flag_off) through which each
// tier hands the waves it could not finish to the next.
inline Plan recall_plan(int B, int H_q, int H_kv, int Q, int N_valid) {
  Plan p = make_plan(B, H_q, Q, N_valid, 16, Q >= 16);
  if (!p.mfma) return p;
  const size_t nt = n_tiles(N_valid);
  p.z_off = round_up(p.ws_bytes, 256);
  p.b_off = round_up(p.z_off + 2 * (size_t)B * H_kv * nt * kTile * kHeadDim * 2, 256);
  p.flag_off = round_up(p.b_off + (size_t)B * H_kv * nt * kTile * sizeof(float), 256);
  const size_t blocks = (size_t)p.row_blocks * p.n_chunks * B * H_q;
  p.flag_count = (blocks + 8) * 2;
  p.ws_bytes = round_up(p.flag_off + 2 * p.flag_count * sizeof(int), 256);
  return p;
}

// Recall of few rows per key (Q < 16, or a batch whose rows alone do not fill
// the GPU): the keys of a KV group are read once for all rows of its query
// heads, 16 nb rows per wave.  Lists of 128 entries (8 bytes) per (row, chunk)
// from offset 0, which the partial lists of the rows redone by `stream` take
// over afterwards; a count per (row, chunk), a gate and a redo flag per row.
struct OncePlan {
  bool use = false;
  int nb = 1, row_blocks = 0, chunk = kTile, n_chunks = 1;
  size_t count_off = 0, tau_off = 0, redo_off = 0, ws_bytes = 0;
  Plan stream;
};
constexpr int kOnceMinChunk = 128;  // keys a wave takes at least
constexpr int kOnceWaves = 4096;    // waves wanted over the whole GPU
constexpr int kOnceMaxRows = 2048;  // rows of 16 or more queries a head that take it
// Whether it is the better path.  Its decision rescores every listed key (25 to
// 45 us per 1,000 rows), so it gains with the key reads that it saves.  us,
// float32 keys, d = 128, this path / the other one; H_q / H_kv x Q, sequences:
//   Q < 16, against one wave per 1 or 4 rows, which takes 0.2 us a key
//     32 / 8 x 1, 1           64 keys 29 / 20    128 keys 33 / 33    300 keys 31 / 71
//     32 / 8 x 2, 16                  46 / 24            55 / 42     256 keys 55 / 76
//     32 / 8 x 2, 64                 120 / 102          139 / 196            144 / 386
//     32 / 8 x 4, 1                   29 / 40            33 / 58              32 / 92
//     32 / 8 x 4, 64                 222 / 135          254 / 200            235 / 321
//     32 / 8 x 15, 4                  66 / 43            77 / 64              75 / 104
//     32 / 8 x 15, 16                206 / 58           234 / 94             216 / 159
//   Q >= 16, against 16 rows a wave    4,096 keys      8,192 keys      16,384 keys
//     32 / 8 x 16, 4 (64 rows a group)   87 / 126                       138 / 394
//     32 / 8 x 64, 1 (256)               96 / 99                        131 / 216
//     28 / 4 x 73, 1 (511)              114 / 109       111 / 140       134 / 242
//     8 / 1 x 64, 1 (512)                89 / 91         77 / 95         74 / 95
//     2 / 1 x 400, 1 (800)              111 / 92        102 / 93         98 / 112
//     1 / 1 x 2,000, 1 (2,000)          163 / 95        157 / 118       147 / 185
//   More rows also gain from 16,384 keys on (28 / 4 x 128: 208 / 308), which
//   kOnceMaxRows leaves to the other path.
inline bool once_better(int H_q, int H_kv, int Q, size_t rows, int N_valid) {
  const size_t group = (size_t)(H_q / H_kv) * Q;
  size_t least;  // keys
  if (Q < 4)
    least = rows <= 1536 ? 129 : 32 * (size_t)Q + 1;
  else if (Q < 16)
    least = rows <= (Q < 8 ? 1024u : 512u) ? 0 : Q < 8 || rows <= 2048 ? 129 : Q < 12 ? 257 : 353;
  else
    least = group <= 384 || rows <= 512 ? 0 : group <= 512 ? 8192 : 16384;
  return (size_t)N_valid >= least;
}
inline OncePlan recall_once_plan(int B, int H_q, int H_kv, int Q, int N_valid) {
  OncePlan o;
  if (Q <= 0 || N_valid <= 0) return o;  // no rows, or none with a key
  const Plan p = recall_plan(B, H_q, H_kv, Q, N_valid);
  const size_t group_rows = (size_t)(H_q / H_kv) * Q, rows = (size_t)B * H_q * Q;
  if (p.mfma && (p.n_chunks == 1 || rows > (size_t)kOnceMaxRows)) return o;
  if (!once_better(H_q, H_kv, Q, rows, N_valid)) return o;
  o.stream = make_plan(B, H_q, Q, N_valid, 16, false);
  o.nb = group_rows > 16 ? 2 : 1;
  o.row_blocks = (int)((group_rows + 16 * o.nb - 1) / (16 * o.nb));
  const size_t per_chunk = (size_t)o.row_blocks * B * H_kv, entry = 1024 + sizeof(int);
  size_t want = (kOnceWaves + per_chunk - 1) / per_chunk;
  // no more workspace than the rows' other path takes
  if (p.mfma) {
    const size_t room = p.ws_bytes / rows > 2 * sizeof(float) ? p.ws_bytes - rows * 2 * sizeof(float) : 0;
    const size_t most = room > 1024 ? (room - 1024) / (rows * entry) : 0;
    if (most < 1) return o;
    if (want > most) want = most;
  }
  size_t chunk = round_up(((size_t)N_valid + want - 1) / want, kTile);
  if (chunk < (size_t)kOnceMinChunk) chunk = kOnceMinChunk;
  o.chunk = (int)chunk;
  o.n_chunks = (int)(((size_t)N_valid + chunk - 1) / chunk);
  size_t lists = rows * o.n_chunks * 1024;
  if (lists < o.stream.ws_bytes) lists = o.stream.ws_bytes;
  o.count_off = round_up(lists, 256);
  o.tau_off = round_up(o.count_off + rows * o.n_chunks * sizeof(int), 256);
  o.redo_off = round_up(o.tau_off + rows * sizeof(float), 256);
  o.ws_bytes = round_up(o.redo_off + rows * sizeof(int), 256);
  if (p.mfma && o.ws_bytes > p.ws_bytes) return o;
  o.use = true;
  return o;
}

}  // namespace saki

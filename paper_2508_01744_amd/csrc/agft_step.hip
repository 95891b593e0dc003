// agft_step.hip -- batched AGFT decide-and-update step for CDNA4 (gfx950).
//
// One workgroup per tuner instance.  Each arm's record (theta_k and the
// packed upper factor S_k of A_k^{-1}) is read by a group of G = d/2 lanes:
// lane j of the group owns factor columns j and d-1-j (d+1 elements
// together) and theta_{2j}, theta_{2j+1}, so it forms two complete entries
// of v = S^T x_t and two terms of theta^T x_t on its own, and the group only
// sums two numbers at the end.  A record's main part is contiguous in HBM
// and its short tail sits beside the tails of the other arms of its block
// (Rec below): for every load instruction the G lanes of a group read G x 16
// contiguous bytes of one record and a wavefront covers whole cache lines,
// and rewriting one arm touches a handful of cache lines instead of one line
// per 16-byte piece.
//
// Per step and instance (Sec. 4.2-4.4):
//   0. read the instance's words, mask, context and reward, all in one
//      memory round trip; with the switch to exploitation on, feed the
//      previous reward to the instance's Page-Hinkley test and switch when
//      the rewards are stable;
//   1. fetch the record of the previous decision's arm (its update waits);
//      with the paper's pruning rules on, drop arms by their reward counts
//      and means; list the other arms in play (in the action space, not
//      pruned);
//   2. every listed arm: m = theta^T x_t, w^2 = |S^T x_t|^2,
//      UCB = m + alpha_t w, LCB = m - alpha_t w  (Eq. 1); an exploiting
//      instance reads only a contiguous copy of theta and scores m (Eq. 2);
//   3. fold the previous decision's reward into its arm: Eq. 3-5 as a
//      square-root rank-1 update of S (below) plus the matching theta
//      update, in LDS, once the arm's record and the stream's first pass,
//      requested together, have landed; the updated arm is scored on x_t from
//      LDS in the same operation order as the stream, and its record is
//      written back at the end of the step (large batches: ahead of the step,
//      in a kernel of its own);
//   4. pruning when due (drop UCB_k < max_j LCB_j), argmax with ties to the
//      lowest arm index; refinement of the action space when due; epilogue.
//
// Square-root update.  Eq. 3 adds x x^T to A, so P = A^{-1} changes by the
// Sherman-Morrison identity P' = P - P x x^T P / (1 + x^T P x).  With P = S S^T
// (S upper triangular) and f = S^T x, P' = S M M^T S^T where M is the upper
// triangular factor of I - f f^T / alpha_d, alpha_j = 1 + f_0^2 + ... + f_j^2
// (alpha_{-1} = 1):
//   M_jj = sqrt(alpha_{j-1} / alpha_j),  M_ij = -f_i f_j / sqrt(alpha_{j-1} alpha_j), i < j,
// so S' = S M column by column:
//   S'_ij = M_jj S_ij - f_j / sqrt(alpha_{j-1} alpha_j) * sum_{i<=k<j} f_k S_ik.
// Eq. 4-5 combine into theta' = theta + g (r - x^T theta) with the gain
// g = P x / (1 + x^T P x) = S f / alpha_{d-1}.
// This is the triangular square-root covariance update of sequential
// estimation (Carlson's form); its fp32 error grows with the square root of
// the condition number of A rather than with the condition number itself.

#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <type_traits>

#include "agft.h"
#include "agft_env_math.h"

namespace {

constexpr uint32_t kMagic = 0x54464741u;  // "AGFT"
constexpr int kWave = 64;
constexpr int kMaxK = 1024;
constexpr int kMaxWords = kMaxK / 32;
constexpr int kMaxWaves = 16;
constexpr size_t kAlign = 256;

// Header at the start of the state buffer (256 bytes).  pending: 0 no decision
// awaits its reward, 1 one does, kPendingFolded between the two launches of a
// step: the decision is pending, its reward already in its arm.
constexpr int kPendingFolded = 2;
struct alignas(16) StateHeader {
    uint32_t magic;
    uint32_t version;
    int32_t B, K, d, chunks, mask_words, pending;
    int64_t t;
    float lambda, alpha0;
    int32_t alpha_sched, prune_rule, prune_period;
    int32_t exploit;      // 1: the buffer holds the theta copy of the switch
    int32_t tail_floats;  // record layout: floats per lane slice of a tail
    int32_t stats_kept;   // 1: the per-arm reward counts and sums are maintained
    uint32_t reserved[44];
};
static_assert(sizeof(StateHeader) == 256, "header is 256 bytes");

size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// Record geometry for context dimension D: G lanes per arm, each owning
// D + 3 positions (D + 1 factor elements and two theta entries).  Positions
// 0..D-1 of every lane form the arm's main part (D/4 float4 chunks per
// lane, lane-interleaved); positions D..D+2 its tail, TF floats per lane.
// NB = 64/D arms make a block: their main parts, then their tails, so that
// every main part starts on a 128-byte line.  With TF = 3 records carry no
// padding (608 bytes at D = 16) and the NB tails fill three whole lines,
// but half of them straddle two; with TF = 4 each tail slice is padded to
// a chunk and every tail sits in one line.  An instance's arms take
// ceil(K/NB) blocks.
template <int D, int TF>
struct Rec {
    static constexpr int G = D / 2;              // lanes per arm
    static constexpr int P = D + 1;              // factor elements per lane
    static constexpr int MQ = D / 4;             // main chunks per lane
    static constexpr int S = MQ + 1;             // register slots per lane (the last holds the tail)
    static constexpr int MAIN = G * MQ;          // main chunks per arm
    static constexpr int TAIL = G * TF / 4;      // tail chunks per arm
    static constexpr int R = MAIN + TAIL;        // chunks per record
    static constexpr int NB = 32 / G;            // arms per block
    static constexpr int BLK = NB * R;           // chunks per block
    static constexpr int NSE = D * (D + 1) / 2;  // packed factor elements
    static constexpr int CAN = D + NSE;          // canonical floats: theta, then packed S
};

int chunks_for(int d, int tf) { return (d / 2) * (d / 4) + (d / 2) * tf / 4; }
int block_arms(int d) { return 64 / d; }
// float4 chunks of one instance's arm records: whole blocks
size_t instance_chunks(int K, int d, int tf) {
    const int nb = block_arms(d);
    return (size_t)((K + nb - 1) / nb) * nb * chunks_for(d, tf);
}

// Packed column-major index of S_ij (i <= j) within the factor part.
__host__ __device__ constexpr int packed(int i, int j) { return j * (j + 1) / 2 + i; }

// Canonical index (theta_0..theta_{D-1}, then packed S) of position e of
// lane j's slice of a record; -1 for padding.
__host__ __device__ constexpr int canon(int D, int j, int e) {
    return e <= j ? D + packed(e, j)
         : e <= D ? D + packed(D - e, D - 1 - j)
         : e == D + 1 ? 2 * j
         : e == D + 2 ? 2 * j + 1
         : -1;
}

// Canonical index of component q of record chunk c; -1 for padding.
__host__ __device__ constexpr int canon_chunk(int D, int TF, int c, int q) {
    const int G = D / 2, MAIN = G * (D / 4);
    if (c < MAIN) return canon(D, c % G, 4 * (c / G) + q);
    const int t = 4 * (c - MAIN) + q;   // tail float: lane t/TF, position D + t%TF
    return t % TF < 3 ? canon(D, t / TF, D + t % TF) : -1;
}

// Float offset, within an arm's record (chunks in record order), of factor
// element S_ij (i <= j) and of theta_i: column j < G sits in lane slice j at
// position i, column j >= G in slice D-1-j at position D-i; theta_i at
// position D+1+(i%2) of slice i/2.  Positions below D are component e%4 of
// main chunk (e/4)*G + slice, the others tail float TF*slice + (e-D).
template <int D, int TF>
__host__ __device__ constexpr int rec_pos_S(int i, int jc) {
    constexpr int G = D / 2, MAIN = G * (D / 4);
    const bool first = jc < G;
    const int sl = first ? jc : D - 1 - jc;
    const int e = first ? i : D - i;
    return e < D ? 4 * ((e >> 2) * G + sl) + (e & 3) : 4 * MAIN + TF * sl + (e - D);
}
template <int D, int TF>
__host__ __device__ constexpr int rec_pos_theta(int i) {
    constexpr int G = D / 2, MAIN = G * (D / 4);
    return 4 * MAIN + TF * (i >> 1) + 1 + (i & 1);
}

// The two offset functions above invert canon_chunk: checked at compile time
// for every record layout the kernels are built for.
template <int D, int TF>
constexpr bool rec_pos_consistent() {
    for (int jc = 0; jc < D; ++jc)
        for (int i = 0; i <= jc; ++i) {
            const int pos = rec_pos_S<D, TF>(i, jc);
            if (canon_chunk(D, TF, pos / 4, pos % 4) != D + packed(i, jc)) return false;
        }
    for (int i = 0; i < D; ++i) {
        const int pos = rec_pos_theta<D, TF>(i);
        if (canon_chunk(D, TF, pos / 4, pos % 4) != i) return false;
    }
    return true;
}
static_assert(rec_pos_consistent<8, 3>() && rec_pos_consistent<8, 4>() && rec_pos_consistent<16, 3>() &&
                  rec_pos_consistent<16, 4>() && rec_pos_consistent<32, 3>() && rec_pos_consistent<32, 4>(),
              "record offsets of the update disagree with the record layout");

// The update walks the factor RP rows apart from one pass to the next.  For
// RP a multiple of 4, row r0 + ps*RP of column jc sits at a fixed per-lane
// base plus ps steps of +G*RP floats (top-down slices, columns < G) or
// -G*RP (bottom-up slices), except row 0 of a bottom-up column, which is its
// slice's tail float; theta_i, RP/2 slices further per pass, moves by TF*RP/2.
// So each pass costs one add of address arithmetic.  Checked at compile time
// against rec_pos_S for every lane and pass of the kernels' shapes.
template <int D, int TF, int RP>
struct RowWalk {
    static constexpr int G = D / 2, MAIN = G * (D / 4);
    static constexpr bool kLinear = RP % 4 == 0;
    __host__ __device__ static constexpr int step(int jc) { return jc < G ? G * RP : -G * RP; }
    __host__ __device__ static constexpr int base(int r0, int jc) {
        const int sl = jc < G ? jc : D - 1 - jc;
        const int e = jc < G ? r0 : D - r0;
        return 4 * ((e >> 2) * G + sl) + (e & 3);
    }
    __host__ __device__ static constexpr int tail(int jc) { return 4 * MAIN + TF * (D - 1 - jc); }
    __host__ __device__ static constexpr int pos(int r0, int jc, int ps) {
        return ps == 0 && r0 == 0 && jc >= G ? tail(jc) : base(r0, jc) + ps * step(jc);
    }
};

template <int D, int TF, int RP>
constexpr bool row_walk_consistent() {
    if constexpr (!RowWalk<D, TF, RP>::kLinear) return true;
    for (int jc = 0; jc < D; ++jc)
        for (int r0 = 0; r0 < RP && r0 < D; ++r0)
            for (int ps = 0; r0 + ps * RP < D; ++ps) {
                const int i = r0 + ps * RP;
                if (i <= jc && RowWalk<D, TF, RP>::pos(r0, jc, ps) != rec_pos_S<D, TF>(i, jc)) return false;
                if (rec_pos_theta<D, TF>(r0) + ps * TF * (RP / 2) != rec_pos_theta<D, TF>(i)) return false;
            }
    return true;
}
// rows per pass: (64 / D) segments per wavefront times 1 or 4 wavefronts
static_assert(row_walk_consistent<8, 3, 8>() && row_walk_consistent<8, 4, 8>() && row_walk_consistent<8, 3, 32>() &&
                  row_walk_consistent<8, 4, 32>() && row_walk_consistent<16, 3, 4>() && row_walk_consistent<16, 4, 4>() &&
                  row_walk_consistent<16, 3, 16>() && row_walk_consistent<16, 4, 16>() &&
                  row_walk_consistent<32, 3, 8>() && row_walk_consistent<32, 4, 8>(),
              "the update's row walk matches the record layout");

// Per-instance block of 32-bit words: previous action, active-arm count,
// non-finite-input count, mode (-1 exploring, else the round exploitation
// began), the Page-Hinkley state (n, mean, m+, min m+, m-, min m-), the round
// of its last alarm, its last margin, the action space (lo, hi, stride), the
// top-two score gap of the last decision that dumped its scores, then the
// stashed context.  Kept together so the epilogue
// writes one or two lines per instance.
constexpr int kInstAprev = 0, kInstKact = 1, kInstBad = 2, kInstMode = 3, kInstPh = 4,
              kInstPhLast = 10, kInstPhMargin = 11, kInstLo = 12, kInstHi = 13, kInstStride = 14,
              kInstGap = 15, kInstX = 16;

int inst_words(int d) { return (kInstX + d + 15) / 16 * 16; }

struct Layout {
    size_t arms, mask, inst, stats, theta, total;
};

// Arms an instance may have in play: K, or with the refinement the larger of
// the coarse grid and the window.
int arms_in_play(const agft_config &c) {
    if (!c.refine) return c.K;
    const int coarse = (c.K - 1) / c.refine_stride + 1, window = 2 * c.refine_half + 1;
    const int k = coarse > window ? coarse : window;
    return k < c.K ? k : c.K;
}

// Bytes an exploring instance streams per step, at most: theta and the
// packed factor of every arm in play.
size_t explore_bytes(const agft_config &c) {
    return (size_t)arms_in_play(c) * 4 * (size_t)(c.d + c.d * (c.d + 1) / 2);
}

// Record layout: packed tails (TF = 3) where an exploring instance streams
// more than 16 KB per step, or more than 8 KB when every step streams every
// record (no pruning rule, no refinement, no switch to exploitation), so
// that the stream moves no padding; padded tails (TF = 4) otherwise, where
// the update's one-record read and write-back weigh more than the stream
// and a tail that straddles two lines costs more than its padding.
// Measured on MI355X (step kernel, packed / padded tails): K=128 d=16
// B=65,536 (76 KB) 853 / 889 us, the same with exploitation 827 / 845 us,
// K=256 d=32 B=1,024 (560 KB) 92.0 / 93.0 us, K=128 d=16 B=65,536 with the
// refinement (13 KB) 186 / 176 us, with the refinement, the rules and the
// switch 190 / 179 us; K=64 d=8 B=4,096 (11 KB) over the whole horizon
// 12.85 / 13.25 us without pruning, 11.6 / 11.25 us with rules 1-8,
// 10.45 / 10.45 us with the refinement, 10.5 / 10.4 us with the switch.
int tail_floats(const agft_config &c) {
    const size_t bytes = explore_bytes(c);
    return bytes > 16384 || (bytes > 8192 && c.prune_rule == 0 && !c.refine && !c.exploit) ? 3 : 4;
}

// The per-arm reward counts and sums are read only by the paper's rules 2-8
// and by the refinement's statistical anchor; without those the update
// skips them (their one-line store per instance and step costs 1.4% of the
// step at K=128 d=16 B=65,536) and they stay at zero.
bool stats_kept(const agft_config &c) { return (c.prune_rule & 14) != 0 || c.refine != 0; }

// theta copy [B][K][d] only with the switch to exploitation (0 bytes otherwise)
Layout layout_for(const agft_config &c) {
    Layout L;
    const size_t b = (size_t)c.B, k = (size_t)c.K;
    const size_t kw = (k + 31) / 32;
    size_t off = sizeof(StateHeader);
    L.arms = off;  off = align_up(off + b * instance_chunks(c.K, c.d, tail_floats(c)) * 16);
    L.mask = off;  off = align_up(off + b * kw * 4);
    L.inst = off;  off = align_up(off + b * (size_t)inst_words(c.d) * 4);
    L.stats = off; off = align_up(off + b * k * 8);
    L.theta = off; off = align_up(off + (c.exploit ? b * k * (size_t)c.d * 4 : 0));
    L.total = off;
    return L;
}

// Dynamic LDS of the step kernel: UCB and LCB per arm, then the arm list.
size_t step_lds_bytes(int K) { return ((size_t)K * (2 * 4 + 2) + 15) / 16 * 16; }

// Workgroup width (wavefronts); one workgroup per instance, looping over its
// arms in passes of 64*w/(d/2).  The step is a chain of dependent phases per
// instance, so narrow workgroups (more instances in flight per CU, cheaper
// barriers) win unless each instance streams many bytes.  The bytes per
// step are estimated from the arms in play (with the refinement, at most the
// larger of the coarse grid and the window) times what each costs (the
// record, or the theta copy once instances exploit): one wavefront up to
// 16 KB, four beyond.  Measured on MI355X with padded 640-byte records
// (step kernel, us, w = 1 / 2 / 4; with the packed blocks, w = 2 stayed
// 2-3% slower than w = 4 at K=128 d=16):
//   K=64 d=8 B=4,096 (12 KB):              21 / 25 / 30
//   K=128 d=16 B=65,536 (80 KB):           895 / 892 / 882
//   the same, exploitation (8 KB):         595 / 602 / 672
//   the same, refinement (13 KB):          190 / 231 / 376
//   K=256 d=32 B=1,024 (590 KB):           31 / 29 / 29
//   the same, exploitation (32 KB):        43 / 34 / 31
int waves_for(const agft_config &c) {
    const size_t bytes = c.exploit ? (size_t)arms_in_play(c) * 4 * c.d : explore_bytes(c);
    return bytes <= 16384 ? 1 : 4;
}

// Before round ph_min_rounds no instance can have switched to exploitation,
// so with the switch on, those steps take the width of an exploring
// instance.  Measured on MI355X (us per step over the whole horizon, one
// width throughout / exploring width before the first possible switch):
// K=128 d=16 B=65,536 566.2 / 557.9, the same with rules 2-8 570.8 / 565.1,
// B=16,384 82.6 / 81.5.
int waves_at(const agft_config &c, int64_t t) {
    if (c.exploit && t < c.ph_min_rounds) return explore_bytes(c) <= 16384 ? 1 : 4;
    return waves_for(c);
}

// Whether the update of the previous decision's arm runs ahead of the stream,
// when its record and the stream's first pass have landed, rather than after
// it: always, except at d = 32 where an instance streams more than 16 KB, since
// the second pass is requested only after it and the longer update holds that
// back (the kernel still runs it first at a step whose list of arms fits in one
// pass).
// Measured on MI355X (step kernel, ahead of / after the stream): K=64 d=8
// B=4,096 19.1 / 20.5 us; K=128 d=16 B=65,536 853 / 857 us, B=16,384 218.4 /
// 220.8 us; K=256 d=32 B=1,024 92.4 / 91.7 us.
bool early_update(const agft_config &c) { return c.d < 32 || explore_bytes(c) <= 16384; }

// Workgroup width of the score kernel after a separate update: one wavefront
// up to 32 KB per instance (96 KB with rules 2-8, which remove most arms in
// the end), four beyond.  Without the update, an instance's chain is short and
// one wavefront carries longer streams, and far more instances when few arms
// are left.  Measured on MI355X with 1.5 GB of records (us per step, one
// wavefront / four, every arm in play, then a quarter of them): d=16 K=32 (19
// KB) 268 / 271 and 106 / 201, K=48 (29 KB) 256 / 243 and 94 / 144, K=64 (39
// KB) 250 / 239 and 88 / 114, K=128 235 / 229 and 80 / 88; d=8 K=128 (23 KB)
// 290 / 298 and 118 / 139, K=192 (34 KB) 281 / 270 and 116 / 121; d=32 K=20
// (45 KB) 295 / 283 and 105 / 146.  With rules 2-8 one wavefront costs up to 4%
// while every arm is in play and halves the step once eight are left; the line
// lies where the former would make the step slower than one launch is (1.3 GB of
// records, one wavefront / four / one launch, every arm in play, then eight):
//   d=16 K=64 (38 KB)   220 / 228 / 250 and 63 / 129 / 174
//        K=128 (76 KB)  218 / 212 / 224 and 40 / 70 / 93
//        K=160 (95 KB)  217 / 211 / 224 and 34 / 59 / 77
//        K=200 (119 KB) 220 / 210 / 222 and 33 / 50 / 64
//        K=256 (152 KB) 219 / 209 / 217 and 30 / 42 / 52
//   d=8  K=512 (88 KB)  246 / 247 / 253 and 49 / 72 / 94
//        K=800 (138 KB) 263 / 248 / 254 and 57 / 61 / 79
//   d=32 K=32 (70 KB)   253 / 254 / 266 and 92 / 138 / 167
//        K=64 (140 KB)  418 / 390 / 407 and 87 / 127 / 153
int score_waves_at(const agft_config &c, int64_t t) {
    const bool may_exploit = c.exploit && t >= c.ph_min_rounds;
    const size_t bytes = may_exploit ? (size_t)arms_in_play(c) * 4 * c.d : explore_bytes(c);
    return bytes <= (size_t)((c.prune_rule & 14) ? 96 : 32) * 1024 ? 1 : 4;
}

// Whether the update of the previous decisions' arms is a kernel of its own,
// ahead of one that only reads the records.  A write-back between the reads of
// a stream at HBM's rate costs far more than its bytes (65,536 of 608 bytes:
// 97 us of a 810 us stream, against 24 us for all of them on their own; a
// 16-byte-per-lane read-only stream of the same 5.1 GB takes 713 us), so large
// batches that stream from HBM are better off with a second launch.  Not where
// the launch costs more than the interference saves: few instances, or records
// that the Infinity Cache (256 MB) holds.  At d = 8, whose records are smallest,
// the gain is mostly the second launch's width: with four wavefronts it is lost
// again between all arms and few, so where arms go those batches need 2 GB; where
// none do, from 24 KB on, 1 GB.  The host does not know how many arms are left:
// with a handful, two launches can cost up to 5 us more than one, with all of
// them they gain 2-10%.  Measured on MI355X (us per step, in one kernel / two,
// every arm in play, then a half, a quarter and eight):
//   d=16 K=128: B=4,096 53.3 / 52.3; B=8,192 105 / 100, 69.2 / 61.9, 47.7 / 45.1,
//     34.0 / 37.1; B=16,384 211 / 197, 135 / 114, 90.8 / 81.8, 65.8 / 66.8;
//     B=65,536 819 / 746, 535 / 438, 354 / 306, 256 / 250; with the refinement
//     (21 arms) B=8,192 25.8 / 27.6, 16,384 47.3 / 46.5, 65,536 179 / 170; mostly
//     exploiting B=8,192 45.8 / 44.9, 65,536 297 / 267; rules 2-8 B=4,096 60.6 /
//     60.6, 16,384 210 / 194
//   d=16 K=64: B=8,192 58.5 / 57.0, 37.8 / 38.6, 28.6 / 31.3, 23.0 / 28.3;
//     B=65,536 433 / 389, 273 / 245, 199 / 200
//   d=8, one wavefront: K=64 B=16,384 (184 MB) 40.0 / 44.4, 65,536 163 / 161;
//     K=128 B=32,768 (738 MB) 146 / 149, -, 82.8 / 63.8, 67.8 / 30.2; K=180
//     B=17,000 (539 MB) 100 / 105, 69.4 / 69.7, 50.0 / 46.0, 38.4 / 20.2
//   d=8, four: K=256 B=16,384 (738 MB) 131 / 133, 84.6 / 93.6, 56.8 / 61.7, 37.9 /
//     38.0; 32,768 (1.5 GB) 268 / 261, 172 / 181, 111 / 117, 70.9 / 68.5; 65,536
//     537 / 495, 349 / 355, 222 / 226, 140 / 130; K=373 B=32,768 (2.15 GB) 381 /
//     366, 242 / 241, 153 / 160, 73.5 / 71.5
//   d=8, no pruning: K=96 (17 KB) 0.55 GB 119 / 115, 1.1 GB 237 / 219; K=128 (23
//     KB) 109 / 112, 218 / 214; K=160 (28 KB) 105 / 109, 211 / 211; K=180 (32 KB)
//     103 / 107, 207 / 208; K=256 (45 KB) 0.7 GB 131 / 133, 1.5 GB 268 / 261
//   d=32, whose update is the longest: K=256 B=2,048 183 / 186, 4,096 374 / 362,
//     with a quarter of the arms B=2,615 69.1 / 77.3; K=32 B=16,384 211 / 213,
//     127 / 129, 95 / 85, 80 / 74 (three); K=64 401 / 398, 219 / 223, 130 / 134,
//     96 / 86; K=96 600 / 574, 318 / 318, 180 / 183, 97 / 88
// With the score dump, whose stores interfere either way, not for streams up to
// 16 KB (us per step, in one kernel / two): refinement B=65,536 185 / 187, K=45
// d=16 (27 KB) 362 / 329, K=128 d=16 887 / 800, mostly exploiting 309 / 301; at
// d = 8 beyond that from 512 MB at either width: K=256 B=16,384 154 / 152, 98.2 /
// 102, 67.6 / 65.4, 56.4 / 53.5.
constexpr int kSplitMinB = 8192;   // (twice that at d = 32)
bool split_update(const agft_config &c, int64_t t, bool dump) {
    const size_t stream = (size_t)c.B * explore_bytes(c);
    if (dump && explore_bytes(c) <= 16384) return false;
    const bool arms_go = c.prune_rule != 0 || c.refine || c.exploit;
    const size_t least_mb = c.d != 8 ? 256
                          : dump ? 512
                          : arms_go ? (score_waves_at(c, t) == 1 ? 512 : 2048)
                          : explore_bytes(c) <= 24 * 1024 ? 512 : 1024;
    return c.B >= (c.d == 32 ? 2 * kSplitMinB : kSplitMinB) && stream >= least_mb << 20;
}

// What lane j of a group multiplies the positions of its record slice with.
// Positions e <= j belong to column j (times x_e), positions e > j to column
// D-1-j (times x_{D-e}).  With j < G = D/2, position 0 is always of the first
// kind and positions G..D always of the second: those take elements of x that
// are the same in every lane, from scalar registers (u), and only positions
// 1..G-1 need a selected pair (a, b; one of the two is 0).
template <int D>
struct SliceX {
    static constexpr int G = D / 2;
    float u[G + 1];      // x_0..x_G
    float a[G], b[G];    // [e], 1 <= e < G: e <= j ? x_e : 0 and e > j ? x_{D-e} : 0
    float t0, t1;        // x_{2j}, x_{2j+1}
};

// Per-lane slice of the Eq. 1 terms from the positions f of one record slice:
// m, the two owned terms of theta^T x, and w2, the squares of the two owned
// entries of S^T x.
template <int D>
__device__ __forceinline__ void slice_terms(const float *f, const SliceX<D> &x, float &m, float &w2) {
    constexpr int G = D / 2;
    float va = f[0] * x.u[0], vb = f[1] * x.b[1];
#pragma unroll
    for (int e = 1; e < G; ++e) va = fmaf(f[e], x.a[e], va);
#pragma unroll
    for (int e = 2; e < G; ++e) vb = fmaf(f[e], x.b[e], vb);
#pragma unroll
    for (int e = G; e <= D; ++e) vb = fmaf(f[e], x.u[D - e], vb);
    m = fmaf(f[D + 2], x.t1, f[D + 1] * x.t0);
    w2 = fmaf(vb, vb, va * va);
}

// v of another lane of the same row, through a DPP lane pattern.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Sum over the G lanes of an aligned group (G = 2, 4, 8, 16), every lane
// ending with the same total: pairs within quads, then the two pairs of a
// quad, then mirrored half rows (8 lanes) and mirrored rows (16 lanes), each
// step a DPP add on the vector unit.
template <int G>
__device__ __forceinline__ float group_sum(float v) {
    static_assert(G == 1 || G == 2 || G == 4 || G == 8 || G == 16, "group of 1..16 lanes");
    if constexpr (G >= 2) v += dpp<0xB1>(v);    // quad_perm [1,0,3,2]
    if constexpr (G >= 4) v += dpp<0x4E>(v);    // quad_perm [2,3,0,1]
    if constexpr (G >= 8) v += dpp<0x141>(v);   // row_half_mirror
    if constexpr (G >= 16) v += dpp<0x140>(v);  // row_mirror
    return v;
}

// Parameters of the paper's pruning rules (bits 2, 4, 8 of the rule mask).
struct Heuristics {
    int32_t mask;          // rule bits 2 | 4 | 8 in use
    int32_t ext_rounds, ext_min_n;
    float ext_thr;
    int32_t hist_after, hist_min_n;
    float hist_kappa;
    int32_t hist_min_arms, cascade_k;
};

// Bits of word w of the action space lo <= k <= hi, (hi - k) % stride == 0.
__device__ inline uint32_t space_bits(int w, int lo, int hi, int stride) {
    const int k0 = 32 * w;
    const int first = lo > k0 ? lo - k0 : 0;
    const int last = hi < k0 + 31 ? hi - k0 : 31;
    if (last < first) return 0u;
    const uint32_t range = last - first == 31 ? 0xffffffffu : ((1u << (last - first + 1)) - 1u) << first;
    if (stride == 1) return range;
    uint32_t grid = 0u;   // positions congruent to hi modulo the stride
    for (int b = (hi - k0) % stride; b < 32; b += stride) grid |= 1u << b;
    return range & grid;
}

// Refinement of the action space after this step's decision (Sec. 4.4).
struct Refine {
    int32_t now;          // refinement due at this step
    int32_t stat;         // statistical anchor (before maturity), else predictive
    int32_t half, min_n;  // window half-width in arms; samples for the statistical anchor
};

// Switch to greedy exploitation after a Page-Hinkley test finds the
// reward sequence stable (Sec. 4.2, Eq. 2).
struct Exploit {
    int32_t on;
    float delta, lambda;
    int32_t window, min_rounds;
};

struct StepArgs {
    float4 *arms;
    uint32_t *mask;
    int32_t *inst;        // [B][IW] per-instance blocks
    int2 *stats;          // [B][K] rewards folded in, their sum (fp32 bits)
    float *theta;         // [B][K][D] copy of theta (exploitation on), else nullptr
    Heuristics h;
    Exploit e;
    Refine rf;
    int64_t t;            // decisions made before this step
    StateHeader *hdr;
    const float *ctx;     // [B][D] or nullptr (flush)
    const float *reward;  // [B] or nullptr
    int32_t *action;      // [B] or nullptr
    float *scores;        // [B][2][K] or nullptr
    int32_t B, K, KW, IW;
    int32_t apply_update;  // a decision is pending
    int32_t prune_now;
    int32_t prune_reset;   // rule 1 starts again from the whole action space (non-sticky)
    int32_t early_update;  // fold the previous reward in before the stream
    int32_t keep_stats;    // maintain the per-arm reward counts and sums
    int32_t sum_waves;     // workgroup width whose order of sums a step after a separate update keeps (1 or 4)
    float alpha;
    int64_t t_next;        // t after this call (header bookkeeping)
};

// Streaming load that bypasses cache retention: every record is read once
// per step and the state of a large batch is many times the cache size.
typedef float nt_f4 __attribute__((ext_vector_type(4)));
// three floats at 4-byte alignment (a record tail slice)
typedef float nt_f3 __attribute__((ext_vector_type(3))) __attribute__((aligned(4)));
// four floats at 4-byte alignment (a caller's output)
typedef float out_f4 __attribute__((ext_vector_type(4))) __attribute__((aligned(4)));
__device__ __forceinline__ float4 ld_nt(const float4 *p) {
    const nt_f4 v = __builtin_nontemporal_load(reinterpret_cast<const nt_f4 *>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}

// The one record per instance that the step kernel's update gathers and writes
// back takes the same non-temporal hint only for d = 16.  Measured per step
// against ordinary accesses: d = 16, -0.9% (65,536 x 128) and -0.4% (16,384 x 128);
// d = 8, +5% (4,096 x 64); d = 32, +3% (1,024 x 256).
// The gather goes from memory to LDS without registers: 16 bytes per lane,
// lane l's to dst[l] (dst the same in every lane).  It has landed once vmcnt
// says so.
template <int D>
__device__ __forceinline__ void load_to_lds(const float4 *src, float4 *dst) {
    constexpr int kNonTemporal = 2;   // gfx9 cache policy bit
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)dst, 16, 0, D == 16 ? kNonTemporal : 0);
}
template <int D>
__device__ __forceinline__ void st_record(float4 *p, float x, float y, float z, float w) {
    if constexpr (D == 16) __builtin_nontemporal_store(nt_f4{x, y, z, w}, reinterpret_cast<nt_f4 *>(p));
    else *p = make_float4(x, y, z, w);
}

// One word of an instance block or of the score dump.  THROUGH: written through the caches at once
// (a store visible to the whole device), not left in them to be evicted
// between the reads of a stream, which costs more: 65,536 lines of 128 bytes
// beside a 5.1 GB stream take 38 us so left and 11 us written through.  Used by
// the score kernel's four-wavefront workgroups, whose streams are long
// (measured on MI355X, us per step, left / through: K=128 d=16 B=65,536 736 /
// 716; with four arms left in play, B=16,384, 63 / 65), not by one-wavefront
// ones (with the refinement, B=65,536, 171 / 172).  The score kernel's dump goes
// through at both widths (us per step with the dump, and the gap word, left /
// through): K=128 d=16 B=65,536 951 / 800, B=16,384 243 / 210, K=64 d=32
// B=20,000 520 / 492, K=45 d=16 B=65,536 335 / 329, K=130 d=8 B=65,536 331 / 320.
template <bool THROUGH>
__device__ __forceinline__ void st_word(int32_t *p, int32_t v) {
    if constexpr (THROUGH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}

// Element `idx` of a register array indexed by a lane-varying value
// (an unrolled select, so the array stays in registers).
template <int N>
__device__ __forceinline__ float pick(const float *v, int idx) {
    float out = 0.0f;
#pragma unroll
    for (int q = 0; q < N; ++q) out = (idx == q) ? v[q] : out;
    return out;
}

struct BestPair {
    float v;
    int k;
};

__device__ inline BestPair better(BestPair a, BestPair b) {
    if (b.v > a.v || (b.v == a.v && b.k < a.k)) return b;
    return a;
}

// Partner value for step s (0..5) of a 64-lane butterfly: quad pairs, quads,
// mirrored half rows, mirrored rows (all DPP, within rows of 16 lanes), then
// rows 16 and 32 lanes apart.  After the six steps of an associative and
// commutative op every lane holds the same result.
template <int STEP>
__device__ __forceinline__ int partner(int v) {
    if constexpr (STEP == 0) return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);
    else if constexpr (STEP == 1) return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);
    else if constexpr (STEP == 2) return __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);
    else if constexpr (STEP == 3) return __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false);
    else if constexpr (STEP == 4) return __shfl_xor(v, 16);
    else return __shfl_xor(v, 32);
}
template <int STEP>
__device__ __forceinline__ float partner(float v) { return __int_as_float(partner<STEP>(__float_as_int(v))); }

// The two values that lanes of neighbouring rows (SPAN 16) or half-waves
// (SPAN 32) hold, in every lane of the pair: a swap on the vector unit,
// without the LDS round trip of a permute.
struct LanePair {
    int lo, hi;
};
template <int SPAN>
__device__ __forceinline__ LanePair lane_pair(int v) {
    if constexpr (SPAN == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
        return LanePair{(int)r[0], (int)r[1]};
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
        return LanePair{(int)r[0], (int)r[1]};
    }
}
template <int SPAN, class T, class Op>
__device__ __forceinline__ T across(T v, Op op) {
    static_assert(sizeof(T) == 4, "one register");
    const LanePair r = lane_pair<SPAN>(__builtin_bit_cast(int, v));
    return op(__builtin_bit_cast(T, r.lo), __builtin_bit_cast(T, r.hi));
}

template <class T, class Op>
__device__ __forceinline__ T wave_reduce(T v, Op op) {
    v = op(v, partner<0>(v));
    v = op(v, partner<1>(v));
    v = op(v, partner<2>(v));
    v = op(v, partner<3>(v));
    v = across<16>(v, op);
    return across<32>(v, op);
}

__device__ __forceinline__ BestPair wave_best(BestPair b) {
    auto step = [&](BestPair o) { b = better(b, o); };
    step(BestPair{partner<0>(b.v), partner<0>(b.k)});
    step(BestPair{partner<1>(b.v), partner<1>(b.k)});
    step(BestPair{partner<2>(b.v), partner<2>(b.k)});
    step(BestPair{partner<3>(b.v), partner<3>(b.k)});
    step(BestPair{partner<4>(b.v), partner<4>(b.k)});
    step(BestPair{partner<5>(b.v), partner<5>(b.k)});
    return b;
}

// What N wavefronts of which wavefront w holds p_w sum to, worked out by one:
// each part by wave_reduce's tree, then part after part.  The parts share the
// tree's later levels, part w in the lanes w modulo N, for 13 (N = 2) and 21
// (N = 4) instructions against 10 for one part and 20 and 40 apart (which cost
// 2 us of a 47 us step, K=128 d=8 B=32,768 with eight arms left).
template <int N>
__device__ __forceinline__ float waves_sum(float p0, float p1, float p2, float p3, int lane) {
    static_assert(N == 2 || N == 4, "two or four parts");
    auto add = [](float a, float b) { return a + b; };
    p0 += dpp<0xB1>(p0);             // quad_perm [1,0,3,2]
    p1 += dpp<0xB1>(p1);
    float v = lane & 1 ? p1 : p0;
    v += dpp<0x4E>(v);               // quad_perm [2,3,0,1]
    if constexpr (N == 4) {
        p2 += dpp<0xB1>(p2);
        p3 += dpp<0xB1>(p3);
        float u = lane & 1 ? p3 : p2;
        u += dpp<0x4E>(u);
        v = lane & 2 ? u : v;
    }
    v += dpp<0x1B>(dpp<0x141>(v));   // the other quad of the half row, same place: mirrored, then each quad reversed
    v += dpp<0x128>(v);              // row_ror:8, the other half row
    v = across<16>(v, add);
    v = across<32>(v, add);
    float total = dpp<0x00>(v) + dpp<0x55>(v);                      // each quad's lanes 0, 1
    if constexpr (N == 4) total = (total + dpp<0xAA>(v)) + dpp<0xFF>(v);   // 2, 3
    return total;
}

// The arm of the wavefront's best pair: the largest value as an ordered
// integer (negative floats with their magnitude bits flipped, -0 as +0), then
// the smallest index that holds it.  Half the instructions of reducing pairs.
// v is never a NaN (better() takes none).
__device__ __forceinline__ int wave_best_arm(BestPair b) {
    auto dpp_op = [](int v, auto ctrl, int identity, auto op) {
        return op(v, __builtin_amdgcn_update_dpp(identity, v, decltype(ctrl)::value, 0xF, 0xF, false));
    };
    auto reduce = [&](int v, int identity, auto op) {
        v = dpp_op(v, std::integral_constant<int, 0xB1>{}, identity, op);
        v = dpp_op(v, std::integral_constant<int, 0x4E>{}, identity, op);
        v = dpp_op(v, std::integral_constant<int, 0x141>{}, identity, op);
        v = dpp_op(v, std::integral_constant<int, 0x140>{}, identity, op);
        v = across<16>(v, op);
        return across<32>(v, op);
    };
    const int bits = __float_as_int(b.v + 0.0f);
    const int key = bits ^ ((bits >> 31) & 0x7fffffff);
    const int top = reduce(key, (int)0x80000000, [](int x, int y) { return x > y ? x : y; });
    return reduce(key == top ? b.k : 0x7fffffff, 0x7fffffff, [](int x, int y) { return x < y ? x : y; });
}

// Inclusive prefix sum of a*b (prod, rounded) within aligned segments of SEG
// lanes (8, 16 or 32): DPP shifts within rows of 16 lanes (zero-filled at row
// edges), masked at the edges of 8-lane segments; for 32 lanes, the first
// row's total is then added to the second row of each half-wavefront.  The
// first addition takes a*b unrounded.
template <int SEG>
__device__ __forceinline__ float segment_scan(float a, float b, float prod, int lane) {
    static_assert(SEG == 8 || SEG == 16 || SEG == 32, "segments of 8, 16 or 32 lanes");
    auto shr = [](float x, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value,
                                                          0xF, 0xF, true));
    };
    const int pos = lane & 7;
    float s = shr(prod, std::integral_constant<int, 0x111>{});    // row_shr:1
    float v = fmaf(a, b, (SEG > 8 || pos >= 1) ? s : 0.0f);
    s = shr(v, std::integral_constant<int, 0x112>{});          // row_shr:2
    v += (SEG > 8 || pos >= 2) ? s : 0.0f;
    s = shr(v, std::integral_constant<int, 0x114>{});          // row_shr:4
    v += (SEG > 8 || pos >= 4) ? s : 0.0f;
    if constexpr (SEG >= 16) v += shr(v, std::integral_constant<int, 0x118>{});   // row_shr:8
    if constexpr (SEG == 32)
        v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x142, 0xA, 0xF, false));  // row_bcast:15
    return v;
}

// Sum over the 64/SEG segments of a wavefront: every lane ends with the
// total of its column (lane % SEG) over the segments.
template <int SEG>
__device__ __forceinline__ float segment_colsum(float v) {
    auto add = [](float a, float b) { return a + b; };
    if constexpr (SEG == 8) v += dpp<0x128>(v);   // row_ror:8, the other half row
    if constexpr (SEG <= 16) v = across<16>(v, add);
    return across<32>(v, add);
}

// Workgroup-wide reductions through one LDS slot per wavefront (a
// one-wavefront workgroup needs neither the slots nor the barriers).
template <class T, class Op>
__device__ T block_reduce(T v, T *red, int lane, int wave, int nwave, Op op) {
    v = wave_reduce(v, op);
    if (nwave == 1) return v;
    if (lane == 0) red[wave] = v;
    __syncthreads();
    T out = red[0];
    for (int w = 1; w < nwave; ++w) out = op(out, red[w]);
    __syncthreads();
    return out;
}

// Wavefronts per SIMD the register allocation must allow (the kernel's W).
// At d = 16 with packed tails (instances that stream more than 16 KB, four
// wavefronts each) the code the compiler gives at six (75 registers) beats
// the one squeezed into seven (72): step kernel 842 vs 848 us at K=128
// B=65,536, 211.7 vs 212.8 us at B=16,384.  Seven wins everywhere else:
// with the paper's rules 2-8, whose pass over the arm statistics gains from
// more instances in flight (918.6 vs 885.2 us at K=128 B=65,536, 186.4 vs
// 177.8 us at B=16,384), and with padded tails (one wavefront per instance):
// 173.6 vs 183.1 us with the refinement, rules and switch, 48.6 vs 49.8 us
// with the refinement alone.
int occupancy_for(const agft_config &c, int tail) {
    if (c.d == 32) return 4;
    return c.d == 16 && tail == 3 && !(c.prune_rule & 14) ? 6 : 7;
}

// Workgroups per compute unit for four-wavefront workgroups at six
// wavefronts per SIMD (d = 16, packed tails, no rules 2-8): 4, enforced by
// the launch's LDS request.  There the chain of phases per instance is short
// beside its stream, and four instances per compute unit keep enough of the
// stream in flight to hold the HBM rate, while more interleave more
// concurrent streams and lose rate.  Measured on MI355X (step kernel, us, at
// 6 / 5 / 4 / 3 workgroups per compute unit): K=128 d=16 B=65,536 823.6 /
// 819.5 / 807.8 / 858.0, B=16,384 199.0 / 197.5 / 197.1 / 209.4.  Not with
// the paper's rules 2-8, whose pass over the arm statistics needs the
// instances in flight (K=128 d=16 B=65,536: 827.7 uncapped, 852.6 at 5,
// 911.1 at 4), nor for one-wavefront workgroups, whose steps are short
// chains with little to stream.
// Nor up to 64 KB per instance, where the chain weighs more: the score kernel
// at 4 / uncapped with 1.5 GB of records, d=16 K=32 324 / 271, K=48 258 / 244,
// K=64 236 / 239, K=96 229 / 231, K=128 (76 KB) 229 / 233, and with a quarter
// of the arms in play 269 / 201, 189 / 144, 147 / 114, 110 / 91, 88 / 82.
int cu_workgroups_for(const agft_config &c, int waves, int simd_waves) {
    return waves == 4 && simd_waves == 6 && explore_bytes(c) > 65536 ? 4 : 0;
}

// The environment's arguments of the fused kernel, read again from the launch's
// argument memory: what is read through this pointer cannot be loaded before
// the point of the call, so that the epilogue's constants hold no scalar
// registers through the stream.
__device__ __forceinline__ const agft_env_detail::EnvArgs &env_args_again() {
    typedef const char __attribute__((address_space(4))) *kernarg_ptr;
    constexpr size_t align = alignof(agft_env_detail::EnvArgs);
    constexpr size_t off = (sizeof(StepArgs) + align - 1) / align * align;   // the kernel's second argument
    kernarg_ptr at = (kernarg_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(at));
    return *(const agft_env_detail::EnvArgs *)(at + off);
}

// What bounds the kernel: HBM's rate where a batch streams many bytes, else
// one instance's chain of dependent phases and the instructions that it
// issues, four cycles each whether vector or scalar (half to two thirds of
// the time of the small batches).  Hence: the previous record goes straight to
// LDS and the first pass is requested beside it, not after it; the list comes
// from the mask words in scalar registers; what every lane multiplies by the
// same element of x takes it from a scalar register; roots are taken once per
// arm in the epilogue, 64 arms at a time, not once per pass by every lane; the
// updated arm takes a slot of the stream's last pass; and one wavefront takes
// the argmax while the others write the record back.  Measured on MI355X
// against none of these (us per step): K=256 d=32 B=1,024 with three arms left
// 9.25 -> 7.04, K=64 d=8 B=4,096 with the environment's kernel 16.44 -> 15.33,
// K=129 d=16 B=1,000 with the score dump 15.22 -> 14.54; batches at HBM's rate
// unchanged.
//
// ENV: the simulator's environment responds in the epilogue (agft_sim_step):
// once the decision is known, the first lanes of wavefront 0 run the
// instance's next window with it, writing the reward and the next context in
// place of the ones read.  The word each of those lanes prefetches costs a
// register: at d = 16 the seven-wavefront form gets six, to fit without
// spilling.
//
// FOLD: the previous decision's reward is folded in by this kernel (else
// agft_update_kernel has done it).
template <int D, int TF, int NW, bool ENV, bool FOLD, int NBUF = 2>
__device__ __forceinline__ void step_body(const StepArgs &p, const agft_env_detail::EnvArgs &env) {
    using R = Rec<D, TF>;
    constexpr int G = R::G, S = R::S;
    // The previous decision's record is fetched and written back by the
    // wavefronts other than 0, which has the list and the argmax to do (one
    // wavefront does it all): thread u0 and up, NQ chunks each.
    constexpr int u0 = NW > 1 ? kWave : 0, NU = NW * kWave - u0;
    constexpr int NQ = (R::R + NU - 1) / NU;
    const int inst = blockIdx.x;
    const int tid = threadIdx.x;
    constexpr int nthr = NW * kWave;   // the launch's workgroup width, fixed per instantiation
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    constexpr int nwave = NW;
    const int K = p.K;
    const int KW = p.KW;
    const int j = tid % G;           // slot of this lane within its arm's group
    const int grp = tid / G;         // group index within the workgroup
    const int apw = nthr / G;        // arms per pass of the workgroup
    const size_t inst_chunks = (size_t)((K + R::NB - 1) / R::NB) * R::BLK;
    const float4 *recs = p.arms + (size_t)inst * inst_chunks;

    // the previous decision's record before and after its update, chunks in
    // record order (the layout of the arm's record in HBM)
    __shared__ float4 s_old4[(R::R + kWave - 1) / kWave * kWave];   // (and slack for load_to_lds)
    __shared__ float4 s_new4[R::R];
    float *s_old = reinterpret_cast<float *>(s_old4);
    float *s_new = reinterpret_cast<float *>(s_new4);
    __shared__ float s_fpart[NW][D];   // per-wavefront partial sums of f = S^T xp
    // per arm, (theta^T x, |S^T x|^2) as the stream leaves them, then (UCB, LCB)
    // where a later phase reads them by arm; and the list of arms to score.
    // Sized by K at launch (step_lds_bytes) so that small arm counts leave room
    // for more workgroups.
    extern __shared__ float s_arm[];
    float2 *s_sc = reinterpret_cast<float2 *>(s_arm);
    short *s_list = reinterpret_cast<short *>(s_arm + 2 * K);
    __shared__ uint32_t s_mask[kMaxWords];
    __shared__ int s_nlist;
    __shared__ float s_red_v[kMaxWaves];
    __shared__ int s_red_k[kMaxWaves];
    __shared__ int s_red_n[kMaxWaves];
    __shared__ uint32_t s_mask2[kMaxWords];
    __shared__ uint32_t s_raw[kMaxWords];   // arms no rule has removed (the global mask words)
    __shared__ float s_red_v2[kMaxWaves];
    __shared__ int s_red_k2[kMaxWaves];

    __shared__ float s_xp[D];   // context of the previous decision, for the update
    __shared__ int s_stu[kWave];   // its arm's reward count and sum (fp32 bits), then slack

    const bool decide = p.ctx != nullptr;
    int32_t *blk = p.inst + (size_t)inst * p.IW;
    // Everything the step reads before it knows the previous decision's arm is
    // requested at once, so that the prologue waits for one memory round trip
    // rather than one per item (the vector loads first: the compiler's waits
    // for the addresses of later ones would hold them back behind the scalar
    // loads).  Vector loads: the context, by every wavefront; by wavefront 0
    // the environment's state of the instance (for the epilogue), the
    // instance's mask words and the previous decision's context.  Scalar
    // loads: the instance's first sixteen words and the reward.
    __shared__ uint32_t s_envw[ENV ? 32 : 1];
    uint32_t env_pre = 0u;
    if constexpr (ENV)
        if (wave == 0) env_pre = agft_env_detail::env_prefetch(env, inst, lane);
    const int lane_d = lane < D ? lane : 0;   // clamped element index
    const uint32_t *mask_at = p.mask + (size_t)inst * KW + (lane < KW ? lane : 0);
    const float *xp_at = reinterpret_cast<const float *>(blk + kInstX) + lane_d;
    uint32_t raw_word = 0u;
    float xp_word = 0.0f;
    if (wave == 0) {
        raw_word = *mask_at;
        if constexpr (FOLD) xp_word = *xp_at;
    }
    const int4 *blk4 = reinterpret_cast<const int4 *>(blk);
    const int4 wa = blk4[0], wb = blk4[1], wc = blk4[2], wd = blk4[3];
    // (no branch around the reward either: without a pending decision the
    // block's first word stands in for it, unused)
    const float r_in = *(p.apply_update ? p.reward + inst : reinterpret_cast<const float *>(blk));
    // The context, element `lane` in lanes < D, without a branch: a flush reads
    // the block's own words in its place, and nothing uses them (x_ok is false,
    // so no arm is listed, scored or stashed).  Non-finite test on the exponent
    // bits.
    const float x_lane = (decide ? p.ctx + (size_t)inst * D : reinterpret_cast<const float *>(blk))[lane_d];
    const bool x_ok = decide & (__ballot((__float_as_uint(x_lane) & 0x7f800000u) == 0x7f800000u) == 0ull);

    __shared__ float4 s_x4[D / 4];   // the context, for its readers below
    float *s_x = reinterpret_cast<float *>(s_x4);
    const int a_prev = p.apply_update ? wa.x : -1;   // word kInstAprev
    const bool has_prev = a_prev >= 0 && a_prev < K;
    // (taken back to a scalar register: the select leaves it in a vector one)
    const float r = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(has_prev ? r_in : 0.0f)));
    const bool upd = has_prev && isfinite(r);
    const bool fold = FOLD && upd;
    const int a_upd = fold ? a_prev : -1;

    // Record of the previous decision's arm, requested as soon as its index is
    // known, straight into LDS (no registers, no staging), with its reward count
    // and sum, so that the end of the step only stores them.  No branch around
    // the loads (lanes past the record repeat its last chunk into the slack of
    // s_old4, a step without an update reads arm 0's), so that the waits for
    // the loads before them do not wait for these too.
    const int rec_blk = fold ? a_prev / R::NB : 0, rec_slot = fold ? a_prev % R::NB : 0;
    const uint32_t rec_main = (uint32_t)(rec_blk * R::BLK + rec_slot * R::MAIN);
    const uint32_t rec_tail = (uint32_t)(rec_blk * R::BLK + R::NB * R::MAIN + rec_slot * R::TAIL - R::MAIN);
    auto rec_at = [&](int c) { return (uint32_t)c + (c < R::MAIN ? rec_main : rec_tail); };
    const bool gathers = FOLD && (NW == 1 || (wave > 0 && (wave - 1) * kWave < R::R));
    if (gathers) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int c = tid - u0 + q * NU;
            load_to_lds<D>(recs + rec_at(c < R::R ? c : R::R - 1), s_old4 + (wave * kWave - u0) + q * NU);
        }
        if (p.keep_stats && wave == u0 / kWave) {
            // (its two words: lanes past 1 repeat the second)
            const int *st = reinterpret_cast<const int *>(p.stats + (size_t)inst * K + (fold ? a_upd : 0));
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(st + (lane < 1 ? 0 : 1)),
                                             (__attribute__((address_space(3))) void *)s_stu, 4, 0, 0);
        }
    }

    // Page-Hinkley test on the instance's rewards and the switch to greedy
    // exploitation (uniform scalar code, single precision, fixed order).
    static_assert(kInstAprev == 0 && kInstKact == 1 && kInstMode == 3 && kInstPh == 4 && kInstPhLast == 10 && kInstPhMargin == 11 && kInstLo == 12 &&
                      kInstHi == 13 && kInstStride == 14,
                  "word order of the instance block");
    int mode = p.e.on ? wa.w : -1;
    float ph[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    int ph_last = 0;
    float ph_margin = 0.0f;
    if (p.e.on) {
        ph[0] = __int_as_float(wb.x);
        ph[1] = __int_as_float(wb.y);
        ph[2] = __int_as_float(wb.z);
        ph[3] = __int_as_float(wb.w);
        ph[4] = __int_as_float(wc.x);
        ph[5] = __int_as_float(wc.y);
        ph_last = wc.z;
        ph_margin = __int_as_float(wc.w);
        if (upd && mode < 0) {
            ph[0] = ph[0] + 1.0f;
            ph[1] = ph[1] + (r - ph[1]) / ph[0];
            ph[2] = ph[2] + ((r - ph[1]) - p.e.delta);
            ph[3] = fminf(ph[3], ph[2]);
            ph[4] = ph[4] + ((ph[1] - r) - p.e.delta);
            ph[5] = fminf(ph[5], ph[4]);
            const float up = ph[2] - ph[3], dn = ph[4] - ph[5];
            ph_margin = p.e.lambda - (up > dn ? up : dn);
            if (up > p.e.lambda || dn > p.e.lambda) {
                ph_last = (int)p.t;
#pragma unroll
                for (int q = 0; q < 6; ++q) ph[q] = 0.0f;
            }
        }
        if (mode < 0 && x_ok && p.t >= p.e.min_rounds && p.t - ph_last >= p.e.window) mode = (int)p.t;
    }
    const bool greedy = mode >= 0;
    // The block's words 3..11 after this step, parked in LDS by the lanes that
    // store them at the end (so they hold no registers through the stream; every
    // wave has read the old words before any lane writes the new ones).
    __shared__ int s_phw[kInstPhMargin + 1 - kInstMode];
    const bool ph_lane = p.e.on && tid >= kInstMode && tid <= kInstPhMargin;
    if (ph_lane)
        s_phw[tid - kInstMode] = tid == kInstMode ? mode
                               : tid == kInstPhLast ? ph_last
                               : tid == kInstPhMargin ? __float_as_int(ph_margin)
                               : __float_as_int(pick<6>(ph, tid - kInstPh));

    // the arms in play: not removed by a pruning rule, inside the action space;
    // at a rule-1 step of the non-sticky reading, every arm of the space
    const int sp_lo = wd.x, sp_hi = wd.y;
    const int sp_st = wd.z > 1 ? wd.z : 1;
    const bool reset = p.prune_reset && !greedy && x_ok;
    uint32_t word = 0u;   // wavefront 0, lane < KW: the arms in play of mask word `lane`
    if (wave == 0) {
        if (lane < KW) {
            word = (reset ? 0xffffffffu : raw_word) & space_bits(lane, sp_lo, sp_hi, sp_st);
            s_raw[lane] = raw_word;
            s_mask[lane] = word;
        }
        if (lane < D) {
            s_x[lane] = x_lane;
            if constexpr (FOLD) s_xp[lane] = xp_word;
        }
    }

    // The paper's pruning rules (Sec. 4.3) on the arms active at step start,
    // with the previous decision's reward already counted.
    if (p.h.mask != 0 && x_ok) {
        __syncthreads();
        const int2 *st = p.stats + (size_t)inst * K;
        const Heuristics &h = p.h;
        auto act0 = [&](int k) { return ((s_mask[k >> 5] >> (k & 31)) & 1u) != 0; };
        // The mean and the spread over the arms are sums in single precision, and
        // the last bit of sigma can decide on an arm: a step after a separate
        // update takes them in the order of the one-launch step's width, whatever
        // its own, and removes the same arms.
        auto fsum = [](float a, float b) { return a + b; };
        auto fmx = [](float a, float b) { return fmaxf(a, b); };
        auto isum = [](int a, int b) { return a + b; };
        auto imx = [](int a, int b) { return a > b ? a : b; };
        auto sum_arms = [&](auto term) {
            if constexpr (!FOLD && NW == 1) {
                // (up to 64 arms the orders are the same)
                if (p.sum_waves == 4 && K > kWave) {
                    if (K <= 2 * kWave)
                        return waves_sum<2>(term(lane, 0.0f), lane + kWave < K ? term(lane + kWave, 0.0f) : 0.0f, 0.0f,
                                            0.0f, lane);
                    float p0 = 0.0f, p1 = 0.0f, p2 = 0.0f, p3 = 0.0f;
                    for (int k = lane; k < K; k += 4 * kWave) {
                        p0 = term(k, p0);
                        if (k + kWave < K) p1 = term(k + kWave, p1);
                        if (k + 2 * kWave < K) p2 = term(k + 2 * kWave, p2);
                        if (k + 3 * kWave < K) p3 = term(k + 3 * kWave, p3);
                    }
                    return waves_sum<4>(p0, p1, p2, p3, lane);
                }
            }
            float part = 0.0f;
            for (int k = tid; k < K; k += nthr) part = term(k, part);
            return block_reduce(part, s_red_v, lane, wave, nwave, fsum);
        };
        // counts (as int bits) and means to s_sc, which the stream rewrites
        int q = 0;
        float qbest = -INFINITY;
        const float qsum = sum_arms([&](int k, float part) {
            const int2 v = st[k];
            int n = v.x;
            float rs = __int_as_float(v.y);
            if (k == a_upd) {
                n += 1;
                rs += r;
            }
            const float mean = n > 0 ? rs / (float)n : 0.0f;
            s_sc[k] = make_float2(__int_as_float(n), mean);
            const bool counts = act0(k) && n >= h.hist_min_n;
            q += counts ? 1 : 0;
            qbest = counts ? fmaxf(qbest, mean) : qbest;
            return counts ? part + mean : part;
        });
        q = block_reduce(q, s_red_n, lane, wave, nwave, isum);
        qbest = block_reduce(qbest, s_red_v, lane, wave, nwave, fmx);
        const bool hist_on = (h.mask & 4) && p.t >= h.hist_after && q >= h.hist_min_arms && q > 0;
        float sigma = 0.0f;
        if (hist_on) {
            const float mu = qsum / (float)q;
            const float acc = sum_arms([&](int k, float part) {
                const int n = __float_as_int(s_sc[k].x);
                const float dev = s_sc[k].y - mu;
                return act0(k) && n >= h.hist_min_n ? fmaf(dev, dev, part) : part;
            });
            sigma = sqrtf(acc / (float)q);
        }
        auto gone = [&](int k) {
            if (!act0(k)) return false;
            const int n = __float_as_int(s_sc[k].x);
            const float mean = s_sc[k].y;
            if ((h.mask & 2) && p.t < h.ext_rounds && n >= h.ext_min_n && mean < h.ext_thr) return true;
            if (hist_on && n >= h.hist_min_n && h.hist_kappa * sigma - (qbest - mean) < 0.0f) return true;
            return false;
        };
        int kstar = -1;
        if (h.mask & 8) {
            for (int k = tid; k < K; k += nthr)
                if (k < h.cascade_k && gone(k)) kstar = k > kstar ? k : kstar;
            kstar = block_reduce(kstar, s_red_n, lane, wave, nwave, imx);
        }
        int left = 0;
        for (int base = 0; base < K; base += nthr) {
            const int k = base + tid;
            const bool stay = k < K && act0(k) && !gone(k) && !(k < kstar);
            left += stay ? 1 : 0;
            const unsigned long long bal = __ballot(stay);
            const int w0 = (base + wave * kWave) >> 5;
            if (lane == 0 && w0 < KW) s_mask2[w0] = (uint32_t)(bal & 0xffffffffull);
            if (lane == 0 && w0 + 1 < KW) s_mask2[w0 + 1] = (uint32_t)(bal >> 32);
        }
        left = block_reduce(left, s_red_n, lane, wave, nwave, isum);
        if (left == 0) {
            // keep the best mean reward among the arms that had rewards, else the first arm
            BestPair bk{-INFINITY, 0x7fffffff};
            int first = 0x7fffffff;
            for (int k = tid; k < K; k += nthr)
                if (act0(k)) {
                    first = k < first ? k : first;
                    if (__float_as_int(s_sc[k].x) > 0) bk = better(bk, BestPair{s_sc[k].y, k});
                }
            bk = wave_best(bk);
            first = wave_reduce(first, [](int a, int b) { return a < b ? a : b; });
            if (lane == 0) {
                s_red_v[wave] = bk.v;
                s_red_k[wave] = bk.k;
                s_red_n[wave] = first;
            }
            __syncthreads();
            if (tid == 0) {
                BestPair all{s_red_v[0], s_red_k[0]};
                int f0 = s_red_n[0];
                for (int w = 1; w < nwave; ++w) {
                    all = better(all, BestPair{s_red_v[w], s_red_k[w]});
                    f0 = s_red_n[w] < f0 ? s_red_n[w] : f0;
                }
                const int keep = all.k != 0x7fffffff ? all.k : f0;
                if (keep < K) s_mask2[keep >> 5] |= 1u << (keep & 31);
            }
        }
        __syncthreads();
        if (wave == 0 && lane < KW) {
            const uint32_t w = s_mask2[lane];
            const uint32_t removed = s_mask[lane] & ~w;
            if (removed != 0u) {
                s_raw[lane] &= ~removed;
                p.mask[(size_t)inst * KW + lane] = s_raw[lane];
            }
            s_mask[lane] = word = w;
        }
        __syncthreads();
    }

    // Active arms other than the one being updated, in index order: 64 arms at
    // a time, the two mask words taken to scalar registers, each arm placed by
    // the count of active lanes below it.  The updated arm, if in play, takes
    // the slot after them: it is scored from LDS, or, folded in ahead of this
    // kernel, like the other arms, except that an exploiting instance still
    // sums its theta terms in the record's order.
    const int a_own = FOLD ? a_upd : greedy && upd ? a_prev : -1;
    int nlist = 0, upd_in = 0;
    if (wave == 0) {
        if (!x_ok) word = 0u;
        if (lane == KW - 1 && (K & 31) != 0) word &= (1u << (K & 31)) - 1u;
        if (a_own >= 0) {
            upd_in = (int)((uint32_t)__builtin_amdgcn_readlane((int)word, a_own >> 5) >> (a_own & 31) & 1u);
            if (lane == a_own >> 5) word &= ~(1u << (a_own & 31));
        }
        for (int k0 = 0; k0 < K; k0 += kWave) {
            // (lanes past the last word hold zeros)
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)word, k0 >> 5);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)word, (k0 >> 5) + 1);
            const unsigned long long bal = (unsigned long long)hi << 32 | lo;
            if (__builtin_amdgcn_inverse_ballot_w64(bal))
                s_list[nlist + (int)__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u))] = (short)(k0 + lane);
            nlist += __popcll(bal);
        }
        if (upd_in && lane == 0) s_list[nlist] = (short)a_own;
        if (NW > 1 && lane == 0) s_nlist = nlist | upd_in << 16;
    }
    if constexpr (NW > 1) {
        __syncthreads();
        const int packed_n = __builtin_amdgcn_readfirstlane(s_nlist);
        nlist = packed_n & 0xffff;
        upd_in = packed_n >> 16;
    } else {
        __syncthreads();   // (one wavefront: orders its LDS accesses)
    }

    // Where the update of an exploring instance runs (early_update on the host):
    // below D = 32 always early; and where the whole list fits in the first
    // pass, no later pass can wait behind the update.
    const bool early = D < 32 || p.early_update || nlist <= apw;
    // arms the stream scores: with the early update, the updated arm as well
    const int total = nlist + (early ? upd_in : 0);
    // whether any group of this wavefront has an arm
    const bool streams = !greedy && wave * (kWave / G) < total;

    // Stream buffers: two sets of S slots per lane, used in turn, so that one
    // pass is scored while the next one's loads are in flight: the lane's
    // main chunks, then its three tail floats.  The first pass is issued now,
    // beside the previous record, so that the two round trips are one.
    float4 buf_a[S], buf_b[S], buf_more[NBUF > 2 ? NBUF - 2 : 1][S];
    const char *rec_bytes = reinterpret_cast<const char *>(recs);
    auto fetch = [&](int slot, float4 *dst) {
        if (slot >= nlist) return;
        const uint32_t k = (uint32_t)s_list[slot];
        const uint32_t b = k / R::NB * (R::BLK * 16), r = k % R::NB;
        const uint32_t main = b + r * (R::MAIN * 16) + (uint32_t)j * 16;
        const uint32_t tail = b + r * (R::TAIL * 16) + (uint32_t)j * (TF * 4) + R::NB * R::MAIN * 16;
#pragma unroll
        for (int sidx = 0; sidx < R::MQ; ++sidx)
            dst[sidx] = ld_nt(reinterpret_cast<const float4 *>(rec_bytes + main + sidx * G * 16));
        const nt_f3 t = __builtin_nontemporal_load(reinterpret_cast<const nt_f3 *>(rec_bytes + tail));
        dst[R::MQ] = make_float4(t.x, t.y, t.z, 0.0f);
    };
    // What this lane multiplies its slice's positions with (slice_terms):
    // uniform elements of x in scalar registers, selected ones from LDS; formed
    // by the wavefronts that stream, just before they do.
    SliceX<D> sx;
    auto selectors = [&]() {
        typedef const float __attribute__((address_space(4))) *scalar_ptr;
        const scalar_ptr xs = (scalar_ptr)(uintptr_t)(p.ctx + (size_t)inst * D);
#pragma unroll
        for (int e = 0; e <= G; ++e) sx.u[e] = xs[e];
#pragma unroll
        for (int e = 1; e < G; ++e) {
            sx.a[e] = e <= j ? s_x[e] : 0.0f;
            sx.b[e] = e > j ? s_x[D - e] : 0.0f;
        }
        const float2 xt = reinterpret_cast<const float2 *>(s_x)[j];
        sx.t0 = xt.x;
        sx.t1 = xt.y;
    };

    // Every wavefront sees the previous decision's record in LDS.
    auto record_ready = [&]() {
        if (gathers) {
            // the loads to LDS have landed (gfx9 encoding: vmcnt 0 only)
            __builtin_amdgcn_s_waitcnt(0x0F70);
        }
        if constexpr (FOLD) __syncthreads();
    };

    // ---- square-root rank-1 update of the previous decision's arm ----
    // Run when the record and the stream's first pass have landed, or after the
    // stream (early_update on the host decides which, and the kernel runs it
    // early whenever the whole list fits in the first pass), in LDS; the updated
    // record is written back as the kernel's last act (write_back below).
    auto update = [&]() {
        // (fused and separate products as written, here and in agft_update_kernel)
#pragma clang fp contract(off)
        if (fold) {
            // Lane l of every wavefront takes column j = l % D of one row per
            // pass (row segments of D lanes; a pass of the workgroup covers RP
            // rows), so that the column sums and the row prefix sums below are
            // segment-wide DPP reductions instead of D-step loops on one lane.
            constexpr int SEGS = kWave / D, RP = NW * SEGS, NP = (D + RP - 1) / RP;
            const int jc = lane % D, seg = lane / D;
            const int r0 = wave * SEGS + seg;   // this lane's row in pass 0
            using Walk = RowWalk<D, TF, RP>;
            const int wbase = Walk::base(r0, jc), wstep = Walk::step(jc), wtail = Walk::tail(jc);
            const int tbase = rec_pos_theta<D, TF>(r0 < D ? r0 : 0);
            auto pos_S = [&](int ps, int i) {
                if constexpr (Walk::kLinear) return ps == 0 && r0 == 0 && jc >= G ? wtail : wbase + ps * wstep;
                else return rec_pos_S<D, TF>(i, jc);
            };
            // f_j = sum_{i<=j} S_ij xp_i: this lane's rows, then the other
            // segments of the wavefront, then the other wavefronts
            float fj = 0.0f;
#pragma unroll
            for (int ps = 0; ps < NP; ++ps) {
                const int i = ps * RP + r0;
                if (i < D && i <= jc) fj = fmaf(s_old[pos_S(ps, i)], s_xp[i], fj);
            }
            fj = segment_colsum<D>(fj);
            if constexpr (NW > 1) {
                if (seg == 0) s_fpart[wave][jc] = fj;
                __syncthreads();
                fj = s_fpart[0][jc];
#pragma unroll
                for (int w = 1; w < NW; ++w) fj += s_fpart[w][jc];
            }
            // alpha_j = 1 + f_0^2 + ... + f_j^2 (prefix over the segment) and the
            // column coefficients of M; alpha_{d-1} from the segment's last lane
            const float f2 = fj * fj;
            const float incl = segment_scan<D>(fj, fj, f2, lane);
            const float al = 1.0f + incl;
            const float al_prev = 1.0f + (incl - f2);
            const float ca = sqrtf(al_prev / al), cb = fj / sqrtf(al_prev * al);
            const float al_last = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(al), D - 1));
            // prediction error r - xp^T theta
            float pred = lane < D ? s_xp[lane] * s_old[rec_pos_theta<D, TF>(lane)] : 0.0f;
            pred = group_sum<D < 16 ? D : 16>(pred);
            if constexpr (D == 32) pred = across<16>(pred, [](float a, float b) { return a + b; });
            const float err = r - __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(pred)));
            // row i of S' = S M:  S'_ij = ca_j S_ij - cb_j g_ij with g_ij the
            // exclusive prefix sum of f_q S_iq along the row; its total is
            // (S f)_i, so the gain is that total / alpha_{d-1} (one reciprocal
            // for all rows: theta carries a 1e-3 tolerance, orders of
            // magnitude above the ulp this gives away)
            const float inv_al = 1.0f / al_last;
#pragma unroll
            for (int ps = 0; ps < NP; ++ps) {
                const int i = ps * RP + r0;
                const bool in_row = i < D && i <= jc;
                const int pos = pos_S(ps, i < D ? i : 0);
                const float sij = in_row ? s_old[pos] : 0.0f;
                const float q = fj * sij;
                const float qi = segment_scan<D>(fj, sij, q, lane);
                if (in_row) s_new[pos] = fmaf(ca, sij, -(cb * (qi - q)));
                if (i < D && jc == D - 1) {
                    const int tp = tbase + ps * TF * (RP / 2);
                    s_new[tp] = fmaf(qi * inv_al, err, s_old[tp]);
                }
            }
            // padded tails: the fourth float of each lane slice's tail stays 0
            if constexpr (TF == 4)
                if (tid < G) s_new[4 * R::MAIN + 4 * tid + 3] = 0.0f;
            __syncthreads();
        } else if (has_prev && !upd && tid == 0) {
            blk[kInstBad] += 1;
        }
    };
    // The updated record, its theta copy and its reward count and sum go out
    // last.  Loads and stores share one completion counter on this
    // architecture, and the compiler's waits for the stream's loads do not
    // follow paths: a store issued before a wait for a load is waited for too,
    // so stores in the middle of the step would hold up the rest of it by
    // their full latency.
    auto write_back = [&]() {
        if (fold) {
            if (gathers) {
                float4 *dst = p.arms + (size_t)inst * inst_chunks;
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    int c = tid - u0 + q * NU;
                    asm("" : "+v"(c));   // the chunk's place again, not kept in a register through the stream
                    if (c < R::R) {
                        const float4 v = s_new4[c];
                        st_record<D>(dst + rec_at(c), v.x, v.y, v.z, v.w);
                    }
                }
            }
            const int ut = tid - u0;
            if (p.theta != nullptr && ut >= 0 && ut < D / 4) {
                float4 *tdst = reinterpret_cast<float4 *>(p.theta + ((size_t)inst * K + a_upd) * D);
                tdst[ut] = make_float4(s_new[rec_pos_theta<D, TF>(4 * ut)], s_new[rec_pos_theta<D, TF>(4 * ut + 1)],
                                       s_new[rec_pos_theta<D, TF>(4 * ut + 2)], s_new[rec_pos_theta<D, TF>(4 * ut + 3)]);
            }
            if (p.keep_stats && ut == 0)
                p.stats[(size_t)inst * K + a_upd] =
                    make_int2(s_stu[0] + 1, __float_as_int(__int_as_float(s_stu[1]) + r));
        }
    };
    // A slice of the updated arm's record from LDS, as the stream holds one.
    auto updated_slice = [&](float4 *c4) {
#pragma unroll
        for (int sidx = 0; sidx < R::MQ; ++sidx) c4[sidx] = s_new4[sidx * G + j];
        const float *tl = s_new + 4 * R::MAIN + TF * j;
        c4[R::MQ] = make_float4(tl[0], tl[1], tl[2], 0.0f);
    };
    auto score_updated = [&]() {
        float4 c4[S];
        updated_slice(c4);
        const float *f = reinterpret_cast<const float *>(c4);
        float m, w2;
        slice_terms<D>(f, sx, m, w2);
        m = group_sum<G>(m);
        w2 = group_sum<G>(w2);
        if (lane == 0) s_sc[a_upd] = make_float2(m, w2);
    };
    // One pass: the arm of this lane's group in slot `slot`.  The updated arm,
    // in slot nlist, is scored from LDS exactly as the others are from HBM.
    auto score = [&](float4 *c4, int slot) {
        if (early && upd_in && slot - grp + apw > nlist) {   // the pass that holds slot nlist
            if (slot == nlist) updated_slice(c4);
        }
        const float *f = reinterpret_cast<const float *>(c4);
        float m, w2;
        slice_terms<D>(f, sx, m, w2);
        m = group_sum<G>(m);
        w2 = group_sum<G>(w2);
        if (slot < total && j == 0) s_sc[s_list[slot]] = make_float2(m, w2);
    };

    if (greedy) {
        // Eq. 2: only theta_k^T x_t, read from the contiguous theta copy by
        // groups of D/4 lanes, one float4 each.  UT passes' loads are issued
        // before any of them is used, so that an instance waits for one load
        // latency per UT passes, the first of them beside the previous record's.
        constexpr int GT = D / 4, APT = nthr / GT, UT = D == 32 ? 4 : 8;
        int t = tid;
        asm("" : "+v"(t));   // (keeps what follows out of the other branch's registers)
        const int jt = t % GT, gt = t / GT;
        const char *th_bytes = reinterpret_cast<const char *>(p.theta) + (size_t)inst * K * D * 4;
        float4 v[UT];
        auto theta_fetch = [&](int base) {
#pragma unroll
            for (int u = 0; u < UT; ++u) {
                const int slot = base + u * APT + gt;
                if (slot < nlist)
                    v[u] = ld_nt(reinterpret_cast<const float4 *>(th_bytes + (uint32_t)s_list[slot] * (D * 4) + jt * 16));
            }
        };
        theta_fetch(0);
        float2 own = make_float2(0.0f, 0.0f);
        if (!FOLD && upd_in && wave == 0)
            own = *reinterpret_cast<const float2 *>(th_bytes + (uint32_t)a_own * (D * 4) + t % G * 8);
        record_ready();
        update();
        const float4 x4 = s_x4[jt];
        for (int base = 0; base < nlist;) {
#pragma unroll
            for (int u = 0; u < UT; ++u) {
                const int slot = base + u * APT + gt;
                float m = fmaf(v[u].w, x4.w, fmaf(v[u].z, x4.z, fmaf(v[u].y, x4.y, v[u].x * x4.x)));
                m = group_sum<GT>(m);
                if (slot < nlist && jt == 0) s_sc[s_list[slot]] = make_float2(m, 0.0f);
            }
            base += UT * APT;
            if (base < nlist) theta_fetch(base);
        }
        // the updated arm, by the theta terms of its record
        if (upd_in && wave == 0) {
            const int jg = t % G;
            const float2 xt = reinterpret_cast<const float2 *>(s_x)[jg];
            if constexpr (FOLD) {
                const float *tl = s_new + 4 * R::MAIN + TF * jg;
                own = make_float2(tl[1], tl[2]);
            }
            const float m = group_sum<G>(fmaf(own.y, xt.y, own.x * xt.x));
            if (lane == 0) s_sc[a_own] = make_float2(m, 0.0f);
        }
    } else {
        if (streams) fetch(grp, buf_a);
        record_ready();
        if (early) update();
        // ---- scoring of every listed arm (Eq. 1), two passes in flight ----
        if (streams) {
            selectors();
            if constexpr (!FOLD) {
                fetch(apw + grp, buf_b);
                for (int u = 2; u < NBUF; ++u) fetch(u * apw + grp, buf_more[u - 2]);
                for (int base = 0;;) {
                    score(buf_a, base + grp);
                    score(buf_b, base + apw + grp);
                    for (int u = 2; u < NBUF; ++u) score(buf_more[u - 2], base + u * apw + grp);
                    base += NBUF * apw;
                    if (base >= total) break;
                    fetch(base + grp, buf_a);
                    fetch(base + apw + grp, buf_b);
                    for (int u = 2; u < NBUF; ++u) fetch(base + u * apw + grp, buf_more[u - 2]);
                }
            } else
            for (int base = 0;;) {
                if (base + apw < nlist) fetch(base + apw + grp, buf_b);
                score(buf_a, base + grp);
                base += apw;
                if (base >= total) break;
                if (base + apw < nlist) fetch(base + apw + grp, buf_a);
                score(buf_b, base + grp);
                base += apw;
                if (base >= total) break;
            }
        }
        if (!early) {
            update();
            if (upd_in && wave == 0) {   // scored on its own, after the stream
                selectors();
                score_updated();
            }
        }
    }

    if (!decide) {
        if (tid == 0) {
            blk[kInstAprev] = -1;
            if (inst == 0) p.hdr->pending = 0;
        }
        if (ph_lane) blk[tid] = s_phw[tid - kInstMode];
        write_back();
        return;
    }

    if (!x_ok) {
        if (p.scores != nullptr) {
            float *sc = p.scores + (size_t)inst * 2 * K;
            for (int q = tid; q < K; q += nthr) {
                sc[q] = -INFINITY;
                sc[K + q] = -INFINITY;
            }
        }
        if (tid == 0) {
            blk[kInstBad] += 1;
            blk[kInstAprev] = -1;
            if (p.action != nullptr) p.action[inst] = -1;
            if (inst == 0) {
                p.hdr->t = p.t_next;
                p.hdr->pending = 1;
            }
        }
        if (ph_lane) blk[tid] = s_phw[tid - kInstMode];
        if constexpr (ENV)
            if (wave == 0) agft_env_detail::env_epilogue(env_args_again(), inst, -1, lane, env_pre, s_envw);
        write_back();
        return;
    }
    // ---- pruning and argmax over the scores in LDS ----
    const bool prune_now = p.prune_now && !greedy;
    const bool stat_anchor = p.rf.now && p.rf.stat;
    float *sc = p.scores != nullptr ? p.scores + (size_t)inst * 2 * K : nullptr;
    // Where nothing asks for the bounds by arm (no rule-1 step, score dump or
    // statistical anchor), wavefront 0 alone walks the list; the others write
    // the updated record back meanwhile and are done.
    const bool by_list = !prune_now && sc == nullptr && !stat_anchor;
    const int nplay = nlist + upd_in;
    auto bounds_of = [&](float2 v) {   // (UCB, LCB); once exploiting both are theta^T x
        const float w = sqrtf(v.y);
        return greedy ? make_float2(v.x, v.x) : make_float2(fmaf(p.alpha, w, v.x), fmaf(-p.alpha, w, v.x));
    };
    if (NW > 1 && by_list && wave > 0) write_back();
    __syncthreads();
    if (NW > 1 && by_list && wave > 0) return;
    if (!by_list) {
        for (int slot = tid; slot < nplay; slot += nthr) {
            const int k = s_list[slot];
            s_sc[k] = bounds_of(s_sc[k]);
        }
        __syncthreads();
    }
    auto is_active = [&](int k) { return k < K && ((s_mask[k >> 5] >> (k & 31)) & 1u) != 0; };
    float lstar = -INFINITY;
    if (prune_now) {
        float l = -INFINITY;
        for (int k = tid; k < K; k += nthr)
            if (is_active(k)) l = fmaxf(l, s_sc[k].y);
        l = wave_reduce(l, [](float a, float b) { return fmaxf(a, b); });
        if (lane == 0) s_red_v[wave] = l;
        __syncthreads();
        for (int w = 0; w < nwave; ++w) lstar = fmaxf(lstar, s_red_v[w]);
        __syncthreads();
    }
    BestPair b{-INFINITY, 0x7fffffff};
    BestPair sb{-INFINITY, 0x7fffffff};   // statistical refinement anchor
    int n = 0;
    float top1 = -INFINITY, top2 = -INFINITY;   // two largest kept scores (with the dump only)
    if (by_list)
        for (int slot = lane; slot < nplay; slot += kWave) {
            const int k = s_list[slot];
            b = better(b, BestPair{bounds_of(s_sc[k]).x, k});
        }
    else
    for (int base = 0; base < K; base += nthr) {
        const int k = base + tid;
        const bool act = is_active(k);
        const float u = act ? s_sc[k].x : -INFINITY;
        const bool keep = act && !(u < lstar);
        n += __popcll(__ballot(keep));   // uniform over the wavefront
        if (keep) {
            b = better(b, BestPair{u, k});
            if (sc != nullptr) {
                top2 = fmaxf(top2, fminf(top1, u));
                top1 = fmaxf(top1, u);
            }
            if (stat_anchor) {
                // best mean reward among the arms with enough rewards (this
                // step's update already counted: the updated arm's count and
                // sum are written back only at the end of the step)
                const int2 v = k == a_upd ? make_int2(s_stu[0] + 1, __float_as_int(__int_as_float(s_stu[1]) + r))
                                          : p.stats[(size_t)inst * K + k];
                if (v.x >= p.rf.min_n) sb = better(sb, BestPair{__int_as_float(v.y) / (float)v.x, k});
            }
        }
        if (sc != nullptr && k < K) {
            st_word<!FOLD>(reinterpret_cast<int32_t *>(sc + k), __float_as_int(u));
            st_word<!FOLD>(reinterpret_cast<int32_t *>(sc + K + k), __float_as_int(act ? s_sc[k].y : -INFINITY));
        }
        if (prune_now) {
            // clear the arms rule 1 removed from the global words (non-sticky:
            // the words become exactly this step's removals, all other arms set)
            const unsigned long long bal = __ballot(keep);
            const int w0 = (base + wave * kWave) >> 5;
            uint32_t *mwo = p.mask + (size_t)inst * KW;
            auto all_arms = [&](int w) {
                return K - 32 * w >= 32 ? 0xffffffffu : (1u << (K - 32 * w)) - 1u;
            };
            if (lane == 0 && w0 < KW) {
                const uint32_t from = reset ? all_arms(w0) : s_raw[w0];
                s_raw[w0] = from & ~(s_mask[w0] & ~(uint32_t)(bal & 0xffffffffull));
                mwo[w0] = s_raw[w0];
            }
            if (lane == 0 && w0 + 1 < KW) {
                const uint32_t from = reset ? all_arms(w0 + 1) : s_raw[w0 + 1];
                s_raw[w0 + 1] = from & ~(s_mask[w0 + 1] & ~(uint32_t)(bal >> 32));
                mwo[w0 + 1] = s_raw[w0 + 1];
            }
        }
    }
    int best_arm = 0x7fffffff;
    if (NW == 1 || by_list) best_arm = wave_best_arm(b);
    else b = wave_best(b);
    if (by_list) n = nplay;
    if (stat_anchor) sb = wave_best(sb);
    __shared__ float s_top[kMaxWaves][2];
    if (sc != nullptr) {
        // the two largest of a pair of (largest, second) pairs
        auto merge = [&](float o1, float o2) {
            top2 = fmaxf(fminf(top1, o1), fmaxf(top2, o2));
            top1 = fmaxf(top1, o1);
        };
        merge(partner<0>(top1), partner<0>(top2));
        merge(partner<1>(top1), partner<1>(top2));
        merge(partner<2>(top1), partner<2>(top2));
        merge(partner<3>(top1), partner<3>(top2));
        merge(partner<4>(top1), partner<4>(top2));
        merge(partner<5>(top1), partner<5>(top2));
        if (lane == 0) {
            s_top[wave][0] = top1;
            s_top[wave][1] = top2;
        }
    }
    // a one-wavefront workgroup has its results in every lane already
    const bool merge_waves = NW > 1 && !by_list;
    if (merge_waves) {
        if (lane == 0) {
            s_red_v[wave] = b.v;
            s_red_k[wave] = b.k;
            s_red_n[wave] = n;
            s_red_v2[wave] = sb.v;
            s_red_k2[wave] = sb.k;
        }
        __syncthreads();
    }
    if (wave == 0) {
        // every lane of wavefront 0 reduces the per-wave results, then the
        // lanes write the instance block (action, count, context) at once
        int cnt = n;
        if (merge_waves) {
            BestPair best{s_red_v[0], s_red_k[0]};
            cnt = s_red_n[0];
            for (int w = 1; w < nwave; ++w) {
                best = better(best, BestPair{s_red_v[w], s_red_k[w]});
                cnt += s_red_n[w];
            }
            best_arm = best.k;
        }
        const int a = best_arm == 0x7fffffff ? -1 : best_arm;
        // refinement after the decision: a window of 2*half+1 arms around the
        // anchor, every arm at full resolution, from the next step on
        int anchor = -1;
        if (p.rf.now && a >= 0) {
            if (p.rf.stat) {
                BestPair sbest = sb;
                if constexpr (NW > 1) {
                    sbest = BestPair{s_red_v2[0], s_red_k2[0]};
                    for (int w = 1; w < nwave; ++w) sbest = better(sbest, BestPair{s_red_v2[w], s_red_k2[w]});
                }
                anchor = sbest.k == 0x7fffffff ? -1 : sbest.k;
            } else {
                anchor = a;
            }
        }
        const int nlo = anchor - p.rf.half > 0 ? anchor - p.rf.half : 0;
        const int nhi = anchor + p.rf.half < K - 1 ? anchor + p.rf.half : K - 1;
        if (anchor >= 0) {
            // arms in play in the new space
            int c2 = lane < KW ? __popc(s_raw[lane] & space_bits(lane, nlo, nhi, 1)) : 0;
            c2 = wave_reduce(c2, [](int a, int c) { return a + c; });
            cnt = c2;
        }
        if (lane == 0) {
            if (p.action != nullptr) p.action[inst] = a;
            if (inst == 0) {
                p.hdr->t = p.t_next;
                p.hdr->pending = 1;
            }
        }
        constexpr bool kThrough = !FOLD && NW == 4;
        if (lane <= kInstKact) st_word<kThrough>(blk + lane, lane == kInstAprev ? a : cnt);
        if (sc != nullptr && lane == kInstGap) {
            float t1 = top1, t2 = top2;   // one wavefront: already merged in every lane
            if constexpr (NW > 1) {
                t1 = s_top[0][0];
                t2 = s_top[0][1];
            }
            for (int w = 1; w < nwave; ++w) {
                t2 = fmaxf(fminf(t1, s_top[w][0]), fmaxf(t2, s_top[w][1]));
                t1 = fmaxf(t1, s_top[w][0]);
            }
            st_word<kThrough>(blk + kInstGap, __float_as_int(t1 - t2));   // +inf with one kept arm
        }
        if (anchor >= 0 && lane >= kInstLo && lane <= kInstStride)
            blk[lane] = lane == kInstLo ? nlo : (lane == kInstHi ? nhi : 1);
        if (ph_lane) st_word<kThrough>(blk + tid, s_phw[tid - kInstMode]);
        if (lane >= kInstX && lane < kInstX + D)
            st_word<kThrough>(blk + lane, __float_as_int(s_x[lane - kInstX]));
        // the context and reward read at the start are dead by now: the
        // environment's response overwrites them in place
        if constexpr (ENV) agft_env_detail::env_epilogue(env_args_again(), inst, a, lane, env_pre, s_envw);
    }
    if (NW == 1 || !by_list) write_back();
}

template <int D, int TF, int W, int NW, bool ENV>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(ENV && D == 16 && W > 6 ? W - 1 : W)))
void agft_step_kernel(StepArgs p, agft_env_detail::EnvArgs env) {
    step_body<D, TF, NW, ENV, true>(p, env);
}

// The step after agft_update_kernel: it only reads the records.  An instance
// has two passes' loads in flight together, three for the four-wavefront
// d = 16 launch of four workgroups per compute unit, which leaves the
// registers for it (K=128 d=16 B=65,536, us per step with the update, before
// st_word's stores: 745 with two, 737 with three or four).
template <int D, int TF, int W, int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(D == 16 && W == 6 && NW == 4 ? 5 : W)))
void agft_score_kernel(StepArgs p) {
    step_body<D, TF, NW, false, false, D == 16 && W == 6 && NW == 4 ? 3 : 2>(p, agft_env_detail::EnvArgs{});
}

// Folds every instance's previous reward into its arm, ahead of the score
// kernel.  A wavefront takes 64/D instances, one per segment of D lanes: lane
// j of a segment holds column j of the factor, so the chain of square roots
// and divisions is worked out once for all of them, and each row of S' is one
// segment prefix sum.  The operations and their order are those of the step
// kernel's own update for workgroups of ORDER wavefronts, so the results are
// the same bits.  Bound by the round trips to the instance's words and then to
// its record, and by HBM: 65,536 instances at d = 16 take 24 us (80 MB of
// records read and written), 16,384 take 8.6 us.  The records go back with the
// non-temporal hint at every d: with nothing else in the kernel it makes no
// difference at d = 8 and 32 (us per step with and without: 65,536 x 128 x 8 284.2
// / 284.8, 16,384 x 64 x 32 399.5 / 399.9, with eight arms left 52.2 / 51.5 and
// 86.4 / 86.4).
constexpr int kUpdateThreads = 256;
template <int D, int TF, int ORDER>
__global__ __launch_bounds__(kUpdateThreads) void agft_update_kernel(StepArgs p) {
#pragma clang fp contract(off)
    using R = Rec<D, TF>;
    constexpr int G = R::G, NI = kWave / D, WV = kUpdateThreads / kWave;
    constexpr int NQ = (NI * R::R + kWave - 1) / kWave;   // loads of 64 chunks per wavefront
    __shared__ float4 s_rec4[WV][NQ * kWave];
    __shared__ float4 s_xp4[WV][NI][D / 4];
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int jc = lane % D, seg = lane / D;
    const int i0 = (blockIdx.x * WV + wave) * NI;
    if (i0 >= p.B) return;
    const int inst = i0 + seg < p.B ? i0 + seg : p.B - 1;   // (past the end: repeats the last, stores nothing)
    const int K = p.K;
    const size_t inst_chunks = (size_t)((K + R::NB - 1) / R::NB) * R::BLK;
    int32_t *blk = p.inst + (size_t)inst * p.IW;
    const int a_prev = blk[kInstAprev];
    const float xp = reinterpret_cast<const float *>(blk)[kInstX + jc];
    const float r = p.reward[inst];
    const bool upd = i0 + seg < p.B && a_prev >= 0 && a_prev < K && isfinite(r);
    const int a = upd ? a_prev : 0;
    const int rec_main = a / R::NB * R::BLK + a % R::NB * R::MAIN;
    const int rec_tail = a / R::NB * R::BLK + R::NB * R::MAIN + a % R::NB * R::TAIL - R::MAIN;
    // chunk q of the wavefront's NI records, in LDS order
    auto place = [&](int q) {
        const int s = q / R::R, c = q - s * R::R;
        const int m = __shfl(rec_main, s * D), t = __shfl(rec_tail, s * D);
        const size_t at = (size_t)(i0 + s < p.B ? i0 + s : p.B - 1) * inst_chunks;
        return at + (uint32_t)(c + (c < R::MAIN ? m : t));
    };
    size_t at[NQ];
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const int q = u * kWave + lane;
        at[u] = place(q < NI * R::R ? q : NI * R::R - 1);
        load_to_lds<D>(p.arms + at[u], s_rec4[wave] + u * kWave);
    }
    int2 st = make_int2(0, 0);
    if (p.keep_stats && jc == 0) st = p.stats[(size_t)inst * K + a];
    reinterpret_cast<float *>(s_xp4[wave][seg])[jc] = xp;
    // the records have landed (gfx9 encoding: vmcnt 0 only), and the wavefront's
    // LDS writes are seen by its other lanes
    __builtin_amdgcn_s_waitcnt(0x0F70);
    auto lds_order = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    lds_order();

    float *rec = reinterpret_cast<float *>(s_rec4[wave] + seg * R::R);
    // column jc, rows 0..jc: top down in slice jc, or bottom up in slice D-1-jc,
    // where row 0 is the tail float
    const bool first = jc < G;
    const int sl = first ? jc : D - 1 - jc;
    auto pos = [&](int i) {
        const int e = first ? i : D - i;
        return e < D ? 4 * ((e >> 2) * G + sl) + (e & 3) : 4 * R::MAIN + TF * sl;
    };
    float col[D], xr[D];
#pragma unroll
    for (int q = 0; q < D / 4; ++q) {
        const float4 v = s_xp4[wave][seg][q];
        xr[4 * q] = v.x;
        xr[4 * q + 1] = v.y;
        xr[4 * q + 2] = v.z;
        xr[4 * q + 3] = v.w;
    }
#pragma unroll
    for (int i = 0; i < D; ++i) col[i] = i <= jc ? rec[pos(i)] : 0.0f;
    // f_j = sum_{i<=j} S_ij xp_i: chains of rows RP apart, summed as the lanes
    // and wavefronts of the step kernel's update sum them
    constexpr int SEGS = kWave / D, RP = ORDER * SEGS;
    float fj = 0.0f;
#pragma unroll
    for (int w = 0; w < ORDER; ++w) {
        float part[SEGS];
#pragma unroll
        for (int g = 0; g < SEGS; ++g) {
            part[g] = 0.0f;
#pragma unroll
            for (int i = w * SEGS + g; i < D; i += RP) part[g] = fmaf(col[i], xr[i], part[g]);
        }
#pragma unroll
        for (int h = 1; h < SEGS; h *= 2)
#pragma unroll
            for (int g = 0; g + h < SEGS; g += 2 * h) part[g] += part[g + h];
        fj = w == 0 ? part[0] : fj + part[0];
    }
    const float f2 = fj * fj;
    const float incl = segment_scan<D>(fj, fj, f2, lane);
    const float al = 1.0f + incl;
    const float al_prev = 1.0f + (incl - f2);
    const float ca = sqrtf(al_prev / al), cb = fj / sqrtf(al_prev * al);
    const float al_last = __shfl(al, lane | (D - 1));
    const int tpos = 4 * R::MAIN + TF * (jc >> 1) + 1 + (jc & 1);
    const float theta = rec[tpos];
    float pred = group_sum<D < 16 ? D : 16>(xp * theta);
    if constexpr (D == 32) pred = across<16>(pred, [](float x, float y) { return x + y; });
    const float err = r - pred;
    const float inv_al = 1.0f / al_last;
#pragma unroll
    for (int i = 0; i < D; ++i) {
        const float q = fj * col[i];
        const float qi = segment_scan<D>(fj, col[i], q, lane);
        if (i <= jc) rec[pos(i)] = fmaf(ca, col[i], -(cb * (qi - q)));
        col[i] = qi;
    }
    // the rows' totals, which the segment's last lane holds: (S f)_i
    if (jc == D - 1) {
#pragma unroll
        for (int q = 0; q < D / 4; ++q)
            s_xp4[wave][seg][q] = make_float4(col[4 * q], col[4 * q + 1], col[4 * q + 2], col[4 * q + 3]);
    }
    lds_order();
    const float gain = reinterpret_cast<const float *>(s_xp4[wave][seg])[jc];
    const float theta_new = fmaf(gain * inv_al, err, theta);
    rec[tpos] = theta_new;
    lds_order();
    const unsigned long long upd_lanes = __ballot(upd);
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const int q = u * kWave + lane;
        const int s = q / R::R;
        if (q < NI * R::R && ((upd_lanes >> (s * D)) & 1ull) != 0) {
            const float4 v = s_rec4[wave][q];
            __builtin_nontemporal_store(nt_f4{v.x, v.y, v.z, v.w}, reinterpret_cast<nt_f4 *>(p.arms + at[u]));
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) p.hdr->pending = kPendingFolded;
    if (upd && p.theta != nullptr) p.theta[((size_t)inst * K + a) * D + jc] = theta_new;
    if (upd && p.keep_stats && jc == 0)
        p.stats[(size_t)inst * K + a] = make_int2(st.x + 1, __float_as_int(__int_as_float(st.y) + r));
}

// ---- initialisation and export ----

struct InitArgs {
    char *base;           // the state buffer
    Layout lay;
    StateHeader h;
    int32_t B, K;
    int32_t stride0;      // stride of the starting action space
    float inv_sqrt_lambda;
};

// A launch takes fewer than 2^32 threads per dimension of its grid, which a
// buffer past 68 GB exceeds at one chunk per thread: workgroups beyond kRow
// take further rows, the last of them part-filled.
constexpr unsigned kRow = 1u << 23;
dim3 rows_of(size_t groups) {
    return groups <= kRow ? dim3((unsigned)groups) : dim3(kRow, (unsigned)((groups + kRow - 1) / kRow));
}
__device__ __forceinline__ uint64_t row_group() { return (uint64_t)blockIdx.y * gridDim.x + blockIdx.x; }

// Record chunks per workgroup of the initialisation.
constexpr int kInitThreads = 256, kInitChunks = kInitThreads;

// Writes every byte of the state buffer (the gaps between regions as zeros).
// Bound by HBM's write rate, so the values have to cost next to nothing: the
// only elements of a record that are not zero are S_ii = 1/sqrt(lambda), at
// positions j and j+1 of lane slice j (columns j and D-1-j), all in the main
// part, and a chunk's place in its block comes from divisions by constants.
// One chunk per thread, each workgroup's contiguous.  Measured on MI355X with
// 65,536 x 128 x 16 (5.17 GB): 5,080 us with the index of every element
// unpacked by a loop behind 64-bit divisions; so, 845 us (6.1 TB/s), 906 us
// with two chunks per thread, 915 us with eight.  1,024 x 256 x 32: 1,040 ->
// 99 us.
template <int D, int TF>
__global__ __launch_bounds__(kInitThreads) void agft_init_kernel(InitArgs p) {
    using R = Rec<D, TF>;
    constexpr int IW = (kInstX + D + 15) / 16 * 16;   // inst_words(D)
    const int tid = threadIdx.x;
    const uint32_t KB = (uint32_t)(p.K + R::NB - 1) / R::NB;
    const uint64_t chunks = (uint64_t)p.B * KB * R::BLK;
    const int tail_arms = p.K % R::NB;   // arms of an instance's last block, if part-filled
    const uint64_t group = row_group();
    const uint64_t c0 = group * kInitChunks;
    const uint64_t blk0 = c0 / R::BLK;
    const uint32_t o0 = (uint32_t)(c0 - blk0 * R::BLK);
    const uint32_t kb0 = (uint32_t)(blk0 % KB);
    float4 *arms = reinterpret_cast<float4 *>(p.base + p.lay.arms) + c0;
    const uint32_t left = c0 >= chunks ? 0u
                        : chunks - c0 < (uint64_t)kInitChunks ? (uint32_t)(chunks - c0) : (uint32_t)kInitChunks;
#pragma unroll
    for (int q = 0; q < kInitChunks / kInitThreads; ++q) {
        const uint32_t c = (uint32_t)(q * kInitThreads + tid);
        const uint32_t b = (o0 + c) / R::BLK, o = (o0 + c) % R::BLK;
        const int cc = (int)(o % R::MAIN), j = cc % R::G, e0 = 4 * (cc / R::G);
        bool arm = o < (uint32_t)(R::NB * R::MAIN);
        if (tail_arms != 0) arm = arm && ((int)(o / R::MAIN) < tail_arms || (kb0 + b) % KB != KB - 1);
        nt_f4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = arm && (e0 + e == j || e0 + e == j + 1) ? p.inv_sqrt_lambda : 0.0f;
        if (c < left) *reinterpret_cast<nt_f4 *>(arms + c) = v;
    }

    const uint64_t gtid = group * kInitThreads + tid;
    const uint64_t gsz = (uint64_t)gridDim.x * gridDim.y * kInitThreads;
    // masks, every arm in play, and the gaps before and after them
    const uint32_t KW = (uint32_t)(p.K + 31) / 32;
    const uint32_t last = p.K % 32 ? (1u << (p.K % 32)) - 1u : 0xffffffffu;
    uint32_t *mask = reinterpret_cast<uint32_t *>(p.base + p.lay.mask);
    const uint64_t nmask = (uint64_t)p.B * KW;
    for (uint64_t idx = gtid; idx < (p.lay.inst - p.lay.mask) / 4; idx += gsz)
        mask[idx] = idx >= nmask ? 0u : last == 0xffffffffu || idx % KW != KW - 1 ? 0xffffffffu : last;
    uint32_t *pad = reinterpret_cast<uint32_t *>(p.base + p.lay.arms) + chunks * 4;
    for (uint64_t idx = gtid; idx < (p.lay.mask - p.lay.arms) / 4 - chunks * 4; idx += gsz) pad[idx] = 0u;
    // instance blocks
    int32_t *inst = reinterpret_cast<int32_t *>(p.base + p.lay.inst);
    const uint64_t ninst = (uint64_t)p.B * IW;
    for (uint64_t idx = gtid; idx < (p.lay.stats - p.lay.inst) / 4; idx += gsz) {
        const int w = (int)(idx % IW);
        const int hi = p.K - 1;
        inst[idx] = idx >= ninst ? 0
                  : w == kInstAprev || w == kInstMode ? -1
                  : w == kInstKact ? hi / p.stride0 + 1   // arms on the starting grid
                  : w == kInstPhMargin ? 0x7f800000       // +inf: no test yet
                  : w == kInstHi ? hi
                  : w == kInstStride ? p.stride0
                  : 0;
    }
    // reward counts and sums, the theta copy: zeros to the end of the buffer
    float4 *zero = reinterpret_cast<float4 *>(p.base + p.lay.stats);
    for (uint64_t idx = gtid; idx < (p.lay.total - p.lay.stats) / 16; idx += gsz)
        zero[idx] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (gtid == 0) *reinterpret_cast<StateHeader *>(p.base) = p.h;
}

// Materialises theta and A^{-1} = S S^T.  A workgroup takes whole blocks of
// records, contiguous in HBM, spreads their factors over LDS (column-major,
// columns D + 4 floats apart, so that four rows are one aligned 16-byte read)
// and each thread forms one 4 x 4 tile of one arm's A^{-1}, starting at the
// tile's own first non-zero column, and writes it as four 16-byte stores.
// Each entry sums its columns in ascending order.  Bound by HBM (a record
// read, 4(d + d^2) bytes written per arm); measured on MI355X for both
// outputs: 4,096 x 128 x 16 3,534 us with one thread per arm and its record
// in scratch memory, 162 us so (0.89 GB, 5.5 TB/s); 1,024 x 256 x 32 300 us
// (5.6 TB/s).
constexpr int kExportThreads = 256;
template <int D, int TF>
__global__ __launch_bounds__(kExportThreads) void agft_export_kernel(const float4 *arms, int B, int K, float *theta,
                                                                     float *ainv) {
    using R = Rec<D, TF>;
    constexpr int TR = D / 4, TILES = TR * TR;          // tiles per row and per arm
    constexpr int AW = kExportThreads / TILES;          // arms per workgroup
    constexpr int BW = AW / R::NB;                      // blocks per workgroup
    static_assert(AW % R::NB == 0, "whole blocks per workgroup");
    constexpr int CS = D + 4, AS = D * CS;              // floats per column, per arm
    __shared__ __attribute__((aligned(16))) float s_S[AW * AS];
    __shared__ __attribute__((aligned(16))) float s_theta[AW * D];
    const int tid = threadIdx.x;
    const uint32_t KB = (uint32_t)(K + R::NB - 1) / R::NB;
    const uint64_t nblk = (uint64_t)B * KB;
    const uint64_t blk0 = row_group() * BW;
    if (blk0 >= nblk) return;
    const int nch = (int)(nblk - blk0 < (uint64_t)BW ? nblk - blk0 : (uint64_t)BW) * R::BLK;
    const float4 *src = arms + blk0 * R::BLK;
#pragma unroll
    for (int c0 = 0; c0 < BW * R::BLK; c0 += kExportThreads) {
        const int c = c0 + tid;
        if (c >= nch) break;
        const float4 v4 = ld_nt(src + c);
        const float v[4] = {v4.x, v4.y, v4.z, v4.w};
        const int b = c / R::BLK, o = c % R::BLK;
        if (o < R::NB * R::MAIN) {
            const int cc = o % R::MAIN, j = cc % R::G, e0 = 4 * (cc / R::G);
            float *S = s_S + (b * R::NB + o / R::MAIN) * AS;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = e0 + q;
                S[e <= j ? j * CS + e : (D - 1 - j) * CS + D - e] = v[q];
            }
        } else {
            const int ot = o - R::NB * R::MAIN;
            const int a = b * R::NB + ot / R::TAIL;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int t = 4 * (ot % R::TAIL) + q, j = t / TF, i = t % TF;
                if (i == 0) s_S[a * AS + (D - 1 - j) * CS] = v[q];   // position D: row 0 of column D-1-j
                else if (i < 3) s_theta[a * D + 2 * j + i - 1] = v[q];
            }
        }
    }
    __syncthreads();
    // where arm `a` of the workgroup goes, B*K if it has no place
    auto place = [&](int a) -> uint64_t {
        const uint64_t blk = blk0 + (uint32_t)(a / R::NB);
        const uint64_t i = blk / KB;
        const uint32_t k = (uint32_t)(blk - i * KB) * R::NB + (uint32_t)(a % R::NB);
        return blk < nblk && k < (uint32_t)K ? i * (uint32_t)K + k : (uint64_t)B * (uint32_t)K;
    };
    if (theta != nullptr)
        for (int t = tid; t < AW * TR; t += kExportThreads) {
            const uint64_t g = place(t / TR);
            if (g < (uint64_t)B * (uint32_t)K) {
                const float4 v = reinterpret_cast<const float4 *>(s_theta)[t];
                *reinterpret_cast<out_f4 *>(theta + g * D + 4 * (t % TR)) = out_f4{v.x, v.y, v.z, v.w};
            }
        }
    if (ainv == nullptr) return;
    const int a = tid / TILES, tr = tid % TILES / TR, tc = tid % TR;
    const uint64_t g = place(a);
    if (g >= (uint64_t)B * (uint32_t)K) return;
    const float *S = s_S + a * AS;
    const int r0 = 4 * tr, q0 = 4 * tc, first = r0 > q0 ? r0 : q0;
    float acc[4][4] = {};
    // the tile's first four columns hold the diagonal: S_ij with i > j is no element
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int jc = first + u;
        const float4 ra = *reinterpret_cast<const float4 *>(S + jc * CS + r0);
        const float4 qa = *reinterpret_cast<const float4 *>(S + jc * CS + q0);
        const float rv[4] = {ra.x, ra.y, ra.z, ra.w}, qv[4] = {qa.x, qa.y, qa.z, qa.w};
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc[r][q] = jc >= r0 + r && jc >= q0 + q ? fmaf(rv[r], qv[q], acc[r][q]) : acc[r][q];
    }
    for (int jc = first + 4; jc < D; ++jc) {
        const float4 ra = *reinterpret_cast<const float4 *>(S + jc * CS + r0);
        const float4 qa = *reinterpret_cast<const float4 *>(S + jc * CS + q0);
        const float rv[4] = {ra.x, ra.y, ra.z, ra.w}, qv[4] = {qa.x, qa.y, qa.z, qa.w};
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[r][q] = fmaf(rv[r], qv[q], acc[r][q]);
    }
    float *out = ainv + g * D * D + r0 * D + q0;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        *reinterpret_cast<out_f4 *>(out + r * D) = out_f4{acc[r][0], acc[r][1], acc[r][2], acc[r][3]};
}

}  // namespace

// ---- C ABI ----

struct agft_handle {
    agft_config cfg;
    Layout lay;
    char *base;
    hipStream_t stream;
    int64_t t;
    int pending;
    int folded;   // 1: the pending reward is in its arm already, by a step whose update ran and whose score launch failed
};

namespace {

bool config_ok(const agft_config *c) {
    if (c == nullptr) return false;
    if (c->B < 1 || c->K < 1 || c->K > kMaxK) return false;
    if (!std::isfinite(c->lambda) || !(c->lambda > 0.0f)) return false;
    if (!std::isfinite(c->alpha0) || c->alpha0 < 0.0f) return false;
    if (c->alpha_sched != 0 && c->alpha_sched != 1) return false;
    if (c->prune_rule < 0 || c->prune_rule > 15) return false;
    if (c->prune_period < 1) return false;
    if (c->prune_sticky != 0 && c->prune_sticky != 1) return false;
    if ((c->prune_rule & 2) && (c->ext_rounds < 0 || c->ext_min_n < 1 || !std::isfinite(c->ext_thr)))
        return false;
    if ((c->prune_rule & 4) && (c->hist_after < 0 || c->hist_min_n < 1 || c->hist_min_arms < 1 ||
                                !std::isfinite(c->hist_kappa) || c->hist_kappa < 0.0f))
        return false;
    if ((c->prune_rule & 8) && (c->cascade_k < 0 || c->cascade_k > c->K)) return false;
    if (c->exploit != 0 && c->exploit != 1) return false;
    if (c->refine != 0 && c->refine != 1) return false;
    if (c->refine && (c->refine_period < 1 || c->refine_stride < 1 || c->refine_half < 0 ||
                      c->refine_mature < 0 || c->refine_min_n < 1))
        return false;
    if (c->exploit && (!std::isfinite(c->ph_delta) || !std::isfinite(c->ph_lambda) || c->ph_lambda < 0.0f ||
                       c->ph_window < 0 || c->ph_min_rounds < 0))
        return false;
    if ((c->flags & ~AGFT_ADOPT_STATE) != 0) return false;
    return true;
}

// Context dimensions the kernels are built for; a non-sticky rule 1 only on
// its own (the paper's rules 2-8 remove arms for good, and one mask cannot
// hold both kinds of removal).
bool supported(const agft_config *c) {
    return (c->d == 8 || c->d == 16 || c->d == 32) && (c->prune_sticky || !(c->prune_rule & 14));
}

int hip_status(hipError_t e) { return e == hipSuccess ? AGFT_OK : AGFT_E_HIP; }

StateHeader make_header(const agft_config *c) {
    StateHeader h;
    std::memset(&h, 0, sizeof(h));
    h.magic = kMagic;
    h.version = AGFT_ABI_VERSION;
    h.B = c->B;
    h.K = c->K;
    h.d = c->d;
    h.chunks = chunks_for(c->d, tail_floats(*c));
    h.tail_floats = tail_floats(*c);
    h.stats_kept = stats_kept(*c) ? 1 : 0;
    h.mask_words = (c->K + 31) / 32;
    h.pending = 0;
    h.t = 0;
    h.lambda = c->lambda;
    h.alpha0 = c->alpha0;
    h.alpha_sched = c->alpha_sched;
    h.prune_rule = c->prune_rule;
    h.prune_period = c->prune_period;
    h.exploit = c->exploit;
    return h;
}

template <class T>
T *at(char *base, size_t off) {
    return reinterpret_cast<T *>(base + off);
}

// fn(d, tail floats) with both as compile-time constants, for a supported d.
template <class Fn>
void for_layout(int d, int tf, Fn fn) {
    auto with_d = [&](auto dc) {
        if (tf == 3) fn(dc, std::integral_constant<int, 3>{});
        else fn(dc, std::integral_constant<int, 4>{});
    };
    if (d == 8) with_d(std::integral_constant<int, 8>{});
    else if (d == 16) with_d(std::integral_constant<int, 16>{});
    else with_d(std::integral_constant<int, 32>{});
}

// agft_sim_step runs the environment in the step kernel's epilogue up to
// this many instances, and launches the step and environment kernels above.
constexpr int kFusedMaxB = 3072;
static_assert(kFusedMaxB < kSplitMinB, "a batch in the single launch has no update of its own");

// Dynamic LDS that caps a kernel at `cap` workgroups per compute unit: a
// 1/cap share of the unit's LDS less the kernel's static LDS, lowered in
// 512-byte steps until the occupancy calculator admits exactly cap
// workgroups (allocation granules round a request up).  Worked out once per
// kernel and device; a share the calculator does not confirm, or below what
// the kernel needs, leaves the launch uncapped.  Only host queries, no
// allocation; the error of a failed query is cleared so that the launch's
// own error check does not see it.
constexpr int kMaxDevices = 64;
template <int D, int TF, int W, int NW, bool ENV>
std::atomic<int64_t> *capped_lds_cache() {
    static std::atomic<int64_t> cache[kMaxDevices];   // 0: not worked out; else bytes + 1
    return cache;
}

size_t capped_lds(const void *kernel, int threads, size_t need, int cap, std::atomic<int64_t> *cache) {
    if (cap <= 0) return need;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return need;
    }
    if (dev < 0 || dev >= kMaxDevices) return need;
    int64_t v = cache[dev].load(std::memory_order_relaxed);
    if (v == 0) {
        int64_t dyn = 0;   // 0: uncapped
        int per_cu = 0;
        hipFuncAttributes fa;
        bool failed = hipDeviceGetAttribute(&per_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) !=
                          hipSuccess ||
                      hipFuncGetAttributes(&fa, kernel) != hipSuccess;
        if (!failed && per_cu > 0) {
            const int64_t max_dyn = 64 * 1024 - (int64_t)fa.sharedSizeBytes;
            for (int64_t d = (per_cu / cap - (int64_t)fa.sharedSizeBytes) / 16 * 16; d >= (int64_t)need && d > 0;
                 d -= 512) {
                if (d > max_dyn) continue;
                int blocks = 0;
                if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, kernel, threads, (size_t)d) != hipSuccess) {
                    failed = true;
                    break;
                }
                if (blocks == cap) {
                    dyn = d;
                    break;
                }
                if (blocks > cap) break;
            }
        }
        if (failed) (void)hipGetLastError();
        v = dyn + 1;
        cache[dev].store(v, std::memory_order_relaxed);
    }
    // (a share worked out for a smaller need than this launch's is not used)
    return v > 1 && (size_t)(v - 1) >= need ? (size_t)(v - 1) : need;
}

// The step kernel for one or four wavefronts per workgroup (the two widths
// waves_for chooses), each compiled for its width.
template <int D, int TF, int W, bool ENV>
void launch_width(int waves, int cap, unsigned grid, size_t lds, hipStream_t stream, const StepArgs &p,
                  const agft_env_detail::EnvArgs &e) {
    if (waves == 1) {
        hipLaunchKernelGGL((agft_step_kernel<D, TF, W, 1, ENV>), dim3(grid), dim3(kWave), lds, stream, p, e);
    } else {
        lds = capped_lds(reinterpret_cast<const void *>(&agft_step_kernel<D, TF, W, 4, ENV>), 4 * kWave, lds, cap,
                         capped_lds_cache<D, TF, W, 4, ENV>());
        hipLaunchKernelGGL((agft_step_kernel<D, TF, W, 4, ENV>), dim3(grid), dim3(4 * kWave), lds, stream, p, e);
    }
}

// The score kernel, likewise.
template <int D, int TF, int W>
void launch_score(int waves, int cap, unsigned grid, size_t lds, hipStream_t stream, const StepArgs &p) {
    if (waves == 1) {
        hipLaunchKernelGGL((agft_score_kernel<D, TF, W, 1>), dim3(grid), dim3(kWave), lds, stream, p);
    } else {
        static std::atomic<int64_t> cache[kMaxDevices];
        lds = capped_lds(reinterpret_cast<const void *>(&agft_score_kernel<D, TF, W, 4>), 4 * kWave, lds, cap, cache);
        hipLaunchKernelGGL((agft_score_kernel<D, TF, W, 4>), dim3(grid), dim3(4 * kWave), lds, stream, p);
    }
}

// The update on its own, for the order of sums of workgroups of `waves`; the
// launch's own status.
template <int D, int TF>
hipError_t launch_update(int waves, hipStream_t stream, StepArgs p) {
    constexpr int per_group = kUpdateThreads / D;
    const dim3 grid((unsigned)(((int64_t)p.B + per_group - 1) / per_group)), block(kUpdateThreads);
    const void *kernel = waves == 1 ? reinterpret_cast<const void *>(&agft_update_kernel<D, TF, 1>)
                                    : reinterpret_cast<const void *>(&agft_update_kernel<D, TF, 4>);
    void *args[] = {&p};
    return hipLaunchKernel(kernel, grid, block, args, 0, stream);
}

// One decision for every instance of handle h (and, with env, the
// environment's response): arguments checked by the caller.
int launch_step(agft_handle *h, const float *d_ctx, const float *d_reward, int32_t *d_action, float *d_scores,
                const agft_env_detail::EnvArgs *env) {
    const agft_config &c = h->cfg;
    StepArgs p;
    p.arms = at<float4>(h->base, h->lay.arms);
    p.mask = at<uint32_t>(h->base, h->lay.mask);
    p.inst = at<int32_t>(h->base, h->lay.inst);
    p.stats = at<int2>(h->base, h->lay.stats);
    p.theta = c.exploit ? at<float>(h->base, h->lay.theta) : nullptr;
    p.h.mask = c.prune_rule & 14;
    p.h.ext_rounds = c.ext_rounds;
    p.h.ext_min_n = c.ext_min_n;
    p.h.ext_thr = c.ext_thr;
    p.h.hist_after = c.hist_after;
    p.h.hist_min_n = c.hist_min_n;
    p.h.hist_kappa = c.hist_kappa;
    p.h.hist_min_arms = c.hist_min_arms;
    p.h.cascade_k = c.cascade_k;
    p.t = h->t;
    p.e.on = c.exploit;
    p.e.delta = c.ph_delta;
    p.e.lambda = c.ph_lambda;
    p.e.window = c.ph_window;
    p.e.min_rounds = c.ph_min_rounds;
    p.rf.now = (c.refine && d_ctx != nullptr && h->t > 0 && h->t % c.refine_period == 0) ? 1 : 0;
    p.rf.stat = h->t < c.refine_mature ? 1 : 0;
    p.rf.half = c.refine_half;
    p.rf.min_n = c.refine_min_n;
    p.hdr = at<StateHeader>(h->base, 0);
    p.ctx = d_ctx;
    p.reward = d_reward;
    p.action = d_ctx != nullptr ? d_action : nullptr;
    p.scores = d_ctx != nullptr ? d_scores : nullptr;
    p.B = c.B;
    p.K = c.K;
    p.KW = (c.K + 31) / 32;
    p.IW = inst_words(c.d);
    p.apply_update = h->pending;
    const int64_t t = h->t;
    p.prune_now = (d_ctx != nullptr && (c.prune_rule & 1) && t > 0 && t % c.prune_period == 0) ? 1 : 0;
    p.prune_reset = p.prune_now && !c.prune_sticky ? 1 : 0;
    p.alpha = c.alpha_sched == 0 ? c.alpha0 : (float)((double)c.alpha0 / std::sqrt((double)t + 1.0));
    p.t_next = d_ctx != nullptr ? t + 1 : t;
    agft_launch_shape shape;
    agft_launch_shape_for(&c, &shape);
    const int waves = waves_at(c, t);
    p.early_update = shape.early_update;
    p.keep_stats = stats_kept(c) ? 1 : 0;
    p.sum_waves = waves;
    if (waves != 1 && waves != 4) return AGFT_E_UNSUPPORTED;
    const unsigned grid = (unsigned)c.B;
    const size_t lds = step_lds_bytes(c.K);
    const bool packed_tails = shape.tail_floats == 3;
    hipStream_t s = h->stream;
    agft_env_detail::EnvArgs e{};
    if (env != nullptr) e = *env;
    // The simulator's single launch runs uncapped: the environment's
    // response at the end of each workgroup wants more instances in flight
    // (K=128 d=16, us per fused step, uncapped / at 4, measured when larger
    // batches took the single launch too: B=65,536 881.5 / 891.0, B=16,384
    // 211.9 / 218.0).
    const int cap = env != nullptr ? 0 : cu_workgroups_for(c, waves, shape.simd_waves);
    const int score_cap = cu_workgroups_for(c, score_waves_at(c, t), shape.simd_waves);
    // the update ahead of the step, where that pays (never for the simulator's
    // single launch, whose batches are small, nor for a flush); a step or flush
    // that finds the reward folded in already only takes what follows the update
    const bool split = env == nullptr && h->pending &&
                       (h->folded || (d_ctx != nullptr && split_update(c, t, d_scores != nullptr)));
    const int score_waves = score_waves_at(c, t);
    if (split && !h->folded) {
        hipError_t ran = hipErrorUnknown;
        for_layout(c.d, shape.tail_floats,
                   [&](auto dc, auto tf) { ran = launch_update<dc.value, tf.value>(waves, s, p); });
        if (ran == hipSuccess) h->folded = 1;
        if (hipGetLastError() != hipSuccess || ran != hipSuccess) return AGFT_E_HIP;
    }
#define AGFT_LAUNCH(D_, TF_, W_)                                                          \
    (env != nullptr ? launch_width<D_, TF_, W_, true>(waves, cap, grid, lds, s, p, e)    \
     : split        ? launch_score<D_, TF_, W_>(score_waves, score_cap, grid, lds, s, p) \
                    : launch_width<D_, TF_, W_, false>(waves, cap, grid, lds, s, p, e))
    switch (c.d) {
        case 8:
            if (packed_tails) AGFT_LAUNCH(8, 3, 7);
            else AGFT_LAUNCH(8, 4, 7);
            break;
        case 16:
            if (packed_tails && shape.simd_waves == 6) AGFT_LAUNCH(16, 3, 6);
            else if (packed_tails) AGFT_LAUNCH(16, 3, 7);
            else AGFT_LAUNCH(16, 4, 7);
            break;
        case 32:
            if (packed_tails) AGFT_LAUNCH(32, 3, 4);
            else AGFT_LAUNCH(32, 4, 4);
            break;
        default: return AGFT_E_UNSUPPORTED;
    }
#undef AGFT_LAUNCH
    if (hipGetLastError() != hipSuccess) return AGFT_E_HIP;
    h->folded = 0;
    if (d_ctx != nullptr) {
        h->t = t + 1;
        h->pending = 1;
    } else {
        h->pending = 0;
    }
    return AGFT_OK;
}

}  // namespace

extern "C" {

size_t agft_state_bytes(const agft_config *cfg) {
    if (!config_ok(cfg) || !supported(cfg)) return 0;
    return layout_for(*cfg).total;
}

int agft_create(const agft_config *cfg, void *d_state, size_t nbytes, void *stream, agft_handle **out) {
    if (out == nullptr) return AGFT_E_INVAL;
    *out = nullptr;
    if (!config_ok(cfg) || d_state == nullptr) return AGFT_E_INVAL;
    if (!supported(cfg)) return AGFT_E_UNSUPPORTED;
    if (reinterpret_cast<uintptr_t>(d_state) % kAlign != 0) return AGFT_E_INVAL;
    const Layout lay = layout_for(*cfg);
    if (nbytes < lay.total) return AGFT_E_INVAL;
    agft_handle *h = new (std::nothrow) agft_handle;
    if (h == nullptr) return AGFT_E_INVAL;
    h->cfg = *cfg;
    h->lay = lay;
    h->base = static_cast<char *>(d_state);
    h->stream = static_cast<hipStream_t>(stream);
    h->t = 0;
    h->pending = 0;
    h->folded = 0;
    const StateHeader want = make_header(cfg);
    if (cfg->flags & AGFT_ADOPT_STATE) {
        StateHeader got;
        hipError_t e = hipMemcpyAsync(&got, d_state, sizeof(got), hipMemcpyDeviceToHost, h->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
        if (e != hipSuccess) {
            delete h;
            return AGFT_E_HIP;
        }
        if (got.magic != kMagic || got.version != want.version || got.B != want.B || got.K != want.K ||
            got.d != want.d || got.chunks != want.chunks || got.tail_floats != want.tail_floats ||
            got.stats_kept != want.stats_kept ||
            got.exploit != want.exploit || got.t < 0 ||
            got.pending < 0 || got.pending > kPendingFolded) {
            delete h;
            return AGFT_E_STATE;
        }
        h->t = got.t;
        h->pending = got.pending != 0 ? 1 : 0;
        h->folded = got.pending == kPendingFolded ? 1 : 0;
        *out = h;
        return AGFT_OK;
    }
    InitArgs a;
    a.base = h->base;
    a.lay = lay;
    a.h = want;
    a.B = cfg->B;
    a.K = cfg->K;
    a.stride0 = cfg->refine ? cfg->refine_stride : 1;
    a.inv_sqrt_lambda = (float)(1.0 / std::sqrt((double)cfg->lambda));
    const size_t chunks = (size_t)cfg->B * instance_chunks(cfg->K, cfg->d, want.tail_floats);
    const dim3 grid = rows_of((chunks + kInitChunks - 1) / kInitChunks), block(kInitThreads);
    for_layout(cfg->d, want.tail_floats, [&](auto d, auto tf) {
        hipLaunchKernelGGL((agft_init_kernel<d.value, tf.value>), grid, block, 0, h->stream, a);
    });
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        delete h;
        return AGFT_E_HIP;
    }
    *out = h;
    return AGFT_OK;
}

int agft_step(agft_handle *h, const float *d_ctx, const float *d_reward, int32_t *d_action, float *d_scores) {
    if (h == nullptr) return AGFT_E_INVAL;
    if (h->pending && d_reward == nullptr) return AGFT_E_STATE;
    return launch_step(h, d_ctx, d_reward, d_action, d_scores, nullptr);
}

int agft_sim_step(agft_handle *h, const agft_env_config *env_cfg, void *d_env, size_t env_nbytes,
                  const int32_t *d_arrivals, const float *d_noise, float *d_ctx, float *d_reward,
                  int32_t *d_action, float *d_scores) {
    using namespace agft_env_detail;
    if (h == nullptr || !env_config_ok(env_cfg)) return AGFT_E_INVAL;
    if (env_cfg->B != h->cfg.B || env_cfg->K != h->cfg.K || env_cfg->d != h->cfg.d) return AGFT_E_INVAL;
    if (d_env == nullptr || d_arrivals == nullptr || d_noise == nullptr || d_ctx == nullptr ||
        d_reward == nullptr || d_action == nullptr)
        return AGFT_E_INVAL;
    if (reinterpret_cast<uintptr_t>(d_ctx) % 16 != 0) return AGFT_E_INVAL;
    if (reinterpret_cast<uintptr_t>(d_env) % agft_env_detail::kAlign != 0 || env_nbytes < env_layout(env_cfg->B).total)
        return AGFT_E_INVAL;
    if (h->t >= env_cfg->T) return AGFT_E_STATE;   // the draws end at window T
    // Large batches take the step kernel and then the environment kernel:
    // there the epilogue's per-instance stores to the environment's
    // structure-of-arrays state cost more than the launch they save.
    // Measured on MI355X (us per simulator step, fused / two launches, at
    // B = 1,024, 3,072, 4,096 and 8,192):
    //   d=8 K=64    8.4 / 9.7    12.3 / 12.9    15.3 / 14.7    27.6 / 24.5
    //   d=8 K=200   11.7 / 13.6  26.0 / 26.2    33.5 / 32.2    62.5 / 56.4
    //   d=16 K=128  17.3 / 18.0  42.6 / 45.1    58.6 / 57.7    110.8 / 102.7
    //     the same with rules 2-8  18.8 / 20.0  47.2 / 47.7    62.2 / 59.5    115.9 / 108.9
    //     with the refinement      9.6 / 11.7   12.7 / 14.6    15.3 / 16.2    28.9 / 28.5
    //     mostly exploiting        15.6 / 17.5  19.1 / 20.3    21.7 / 22.0    35.4 / 36.6
    //   d=32 K=256  42.1 / 44.3  116.8 / 116.3  155.7 / 153.1  307.2 / 301.9
    //     late in a run            10.8 / 13.3  25.6 / 26.7    31.2 / 30.8    56.0 / 51.6
    if (h->cfg.B > kFusedMaxB) {
        const int64_t t = h->t;
        const int rc = launch_step(h, d_ctx, d_reward, d_action, d_scores, nullptr);
        if (rc != AGFT_OK) return rc;
        return agft_env_step(env_cfg, d_env, env_nbytes, (int32_t)t, d_action, d_arrivals, d_noise, d_reward, d_ctx,
                             h->stream);
    }
    EnvArgs e = make_args(env_cfg, d_env);
    e.arrivals = d_arrivals;
    e.noise = d_noise;
    e.action = d_action;
    e.reward = d_reward;
    e.ctx = d_ctx;
    e.w = (int32_t)h->t + 1;
    const double tau = env_cfg->T > 1 ? (double)h->t / (double)(env_cfg->T - 1) : 0.0;
    e.scale = (float)(1.0 + (double)env_cfg->drift * tau);
    e.reset = 0;
    return launch_step(h, d_ctx, d_reward, d_action, d_scores, &e);
}

int agft_launch_shape_for(const agft_config *cfg, agft_launch_shape *out) {
    if (out == nullptr || !config_ok(cfg)) return AGFT_E_INVAL;
    if (!supported(cfg)) return AGFT_E_UNSUPPORTED;
    out->waves = waves_for(*cfg);
    out->tail_floats = tail_floats(*cfg);
    out->simd_waves = occupancy_for(*cfg, out->tail_floats);
    out->early_update = early_update(*cfg) ? 1 : 0;
    out->cu_workgroups = cu_workgroups_for(*cfg, out->waves, out->simd_waves);
    return AGFT_OK;
}

int agft_get_state(const agft_handle *h, agft_state_view *out) {
    if (h == nullptr || out == nullptr) return AGFT_E_INVAL;
    out->t = h->t;
    out->pending = h->pending;
    out->B = h->cfg.B;
    out->K = h->cfg.K;
    out->d = h->cfg.d;
    out->tail_floats = tail_floats(h->cfg);
    out->chunks = chunks_for(h->cfg.d, out->tail_floats);
    out->block_arms = block_arms(h->cfg.d);
    out->mask_words = (h->cfg.K + 31) / 32;
    out->arms = h->base + h->lay.arms;
    out->mask = at<uint32_t>(h->base, h->lay.mask);
    out->inst = at<int32_t>(h->base, h->lay.inst);
    out->inst_words = inst_words(h->cfg.d);
    out->stats = at<int32_t>(h->base, h->lay.stats);
    out->theta = h->cfg.exploit ? at<float>(h->base, h->lay.theta) : nullptr;
    return AGFT_OK;
}

int agft_export(agft_handle *h, float *d_theta, float *d_ainv) {
    if (h == nullptr) return AGFT_E_INVAL;
    if (d_theta == nullptr && d_ainv == nullptr) return AGFT_OK;
    const agft_config &c = h->cfg;
    const float4 *arms = at<float4>(h->base, h->lay.arms);
    for_layout(c.d, tail_floats(c), [&](auto d, auto tf) {
        constexpr int D = d.value, TF = tf.value;
        constexpr int arms_per_wg = kExportThreads / (D / 4 * (D / 4)), blocks_per_wg = arms_per_wg / Rec<D, TF>::NB;
        const size_t blocks = (size_t)c.B * (size_t)((c.K + Rec<D, TF>::NB - 1) / Rec<D, TF>::NB);
        hipLaunchKernelGGL((agft_export_kernel<D, TF>), rows_of((blocks + blocks_per_wg - 1) / blocks_per_wg),
                           dim3(kExportThreads), 0, h->stream, arms, c.B, c.K, d_theta, d_ainv);
    });
    return hip_status(hipGetLastError());
}

int agft_set_stream(agft_handle *h, void *stream) {
    if (h == nullptr) return AGFT_E_INVAL;
    h->stream = static_cast<hipStream_t>(stream);
    return AGFT_OK;
}

int agft_destroy(agft_handle *h) {
    delete h;
    return AGFT_OK;
}

const char *agft_strerror(int code) {
    switch (code) {
        case AGFT_OK: return "ok";
        case AGFT_E_INVAL: return "invalid argument";
        case AGFT_E_UNSUPPORTED: return "unsupported configuration";
        case AGFT_E_STATE: return "call not valid in the current state";
        case AGFT_E_HIP: return "HIP runtime error";
        default: return "unknown status";
    }
}

int agft_abi_version(void) { return AGFT_ABI_VERSION; }

}  // extern "C"

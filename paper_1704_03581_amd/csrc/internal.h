// Internal declarations shared by the kernels and the C ABI (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <utility>
#include <vector>

namespace pulda {

// device buffers of one model, carved from the caller's workspace
struct DevModel {
    int32_t K, V, L;
    double beta;
    uint32_t key0, key1;
    const double *alpha;          // [K]
    // counts of the current state (word-major dense: n[v*K + k])
    int32_t *n;
    unsigned long long *nk;       // [K]
    // Phi-step
    unsigned long long *S;        // [K] row sums
    // The urn's draws gamma_kv: each word's row has the narrowest of three
    // formats that holds its largest draw (ROW_8, ROW_16 or ROW_32 in the
    // word's record), topic k at k << format.  A row of format f starts at
    // byte row_base[f] + v row_step[f] of gam: three tables while they end
    // within 4 GiB of gam, the reach of a 32-bit offset, so that the narrow
    // rows lie close together; past that one table, a word's row at the
    // start of its 32-bit one's space whatever the format.  phi_kv is
    // fp32(RN64(gamma_kv / S_k)); fp32(gamma_kv * R_k) with
    // R_k = RN64(1 / S_k) equals it bit for bit for gamma < 2^16 and
    // S_k < 2^27, where no fp32 rounding midpoint lies within the product's
    // error of the quotient.
    uint8_t *gam;
    uint32_t row_base[3], row_step[3];
    int32_t ks16;                 // K rounded up to 64
    // Phi has no integer draws (Algorithm 1's, or one loaded as values): the
    // rows are phid's fp32 values, format ROW_32
    int32_t values;
    float *phid;                  // [V*K]
    double *Rd;                   // [K] RN64(1 / S_k) (0 for an empty row)
    // Algorithm 1's Phi-step (phi_k ~ Dir(n_k + beta)): Gamma draws
    // (word-major dense, fp64), their row sums, and per-block partial sums
    double *gamd;                 // [V*K]
    double *Sd;                   // [K]
    double *dpart;                // [ceil(V / ROWSUM_COLS) * K]
    int32_t phi_method;           // of the last Phi-step: 0 Polya urn, 1 Dirichlet
    int32_t *colcnt;              // [V]
    int32_t *longcol;             // columns with long alias tables, in order; [V]: their number
    int32_t *colptr;              // [V+1]
    uint16_t *ctopic;             // [cap + COL_PAD] CSC by word, ascending topic
    float *cphi;                  // [cap + COL_PAD]
    uint64_t *calias;             // [cap] thr | topic << 32 | alias_topic << 48
    double *sigma_a;              // [V]
    // where Phi has draws: row format << 30; where it is values (all ROW_32):
    // bits of the largest phi of the word's column, any float
    uint32_t *phimax;             // [V]
    // per word, what a z-step token needs of its word in one 16-byte load:
    // {first CSC entry, column length | row format << 30, fp32(sigma_a),
    // largest phi} (as bits)
    uint4 *wrec;                  // [V]
    // the corpus's most frequent words, whose count increments the z-step
    // gathers per block in LDS when K is small (hot[v]: the word's index
    // among them, or -1; hot_word[h]: the word of index h)
    int32_t *hot;                 // [V]
    int32_t *hot_word;            // [HOT_MAX]
    int32_t n_hot;
    const uint64_t *pois;         // Poisson alias tables, thr | x_alias << 32
    const int32_t *pois_off;      // [L+2]
    // per-word priors (null: the symmetric beta); zero-truncated
    // Pois(beta_v) thresholds floor(2^32 P(X <= x | X >= 1)), x = 1.., one row
    // per word in ztp_tab from ztp_off (null: one row of ztp_n for beta)
    const double *beta_v;         // [V]
    const uint32_t *ztp_tab;
    const int32_t *ztp_off;       // [V+1]
    int32_t ztp_n;
    double beta_sum;              // sum_v beta_v (V beta for the symmetric prior)
    // log-joint terms for integer counts x < LG_TABLE:
    //   lg_beta[x] = lgamma(x + beta) - lgamma(beta),
    //   lg_alpha[x] = lgamma(x + alpha) - lgamma(alpha) (symmetric alpha only, else null),
    //   lg_A[x] = lgamma(A) - lgamma(x + A), A = sum_k alpha_k
    const double *lg_beta, *lg_alpha, *lg_A;
    const uint32_t *tptr;         // sweep number t, read on the device
    long long *scratch;           // scan scratch: ceil(max(V, D) / 1024) + 2 entries
};

struct DevCorpus {
    int64_t D, N;
    const int64_t *doc_off;
    const int32_t *words;
    uint16_t *z;
    const int32_t *doc_order;     // documents by decreasing length
    int32_t longest;              // tokens of the longest
};

// a unit of z-step work: `count` documents of doc_order starting at `first`,
// processed by groups of `group` lanes
struct WorkItem {
    int32_t first, count, group;
};

// The z-step's slots per lane: a draw handles up to SLOTS_MAX a lane with
// the kernel's fixed counts of them; longer topic lists turn dense
constexpr int32_t SLOTS_MAX = 16;
constexpr int32_t SLOTS_FEW = 6;           // the most of the kernels for short lists
constexpr size_t LDS_BYTES = 160 * 1024;   // per CU, and the most a block takes
// the row that a word's b-terms are gathered from, by the word's largest
// draw: 8-bit, 16-bit or 32-bit draws (ROW_32 also for phi itself, where Phi
// has no draws: Algorithm 1's, or one loaded as values).  log2 of the bytes per topic, held in the top two bits
// of wrec[v].y (a column has at most 4096 entries).
constexpr uint32_t ROW_8 = 0, ROW_16 = 1, ROW_32 = 2;
constexpr int32_t COL_PAD = 8;             // entries of a column read at once
constexpr uint32_t WREC_LOW = 0x3FFFFFFFu;

// LDS of one group of lanes with a document of at most `longest` tokens:
// counts by topic, counts by slot (groups under 64 lanes), the block's draw
// records, a bit per topic, the slots' topics, the list entries before each
// chunk of topics, the drawn slots
struct SlotLds {
    int32_t slots;                                   // the most per lane
    int32_t wide;                                    // counts by topic of 2 bytes, not 1
    int32_t o_ms, o_tok, o_p, o_lst, o_pre, o_out;   // byte offsets (counts by topic at 0)
    int32_t group_bytes;
    int32_t p_words;                                 // 32-bit words of topic bits
    int32_t log_b, chunks, ch_lane;                  // topics per chunk (log2), chunks, chunks per lane
};

inline SlotLds slot_lds(int32_t G, int32_t K, int32_t longest)
{
    SlotLds A{};
    // a block's slots: topics of the document and of G staged a-parts
    const int32_t most = K < longest + G ? K : longest + G;
    const int32_t need = (most + G - 1) / G;
    static const int32_t sizes[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16};
    A.slots = SLOTS_MAX;
    for (int32_t x : sizes)
        if (x >= need) {
            A.slots = x;
            break;
        }
    A.wide = longest > 255;
    A.p_words = (K + 31) / 32;
    A.log_b = 0;
    while (A.log_b < 5 && ((int64_t)G << A.log_b) < K) ++A.log_b;
    A.chunks = (K + (1 << A.log_b) - 1) >> A.log_b;
    A.ch_lane = (A.chunks + G - 1) / G;
    auto up = [](int32_t x) { return (x + 15) / 16 * 16; };
    A.o_ms = up((K + 1) << A.wide);   // (and a place for slots past the list)
    A.o_tok = A.o_ms + (G == 64 ? 0 : A.slots * G * 4);
    A.o_p = A.o_tok + (G == 64 ? (64 + 8) * 32 : (G + 2) * 16);
    A.o_lst = A.o_p + up(A.p_words * 4);
    A.o_pre = A.o_lst + up(A.slots * G * 2);
    A.o_out = A.o_pre + up(A.chunks * 2);
    A.group_bytes = A.o_out + up((G == 64 ? 128 : G) * 2);   // (64 lanes: a place each for no result)
    return A;
}

// a document's topics and the block's a-parts fit the slots of G lanes
inline bool slots_fit(int32_t G, int32_t K, int32_t longest)
{
    return (K < longest + G ? K : longest + G) <= SLOTS_MAX * G;
}

// They do for as many topics as tokens of uniform topics are expected to hold:
// lanes for fold-in and held-out documents (a list that passes its slots all
// the same is drawn slowly)
inline bool slots_likely(int32_t G, int32_t K, int32_t tokens)
{
    return K * (1.0 - exp(-(double)tokens / K)) + G <= (double)(SLOTS_MAX * G);
}

// a z-step group size fits documents of at most `longest` tokens when their
// slots do (groups of 8 take documents shorter than 256 tokens; 64 lanes
// take every document); one document per lane (group 1) keeps a list of at
// most 127 topics with 8-bit counts (every list fits when K <= 127; a count
// stays below 256)
inline bool z_group_fits(int32_t group, int32_t K, int32_t longest)
{
    if (group == 1) return longest < 128 || (K <= 127 && longest < 256);
    if (group == 64) return true;
    if (group == 8 && longest >= 256) return false;
    return slots_fit(group, K, longest) &&
           (size_t)(K * 4 + 15) / 16 * 16 + 4 * (64 / group) * (size_t)slot_lds(group, K, longest).group_bytes <=
               LDS_BYTES;
}

// LDS for the per-block counts of the frequent words (hot words) and the
// fewest such words worth it
constexpr int32_t HOT_BYTES = 16384;
constexpr int32_t HOT_MIN = 16;
constexpr int32_t HOT_MAX = HOT_BYTES / 4;

// ST_TOKENS counts z-step launches since the last statistics read
constexpr int32_t LG_TABLE = 65536;

// work-item queues of a z-step: one atomic counter per class, cleared by
// launch_z_prepare
constexpr int32_t Z_QUEUES = 16;

enum StatIndex { ST_DEGENERATE = 0, ST_SUM_J = 1, ST_SUM_A = 2, ST_NNZ_PHI = 3, ST_EMPTY_ROWS = 4, ST_TOKENS = 5,
                 ST_SUM_JB = 6, ST_FALLBACK = 7, ST_COUNT = 8 };

// launchers (stream-ordered; return the launch status)
hipError_t launch_fill_u32(uint32_t *p, uint32_t value, int64_t count, hipStream_t s);
hipError_t launch_fill_u64(unsigned long long *p, unsigned long long value, int64_t count, hipStream_t s);
hipError_t launch_validate(const DevCorpus &c, int32_t V, int32_t *err, hipStream_t s);
hipError_t launch_init_z(const DevCorpus &c, int32_t K, uint32_t key0, uint32_t key1, hipStream_t s);
hipError_t launch_count_rebuild(const DevCorpus &c, const DevModel &m, hipStream_t s);
hipError_t launch_row_sums(const int32_t *dense, int32_t V, int32_t K, unsigned long long *out, hipStream_t s);
hipError_t launch_phi_step(const DevModel &m, unsigned long long *stats, int32_t n_cu, hipStream_t s);
// Algorithm 1's Phi-step into the same Phi tables (m.phi_method must be 1)
hipError_t launch_phi_step_dirichlet(const DevModel &m, unsigned long long *stats, int32_t n_cu, hipStream_t s);
constexpr int32_t ROWSUM_COLS = 256;      // words per block of the row-sum kernels
// z-step: launch_z_prepare clears n and the Z_QUEUES work queues; then one
// persistent kernel per work-item class (group size 8 to 64 and count
// width, or one document per lane) over that class's items.
// With ll_doc non-null (symmetric alpha) the z-step also writes each
// document's term of the log joint for the state it leaves.
hipError_t launch_z_prepare(const DevModel &m, int32_t *queues, unsigned long long *stats, hipStream_t s);
// longest: no document of the items has more tokens.  The grid is as many
// blocks as n_cu compute units hold at once.
hipError_t launch_z_class(const DevCorpus &c, const DevModel &m, int32_t group, int32_t longest,
                          const WorkItem *items, int32_t n_items, int32_t n_cu, int32_t *queue, unsigned long long *stats,
                          double *ll_doc, hipStream_t s);
// working space of the log joint
struct LLSpace {
    int32_t max_words, max_docs;   // most blocks of the words' part, of the documents'
    unsigned long long *part_nk;   // [max_words * K]
    double *part;                  // [max_words + max_docs + ceil(K / 16)]
    uint32_t *done;
};
// sweep number t, history index 0
hipError_t launch_set_sweep(uint32_t *tptr, uint32_t t, uint32_t *hist_idx, hipStream_t s);
// log joint of the current state; with ll_doc non-null the document terms
// are taken from it (written by the z-step) instead of recounted from z.
// With advance_t non-null the sweep number there and the history index move
// on by one afterwards.
hipError_t launch_loglik(const DevCorpus &c, const DevModel &m, const LLSpace &space, const double *ll_doc, double *out,
                         double *hist, uint32_t *hist_idx, uint32_t *advance_t, hipStream_t s);
hipError_t launch_n_colcount(const DevModel &m, int64_t *cnt, hipStream_t s);
// rebuild the per-word records from colptr, sigma_a and phimax
hipError_t launch_word_records(const DevModel &m, hipStream_t s);
hipError_t launch_export_phi(const DevModel &m, int64_t *colptr64, uint16_t *topic, int32_t *gam_e, float *phi_e,
                             uint32_t *thr, uint16_t *alias_topic, hipStream_t s);
hipError_t launch_import_phi(const DevModel &m, const int64_t *colptr64, const uint16_t *topic, const float *phi_e,
                             const uint32_t *thr, const uint16_t *alias_topic, hipStream_t s);
hipError_t launch_counts_csc(const DevModel &m, const int64_t *colptr64, uint16_t *topic, int32_t *cnt,
                             int32_t *colcnt_scratch, hipStream_t s);
hipError_t launch_counts_m(const DevCorpus &c, int32_t K, int64_t *rowcnt_or_ptr, uint16_t *topic, int32_t *cnt,
                           int pass, hipStream_t s);
hipError_t launch_check_u16_below(const uint16_t *x, int64_t n, uint32_t limit, int32_t *err, hipStream_t s);
hipError_t launch_check_phi(const int64_t *colptr, int32_t V, const uint16_t *topic, const uint16_t *alias_topic,
                            uint32_t K, int32_t *err, hipStream_t s);
hipError_t launch_scan_i64(const int64_t *in, int64_t *out_excl, int64_t n, long long *scratch, hipStream_t s);

// fold-in
// host-written control of a resident request
struct FoldSlot {
    int32_t arena_off;  // first token of the slot's region in the arena
    int32_t len;        // request length
    uint32_t req;       // request id
    int32_t fresh;      // 1 on the request's first step (drop tokens, draw initial topics)
    int32_t budget;     // token draws to run in this step
    int32_t pad[3];
};

struct DevFoldin {
    int32_t sweeps, burn_in, group;
    // the step's requests whose topics are not likely to fit the slots of
    // `group` lanes (32): the first n_wide active ones, on 64 lanes; longest
    // request of them, of the others
    int32_t n_wide, wide_len, max_len;
    uint32_t key0, key1;
    double A;
    const FoldSlot *slots;  // [max_slots] control, written by the host
    int32_t *kept;          // [2*max_slots] kept, dropped: written by the device
    int32_t *prog;          // [2*max_slots] sweeps done, next token of the current sweep: device-written
    int32_t *words;         // arena [arena_tokens]
    int32_t *pos;           // arena: kept positions
    uint16_t *z;            // arena
    uint32_t *acc;          // [max_slots*K]
    float *theta;           // [max_slots*K]
    double *ll;             // [max_slots]
    int64_t *fin;           // [max_slots] the step that finished the request
                            // (written after theta and ll; 0 until then)
    int64_t step_no;        // this launch's step number (from 1)
};

hipError_t launch_foldin_step(const DevModel &m, const DevFoldin &f, const int32_t *active, int32_t n_active,
                              int32_t n_cu, hipStream_t s);

// held-out log-likelihood of new documents (left-to-right estimate): the
// region of document d's particle r in kw, z and Zs starts at
// doc_off[d] * R + r * N_d (N_d = the document's length)
struct DevHeldout {
    int64_t D;
    int32_t R, group;
    // the documents whose topics are not likely to fit the slots of `group`
    // lanes (32): the first n_wide of the order, on 64 lanes; tokens of the
    // longest of them, of the others
    int64_t n_wide;
    int32_t wide_len, longest;
    uint32_t key0, key1;
    double A;                  // sum_k alpha_k
    const int64_t *doc_off;    // [D+1]
    const int32_t *words;      // [N]
    const uint32_t *req;       // [D] request ids (keys of the random numbers)
    const int32_t *order;      // [D] documents by decreasing length (longest chains start first)
    int32_t *kw;               // [R*N] each particle's kept words
    uint16_t *z;               // [R*N] each particle's topics
    double *Zs;                // [R*N] Z_n of each particle and step
    int32_t *kept;             // [D]
    double *ll;                // [D]
};

hipError_t launch_heldout(const DevModel &m, const DevHeldout &h, hipStream_t s);

}  // namespace pulda

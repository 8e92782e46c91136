// Launchers of the device kernels (one per .hip file), called by the host
// library.  All return the launch status; none synchronises.
#pragma once
#include "common.h"

namespace rp {

uint32_t sort_tile_size();
uint32_t conf_tile_size();

// count_lo: generation stores per-chunk counts of key bits [count_lo,
// count_lo + rb) (the first pass's digit) in item_hist; -1 for none
hipError_t launch_gen(int rb, const GenItem* items, uint32_t n_items, const Job* jobs,
                      const SortSeg* segs, uint64_t* recs, uint32_t* item_hist, int count_lo,
                      hipStream_t s);
// generation items and sort chunks: chunk c of segment s covers its records
// [(c - chunk_beg) * chunk_len, ...) up to the segment's end
hipError_t launch_items(const Job* jobs, const SortSeg* segs, uint32_t nseg, uint32_t nchunks,
                        uint64_t chunk_len, GenItem* items, SortChunk* chunks, hipStream_t s);
// dig: each record's digit of this pass (1 byte for 8-bit digits, else 2),
// as the previous pass's scatter wrote it; unused when counts_ready (pass 0
// takes its counts from record generation)
// n_cblk column blocks over all segments (each segment's from its cblk_beg),
// at most max_cblk in one segment; part: [n_cblk][2^rb] scratch
hipError_t launch_sort_scan(int rb, const void* dig, const SortSeg* segs, uint32_t nseg,
                            const SortChunk* chunks, uint32_t nchunks, uint32_t n_cblk,
                            uint32_t max_cblk, uint32_t* cnt, uint64_t* tot, uint64_t* part,
                            uint64_t* off, uint32_t* ticket, bool counts_ready, hipStream_t s);
// The pass sorts by key bits [lo, lo + rb) above each segment's key shift;
// the next pass's digit, key bits [nlo, nlo + nbits), is stored per output
// record in dnext (1 byte for up to 8 bits, else 2; NULL after the last
// pass); ticket: one device word, set to zero by launch_sort_scan of the
// same pass; pass: the pass's index in execution order (its tile shape)
hipError_t launch_sort_scatter(int rb, int pass, const uint64_t* in, uint64_t* out,
                               const SortSeg* segs, const SortChunk* chunks, uint32_t nchunks,
                               int lo, int nlo, int nbits, const uint64_t* off, uint32_t* ticket,
                               uint32_t* err, void* dnext, hipStream_t s);
// Radix-scatter tile shapes 0..SCATTER_SHAPE_MAX; the per-pass shapes'
// default (every pass on the common shape)
constexpr int SCATTER_SHAPE_MAX = 9;
constexpr int PASS_SHAPES_DEFAULT = 0x0FFFFFFF;
constexpr int IVL_RESOLVE = 0, IVL_CHECK = 1, IVL_ZERO = 2;
hipError_t launch_ivl(const Job* jobs, uint32_t njobs, int mode, hipStream_t s);
hipError_t launch_save_j0(const Job* jobs, uint32_t njobs, hipStream_t s);
// Lays out the round's tiles over the logs of running jobs: ctile_beg of
// each segment, the total in *tiles.
hipError_t launch_conf_tiles(const Job* jobs, ConfSeg* segs, int nseg, uint32_t* tiles,
                             hipStream_t s);
// Every racing pair under x over the tiles laid out by launch_conf_tiles.
hipError_t launch_conf(const Job* jobs, const ConfSeg* segs, int nseg, uint32_t max_points,
                       const uint32_t* tiles, hipStream_t s);
// First partners with no barrier enabled, into minj (cleared beforehand).
// lo32: the point and id fields of every record lie in its low 32 bits
// (thread, block and point bits together at most 32, in every job)
hipError_t launch_j0(const Job* jobs, const ConfSeg* segs, int nseg, uint32_t max_points,
                     bool lo32, const uint32_t* tiles, hipStream_t s);
// First partners of the PF_CLOSED points, into j0 (every row of a job that has
// no records).  form: the narrowest one that every closed array of every job
// fits (FORM_*).
hipError_t launch_first_closed(const Job* jobs, uint32_t njobs, uint32_t max_points, int form,
                               const CallBlock& call, hipStream_t s);
// First partners under its assignment of one job that has no records, into
// minj; the last kernel of its call.
hipError_t launch_first_under(const Job* job, uint32_t points, int form, const CallBlock& call,
                              hipStream_t s);
// Racing pairs of the PF_CLOSED points of one job under its assignment: bitmap
// rows, and their counts in minj (every row of a job that
// has no records).
hipError_t launch_all_closed(const Job* job, uint32_t points, int form, const CallBlock& call,
                             hipStream_t s);
// The bitmap of one job as a pair list in (level, i, j) order.  counted: the
// row counts are in minj already.
hipError_t launch_pairs(const Job* job, uint32_t points, bool counted, rp_pair* out,
                        uint64_t* total, const CallBlock& call, hipStream_t s);
// The rounds of Alg. 1 on every running job.  RD_BUILD: the job's clause tables
// from j0 first (a packed job, see PACKED_TESTS, works out
// j0 itself; RD_FIRST: every job is one, and no first-partner launch has
// come before); RD_SOLVE: one Solve first; RD_LOOP: rounds, at most limit of
// them (0: until a verdict); RD_LEARN: Verify and GenerateClause under the
// job's assignment only; RD_TIMED: the phases' clock ticks into the job state.
constexpr int RD_BUILD = 1, RD_SOLVE = 2, RD_LOOP = 4, RD_LEARN = 8, RD_TIMED = 16,
              RD_FIRST = 32;
// Most points, and most pair tests by the plan's bound, of a job whose first
// partners the rounds kernel works out (Job::packed).  Its one workgroup tests
// 256 pairs at a time, a test 1.6 to 2.8 us there (nothing else hides its
// latency), where the launch of first_kernel costs a lone job 5 to 8 us and
// spreads the rows over the chip: 128 points of one array that never conflict
// 64 and 12 + 5 us over one view, 189 and 12 + 8 us over two, and 15 ms and 0.3
// ms where a pair's walk meets 256 values; 32 points over one view 40 and 37 us
// a call.  In batches the launch is shared and the line matters less: 512
// programs together 104 us with the line at 128, 512 or 1,024 and 101 us with all
// up to 128 points packed, 128 batched kernels 154 us up to 2,048 and 162 us
// with all (means over eight seeds).
constexpr uint32_t PACKED_POINTS = 128;
constexpr double PACKED_TESTS = 512;
hipError_t launch_rounds(const Job* jobs, uint32_t njobs, int form, int flags, uint32_t limit,
                         const CallBlock& call, hipStream_t s);

}  // namespace rp

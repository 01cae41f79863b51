// The library as one translation unit, hence one device code object.  The units below can be compiled each by itself,
// in 90 s side by side instead of 220, but then every one is a code object of its own, and where it lands on the GPU is
// left to chance.  A program that alternates between kernels notices (see proj_kernels.hpp): absorbed query, decode and
// output projection one behind the other (24 sequences of 200 to 6000 tokens, two latent heads) took 142.3 and 143.7 us per
// round in two builds of five code objects (105 now, with faster kernels).  The decode alone, again and again, takes the same time wherever it lies.
#include "gla_decode.hip"
#include "tuned_128.hip"
#include "tuned_256.hip"
#include "tuned_512.hip"
#include "wide.hip"
